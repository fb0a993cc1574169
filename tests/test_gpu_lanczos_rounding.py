"""Rounding of the Lanczos scalars on states whose reductions run over many
workgroups: the off-diagonal entry of a two-vector tridiagonal matrix is
(theta_2 - theta_1) / 2 up to the small diagonal, and its error is that of the
sums of ||psi||^2 and ||w||^2 (the products' own rounding averages out over the
rows).

Expected rms at 2^16 rows: half of 7.7e-17 for each of the two sums added
pairwise, 4.6e-17 for the square root, 1.5e-16 for the 2 x 2 eigenvalues, together
1.7e-16; with the 256 workgroup sums added one after another 2.7e-16."""
import numpy as np
import pytest
import torch

from paper_2002_05725_amd import api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _norm2(x):
    x = x.cpu().numpy()
    return np.sum(x.real.astype(np.longdouble) ** 2) + np.sum(x.imag.astype(np.longdouble) ** 2)


def test_beta_is_as_accurate_as_pairwise_sums():
    N, n = 32, 300
    T = api.Terms(N, inputs.couplings(N, 4))
    g = torch.Generator(device=DEV).manual_seed(5)
    err = []
    for _ in range(n):
        x = torch.randn(T.dim, dtype=torch.complex128, device=DEV, generator=g)
        ev, _ = api.lowest_eigenvalues(T, x, k=2, m=2)
        w = api.apply_H(T, x)
        p, q = x.cpu().numpy(), w.cpu().numpy()
        nx = _norm2(x)
        a0 = np.sum(p.real.astype(np.longdouble) * q.real + p.imag.astype(np.longdouble) * q.imag) / nx
        b = np.sqrt(_norm2(w) / nx - a0 * a0)
        # the second diagonal entry from the trace: theta_1 + theta_2 = a0 + a1
        a1 = np.longdouble(ev[0]) + np.longdouble(ev[1]) - a0
        ref = np.sqrt(((a0 - a1) / 2) ** 2 + b * b)
        got = (np.longdouble(ev[1]) - np.longdouble(ev[0])) / 2
        err.append(float((got - ref) / ref))
    rms = float(np.sqrt(np.mean(np.square(err))))
    print(f"[rounding] rms relative error of beta over {n} states: {rms:.3g}", flush=True)
    assert rms <= 2.0e-16
    T.close()
