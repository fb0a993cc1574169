"""The 16-row apply kernel (states of at least 2^13 rows) against the checker on
sampled rows: two tiles, one and two row layouts on both sides of their
threshold, split and unsplit launches, columns of several realisations and
parity sectors; its complex64 sums stay as accurate as short FP32 sums allow."""
import numpy as np
import pytest
import torch

from oracle import native
from paper_2002_05725_amd import api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("N,nvec", [(26, 2), (28, 64), (36, 16), (38, 1), (40, 1), (42, 2), (46, 1), (48, 1)])
def test_rows_match_checker(N, nvec):
    Js = np.stack([inputs.couplings(N, 60 + r) for r in range(min(nvec, 2))])
    real = np.array([c % len(Js) for c in range(nvec)], dtype=np.int32)
    psi = [inputs.typical_state(N, 600 + c) for c in range(min(nvec, 2))]
    x = torch.from_numpy(np.stack([psi[c % len(psi)] for c in range(nvec)])).to(DEV)
    D = x.shape[1]
    rows = np.unique(np.concatenate([inputs.row_sample(N, 5, 256), [0, 255, 256, 4095, 4096, D - 1]]))
    idx = torch.from_numpy(rows).to(DEV)
    T = api.Terms(N, Js)
    for dtype, tol in ((torch.complex128, 1e-12), (torch.complex64, 5e-7)):
        y = api.apply_H(T, x.to(dtype), real_of_col=real)
        for c in sorted({0, nvec - 1}):
            ref = native.apply_rows(N, Js[real[c]], psi[c % len(psi)], rows)
            print(f"[groups] N={N} column {c} of {nvec} {dtype}", flush=True)
            assert _rel(y[c][idx].cpu().numpy().astype(np.complex128), ref) <= tol
    T.close()
