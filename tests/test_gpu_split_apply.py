"""apply_H of small states against the checker.  Up to 2^12 rows and a few
columns the product runs from a coefficient table (fewer rows than a
workgroup's 16, the largest state, and blocks at which the table gives way);
above, the masks are split over several workgroups per tile and summed by a
second kernel: one tile (N = 22), a few tiles, masks that flip only qubits above the tile (N = 34, 36), two row
layouts (N = 38), columns that do not pair up, and parity sectors."""
import numpy as np
import pytest
import torch

from oracle import native
from paper_2002_05725_amd import api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TOL = {torch.complex128: 1e-12, torch.complex64: 2e-6}


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("dtype", list(TOL))
@pytest.mark.parametrize("N,nvec", [(4, 1), (6, 3), (8, 2), (20, 10), (22, 70), (24, 1), (24, 3), (26, 33), (34, 1), (36, 2), (38, 1)])
def test_split_product_matches_checker(N, nvec, dtype):
    Js = np.stack([inputs.couplings(N, 40 + r) for r in range(min(nvec, 2))])
    real = np.array([c % len(Js) for c in range(nvec)], dtype=np.int32)
    psis = np.stack([inputs.typical_state(N, 400 + c) for c in range(nvec)])
    T = api.Terms(N, Js)
    y = api.apply_H(T, torch.from_numpy(psis).to(DEV).to(dtype), real_of_col=real).cpu().numpy()
    for c in sorted({0, nvec - 1}):
        if N <= 26:
            ref, got = native.apply_full(N, Js[real[c]], psis[c]), y[c]
        else:
            rows = np.unique(np.concatenate([inputs.row_sample(N, 7, 512), [0, 2047, 2048, psis.shape[1] - 1]]))
            ref, got = native.apply_rows(N, Js[real[c]], psis[c], rows), y[c][rows]
        print(f"[split] N={N} nvec={nvec} column {c} {dtype}", flush=True)
        assert _rel(got.astype(np.complex128), ref) <= TOL[dtype]
    T.close()


@pytest.mark.parametrize("N", [6, 20, 24, 26, 36])
def test_split_product_of_a_sector_matches_the_full_one(N):
    M = N // 2
    T = api.Terms(N, inputs.couplings(N, 3))
    u = np.arange(1 << (M - 1), dtype=np.int64)
    par = np.array([bin(v).count("1") & 1 for v in u])
    for s in (0, 1):
        rows = u + ((par ^ s) << (M - 1))
        x = inputs.typical_sector_state(N, s, 11)
        full = np.zeros(1 << M, dtype=np.complex128)
        full[rows] = x
        ref = api.apply_H(T, torch.from_numpy(full).to(DEV)).cpu().numpy()[rows]
        got = api.apply_H(T, torch.from_numpy(x).to(DEV), sector=s).cpu().numpy()
        assert _rel(got, ref) <= 1e-12
    T.close()
