"""The 16-row apply kernel on parity-sector states, unsplit with two row layouts
(2^18 to 2^20 rows), against the oracle on sampled rows of the full space; several
columns of two realisations, both precisions."""
import numpy as np
import pytest
import torch

from oracle import native
from paper_2002_05725_amd import api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("N,sector,nvec", [(38, 0, 9), (38, 1, 16), (40, 1, 5), (42, 0, 3)])
def test_sector_rows_match_oracle(N, sector, nvec):
    M = N // 2
    Js = np.stack([inputs.couplings(N, 80 + r) for r in range(2)])
    real = np.array([c % 2 for c in range(nvec)], dtype=np.int32)
    states = [inputs.typical_sector_state(N, sector, 800 + c) for c in range(2)]
    D = states[0].size
    u = np.unique(np.concatenate([np.random.default_rng(N).integers(0, D, 192), [0, 255, 4095, 4096, D - 1]]))
    pop = np.zeros(u.shape, dtype=np.int64)
    for b in range(M - 1):
        pop += (u >> b) & 1
    rows = u + (((pop & 1) ^ sector) << (M - 1))            # the full rows the sector rows stand for
    allu = np.arange(D, dtype=np.int64)
    par = np.zeros(D, dtype=np.int64)
    for b in range(M - 1):
        par ^= (allu >> b) & 1
    allrows = allu + ((par ^ sector) << (M - 1))
    refs = []
    for c in range(2):
        full = np.zeros(1 << M, dtype=np.complex128)
        full[allrows] = states[c]
        refs.append(native.apply_rows(N, Js[c], full, rows))
    x = torch.from_numpy(np.stack([states[c % 2] for c in range(nvec)])).to(DEV)
    idx = torch.from_numpy(u).to(DEV)
    T = api.Terms(N, Js)
    for dtype, tol in ((torch.complex128, 1e-12), (torch.complex64, 5e-7)):
        y = api.apply_H(T, x.to(dtype), real_of_col=real, sector=sector)
        print(f"[group-sectors] N={N} sector {sector} {nvec} columns {dtype}", flush=True)
        for c in sorted({0, 1, nvec - 1}):
            got = y[c][idx].cpu().numpy().astype(np.complex128)
            assert np.linalg.norm(got - refs[c % 2]) <= tol * np.linalg.norm(refs[c % 2])
    T.close()
