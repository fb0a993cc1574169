"""apply_H by another route than a call's own: the allocation-free entry and calls
under graph capture run from the tables that an earlier product of another block
width, or of columns that pair up otherwise, has built; and the routes of the
allocation-free entry that give syk_apply_H's bits: two columns per workgroup,
and the coefficient table of small states; and automatic tiles with the columns
per workgroup and the tile order set by the caller."""
import numpy as np
import pytest
import torch

from paper_2002_05725_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TOL = {torch.complex128: 1e-12, torch.complex64: 2e-6}


def _handle(N):
    return api.Terms(N, np.stack([inputs.couplings(N, 70 + r) for r in range(2)]))


def _states(N, nvec, dtype, seed=0):
    g = torch.Generator(device=DEV).manual_seed(100 * N + nvec + seed)
    x = torch.randn((nvec, 1 << (N // 2)), dtype=dtype, device=DEV, generator=g)
    return x / x.norm(dim=-1, keepdim=True)


def _cols(nvec, paired):
    return np.array([c // 2 % 2 if paired else c % 2 for c in range(nvec)], dtype=np.int32)


def _ref(N, x, real):
    """The product on a handle of its own, by the call's own route."""
    T = _handle(N)
    y = api.apply_H(T, x, real_of_col=real)
    T.close()
    return y


# (N, width and pairing of the warm-up, of the call): table and split 8-row kernel,
# split 16-row kernel, its split and unsplit launches, one and two layouts, and the
# complex64 window in which paired columns run two per workgroup
CASES = [(20, 1, 0, 16, 0), (20, 33, 0, 4, 0), (24, 1, 0, 64, 0), (24, 8, 0, 1, 0), (24, 8, 0, 33, 0), (26, 1, 0, 64, 0),
         (26, 5, 0, 1, 0), (30, 2, 0, 33, 0), (34, 1, 0, 4, 0), (36, 8, 0, 8, 1), (36, 8, 1, 8, 0), (36, 1, 0, 3, 0),
         (38, 8, 1, 4, 0)]


# paired complex64 blocks wide enough for two columns per workgroup
PAIRED = [(36, 32, 0, 32, 1), (38, 16, 0, 16, 1), (38, 16, 1, 4, 0)]


@pytest.mark.parametrize("N,na,pa,nb,pb,dtype", [c + (d,) for d in TOL for c in CASES] + [c + (torch.complex64,) for c in PAIRED])
def test_noalloc_after_another_width_or_pairing(N, na, pa, nb, pb, dtype):
    x, real = _states(N, nb, dtype), _cols(nb, pb)
    ref = _ref(N, x, real)
    T = _handle(N)
    api.apply_H(T, _states(N, na, dtype, 7), real_of_col=_cols(na, pa))
    print(f"[routes] N={N} {dtype} after width {na}: width {nb}", flush=True)
    out = torch.full_like(x, complex(float("nan"), float("nan")))
    api.apply_H_noalloc(T, x, out, real_of_col=real)
    err = ((out - ref).norm(dim=-1) / ref.norm(dim=-1)).max().item()
    assert err <= TOL[dtype]
    T.close()


@pytest.mark.parametrize("N,nvec,paired,dtype", [(36, 8, 1, torch.complex64), (36, 8, 0, torch.complex64),
                                                 (36, 32, 1, torch.complex64), (38, 16, 1, torch.complex64),
                                                 (16, 1, 0, torch.complex128), (20, 5, 0, torch.complex64),
                                                 (24, 1, 0, torch.complex128), (24, 6, 0, torch.complex128),
                                                 (4, 3, 0, torch.complex128)])
def test_noalloc_after_the_same_call_gives_its_bits(N, nvec, paired, dtype):
    T = _handle(N)
    x, real = _states(N, nvec, dtype), _cols(nvec, paired)
    ref = api.apply_H(T, x, real_of_col=real)
    out = torch.full_like(x, complex(float("nan"), float("nan")))
    api.apply_H_noalloc(T, x, out, real_of_col=real)
    assert torch.equal(out, ref)
    T.close()


def test_noalloc_needs_a_product_of_its_dtype():
    for N in (16, 26):
        T = _handle(N)
        api.apply_H(T, _states(N, 1, torch.complex128))
        x = _states(N, 1, torch.complex64)
        with pytest.raises(_lib.SykError) as e:
            api.apply_H_noalloc(T, x, torch.empty_like(x))
        assert e.value.status == _lib.SYK_EINVAL and "tables" in str(e.value)
        T.close()


@pytest.mark.parametrize("dtype", list(TOL))
@pytest.mark.parametrize("N,warm,nvec", [(16, 1, 1), (20, 1, 33), (24, 8, 1), (26, 1, 1), (26, 1, 5), (32, 1, 1), (34, 4, 2)])
def test_captured_product_outlives_wider_calls(N, warm, nvec, dtype):
    """A product captured after a warm-up of width `warm`, replayed between eager
    products of larger and smaller blocks on the same handle (whose scratch grows)."""
    T = _handle(N)
    api.apply_H(T, _states(N, warm, dtype, 3), real_of_col=_cols(warm, 0))
    x, real = _states(N, nvec, dtype), _cols(nvec, 0)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        api.apply_H(T, x, y, real_of_col=real)
    for k, width in enumerate((1, 9, 3)):
        x.copy_(_states(N, nvec, dtype, 20 + k))
        y.fill_(complex(float("nan"), float("nan")))
        ref = _ref(N, x, real)
        wide = _states(N, width, dtype, 40 + k)
        got = api.apply_H(T, wide, real_of_col=_cols(width, 0))
        wref = _ref(N, wide, _cols(width, 0))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        err = ((y - ref).norm(dim=-1) / ref.norm(dim=-1)).max().item()
        assert err <= TOL[dtype], k
        assert ((got - wref).norm(dim=-1) / wref.norm(dim=-1)).max().item() <= TOL[dtype]
    T.close()


@pytest.mark.parametrize("dtype", list(TOL))
@pytest.mark.parametrize("N,nvec", [(20, 4), (26, 6), (32, 64), (36, 8)])
def test_automatic_tiles_with_columns_asked_for(N, nvec, dtype):
    """Two columns per workgroup on automatic tiles is the 2^11-row kernel (bit for
    bit, where neither launch is split); one column and the other tile order
    give the same product."""
    x, real = _states(N, nvec, dtype), _cols(nvec, 1)
    T = _handle(N)
    ref = api.apply_H(T, x, real_of_col=real)
    for xcd in (0, 1):
        for cols in (1, 2):
            api.set_apply_tuning(T, 0, xcd, cols)
            y = api.apply_H(T, x, real_of_col=real)
            assert ((y - ref).norm(dim=-1) / ref.norm(dim=-1)).max().item() <= TOL[dtype], (xcd, cols)
    if (nvec << (N // 2)) >> 11 >= 1024:
        api.set_apply_tuning(T, 11, 1, 2)
        assert torch.equal(api.apply_H(T, x, real_of_col=real), y)
    T.close()
