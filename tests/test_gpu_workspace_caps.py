"""Workspace caps that suffice: the smallest caps (to 16 bytes) under which the
one-buffer reductions and the unsplit pairs of the coupling derivatives run each
call.  Faster paths that need more room must not take a call past its cap, and
give the same results."""
import numpy as np
import pytest
import torch

from paper_2002_05725_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _states(N, nvec, dtype):
    g = torch.Generator(device=DEV).manual_seed(1)
    x = torch.randn((nvec, 1 << (N // 2)), dtype=dtype, device=DEV, generator=g)
    return x / x.norm(dim=-1, keepdim=True)


def _expmv(nvec, m, dtype):
    def run(T):
        x = _states(T.N, nvec, dtype)
        api.krylov_expmv(T, x, -1j, 0.1, m=m, dt=0.1)
        return x.cpu().numpy()
    return run


def _one(T):
    return _states(T.N, 1, torch.complex128)[0].contiguous()


def _two_point(T):
    return api.two_point(T, 0, 2.0, [0.0, 0.1], _one(T), m=12, dt=0.1, tau_step=0.5)[0]


def _lowest(T):
    return api.lowest_eigenvalues(T, _one(T), k=2, m=48)[0]


def _overlaps(pairs):
    def run(T):
        x = _one(T)
        return api.coupling_overlaps(T, [(x, x, 1.0)] * pairs)
    return run


def _cheb(grad):
    def run(T):
        o = api.cheb_opts(degree=16, dt=0.1, e_halfwidth=0.06 * T.N + 0.5, keep_segment=False)
        if grad:
            return api.grad_couplings(T, 0, 1, 2.0, 0.1, _one(T), o)[1]
        return np.array([api.cheb_otoc(T, 0, 1, 2.0, 0.1, _one(T), o)])
    return run


C128, C64 = torch.complex128, torch.complex64
CASES = [(8, 19664, _cheb(True)), (16, 295312, _cheb(True)), (22, 2441392, _cheb(True)), (24, 5249952, _cheb(True)),
         (26, 11531488, _cheb(True)), (26, 1180544, _cheb(False)),
         (8, 7104, _overlaps(64)), (20, 259760, _overlaps(32)), (24, 1644352, _overlaps(4)), (24, 1646752, _overlaps(64)),
         (24, 1384112, _expmv(1, 20, C128)), (24, 1352624, _expmv(1, 40, C64)), (24, 55003920, _expmv(64, 12, C128)),
         (26, 1193264, _expmv(1, 8, C128)), (26, 5561536, _expmv(4, 20, C64)), (24, 1056656, _two_point),
         (26, 6437680, _lowest)]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_call_runs_under_its_cap(k):
    N, cap, run = CASES[k]
    J = inputs.couplings(N, 0)
    T = api.Terms(N, J)
    ref = run(T)
    T.close()
    T = api.Terms(N, J)
    api.set_workspace_limit(T, cap)
    got = run(T)
    tol = 2e-6 if got.dtype == np.complex64 else 1e-11
    assert np.abs(got - ref).max() <= tol * max(1.0, np.abs(ref).max())
    T.close()
    # half of it does not suffice, and says so
    T = api.Terms(N, J)
    api.set_workspace_limit(T, cap // 2)
    with pytest.raises(_lib.SykError) as e:
        run(T)
    assert e.value.status == _lib.SYK_ENOMEM
    T.close()
