"""A first product that fails before its coefficient table is filled leaves the
handle without one: the next product builds it.  The failure is a first call on
a stream under graph capture, where the library's wait for the fill is refused."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import native
from paper_2002_05725_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
RELAXED = 2   # hipStreamCaptureModeRelaxed: allocations go through, waits do not


@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-12), (torch.complex64, 2e-6)])
def test_product_after_a_refused_first_call(dtype, tol):
    N = 16
    hip = ctypes.CDLL("libamdhip64.so")
    J = inputs.couplings(N, 2)
    psi = inputs.typical_state(N, 21)
    x = torch.from_numpy(psi).to(DEV).to(dtype)
    y = torch.zeros_like(x)
    # memory the table may be given next holds large values
    junk = torch.full((1 << 22,), 1e3, dtype=torch.float64, device=DEV)
    T = api.Terms(N, J)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    del junk
    torch.cuda.empty_cache()
    st = ctypes.c_void_p(s.cuda_stream)
    graph = ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(st, RELAXED) == 0
    try:
        with torch.cuda.stream(s), pytest.raises(_lib.SykError):
            api.apply_H(T, x, y)
    finally:
        hip.hipStreamEndCapture(st, ctypes.byref(graph))
        if graph.value:
            hip.hipGraphDestroy(graph)
        hip.hipGetLastError()
    api.apply_H(T, x, y)
    ref = native.apply_full(N, J, psi)
    got = y.cpu().numpy().astype(np.complex128)
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert rel <= tol
    T.close()
