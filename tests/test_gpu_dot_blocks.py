"""Column-wise dot products of blocks against numpy: few results, which the
finishing kernel writes to host memory, and many, which are copied (from 2,049
columns on); one and several workgroups per column, and a column count that does
not fill the last workgroup."""
import numpy as np
import pytest
import torch

from paper_2002_05725_amd import api

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("D,nvec", [(2, 1), (16, 3), (256, 2047), (300, 2048), (300, 2049), (1024, 4097), (16, 60001)])
def test_block_dots(D, nvec, dtype):
    g = torch.Generator(device=DEV).manual_seed(D + nvec)
    a = torch.randn((nvec, D), dtype=dtype, device=DEV, generator=g)
    b = torch.randn((nvec, D), dtype=dtype, device=DEV, generator=g)
    got = api.dot(a, b)
    x, y = a.cpu().numpy().astype(np.complex128), b.cpu().numpy().astype(np.complex128)
    ref = np.sum(np.conj(x) * y, axis=1)
    # FP64 sums of D products of entries of size one
    assert np.abs(got - ref).max() <= 1e-15 * D * 4
    assert np.array_equal(api.dot(a, b), got)
