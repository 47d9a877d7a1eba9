"""The largest grids the plan-free solve takes: its tables and workspace fill the
static array only with larger chunk rows than the built-in ones, so those are
taken, with the bits of a plan of the same chunk rows; one plane more is refused."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2005_11806_amd import _abi
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _solve(grid, f, rho, pp, out):
    lib = _abi.load()
    g, _keep = grid._c()
    o = _abi.psv_opts()
    lib.psv_opts_default(C.byref(o))
    ptr = [C.c_void_p(t.data_ptr()) for t in (f, rho, pp, out)]
    return lib.psv_solve_static(C.byref(g), C.byref(o), ptr[0], ptr[1], 0.0, ptr[2], ptr[3], 1,
                                C.c_void_p(torch.cuda.current_stream().cuda_stream))


@pytest.mark.parametrize("nx,ny,nz,kc", [(128, 128, 413, 16), (64, 64, 1621, 16), (256, 64, 420, 16),
                                         (486, 486, 23, 8), (128, 128, 354, 8)])
def test_largest_grids(gpu, nx, ny, nz, kc):
    gen = torch.Generator(device="cuda").manual_seed(61)
    f, u, pp = (torch.randn(nz + 1, ny, nx, generator=gen, device="cuda", dtype=torch.float64) for _ in range(3))
    rho = 1.0 + u.abs()
    grid = gpu.Grid(nx, ny, nz, 1.0, 1.0, 1.0)
    out = torch.full(grid.shape, np.nan, device="cuda", dtype=torch.float64)
    say(f"static {nx}x{ny}x{nz}")
    _abi.check(_solve(grid, f, rho, pp, out))
    a = [t[:nz].contiguous() for t in (f, rho, pp)]
    assert torch.equal(out, gpu.Plan(grid, chunk_rows=kc).solve(a[0], rho=a[1], p_prev=a[2]))
    if nz != 354:  # (354: the most the built-in chunk rows take)
        more = torch.empty(nz + 1, ny, nx, device="cuda", dtype=torch.float64)
        st = _solve(gpu.Grid(nx, ny, nz + 1, 1.0, 1.0, 1.0), f, rho, pp, more)
        assert st == _abi.PSV_ERR_UNSUPPORTED_SIZE
