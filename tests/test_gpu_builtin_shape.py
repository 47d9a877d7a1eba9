"""The built-in x lines of the inverse pass: 8 where they fill the steps of a block
and there are three tiles per CU (FP64), else the forward pass's; the counts on
both sides of each line give the same bits."""
import pytest
import torch

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,prec,eight", [
    (256, 64, 96, "fp64", True), (256, 64, 95, "fp64", False), (256, 48, 512, "fp64", True),
    (256, 36, 512, "fp64", False), (192, 64, 128, "fp64", False), (256, 64, 96, "mixed", False),
    (512, 64, 128, "fp64", False)])
def test_inverse_lines(gpu, nx, ny, nz, prec, eight):
    plan = gpu.Plan(gpu.Grid(nx, ny, nz, 1.0, 1.0, 1.0), precision=prec, method="const")
    sh = plan.get_shape()
    say(f"{prec} {nx}x{ny}x{nz}: {sh}")
    assert sh["lines_x_inv"] == (8 if eight else sh["lines_x"])
    assert not eight or sh["lines_x"] == 4
    f = torch.randn(nz, ny, nx, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(71))
    p = plan.solve(f)
    plan.set_shape(lines_x_inv=4 if sh["lines_x_inv"] == 8 else 2)
    assert torch.equal(plan.solve(f), p)
