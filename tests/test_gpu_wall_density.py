"""Cells of density 0 at the walls, with rho0 given: every face has a positive
density (the mean of its two cells) and no flux crosses a wall, so the step is
finite. Compile-time and runtime x lengths, staged rows and direct loads, two
planes (each next to both walls) and more. Against the oracle at the paths'
tolerances (FP64 1e-11, mixed 1e-8)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev, host, oracle_inputs, rel_max_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz", [(16, 2), (16, 12), (64, 5), (486, 3)])
def test_vacuum_at_the_walls(gpu, nx, nz):
    spec = W.GridSpec(nx, 12, nz, 1.0, 0.8, 0.6)
    g, f, rho, pp = oracle_inputs(W.two_phase_case("vacuum", spec, 1, 51, n_spheres=3))
    rho = rho.copy()
    for k, j, i in ((0, 3, 5), (0, 0, 0), (nz - 1, 7, nx - 1), (nz - 1, 11, 2)):
        rho[k, j, i] = 0.0
    (ref,), _ = O.solve(f, g, rho, pp, rho0=0.5, with_relres=False)
    assert np.isfinite(ref).all()
    f, rho, pp = dev(f), dev(rho), dev(pp)
    grid = gpu.Grid.from_spec(spec)
    for prec, tol in (("fp64", 1e-11), ("mixed", 1e-8)):
        for stencil in ("staged", "direct"):
            say(f"{prec} {stencil} {nx}x12x{nz}")
            plan = gpu.Plan(grid, precision=prec, x_stencil=stencil)
            assert rel_max_err(host(plan.solve(f, rho=rho, p_prev=pp, rho0=0.5)), ref) <= tol
            batch = gpu.Batch([grid], precision=prec, x_stencil=stencil)
            (p,) = batch.solve([f], [rho], [pp], rho0s=[0.5])
            assert rel_max_err(host(p), ref) <= tol
