"""The compile-time transforms of the x and y passes, every length and tile
shape: x tiles of one step per thread and of several, with full and partial
waves, staged rows and direct loads; y tiles with ragged last chunks. Against
the oracle at the paths' tolerances (FP64 1e-11, mixed 1e-8 and relres 1e-10)."""
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev, host, oracle_inputs, rel_max_err, say

pytestmark = pytest.mark.gpu

TOL_FP64 = 1e-11


def _case(nx, ny, nz, seed):
    lz = 0.9
    spec = W.GridSpec(nx, ny, nz, 1.0, 0.8, lz, W.tanh_faces(nz, lz, 1.5))
    return spec, oracle_inputs(W.two_phase_case("lengths", spec, 1, seed, n_spheres=3))


def _check(gpu, spec, inp, shapes):
    g, f, rho, pp = inp
    (ref,), _ = O.solve(f, g, rho, pp, with_relres=False)
    f, rho, pp = dev(f), dev(rho), dev(pp)
    for prec in ("fp64", "mixed"):
        plan = gpu.Plan(gpu.Grid.from_spec(spec), precision=prec)
        for shape in shapes:
            try:
                plan.set_shape(**shape)
            except gpu.PsvError:  # the tile does not fit a block
                continue
            say(f"{prec} {spec.nx}x{spec.ny}x{spec.nz} {plan.get_shape()}")
            p, info = plan.solve(f, rho=rho, p_prev=pp, info=True)
            err = rel_max_err(host(p), ref)
            assert err <= (TOL_FP64 if prec == "fp64" else 1e-8), (shape, err)
            assert info.relres <= (1e-12 if prec == "fp64" else 1e-10), (shape, info.relres)


@pytest.mark.parametrize("nx", [16, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 192, 216, 256, 288,
                                324, 384, 512, 768, 1024])
def test_x_lengths(gpu, nx):
    spec, inp = _case(nx, 48, 3, 31)
    _check(gpu, spec, inp, [dict(lines_x=lb, lines_x_inv=lb, x_staged=st)
                            for lb in (1, 2, 3, 4, 8, 16) for st in (1, 0)])


@pytest.mark.parametrize("ny", [16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256,
                                288, 324, 384, 432, 512, 768, 1024])
def test_y_lengths(gpu, ny):
    spec, inp = _case(8, ny, 19, 32)
    _check(gpu, spec, inp, [dict(chunk_rows=kc) for kc in (4, 8, 16)])
