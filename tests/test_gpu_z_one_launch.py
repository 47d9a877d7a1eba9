"""The wall-normal solve in one launch: every y length it takes, chunk rows 4,
8 and 16, the largest column of each length and the first past it (three
launches), ragged last chunks, fewer rows than a chunk, ragged blocks of
two-dimensional wavenumbers. Against the oracle at the paths' tolerances (FP64
1e-11, mixed 1e-8). relres within 1e-10: with 1024 stretched rows the rounding of
A p alone, 1e-16 x 4 / h_min^2 x |p| / |f|, comes to some 1e-11."""
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev, host, oracle_inputs, rel_max_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [
    (18, 1, 2), (18, 1, 37), (32, 1, 600), (18, 1, 511), (1024, 1, 131), (18, 1, 1024),
    (12, 16, 256), (12, 16, 253), (12, 16, 257), (12, 24, 85), (12, 24, 86), (12, 32, 64), (12, 32, 3),
    (12, 48, 42), (12, 48, 43), (486, 64, 32), (512, 64, 32), (12, 64, 29)])
def test_one_launch(gpu, nx, ny, nz):
    lz = 0.9
    spec = W.GridSpec(nx, ny, nz, 1.0, 0.8, lz, W.tanh_faces(nz, lz, 1.5))
    g, f, rho, pp = oracle_inputs(W.two_phase_case("one_launch", spec, 1, 33, n_spheres=3))
    (ref,), _ = O.solve(f, g, rho, pp, with_relres=False)
    f, rho, pp = dev(f), dev(rho), dev(pp)
    for prec in ("fp64", "mixed"):
        plan = gpu.Plan(gpu.Grid.from_spec(spec), precision=prec)
        for kc in (4, 8, 16):
            plan.set_shape(chunk_rows=kc)
            say(f"{prec} {nx}x{ny}x{nz} {plan.get_shape()}")
            p, info = plan.solve(f, rho=rho, p_prev=pp, info=True)
            err = rel_max_err(host(p), ref)
            assert err <= (1e-11 if prec == "fp64" else 1e-8), (prec, kc, err)
            assert info.relres <= 1e-10, (prec, kc, info.relres)
