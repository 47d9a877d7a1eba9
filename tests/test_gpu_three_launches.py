"""The wall-normal solve in three launches where small grids take one: the y tiles of
every length, the two-dimensional kernels and the checks (jobs) that both carry, at
columns just past the single launch's; and the runtime transforms, long lines with
over 64 KiB of LDS among them. Against the oracle at the paths' tolerances (FP64
1e-11, mixed 1e-8, iterated mixed 1e-7; relres 1e-10, as with hundreds of stretched
rows the rounding of A p alone comes to some 1e-12)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from oracle import converged as C
from paper_2005_11806_amd import _abi
from tests.gpu_util import dev, host, oracle_inputs, rel_max_err, say

pytestmark = pytest.mark.gpu

X_LENGTHS = [16, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 192, 216, 256, 288, 324, 384, 512, 768, 1024]
Y_LENGTHS = [16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256, 288, 324, 384, 432, 512,
             768, 1024]


def _spec(nx, ny, nz, stretched=True):
    lz = 0.9
    return W.GridSpec(nx, ny, nz, 1.0, 0.8 if ny > 1 else 1.0 / nx, lz, W.tanh_faces(nz, lz, 1.5) if stretched else None)


def _past_one_launch(ny):
    """Rows of a ragged column that one launch does not take."""
    return 19 if ny > 64 or ny in (18, 36, 54) else (4096 if ny == 16 else 2048) // ny + 3


@pytest.mark.parametrize("ny", Y_LENGTHS)
def test_y_tiles(gpu, ny):
    spec = _spec(8, ny, _past_one_launch(ny))
    g, f, rho, pp = oracle_inputs(W.two_phase_case("tiles", spec, 1, 91, n_spheres=3))
    (ref,), _ = O.solve(f, g, rho, pp, with_relres=False)
    f, rho, pp = dev(f), dev(rho), dev(pp)
    for prec, tol in (("fp64", 1e-11), ("mixed", 1e-8)):
        plan = gpu.Plan(gpu.Grid.from_spec(spec), precision=prec)
        ran = 0
        for kc in (4, 8, 16):
            try:
                plan.set_shape(chunk_rows=kc)
            except gpu.PsvError as e:
                assert e.status == _abi.PSV_ERR_UNSUPPORTED_SIZE
                continue
            ran += 1
            plan.trace()
            p, info = plan.solve(f, rho=rho, p_prev=pp, info=True)
            names = plan.trace_summary()
            plan.trace(False)
            err = rel_max_err(host(p), ref)
            say(f"{prec} 8x{ny}x{spec.nz} chunk rows {kc}: {err:.1e} {info.relres:.1e}")
            assert any(n.startswith("yz_fwd") for n in names) and not any(n.startswith("z_solve") for n in names)
            assert err <= tol and info.relres <= 1e-10, (prec, kc)
            # without info the checks join the y tiles
            assert rel_max_err(host(plan.solve(f, rho=rho, p_prev=pp)), ref) <= tol
        assert ran >= (1 if ny > 512 else 2)


@pytest.mark.parametrize("nx,ny,nz", [(12, 32, 67), (12, 64, 35), (18, 1, 513)])
def test_iterated(gpu, nx, ny, nz):
    spec = _spec(nx, ny, nz)
    g, f, rho, _ = oracle_inputs(W.converged_case("conv", spec, 1, n_spheres=4))
    F, R = dev(f), dev(rho)
    plan = gpu.Plan(gpu.Grid.from_spec(spec))
    say(f"converged {nx}x{ny}x{nz}")
    for k in (1, 3):
        ref = C.solve(f, rho, g, 0.0, k)
        p, info = plan.solve_converged(F, R, eps_t=0.0, max_iter=k)
        assert info.iterations == k and not info.converged
        assert rel_max_err(host(p), ref.p) <= 1e-11
        assert abs(info.eps - ref.eps[-1]) <= 1e-8 * ref.eps[-1]
    eps_t = 1e-10 * np.abs(f).sum()
    ref = C.solve(f, rho, g, eps_t, 200)
    for prec, tol in (("fp64", 1e-8), ("mixed", 1e-7)):
        p, info = gpu.Plan(gpu.Grid.from_spec(spec), precision=prec).solve_converged(F, R, eps_t=eps_t, max_iter=200)
        assert info.converged and info.eps <= eps_t
        assert rel_max_err(host(p), ref.p) <= tol


def test_two_dimensional_mixed(gpu):
    """The longest column: its planes do not fit one block."""
    spec = _spec(18, 1, 2048, stretched=False)
    g, f, rho, pp = oracle_inputs(W.two_phase_case("tall", spec, 1, 92, n_spheres=3))
    (ref,), _ = O.solve(f, g, rho, pp, with_relres=False)
    plan = gpu.Plan(gpu.Grid.from_spec(spec), precision="mixed", tol=1e-9)
    f, rho, pp = dev(f), dev(rho), dev(pp)
    p, info = plan.solve(f, rho=rho, p_prev=pp, info=True)
    say(f"mixed 18x1x2048: {info}")
    assert rel_max_err(host(p), ref) <= 1e-8
    assert rel_max_err(host(plan.solve(f, rho=rho, p_prev=pp)), ref) <= 1e-8


@pytest.mark.parametrize("nx,ny,nz", [(864, 6, 5), (972, 4, 6), (648, 18, 3), (12, 486, 9), (4, 576, 6), (6, 6, 40)])
def test_runtime_lengths(gpu, nx, ny, nz):
    spec = _spec(nx, ny, nz)
    g, f, rho, pp = oracle_inputs(W.two_phase_case("runtime", spec, 1, 93, n_spheres=3))
    (ref,), _ = O.solve(f, g, rho, pp, with_relres=False)
    f, rho, pp = dev(f), dev(rho), dev(pp)
    grid = gpu.Grid.from_spec(spec)
    for prec, tol in (("fp64", 1e-11), ("mixed", 1e-8)):
        for stencil in ("staged", "direct"):
            p, info = gpu.Plan(grid, precision=prec, x_stencil=stencil).solve(f, rho=rho, p_prev=pp, info=True)
            err = rel_max_err(host(p), ref)
            say(f"{prec} {stencil} {nx}x{ny}x{nz}: {err:.1e} {info.relres:.1e}")
            assert err <= tol and info.relres <= 1e-10
        (p,) = gpu.Batch([grid], precision=prec).solve([f], [rho], [pp])
        assert rel_max_err(host(p), ref) <= tol


def test_every_length_has_a_shape(gpu):
    """One line per x block and four planes per y tile are taken at every length, with
    the built-in shape's result."""
    gen = torch.Generator(device="cuda").manual_seed(94)
    for nx, ny in [(n, 12) for n in X_LENGTHS] + [(12, n) for n in Y_LENGTHS]:
        f, u, pp = torch.randn(3, 5, ny, nx, generator=gen, device="cuda", dtype=torch.float64)
        rho = 1.0 + u.abs()
        for prec, tol in (("fp64", 1e-12), ("mixed", 1e-9)):
            plan = gpu.Plan(gpu.Grid(nx, ny, 5, 1.0, 1.0, 1.0), precision=prec)
            ref = host(plan.solve(f, rho=rho, p_prev=pp))
            plan.set_shape(lines_x=1, lines_x_inv=1, chunk_rows=4)
            say(f"{prec} {nx}x{ny}x5 {plan.get_shape()}")
            assert rel_max_err(host(plan.solve(f, rho=rho, p_prev=pp)), ref) <= tol
