"""Rounding of the wall-normal solve at a low wavenumber of a fine column, where
the system is nearly singular: one x mode against the same FP64 system solved in
extended precision. A right-hand side of one mode leaves two roundings of 2^-53
for each interface row (2 nz / chunk_rows) and each chunk row, a few of them for
the transforms and the other modes (together 1e-14 with room). Three launches
(ny 4), uniform and stretched, and the single launch (ny 16)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle.tridiag import thomas, z_coefficients
from tests.gpu_util import dev, host, rel_max_err, say

pytestmark = pytest.mark.gpu

LD = np.longdouble


def _thomas_ld(a, b, c, d):
    """oracle.tridiag.thomas in extended precision, one right-hand side."""
    nz = len(d)
    cp, dp = np.zeros(nz, LD), np.zeros(nz, LD)
    for k in range(nz):
        piv = b[k] - (a[k] * cp[k - 1] if k else LD(0))
        cp[k] = c[k] / piv
        dp[k] = (d[k] - (a[k] * dp[k - 1] if k else LD(0))) / piv
    for k in range(nz - 2, -1, -1):
        dp[k] -= cp[k] * dp[k + 1]
    return dp


@pytest.mark.parametrize("ny,nz,lz,stretch", [(4, 1024, 1.0, 0.0), (4, 512, 1.0, 1.5), (16, 256, 0.25, 0.0)])
def test_lowest_mode(gpu, ny, nz, lz, stretch):
    nx = 64
    spec = W.GridSpec(nx, ny, nz, 1.0, 1.0, lz, W.tanh_faces(nz, lz, stretch) if stretch else None)
    g = O.Grid.from_spec(spec)
    a, b, c = z_coefficients(g)
    lam = np.float64(-4 * np.sin(LD(np.pi) / nx + LD(1.2246467991473532e-16) / nx) ** 2 * nx * nx)
    z = (np.arange(nz) + 0.5) / nz
    col = sum(np.cos(j * np.pi * z + j * j) / (1 + j * j) for j in range(6))
    x = _thomas_ld(a.astype(LD), (b + lam).astype(LD), c.astype(LD), col.astype(LD)).astype(np.float64)
    wave = np.cos(2 * np.pi * (np.arange(nx) + 0.5) / nx)
    f = np.broadcast_to(col[:, None, None] * wave, (nz, ny, nx)).copy()
    ref = np.broadcast_to(x[:, None, None] * wave, (nz, ny, nx))
    assert rel_max_err(thomas(a, b + lam, c, col), x) <= 1e-12  # the reference is that system's
    plan = gpu.Plan(gpu.Grid.from_spec(spec), method="const")
    for kc in (4, 8, 16):
        plan.set_shape(chunk_rows=kc)
        err = rel_max_err(host(plan.solve(dev(f))), ref)
        say(f"{nx}x{ny}x{nz} lz {lz} chunk rows {kc}: {err:.2e}")
        assert err <= (2 * nz / kc + kc) * 2.0 ** -52 + 1e-14, (kc, err)


@pytest.mark.parametrize("ny,nz", [(4, 64), (16, 37), (1, 50)])
def test_eigenvalue_below_the_rounding_of_the_diagonal(gpu, ny, nz):
    """A domain 1e-8 thick: the lowest modes' eigenvalue sums vanish in the diagonals
    of the wall-normal systems, which are then singular as rounded. Their part of the
    result hangs on rounding, but no factor is infinite and the result is finite."""
    nx = 16
    x = np.cos(2 * np.pi * (np.arange(nx) + 0.5) / nx)
    f = np.broadcast_to(x, (nz, ny, nx)).copy()
    for prec in ("fp64", "mixed"):
        plan = gpu.Plan(gpu.Grid(nx, ny, nz, 1.0, 1.0, 1e-8), method="const", precision=prec)
        for kc in (4, 8, 16):
            plan.set_shape(chunk_rows=kc)
            p = host(plan.solve(dev(f)))
            say(f"thin {prec} {nx}x{ny}x{nz} chunk rows {kc}: {np.abs(p).max():.2e}")
            assert np.isfinite(p).all()
