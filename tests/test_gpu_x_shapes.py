"""The three launch shapes of the x passes (wide, mid, small: x_shape in
csrc/pipeline.h) at the sizes where a block is ragged: lines that do not fill
the last block, node pairs that do not fill a wavefront, and column counts
around the batches in which the block's wavefronts share the Arnoldi
products."""

import numpy as np
import pytest
import torch

import llg_workloads as W
import paper_2607_15290_amd as P
from oracle import operators, steppers
from oracle.grid import Grid
from tests.gpu_util import announce, assert_elem, both_params, dev, host, unit_field

pytestmark = pytest.mark.gpu

# (nx, ny, nz): shape of the float64 x passes
SHAPES = [
    (4, 6, 1),       # small, 6 lines of 2 pairs in one block
    (24, 10, 6),     # small, 5 lines of 12 pairs
    (40, 10, 1),     # small, 20-pair lines: 3 per block, the last block with one
    (320, 6, 1),     # small, one 160-pair line per block (not a multiple of 64)
    (48, 48, 48),    # mid, 10 lines of 24 pairs, the last block with 4
    (80, 40, 24),    # mid, 6 lines of 40 pairs
    (512, 96, 4),    # mid, one 256-pair line per block
    (32, 160, 128),  # wide in float64 (320 blocks of 64 lines)
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("nb", [1, 3, 4, 5, 17, 32])
def test_products_in_every_shape(shape, nb):
    """M^{-1} A x and its products with nb basis vectors, in float64 and in the
    flexible float32 form: y against the oracle (1e-13; the float32 bound one
    unit roundoff per butterfly level as in the operator tests), the
    products against numpy's on the library's own y (1e-13 of the sum of
    absolute terms)."""
    nx, ny, nz = shape
    announce(f"x shapes {shape} nb={nb}")
    dt = W.dt_explicit_multiple(13.3, 0.02, max(nx, ny, nz), 2 if nz == 1 else 3)
    prm, op = both_params(alpha=0.02, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
    g = Grid(nx, ny, nz, h=1.0 / nx)
    m = unit_field((nz, ny, nx), 41, smooth=40.0)
    x = np.random.default_rng(42).standard_normal((4, nz, ny, nx))
    ctx = P.Context(nx, ny, nz, 1.0 / nx, 0)
    torch.manual_seed(43)
    basis = torch.randn((nb, 4, nz, ny, nx), dtype=torch.float64, device="cuda:0")
    bh = host(basis).reshape(nb, -1)

    def check_dots(y, dots, what):
        yh = host(y).ravel()
        scale = np.abs(bh * yh).sum(axis=1)
        err = np.abs(host(dots)[:nb] - bh @ yh) / scale
        print(f"  {what} products {err.max():.2e}", flush=True)
        assert err.max() <= 1e-13

    y, dots = P.llg_precond_op(ctx, prm, dev(m), dev(x), basis=basis)
    assert_elem(host(y), operators.precond_op(g, op, m, x), 1e-13, "M^-1 A")
    check_dots(y, dots, "float64")
    mf = dev(m, torch.float32)
    z = torch.empty((4, nz, ny, nx), dtype=torch.float32, device="cuda:0")
    y, dots = P.llg_precond_op_f32(ctx, prm, mf, dev(x), side=1, z=z, basis=basis)
    lev = sum(2 * int(np.ceil(np.log2(n))) for n in (nx, ny, nz) if n > 1) + 16
    zr = operators.hss_apply(g, op, host(mf), x.astype(np.float32).astype(np.float64))
    assert_elem(host(z), zr, lev * 2.0 ** -24, "z float32")
    check_dots(y, dots, "flexible float32")
    ctx.close()


@pytest.mark.parametrize("shape", [
    (16, 8, 1),       # one update block, pass-1 products and the pass-2 reduction both carried along
    (512, 512, 1),    # the largest grid whose pass-2 reduction rides (1024 update blocks)
    (128, 64, 48),    # 1536 update blocks: reductions of their own, operator still launched ahead
])
@pytest.mark.parametrize("prec", ["fp64", "fp32_ir", "fp32_ir_left"])
def test_cycles_across_reduction_rules(shape, prec):
    """Solves on both sides of the rules that say where an Arnoldi step's
    inner products are reduced, against the oracle's GMRES: solutions within
    1e-8 (rtol 1e-10), float64 iteration counts within one."""
    nx, ny, nz = shape
    announce(f"reduction rules {shape} {prec}")
    dt = W.dt_explicit_multiple(13.3, 0.05, max(nx, ny, nz), 2 if nz == 1 else 3)
    prm, op = both_params(alpha=0.05, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
    g = Grid(nx, ny, nz, h=1.0 / nx)
    m = unit_field((nz, ny, nx), 51, smooth=12.0)
    b = steppers.rhs(g, op, m)
    xr, ir = steppers.solve_saddle(g, op, m, b, rtol=1e-10)
    ctx = P.Context(nx, ny, nz, 1.0 / nx, 0)
    x, st = P.gmres_solve(ctx, prm, dev(m), dev(b), rtol=1e-10, prec=prec, inner_rtol=1e-3)
    ctx.close()
    assert st["converged"] == 1
    if prec == "fp64":
        assert abs(st["iters"] - ir["iters"]) <= 1, (st, ir)
    assert_elem(host(x), xr, 1e-8, "x")


@pytest.mark.parametrize("n", [64, 128, 160, 192, 256, 320, 384, 512])
@pytest.mark.parametrize("axis", ["y", "z"])
def test_wide_axis_passes(n, axis):
    """Axis lengths with two launch shapes, on grids with enough blocks for the
    wide one (the operator tests' small grids take the narrow one): A x and
    M^{-1} x in float64 (1e-12) and float32 (one unit roundoff per butterfly
    level)."""
    nx, ny, nz = (32, n, 96) if axis == "y" else (32, 96, n)
    announce(f"wide axis passes {axis} {n}")
    dt = W.dt_explicit_multiple(13.3, 0.02, max(nx, ny, nz), 3)
    prm, op = both_params(alpha=0.02, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
    g = Grid(nx, ny, nz, h=1.0 / nx)
    m = unit_field((nz, ny, nx), 61, smooth=40.0)
    x = np.random.default_rng(62).standard_normal((4, nz, ny, nx))
    ctx = P.Context(nx, ny, nz, 1.0 / nx, 0)
    assert_elem(host(P.llg_matvec(ctx, prm, dev(m), dev(x))), operators.matvec(g, op, m, x), 1e-12, "A x")
    assert_elem(host(P.fft_hss_apply(ctx, prm, dev(m), dev(x))), operators.hss_apply(g, op, m, x), 1e-12, "M^-1 x")
    mf, xf = dev(m, torch.float32), dev(x, torch.float32)
    tol = (sum(2 * int(np.ceil(np.log2(k))) for k in (nx, ny, nz)) + 16) * 2.0 ** -24
    assert_elem(host(P.fft_hss_apply_f32(ctx, prm, mf, xf)), operators.hss_apply(g, op, host(mf), host(xf)), tol,
                "M^-1 x float32")
    ctx.close()


PLANE_LENGTHS = [4, 6, 8, 10, 12, 16, 20, 24, 32]


@pytest.mark.parametrize("ny", PLANE_LENGTHS)
def test_plane_kernel(ny):
    """The one-kernel axis passes of small 3-D grids on every pair of lengths
    they take (and, at the larger pairs, on the three passes just above the
    rule): M^{-1} x in float64 (1e-12) and float32 (one unit roundoff per
    butterfly level)."""
    nx = 12
    for nz in PLANE_LENGTHS:
        announce(f"plane kernel {nx}x{ny}x{nz}")
        dt = W.dt_explicit_multiple(13.3, 0.02, max(nx, ny, nz), 3)
        prm, op = both_params(alpha=0.02, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
        g = Grid(nx, ny, nz, h=1.0 / nx)
        m = unit_field((nz, ny, nx), 81, smooth=40.0)
        x = np.random.default_rng(82).standard_normal((4, nz, ny, nx))
        ctx = P.Context(nx, ny, nz, 1.0 / nx, 0)
        assert_elem(host(P.fft_hss_apply(ctx, prm, dev(m), dev(x))), operators.hss_apply(g, op, m, x), 1e-12, "f64")
        mf, xf = dev(m, torch.float32), dev(x, torch.float32)
        tol = (sum(2 * int(np.ceil(np.log2(k))) for k in (nx, ny, nz)) + 16) * 2.0 ** -24
        assert_elem(host(P.fft_hss_apply_f32(ctx, prm, mf, xf)), operators.hss_apply(g, op, host(mf), host(xf)), tol,
                    "f32")
        ctx.close()
