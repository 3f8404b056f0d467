"""Solves whose pass-2 reduction rides in a wide x-forward pass: short x lines,
many of them, few enough nodes (the mid and small shapes carry it in the other
tests' grids)."""

import pytest

import llg_workloads as W
import paper_2607_15290_amd as P
from oracle import steppers
from oracle.grid import Grid
from tests.gpu_util import announce, assert_elem, both_params, dev, host, unit_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 160, 128), (12, 192, 96)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_ir", "fp32_ir_left"])
def test_reduction_rides_in_a_wide_pass(shape, prec):
    """Against the oracle's GMRES: solutions within 1e-8 (rtol 1e-10), float64
    iteration counts within one."""
    nx, ny, nz = shape
    announce(f"ride {shape} {prec}")
    dt = W.dt_explicit_multiple(13.3, 0.05, nx, 3)
    prm, op = both_params(alpha=0.05, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
    g = Grid(nx, ny, nz, h=1.0 / nx)
    m = unit_field((nz, ny, nx), 53, smooth=12.0)
    b = steppers.rhs(g, op, m)
    xr, ir = steppers.solve_saddle(g, op, m, b, rtol=1e-10)
    ctx = P.Context(nx, ny, nz, 1.0 / nx, 0)
    x, st = P.gmres_solve(ctx, prm, dev(m), dev(b), rtol=1e-10, prec=prec, inner_rtol=1e-3)
    ctx.close()
    assert st["converged"] == 1 and st["iters"] > 5
    if prec == "fp64":
        assert abs(st["iters"] - ir["iters"]) <= 1, (st, ir)
    assert_elem(host(x), xr, 1e-8, "x")
