"""Wavefront reductions (csrc/wave.h) at the value counts where their halving
steps change shape: classic CGS2 cycles reduce 8, 16, 32 or 64 values per
wavefront, by the number of directions."""

import numpy as np
import pytest

import llg_workloads as W
import paper_2607_15290_amd as P
from oracle import steppers
from oracle.grid import Grid
from tests.gpu_util import announce, assert_elem, both_params, dev, host, unit_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [1, 8, 9, 17, 33, 62])
def test_classic_cgs2_cycles_match_oracle(restart):
    """A stiff 24 x 16 system run through cycles of the given length: the
    iteration counts follow the oracle's modified Gram-Schmidt, the solution
    agrees to 1e-8 (rtol 1e-11 on a system with condition below 1e3)."""
    announce(f"classic CGS2 restart {restart}")
    g = Grid(24, 16, 1, h=1.0 / 24)
    dt = W.dt_explicit_multiple(100.0, 0.1, 24, 2)
    prm, op = both_params(alpha=0.1, cexc=1.0, dt=dt, theta=1.0, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
    m = unit_field((1, 16, 24), 31, smooth=6.0)
    b = steppers.rhs(g, op, m)
    xr, ir = steppers.solve_saddle(g, op, m, b, rtol=1e-11, restart=restart, maxiter=4000)
    ctx = P.Context(24, 16, 1, 1.0 / 24, 0)
    x, st = P.gmres_solve(ctx, prm, dev(m), dev(b), rtol=1e-11, restart=restart, maxiter=4000, orth="cgs2",
                          check=False)
    ctx.close()
    assert bool(st["converged"]) == ir["converged"]
    assert abs(st["iters"] - ir["iters"]) <= max(1, ir["iters"] // 100), (st["iters"], ir["iters"])
    if ir["converged"]:
        assert_elem(host(x), xr, 1e-8, "x")
