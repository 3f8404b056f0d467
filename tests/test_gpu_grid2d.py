"""The one-kernel pipeline of small 2-D grids (k_grid2d) on every pair of
lengths it takes, and on the three passes just above its rule."""

import numpy as np
import pytest
import torch

import llg_workloads as W
import paper_2607_15290_amd as P
from oracle import operators, steppers
from oracle.grid import Grid
from tests.gpu_util import announce, assert_elem, both_params, dev, host, unit_field

pytestmark = pytest.mark.gpu

LENGTHS_X = [4, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64]
LENGTHS_Y = [4, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64]


@pytest.mark.parametrize("nx", LENGTHS_X)
def test_one_kernel_pipeline(nx):
    """The kernel's modes against the oracle: A x, A^T x, M^{-1} x, M^{-T} x and
    the right-hand side with a spatial field in float64 (1e-12), the first
    four in float32 (one unit roundoff per butterfly level)."""
    for ny in LENGTHS_Y:
        announce(f"one-kernel pipeline {nx}x{ny}")
        dt = W.dt_explicit_multiple(13.3, 0.02, max(nx, ny), 2)
        hf = 0.1 * np.random.default_rng(93).standard_normal((3, 1, ny, nx))
        kw = dict(alpha=0.02, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.0, 0.0, 1.0))
        prm, op = both_params(**kw)
        g = Grid(nx, ny, 1, h=1.0 / nx)
        m = unit_field((1, ny, nx), 91, smooth=40.0)
        x = np.random.default_rng(92).standard_normal((4, 1, ny, nx))
        ctx = P.Context(nx, ny, 1, 1.0 / nx, 0)
        md, xd = dev(m), dev(x)
        ops = [("A x", P.llg_matvec, P.llg_matvec_f32, operators.matvec, dict()),
               ("A^T x", P.llg_matvec, P.llg_matvec_f32, operators.matvec_transpose, dict(transpose=True)),
               ("M^-1 x", P.fft_hss_apply, P.fft_hss_apply_f32, operators.hss_apply, dict()),
               ("M^-T x", P.fft_hss_apply, P.fft_hss_apply_f32,
                lambda *a: operators.hss_apply(*a, transpose=True), dict(transpose=True))]
        mf, xf = dev(m, torch.float32), dev(x, torch.float32)
        tol = (sum(2 * int(np.ceil(np.log2(k))) for k in (nx, ny)) + 16) * 2.0 ** -24
        for what, f64, f32, ref, opt in ops:
            assert_elem(host(f64(ctx, prm, md, xd, **opt)), ref(g, op, m, x), 1e-12, what)
            assert_elem(host(f32(ctx, prm, mf, xf, **opt)), ref(g, op, host(mf), host(xf)), tol, what + " float32")
        prm_h = P.Params(**kw, h_field=dev(hf))
        op_h = operators.Params(**kw, h_field=hf)
        assert_elem(host(P.llg_rhs(ctx, prm_h, md)), steppers.rhs(g, op_h, m), 1e-12, "rhs")
        # the result in the input's place
        P.fft_hss_apply(ctx, prm, md, xd, z=xd)
        assert_elem(host(xd), operators.hss_apply(g, op, m, x), 1e-12, "M^-1 x in place")
        ctx.close()
