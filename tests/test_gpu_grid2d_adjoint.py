"""The left-preconditioned adjoint step on grids whose pipelines run as one
kernel (k_grid2d: the transposed Jacobian, the transposed preconditioner and
the Laplacian of the gradient), the largest of them and one just above."""

import numpy as np
import pytest
import torch

import llg_workloads as W
import paper_2607_15290_amd as P
from oracle import adjoint, steppers
from oracle.grid import Grid
from oracle.operators import Params as OP
from tests.gpu_util import announce, assert_elem, dev, host, unit_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4), (20, 12), (32, 32), (40, 32), (48, 32)])
@pytest.mark.parametrize("orth", ["cgs2", "dcgs2"])
def test_adjoint_step_on_small_grids(shape, orth):
    """Gradients of one midpoint step with a spatial field against the oracle's
    (1e-10: adjoint solves to 1e-13, a preconditioned condition number of
    order 10)."""
    nx, ny = shape
    announce(f"small adjoint {shape} {orth}")
    h = 1.0 / nx
    dt = W.dt_explicit_multiple(13.3, 0.1, max(nx, ny), 2)
    kw = dict(alpha=0.1, cexc=1.0, dt=dt, theta=0.5, shift=0.5, h_uniform=(0.1, -0.2, 1.0))
    hf = 0.1 * np.random.default_rng(101).standard_normal((3, 1, ny, nx))
    g = Grid(nx, ny, 1, h=h)
    op = OP(h_field=hf, **kw)
    m_n = unit_field((1, ny, nx), 102, smooth=10.0)
    m1, v, r, _ = steppers.midpoint_step(g, op, m_n, rtol=1e-14, picard_tol=1e-13, picard_max=100)
    gbar = np.random.default_rng(103).standard_normal(m1.shape)
    gb_ref, hf_ref, hu_ref, _, _ = adjoint.step_adjoint(g, op, m_n, v, r, gbar, rtol=1e-14)
    ctx = P.Context(nx, ny, 1, h, 0)
    prm = P.Params(h_field=dev(hf), **kw)
    gb = dev(gbar)
    hbf = torch.zeros_like(gb)
    hu, st = P.llg_step_midpoint_adjoint(ctx, prm, dev(m_n), dev(v), dev(r), gb, hbf, [0.0, 0.0, 0.0], rtol=1e-13,
                                         orth=orth)
    assert st["converged"] == 1
    assert_elem(host(gb), gb_ref, 1e-10, "gbar")
    assert_elem(host(hbf), hf_ref, 1e-10, "hbar_field")
    assert_elem(np.array(hu), np.array(hu_ref), 1e-10, "hbar_uniform")
    ctx.close()
