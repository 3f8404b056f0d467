"""The lower-order field's fused axis pass (k_axis_field) on every line length
it is instantiated for, as the y pass of a 2-D grid and the z pass of a 3-D
one, with half spectra that do not fill the last block of columns: the
right-hand side and the energy against the oracle's full complex FFTs."""

import numpy as np
import pytest

import paper_2607_15290_amd as P
from oracle import steppers
from oracle.grid import Grid
from oracle.operators import Params as OP
from tests.gpu_util import announce, assert_elem, dev, host, unit_field

pytestmark = pytest.mark.gpu

LENGTHS = [4, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512]


@pytest.mark.parametrize("n", LENGTHS)
def test_field_pass_lengths(n):
    """float64, element-wise 1e-12 of the largest value (a few units of
    roundoff per butterfly level, times the cancellation of the Laplacian's
    large wave numbers in the relative measure)."""
    for nx, ny, nz in ((24, n, 1), (16, 6, n)):
        announce(f"field pass {nx}x{ny}x{nz}")
        g = Grid(nx, ny, nz, h=1.0 / nx)
        hf = 0.1 * np.random.default_rng(71).standard_normal((3, nz, ny, nx))
        kw = dict(alpha=0.2, cexc=1.0, dt=1e-3, theta=1.0, shift=0.5, h_uniform=(0.05, -0.1, 0.2), demag=1.0,
                  aniso_k=0.3, aniso_axis=(1 / 3, 2 / 3, 2 / 3))
        op = OP(h_field=hf, **kw)
        prm = P.Params(h_field=dev(hf), **kw)
        m = unit_field((nz, ny, nx), 72)
        ctx = P.Context(nx, ny, nz, 1.0 / nx, 0)
        assert_elem(host(P.llg_rhs(ctx, prm, dev(m))), steppers.rhs(g, op, m), 1e-12, "rhs")
        e, er = P.llg_energy(ctx, prm, dev(m)), steppers.energy(g, op, m)
        assert abs(e - er) <= 1e-12 * abs(er), (e, er)
        ctx.close()
