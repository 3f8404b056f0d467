"""Calls that wait for the device: the same results behind a long queue of the
caller's work, and the stream drained at every return, failing ones included
(the workspace may go to another stream then)."""

import pytest
import torch

import paper_2607_15290_amd as P
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

NX, NY, NZ = 128, 128, 64  # the largest grid that queues an operator ahead of the host's wait


def _field():
    m = torch.zeros((3, NZ, NY, NX), dtype=torch.float64, device="cuda:0")
    x = torch.arange(NX, dtype=torch.float64, device="cuda:0") / NX
    m[0] = 0.3 * torch.cos(2 * torch.pi * x)
    m[2] = 1.0
    return m / torch.sqrt((m * m).sum(0, keepdim=True))


def _drained():
    return torch.cuda.current_stream().query()


@pytest.mark.parametrize("prec", ["fp64", "fp32_ir", "fp32_ir_left"])
def test_results_behind_a_queue(prec):
    announce(f"waits {prec}")
    ctx = P.Context(NX, NY, NZ, 1.0 / NX, 0)
    prm = P.Params(alpha=0.1, dt=1e-5, theta=1.0, shift=0.5, h_uniform=(0.1, 0.0, 1.0))
    m = _field()
    e0 = P.llg_energy(ctx, prm, m)
    assert _drained()
    g = torch.Generator(device="cuda:0").manual_seed(5)
    b = torch.randn((4, NZ, NY, NX), dtype=torch.float64, device="cuda:0", generator=g)
    x0, s0 = P.gmres_solve(ctx, prm, m, b, prec=prec)
    assert _drained()
    torch.cuda._sleep(20_000_000)
    assert P.llg_energy(ctx, prm, m) == e0 and _drained()
    torch.cuda._sleep(20_000_000)
    x1, s1 = P.gmres_solve(ctx, prm, m, b, prec=prec)
    assert _drained()
    assert s1["iters"] == s0["iters"] and torch.equal(x0, x1)
    ctx.close()


def test_failing_calls_leave_the_stream_drained():
    """Exchange constants beyond float32 make the precision form's inner
    operator non-finite, found while the next operator is queued: LLG_ENAN with
    nothing left on the stream.  An iteration limit: LLG_ENOCONV, the same."""
    announce("waits: failing calls")
    ctx = P.Context(NX, NY, NZ, 1.0 / NX, 0)
    m0 = _field()
    big = P.Params(alpha=0.1, cexc=1e44, dt=1e-5, theta=0.5, shift=0.5, h_uniform=(0.1, 0.0, 1.0))
    for step in (P.llg_step_euler, P.llg_step_midpoint):
        m = m0.clone()
        ctx.workspace(30, "fp32_ir")
        torch.cuda.synchronize()
        st = step(ctx, big, m, prec="fp32_ir", check=False)
        done = _drained()
        assert st["status"] == "LLG_ENAN", st
        assert done, step.__name__
    prm = P.Params(alpha=0.1, dt=1e-5, theta=0.5, shift=0.5, h_uniform=(0.1, 0.0, 1.0))
    m = m0.clone()
    st = P.llg_step_euler(ctx, prm, m, maxiter=2, rtol=1e-13, check=False)
    done = _drained()
    assert st["status"] == "LLG_ENOCONV" and done
    ctx.close()
