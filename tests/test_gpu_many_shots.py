"""GPU: batches of very many shots on the smallest grid.  Parts of a step that share a launch count
their shots' planes together and a launch has at most 65536 of them, so these batches take a launch
per part: tangent-linear data of 32768 shots (the most that one field's planes leave room for is
65535) equal those of a small batch, and density gradients of the forced two-launch
reverse step equal those of the five-launch one, bitwise."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import say

pytestmark = pytest.mark.gpu


def _batch(nshot, nt):
    import torch
    from paper_2311_02293_amd import binding as B
    job = I.config2(n1=8, n2=8, nt=nt, nshot=1, box=0)
    g = job.grid
    g.nb, g.order, g.fm = 4, 4, 7.0
    g.vpmin, g.vpmax = float(job.vp.min()), float(job.vp.max())
    src = np.tile([[20.0, 30.0, 0.0]], (nshot, 1))
    src[1::2, 1] = 50.0
    acq = I.Acquisition(src, np.arange(nshot + 1, dtype=np.int32),
                        np.tile([[20.0, 40.0, 0.0]], (nshot, 1)))
    vp, rho = (torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in (job.vp, job.rho))
    stf = torch.cos(0.3 * torch.arange(nt, device="cuda")).repeat(nshot, 1).contiguous()
    return B.Context(0), g, acq, vp, rho, stf


def test_tangent_linear_of_32768_shots():
    import torch
    out = []
    for nshot in (2, 32768):
        ctx, g, acq, vp, rho, stf = _batch(nshot, 12)
        dk = 1e-3 * vp * vp * rho
        out.append(ctx.born(g, acq, vp, rho, stf, dk).view(nshot, g.nt))
        ctx.poll_status()
    small, many = out
    say("tangent-linear, 2 and 32768 shots: max", float(small.abs().max()))
    assert float(small.abs().max()) > 0
    assert torch.equal(many.view(-1, 2, many.shape[1]), small.expand(16384, 2, -1))


def test_density_gradient_of_12000_shots():
    import torch
    from paper_2311_02293_amd import binding as B
    ctx, g, acq, vp, rho, stf = _batch(12000, 12)
    gen = torch.Generator(device="cuda").manual_seed(4)
    d = 1e-7 * torch.randn(12000 * g.nt, generator=gen, device="cuda")
    out = []
    for form in (2, 1):
        ctx.set_option(B.OPT_REVERSE, form)
        out.append([t.cpu().numpy() for t in ctx.fwi_grad(g, acq, vp, rho, stf, d, rho_grad=True)[:3]])
        ctx.poll_status()
    same = [bool(np.array_equal(a, b)) for a, b in zip(*out)]
    say("12000 shots, forced two-launch against five-launch reverse: bitwise", same)
    assert np.abs(out[0][1]).max() > 0 and all(same)
