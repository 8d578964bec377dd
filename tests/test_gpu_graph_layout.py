"""GPU: captured loops (SMI_OPT_GRAPH) over one buffer given as workspaces of two sizes.  The layout
of a 2D workspace depends on whether the rows of the two-step launches fit, so a loop captured for
one size is not replayed for the other: seismograms and gradients stay bitwise those without
graphs, and nothing is written past the smaller workspace."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,dr", [(8, 1), (8, 3), (4, 1)])
def test_replay_knows_the_layout(order, dr):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=70, n2=150, nt=240, nshot=2)
    job.grid.order, job.grid.dr = order, dr
    job.grid.fm = 15.0 if order == 8 else 7.0
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    R = int(job.acq.rec_off[-1])
    gen = torch.Generator(device="cuda").manual_seed(3)
    adj = 1e-7 * torch.randn(job.grid.nt * R, generator=gen, device="cuda")
    dcal = torch.empty(job.grid.nt * R, device="cuda")
    full = ctx.workspace_bytes(job.grid, job.acq, B.JOB_FORWARD_SAVE)
    buf = torch.empty(full + 4096, dtype=torch.uint8, device="cuda")

    def run(nbytes):
        buf.fill_(0x5A)
        state = ctx.forward(job.grid, job.acq, vp, rho, stf, save=True, dcal=dcal, ws=buf[:nbytes])[2]
        out = ctx.adjoint_reconstruct(state, adj, grad=True, grad_rho=True)
        ctx.poll_status()
        assert bool((buf[nbytes:] == 0x5A).all())
        flat = out.values() if isinstance(out, dict) else out
        return [dcal.cpu().numpy()] + [t.cpu().numpy() for t in flat if t is not None]

    want = run(full)
    assert all(np.array_equal(a, b) for a, b in zip(run(full - 1), want))
    ctx.set_option(B.OPT_GRAPH, 1)
    try:
        for nbytes in (full, full - 1, full, full - 1):
            got = run(nbytes)
            say(f"order {order} dr {dr} workspace {nbytes}:",
                [bool(np.array_equal(a, b)) for a, b in zip(got, want)])
            for a, b in zip(got, want):
                assert np.abs(b).max() > 0 and np.array_equal(a, b)
    finally:
        ctx.set_option(B.OPT_GRAPH, 0)
