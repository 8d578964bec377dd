"""GPU: 2D reverse steps of small launches (two cells per lane up to 0.8 M padded cells) against the
five-launch step, which keeps four cells per lane: the same arithmetic per cell, so gradients,
density gradients, images and illumination are bitwise equal.  Column counts that leave a lane with
one cell, receivers between the nodes, a free surface, decimated bands, shot groups, and a batch on
each side of the line."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n1,n2,nshot,box,freesurf,dr,group,offgrid", [
    (8, 61, 101, 1, 0, 0, 1, 0, False), (4, 64, 102, 3, 1, 1, 1, 0, True),
    (8, 120, 203, 2, 1, 1, 1, 0, True), (8, 65, 99, 2, 0, 0, 3, 1, False),
    (8, 250, 701, 3, 1, 0, 1, 0, False), (8, 250, 701, 4, 1, 0, 1, 0, False)])
def test_two_cells_per_lane_equal_four_in_reverse(order, n1, n2, nshot, box, freesurf, dr, group,
                                                  offgrid):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=n1, n2=n2, nt=200, nshot=nshot, box=box)
    g = job.grid
    g.order, g.freesurf, g.dr, g.nb = order, freesurf, dr, 10
    if order == 4:
        g.fm = 7.0
    if offgrid:
        job.acq.rec[:, 0] += 0.37 * g.d1
        job.acq.rec[:, 1] = np.minimum(job.acq.rec[:, 1] + 0.41 * g.d2, (n2 - 1) * g.d2)
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    gen = torch.Generator(device="cuda").manual_seed(9)
    d = 1e-7 * torch.randn(g.nt * int(job.acq.rec_off[-1]), generator=gen, device="cuda")
    ctx.set_option(B.OPT_REV_GROUP, group)
    out = []
    for form in (2, 1):
        ctx.set_option(B.OPT_REVERSE, form)
        r = [*ctx.fwi_grad(g, job.acq, vp, rho, stf, d, rho_grad=True)[:2],
             ctx.fwi_grad(g, job.acq, vp, rho, stf, d)[0],
             *ctx.rtm_image(g, job.acq, vp, rho, stf, d)[:2]]
        ctx.poll_status()
        out.append([t.cpu().numpy() for t in r])
    for k, (a, b) in enumerate(zip(*out)):
        say(f"order {order} {n1}x{n2} x{nshot} output {k}: bitwise {np.array_equal(a, b)}")
        assert np.abs(a).max() > 0 and np.array_equal(a, b)
