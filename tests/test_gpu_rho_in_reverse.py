"""GPU: the density face sums carried by the two-launch 2D reverse step (SMI_OPT_REVERSE 1) against
their own launch beside the five-launch step (2): the same sums in the same order, bitwise, with
extents around the 64 x 4 blocks, boxes on and off, free surface, decimated bands and groups."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n1,n2,nshot,box,freesurf,dr,group", [
    (8, 63, 99, 1, 0, 0, 1, 0), (8, 64, 100, 3, 1, 0, 1, 2), (4, 65, 101, 2, 1, 1, 1, 0),
    (4, 127, 40, 2, 0, 0, 3, 1), (8, 30, 12, 1, 0, 0, 1, 0)])
def test_density_sums_in_the_reverse_step(order, n1, n2, nshot, box, freesurf, dr, group):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=n1, n2=n2, nt=250, nshot=nshot, box=box)
    g = job.grid
    g.order, g.freesurf, g.dr, g.nb = order, freesurf, dr, 10
    if order == 4:
        g.fm = 7.0
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    gen = torch.Generator(device="cuda").manual_seed(4)
    d = 1e-7 * torch.randn(g.nt * int(job.acq.rec_off[-1]), generator=gen, device="cuda")
    ctx.set_option(B.OPT_REV_GROUP, group)
    out = []
    for form in (2, 1):
        ctx.set_option(B.OPT_REVERSE, form)
        r = ctx.fwi_grad(g, job.acq, vp, rho, stf, d, rho_grad=True)[:2]
        ctx.poll_status()
        out.append([t.cpu().numpy() for t in r])
    for k, (a, b) in enumerate(zip(*out)):
        say(f"order {order} {n1}x{n2} output {k}: bitwise {np.array_equal(a, b)}")
        assert np.abs(a).max() > 0 and np.array_equal(a, b)
