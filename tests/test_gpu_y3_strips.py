"""GPU: the 3D y-marching default, whose strips of y-planes get shorter (32 down to 4) where a launch
has few tiles, against strips of 64 planes at order 8 and 32 at order 4 (SMI_OPT_KERNEL 5): every
cell's arithmetic is the same whatever the strip, so seismograms and gradients are bitwise equal.
Extents along y around a strip's 4 planes, boxes on and off, free surface."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n3,box,freesurf", [(8, 24, 1, 0), (8, 25, 0, 0), (8, 27, 1, 1),
                                                   (4, 24, 0, 0), (4, 29, 1, 1)])
def test_short_strips_equal_long_ones(order, n3, box, freesurf):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config4(n=32, nt=80, dr=1, nshot=2)
    g = job.grid
    g.order, g.box, g.freesurf, g.nb, g.n3 = order, box, freesurf, 8, n3
    if order == 4:
        g.fm = 7.0
    job.vp = np.ascontiguousarray(job.vp[:n3])
    job.rho = np.ascontiguousarray(job.rho[:n3])
    job.acq.src[:, 2] = np.minimum(job.acq.src[:, 2], (n3 - 1) * g.d3)
    job.acq.rec[:, 2] = np.minimum(job.acq.rec[:, 2], (n3 - 1) * g.d3)
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    gen = torch.Generator(device="cuda").manual_seed(7)
    d = 1e-7 * torch.randn(g.nt * int(job.acq.rec_off[-1]), generator=gen, device="cuda")
    out = []
    for kernel, chunk in ((5, 464 if order == 8 else 432), (0, 0)):
        ctx.set_option(B.OPT_KERNEL, kernel)
        ctx.set_option(B.OPT_CHUNK, chunk)
        r = ctx.fwi_grad(g, job.acq, vp, rho, stf, d, want_dcal=True, rho_grad=True)
        im = ctx.rtm_image(g, job.acq, vp, rho, stf, d, norm=True)
        out.append([t.cpu().numpy() for t in (*r, *im)])
        ctx.poll_status()
    for k, (a, b) in enumerate(zip(*out)):
        say(f"order {order} n3 {n3} box {box} fs {freesurf} output {k}: bitwise {np.array_equal(a, b)}")
        assert np.abs(a).max() > 0 and np.array_equal(a, b)
