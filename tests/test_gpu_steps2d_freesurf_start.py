"""GPU: two-step 2D launches below a free surface whose boxes reach the surface from below.  With 24
to 26 absorbing rows a storage line starts at the surface or up to two rows above it, so the first
strip of a launch can start there, with some of the image rows above its first lane.  Sources too deep to reach the
surface at once, computing boxes on, with the default margin and a small one: seismograms and
gradients are bitwise those of the half-step kernels (SMI_OPT_KERNEL 3)."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,nb", [(8, 24), (8, 25), (8, 26), (8, 27), (8, 28), (4, 24), (4, 25), (4, 26), (8, 56)])
@pytest.mark.parametrize("margin", [-1, 1])
def test_images_above_the_first_strip(order, nb, margin):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=60, n2=104, nt=220, nshot=2, box=1)
    g = job.grid
    g.order, g.nb, g.freesurf, g.box_margin = order, nb, 1, margin
    g.fm = 15.0 if order == 8 else 7.0
    off = 3.3 if order == 8 else 0.0
    job.acq.src[:, 0] = [250.0 + off, 310.0 + off]
    job.acq.src[:, 1] += off
    # (strong from the first step on, so that the first rows a box reaches hold values)
    job.stf = np.tile(np.cos(0.3 * np.arange(g.nt)).astype(np.float32), (2, 1))
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    gen = torch.Generator(device="cuda").manual_seed(2)
    d = 1e-7 * torch.randn(g.nt * int(job.acq.rec_off[-1]), generator=gen, device="cuda")
    out = []
    for opts in ((3, 4, 1), (0, 0, 0)):
        for k, v in zip((B.OPT_KERNEL, B.OPT_CHUNK, B.OPT_TILEMAP), opts):
            ctx.set_option(k, v)
        r = [ctx.forward(g, job.acq, vp, rho, stf)[0],
             *ctx.fwi_grad(g, job.acq, vp, rho, stf, d, want_dcal=True)]
        ctx.poll_status()
        out.append([t.cpu().numpy() for t in r])
    same = [bool(np.array_equal(a, b)) for a, b in zip(*out)]
    say(f"order {order} nb {nb} margin {margin}: bitwise {same}, seismogram difference "
        f"{np.abs(out[0][0] - out[1][0]).max():.2e} of {np.abs(out[0][0]).max():.2e}")
    assert np.abs(out[0][0]).max() > 0 and all(same)
