"""GPU: 2D forward half steps of small launches (two cells per lane up to 1.2 M padded cells)
against four cells per lane (SMI_OPT_KERNEL 3): the same arithmetic per cell, so seismograms and the
gradients of jobs whose forward pass saved bands are bitwise equal.  Odd column counts, and a batch
on each side of the line."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,nshot,freesurf,box", [(61, 101, 1, 0, 0), (120, 203, 3, 1, 1),
                                                      (250, 700, 5, 0, 1), (250, 700, 6, 0, 1)])
def test_two_cells_per_lane_equal_four(n1, n2, nshot, freesurf, box):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=n1, n2=n2, nt=200, nshot=nshot, box=box)
    job.grid.freesurf = freesurf
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    gen = torch.Generator(device="cuda").manual_seed(1)
    d = 1e-7 * torch.randn(job.grid.nt * int(job.acq.rec_off[-1]), generator=gen, device="cuda")
    out = []
    for opts in ((3, 4, 1), (0, 0, 0)):
        for k, v in zip((B.OPT_KERNEL, B.OPT_CHUNK, B.OPT_TILEMAP), opts):
            ctx.set_option(k, v)
        r = [ctx.forward(job.grid, job.acq, vp, rho, stf)[0],
             *ctx.fwi_grad(job.grid, job.acq, vp, rho, stf, d, want_dcal=True)]
        ctx.poll_status()
        out.append([t.cpu().numpy() for t in r])
    for k, (a, b) in enumerate(zip(*out)):
        say(f"{n1}x{n2} x{nshot} fs {freesurf} output {k}: bitwise {np.array_equal(a, b)}")
        assert np.abs(a).max() > 0 and np.array_equal(a, b)
