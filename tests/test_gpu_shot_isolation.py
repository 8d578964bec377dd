"""GPU: a shot whose field becomes non-finite leaves the other shots of its batch alone: their
seismograms are those of the batch with a quiet shot in its place, bitwise, under the default kernels
and the half-step kernels (SMI_OPT_KERNEL 3), and the status reports the non-finite field.  Padded widths that leave the
two-step launches of order 8 and 4 with rounded-up last runs, so that their loads pass the
right edge of a shot's field."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n2,freesurf", [(8, 97, 0), (8, 98, 0), (8, 99, 1), (8, 100, 0), (8, 101, 0),
                                               (4, 97, 0), (4, 98, 1), (4, 99, 0)])
def test_non_finite_shot_stays_alone(order, n2, freesurf):
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=40, n2=n2, nt=260, nshot=3, box=0)
    g = job.grid
    g.order, g.nb, g.freesurf = order, 4, freesurf
    g.fm = 15.0 if order == 8 else 7.0
    off = 3.3 if order == 8 else 0.0
    job.acq.src[:, 0] = 100.0 + off
    job.acq.src[:, 1] = [700.0 + off, 40.0 + off, 700.0 + off]
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    quiet, loud = stf.clone(), stf.clone()
    quiet[1] = 0.0
    loud[1, 5] = float("nan")
    for opts in ((3, 4, 1), (0, 0, 0)):
        for k, v in zip((B.OPT_KERNEL, B.OPT_CHUNK, B.OPT_TILEMAP), opts):
            ctx.set_option(k, v)
        want = [d.cpu().numpy() for d in B.split_dcal(ctx.forward(g, job.acq, vp, rho, quiet)[0], job.acq, g.nt)]
        ctx.poll_status()
        got = [d.cpu().numpy() for d in B.split_dcal(ctx.forward(g, job.acq, vp, rho, loud)[0], job.acq, g.nt)]
        with pytest.raises(B.SmiError):
            ctx.poll_status()
        same = [bool(np.array_equal(got[s], want[s])) for s in (0, 2)]
        say(f"order {order} n2 {n2} fs {freesurf} kernels {opts[0]}: shots 0 and 2 bitwise {same}")
        assert np.isnan(got[1]).any() and np.abs(want[0]).max() > 0 and all(same)
