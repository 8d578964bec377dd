"""GPU: receivers at the first columns under the two-step 2D forward launches with thin absorbing
layers.  The launches keep the receivers' rows of every shot and level side by side, so a store past
the end of one row lands in the first columns of the next.  Padded widths of every remainder modulo
the unrolled block (8 columns at order 8, 4 at order 4), one shot and two, points on the first
column and off the grid beside it: bitwise the half-step kernels (SMI_OPT_KERNEL 3), and within the
1e-4 of the other parity tests of the oracle."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, oracle_dcal, rel_l2, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,nb,n2,nshot",
                         [(8, 4, 96 + k, 1 + k % 2) for k in range(8)] +
                         [(8, 5, 105, 2), (8, 6, 89, 1), (8, 8, 99, 2)] +
                         [(4, 4, 96 + k, 2) for k in range(4)])
def test_receivers_at_the_first_columns(order, nb, n2, nshot):
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=40, n2=n2, nt=320, nshot=nshot, box=0)
    g = job.grid
    g.order, g.nb = order, nb
    g.fm = 15.0 if order == 8 else 7.0
    off = 3.3 if order == 8 else 0.0
    x = np.concatenate([np.arange(8) * g.d2, [2.3, 7.1, 12.6], (n2 - 1 - np.arange(3)) * g.d2])
    spread = np.stack([np.full(len(x), 20.0 + off), x, np.zeros(len(x))], 1)
    job.acq.src[:, 0] = 60.0 + off
    job.acq.src[:, 1] = 60.0 + 10.0 * np.arange(nshot) + off
    job.acq.rec = np.tile(spread, (nshot, 1))
    job.acq.rec_off = (len(x) * np.arange(nshot + 1)).astype(np.int32)
    job.stf *= (1.0 + np.arange(nshot))[:, None].astype(np.float32)     # shots of their own
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    out = []
    for opts in ((3, 4, 1), (0, 0, 0)):
        for k, v in zip((B.OPT_KERNEL, B.OPT_CHUNK, B.OPT_TILEMAP), opts):
            ctx.set_option(k, v)
        out.append(ctx.forward(g, job.acq, vp, rho, stf)[0])
        ctx.poll_status()
    want, got = (t.cpu().numpy() for t in out)
    ref = oracle_dcal(job)
    for s, d in enumerate(B.split_dcal(out[1], job.acq, g.nt)):
        d = d.cpu().numpy()
        say(f"order {order} nb {nb} n2 {n2} shot {s}: bitwise {np.array_equal(got, want)}, "
            f"oracle rel L2 {rel_l2(d, ref[s]):.2e}")
        peak = np.abs(d[:, :11]).max(0)        # the receivers at the first columns
        assert (peak > 0.01 * peak.max()).all()
        assert rel_l2(d, ref[s]) <= 1e-4
    assert np.array_equal(got, want)
