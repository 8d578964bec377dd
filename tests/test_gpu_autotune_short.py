"""GPU: the autotuner on schedules shorter than its timing windows of 8 steps (odd ones among them,
where a launch of two steps would pass the last step): untuned and tuned results are bitwise
equal, for seismograms and for gradients whose forward pass runs on past the last step."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", [1, 2, 3, 5, 7, 8, 9])
@pytest.mark.parametrize("order", [4, 8])
def test_tuned_short_schedules(nt, order):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=40, n2=72, nt=nt, nshot=2)
    job.grid.order = order
    job.grid.fm = 15.0 if order == 8 else 7.0
    # (a wavelet that is strong from the first step on)
    job.stf = np.tile(np.cos(np.arange(nt)).astype(np.float32), (2, 1))
    job.acq.rec[:, 1] = job.acq.src[0, 1] + (np.arange(len(job.acq.rec)) % 3) * job.grid.d2
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    d = torch.zeros(nt * int(job.acq.rec_off[-1]), device="cuda")

    def run():
        out = [ctx.forward(job.grid, job.acq, vp, rho, stf)[0]]
        for dr in (1, 2):
            job.grid.dr = dr
            out += ctx.fwi_grad(job.grid, job.acq, vp, rho, stf, d, want_dcal=True)[:3]
        job.grid.dr = 1
        ctx.poll_status()
        return [t.cpu().numpy() for t in out if t is not None]

    want = run()
    ctx.set_option(B.OPT_AUTOTUNE, 1)
    for call in range(2):
        got = run()
        say(f"nt {nt} order {order} call {call}:", ctx.tuning_report())
        for a, b in zip(got, want):
            assert np.isfinite(b).all() and np.array_equal(a, b)
    assert np.abs(want[0]).max() > 0
