"""GPU: what the autotuner picks for one acquisition is not run where it cannot be.  The two-step 2D
launches keep the receivers' rows in the workspace: on the context that tuned a surface spread,
receivers over more rows than they keep and a workspace without room for those rows still give the
untuned seismograms, bitwise."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [4, 8])
def test_pick_of_another_acquisition(order):
    import copy
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    job = I.config2(n1=96, n2=200, nt=240, nshot=2)
    job.grid.order = order
    job.grid.fm = 15.0 if order == 8 else 7.0
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    well = copy.deepcopy(job.acq)
    well.rec[:, 0] = (np.arange(len(well.rec)) % 40 + 3) * job.grid.d1
    full = ctx.workspace_bytes(job.grid, job.acq, B.JOB_FORWARD)
    calls = [("surface spread", job.acq, full), ("receivers over 40 rows", well, None),
             ("workspace without the rows", job.acq, full - 1)]
    keep = torch.empty(2 * full, dtype=torch.uint8, device="cuda")

    def run(acq, nbytes):
        ws = keep[:nbytes] if nbytes else None
        d = ctx.forward(job.grid, acq, vp, rho, stf, ws=ws)[0].cpu().numpy()
        ctx.poll_status()
        return d

    want = [run(a, n) for _, a, n in calls]
    ctx.set_option(B.OPT_AUTOTUNE, 2)
    ctx.set_option(B.OPT_AUTOTUNE, 1)
    try:
        for rep in range(2):
            for (name, a, n), w in zip(calls, want):
                got = run(a, n)
                say(f"order {order} {name}, call {rep}: bitwise {np.array_equal(got, w)};",
                    ctx.tuning_report())
                assert np.abs(w).max() > 0 and np.array_equal(got, w)
    finally:
        ctx.set_option(B.OPT_AUTOTUNE, 0)
