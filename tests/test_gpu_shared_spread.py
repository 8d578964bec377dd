"""GPU: shots that share the receiver spread of the shot before take over its point operators and
adjoint-source gather; each shot of a batch whose spreads repeat, change, are empty and repeat
again gives bitwise the seismograms and gradients it gives in a call of its own."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,off", [(2, 0), (2, 1), (3, 1)])
def test_repeated_spreads_equal_single_shots(ndim, off):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    if ndim == 2:
        job = I.config3(n1=70, n2=130, nt=260, nshot=6)
    else:
        job = I.config4(n=36, nt=90, dr=1, nshot=4)
    ns = job.acq.nshot
    one = job.acq.rec[:int(job.acq.rec_off[1])][::3].copy()
    if off:
        one[:, 0] += 0.37 * job.grid.d1
        one[:, 1] = np.minimum(one[:, 1] + 0.41 * job.grid.d2, (job.grid.n2 - 1) * job.grid.d2)
    other = one[::-1].copy()
    spreads = [one, one, other, other, one[:0], one][:ns]
    off_ = np.concatenate([[0], np.cumsum([len(s) for s in spreads])]).astype(np.int32)
    acq = I.Acquisition(job.acq.src, off_, np.concatenate(spreads))
    job.acq = acq
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    nt = job.grid.nt
    gen = torch.Generator(device="cuda").manual_seed(3)
    d = 1e-7 * torch.randn(nt * int(off_[-1]), generator=gen, device="cuda")
    ctx.set_shot_groups(np.arange(ns + 1))
    grad, J, dcal = ctx.fwi_grad(job.grid, acq, vp, rho, stf, d, want_dcal=True)
    ctx.set_shot_groups(None)
    ctx.poll_status()
    grad = grad.view(ns, -1).cpu().numpy()
    dcal = [x.cpu().numpy() for x in B.split_dcal(dcal, acq, nt)]
    ds = B.split_dcal(d, acq, nt)
    for s in range(ns):
        if len(spreads[s]) == 0:
            continue
        g1, J1, d1 = ctx.fwi_grad(job.grid, acq.shot(s), vp, rho, stf[s:s + 1].contiguous(),
                                  ds[s].contiguous().view(-1), want_dcal=True)
        same = [np.array_equal(d1.cpu().numpy().ravel(), dcal[s].ravel()),
                np.array_equal(g1.cpu().numpy(), grad[s]), float(J1[0]) == float(J[s])]
        say(f"{ndim}D off-grid {off} shot {s} ({len(spreads[s])} receivers): {same}")
        assert all(same)
