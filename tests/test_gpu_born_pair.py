"""GPU: the tangent-linear step of the default path (2D: background and perturbation in two
launches per step; 3D: the perturbation on the y-marching half steps) against the one-cell-per-lane
kernels (SMI_OPT_KERNEL 4), at sizes around the edges of their tiles: bitwise in 2D (the same
arithmetic per cell), 1e-6 in 3D, the bound that the y-marching kernels are held to elsewhere."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, rel_l2, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,order,freesurf,off,box,n,nshot", [
    (2, 8, 0, 0, 1, (96, 261), 3),
    (2, 4, 0, 0, 0, (240, 97), 2),       # 256 padded rows with the 8 layers per side
    (2, 4, 1, 0, 0, (241, 98), 1),
    (2, 8, 1, 1, 1, (120, 203), 2),
    (3, 8, 0, 1, 1, (40, 40, 40), 2),
    (3, 4, 1, 0, 0, (30, 30, 30), 1),
])
def test_tangent_linear_step_equals_the_sweep_kernels(ndim, order, freesurf, off, box, n, nshot):
    import torch
    from paper_2311_02293_amd import binding as B
    ctx = B.Context(0)
    if ndim == 2:
        job = I.config2(n1=n[0], n2=n[1], nt=240, nshot=nshot, box=box)
    else:
        job = I.config4(n=n[0], nt=60, dr=1, nshot=nshot)
        job.grid.box = box
    job.grid.order = order
    job.grid.freesurf = freesurf
    job.grid.nb = 8
    if order == 4:
        job.grid.fm = 7.0
    if off:
        job.acq.src[:, 0] += 4.5
        job.acq.rec[:, 0] += 3.7
    job = with_bounds(job)
    vp, rho, stf = dev(job)
    gen = torch.Generator(device="cuda").manual_seed(2)
    dk = 0.05 * rho * vp * vp * torch.rand(vp.shape, generator=gen, device="cuda")
    out = []
    for kernel in (4, 0):
        ctx.set_option(B.OPT_KERNEL, kernel)
        out.append(ctx.born(job.grid, job.acq, vp, rho, stf, dk.contiguous()).cpu().numpy())
        ctx.poll_status()
    e = rel_l2(out[1], out[0])
    same = np.array_equal(out[0], out[1])
    say(f"born {ndim}D order {order} fs {freesurf} off {off} box {box} {n}: rel L2 {e:.2e} bitwise {same}")
    assert np.abs(out[0]).max() > 0 and e <= 1e-6 and (same or ndim == 3)
