"""GPU: the two-step 2D forward launches (the default of order 4 and of off-grid sources) against
the half-step kernels (SMI_OPT_KERNEL 3): every cell's arithmetic is the same, so seismograms,
gradients whose forward pass saved bands, and images are bitwise equal.  Sizes around the edges of
its strips of 64 to 512 rows and its runs of columns, step counts with every remainder, and the
cases it leaves to the half-step kernels (snapshots, receivers over many rows, a workspace without
room for its receiver rows)."""
import numpy as np
import pytest

from paper_2311_02293_amd import inputs as I
from helpers import dev, say, with_bounds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2311_02293_amd import binding as B
    return B.Context(0)


def _half_steps(ctx, fn):
    from paper_2311_02293_amd import binding as B
    for k, v in ((B.OPT_KERNEL, 3), (B.OPT_CHUNK, 4), (B.OPT_TILEMAP, 1)):
        ctx.set_option(k, v)
    try:
        return fn()
    finally:
        for k in (B.OPT_KERNEL, B.OPT_CHUNK, B.OPT_TILEMAP):
            ctx.set_option(k, 0)


def _same(ctx, name, fn):
    ref = _half_steps(ctx, fn)
    got = fn()
    ctx.poll_status()
    for k, (a, b) in enumerate(zip(got, ref)):
        a, b = a.cpu().numpy(), b.cpu().numpy()
        say(f"{name} output {k}: bitwise {np.array_equal(a, b)}, max {np.abs(b).max():.3e}")
        assert np.isfinite(b).all() and np.array_equal(a, b)


def _job(n1, n2, nt, nshot, order, freesurf, off, box):
    job = I.config2(n1=n1, n2=n2, nt=nt, nshot=nshot, box=box)
    job.grid.order = order
    job.grid.freesurf = freesurf
    job.grid.nb = 20 if min(n1, n2) > 30 else (8 if n1 > 8 else 4)
    if order == 4:
        job.grid.fm = 7.0
    if off:
        xmax = (n2 - 1) * job.grid.d2
        job.acq.src[:, 0] += 4.5
        job.acq.src[:, 1] += 3.1
        job.acq.rec[:, 0] += 3.7
        job.acq.rec[:, 1] = np.minimum(job.acq.rec[:, 1] + 2.3, xmax)
    return with_bounds(job)


# 60 x 200 pads to 100 rows (two wavefronts), 464 / 465 to 504 / 505 (one strip of 512 lanes with its
# 8 ghost rows just holds the first), 700 to several strips; 8 x 8 with 4 layers is the smallest grid
@pytest.mark.parametrize("n1,n2,nt,nshot,order,freesurf,off,box", [
    (8, 8, 9, 1, 4, 0, 0, 0),
    (20, 24, 50, 1, 8, 0, 1, 1),
    (60, 200, 301, 3, 4, 0, 0, 1),
    (201, 201, 402, 1, 4, 0, 0, 0),
    (464, 150, 203, 1, 4, 1, 0, 0),
    (465, 150, 204, 2, 8, 0, 1, 0),
    (700, 333, 300, 2, 4, 1, 1, 0),
    (263, 611, 500, 2, 8, 1, 1, 1),
    (120, 900, 400, 5, 4, 0, 1, 1),
])
def test_two_step_launches_equal_half_steps(ctx, n1, n2, nt, nshot, order, freesurf, off, box):
    import torch
    job = _job(n1, n2, nt, nshot, order, freesurf, off, box)
    vp, rho, stf = dev(job)
    name = f"{n1}x{n2} nt {nt} order {order} fs {freesurf} off {off} box {box}"
    _same(ctx, name, lambda: [ctx.forward(job.grid, job.acq, vp, rho, stf)[0]])
    gen = torch.Generator(device="cuda").manual_seed(5)
    d = 1e-7 * torch.randn(nt * int(job.acq.rec_off[-1]), generator=gen, device="cuda")
    for dr in (1, 3):
        job.grid.dr = dr
        _same(ctx, name + f" gradient dr {dr}",
              lambda: list(ctx.fwi_grad(job.grid, job.acq, vp, rho, stf, d, want_dcal=True,
                                        rho_grad=True)))


@pytest.mark.parametrize("order,off,nb", [(4, 0, 20), (8, 1, 8)])
def test_long_run_through_the_absorbing_layers(ctx, order, off, nb):
    """Long enough for what the layers let through to come back from their outer corners to the
    receivers: memory variables there stay those of the half-step kernels."""
    job = _job(60, 64, 1500, 1, order, 0, off, 0)
    job.grid.nb = nb
    vp, rho, stf = dev(job)
    _same(ctx, f"long run order {order}", lambda: [ctx.forward(job.grid, job.acq, vp, rho, stf)[0]])


@pytest.mark.parametrize("nrow", [16, 17])
def test_receiver_rows_up_to_the_limit(ctx, nrow):
    """Receivers spread over 16 rows (kept by the launches) and 17 (the half-step kernels)."""
    job = _job(96, 200, 302, 2, 4, 0, 0, 1)
    n = len(job.acq.rec)
    job.acq.rec[:, 0] = (np.arange(n) * 7 % nrow + 3) * job.grid.d1
    vp, rho, stf = dev(job)
    _same(ctx, f"{nrow} receiver rows", lambda: [ctx.forward(job.grid, job.acq, vp, rho, stf)[0]])


def test_small_workspace_graph_snapshots_and_groups(ctx):
    """A workspace without room for the receiver rows, graph replay, snapshots and shot groups give
    the same seismograms."""
    import torch
    from paper_2311_02293_amd import binding as B
    job = _job(150, 260, 403, 4, 4, 0, 1, 1)
    vp, rho, stf = dev(job)
    want = ctx.forward(job.grid, job.acq, vp, rho, stf)[0].cpu().numpy()
    full = ctx.workspace_bytes(job.grid, job.acq, B.JOB_FORWARD)
    small = torch.empty(full - 1, dtype=torch.uint8, device="cuda")
    got = ctx.forward(job.grid, job.acq, vp, rho, stf, ws=small)[0].cpu().numpy()
    assert np.array_equal(got, want)
    got = ctx.forward(job.grid, job.acq, vp, rho, stf, snaps=[77])[0].cpu().numpy()
    assert np.array_equal(got, want)
    ctx.set_option(B.OPT_FWD_GROUP, 3)
    got = ctx.forward(job.grid, job.acq, vp, rho, stf)[0].cpu().numpy()
    ctx.set_option(B.OPT_FWD_GROUP, 0)
    assert np.array_equal(got, want)
    ctx.set_option(B.OPT_GRAPH, 1)
    try:
        out = torch.empty(want.size, device="cuda")
        ws = torch.empty(full, dtype=torch.uint8, device="cuda")
        for _ in range(3):
            out.fill_(7.0)
            ctx.forward(job.grid, job.acq, vp, rho, stf, dcal=out, ws=ws)
            assert np.array_equal(out.cpu().numpy(), want)
    finally:
        ctx.set_option(B.OPT_GRAPH, 0)
