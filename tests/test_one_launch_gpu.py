"""The prepass and the three sweeps of a small block in one launch, and the sum that follows,
against the sequential launches that a block runs once the caller has set its tiles.  The shapes are the
same, so every partial sum is, and they are added in the same order: the right-hand side and
the RK stages (host, device and per-point time steps) agree bit for bit, up to the sizes where
the form ends (300k points in FP64, 600k in mixed precision)."""
import numpy as np
import pytest

from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,viscous,precision", [
    (size, viscous, precision)
    for size, viscous in (((7, 9, 8), True), ((33, 31, 17), True), ((59, 16, 15), False), ((67, 67, 66), True))
    for precision in (B.CFD_FP64, B.CFD_MIXED)] + [((85, 84, 84), True, B.CFD_MIXED)])
def test_one_launch_matches_sequential_sweeps(size, viscous, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = W.vortex_wavy(size[0], nj=size[1], nk=size[2], viscous=viscous)
    a, b = DevBlock(wl, precision=precision), DevBlock(wl, precision=precision)
    try:
        # shapes of the one launch (the default zeta shape of mixed blocks has the same bits)
        tiles = [5, 6, 6] if precision == B.CFD_FP64 else [5, 2, 2]
        B.cfd_block_set_tiles(b.h, tiles)
        np.testing.assert_array_equal(a.rhs(), b.rhs())
        dt = 1e-3
        for d in (a, b):
            d.step(dt)
        np.testing.assert_array_equal(a.host(a.q), b.host(b.q))
        dt_dev = torch.tensor([2e-3], dtype=torch.float64, device="cuda")
        for d in (a, b):
            B.cfd_rk_stage_dev(d.h, 0, dt_dev, d.q, d.q, d.qa)
            local = B.state_tensor(d.desc, 1)
            B.cfd_dt_local([d.h], [d.q], 0.5, [local])
            B.cfd_block_set_local_dt(d.h, local)
            d.halo(d.qa)
            B.cfd_rk_stage(d.h, 1, dt, d.q, d.qa, d.qb)
            B.cfd_block_set_local_dt(d.h, None)
        np.testing.assert_array_equal(a.host(a.qa), b.host(b.qa))
        np.testing.assert_array_equal(a.host(a.qb), b.host(b.qb))
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("precision", [B.CFD_FP64, B.CFD_MIXED])
def test_one_launch_between_walls(precision):
    # the viscous ghosts of the walls are filled between the launch and the sum, and the split
    # form takes them from the fluxes that it is given
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = W.channel(37, 30, 19)
    a, b = DevBlock(wl, precision=precision), DevBlock(wl, precision=precision)
    try:
        B.cfd_block_set_tiles(b.h, [5, 6, 6] if precision == B.CFD_FP64 else [5, 2, 2])
        want = b.rhs()
        np.testing.assert_array_equal(a.rhs(), want)
        inviscid = B.CFD_ALL & ~B.CFD_TERM_VIS
        np.testing.assert_array_equal(a.rhs(inviscid), b.rhs(inviscid))
        B.cfd_viscous_fluxes(a.h, a.q)
        a.r.zero_()
        B.cfd_rhs_sweeps(a.h, a.q, a.r)
        np.testing.assert_array_equal(a.host(a.r), want)
        for d in (a, b):
            d.step(1e-3)
        np.testing.assert_array_equal(a.host(a.q), b.host(b.q))
    finally:
        a.close()
        b.close()
