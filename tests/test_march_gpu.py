"""The marching form of the FP64 eta and zeta sweeps (lines of a block large enough for it)
against the general path, the tile kernels, which a block runs once the caller has set its
tiles: line counts that are no multiple of a workgroup, chunks of odd and even length with a
shorter last one, short and long lines, with and without viscous terms and earlier partial
sums, and a uniform stream.

Both forms take the smoothness indicators from squared differences, so they differ by
roundings of the fluxes alone: about ten of 1.1e-16 on fluxes whose differences between nodes,
with perturbations of 1e-3 per node, are 1e-3 of them, 1e-12 of the largest value.  What a
uniform stream leaves is all rounding: its root mean square is at most 1.25 of the tiles'.
"""
import numpy as np
import pytest

import oracle as O
from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock, normwise
from tests.test_closure_gpu import axis_channel

pytestmark = pytest.mark.gpu

ALL_INV = 7 | B.CFD_TERM_INV


def rms(r):
    return float(np.sqrt(np.mean(r[:, 3:-3, 3:-3, 3:-3] ** 2)))


@pytest.mark.parametrize("size,mask", [
    ((129, 131, 127), B.CFD_ALL), ((67, 257, 129), B.CFD_ALL), ((1203, 150, 13), B.CFD_ALL),
    ((150, 11, 1203), B.CFD_ALL), ((129, 131, 127), ALL_INV),
    # eta first (no partial sum before it), xi last; zeta first, eta last
    ((161, 160, 128), B.CFD_DIR_XI | B.CFD_DIR_ETA | B.CFD_TERM_INV | B.CFD_TERM_VIS),
    ((161, 160, 128), B.CFD_DIR_ETA | B.CFD_DIR_ZETA | B.CFD_TERM_INV)])
def test_march_agrees_with_tiles(size, mask):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = W.vortex_wavy(size[0], nj=size[1], nk=size[2])
    uniform = W.uniform_state(wl.blocks[0].q.shape[1:], u=0.5, v=-0.2, w=0.1)
    dev = DevBlock(wl)
    try:
        got = dev.rhs(mask)
        uniform = torch.from_numpy(uniform).cuda()
        free = rms(dev.rhs(q=uniform))
        B.cfd_block_set_tiles(dev.h, B.cfd_block_tiles(dev.h))
        err = normwise(got, dev.rhs(mask))
        free_tiles = rms(dev.rhs(q=uniform))
    finally:
        dev.close()
    print(size, mask, err, free, free_tiles)
    assert np.all(err < 1e-12), err
    assert free <= 1.25 * free_tiles


@pytest.mark.parametrize("case", ["original", "original Euler", "one-sided j walls", "one-sided k walls",
                                  "one-sided j walls, original"])
def test_march_of_other_forms_agrees_with_tiles(case):
    """The original scheme, and the one-sided closure at walls across the marched direction
    (chunks that start or end at a wall, and lines whose both ends are walls)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    scheme = B.CFD_AFWENO_ORIGINAL if "original" in case else B.CFD_AFWENO_MODIFIED
    if "one-sided" in case:
        wl = axis_channel(1, shape=(163, 137, 97)) if "j walls" in case else axis_channel(2, shape=(131, 127, 139))
        c = O.cfg_from_workload(wl)
        q = O.bc_fill(c, O.periodic_wrap(c, O.wall_reset(c, wl.blocks[0].q)))
    else:
        wl, q = W.vortex_wavy(129, nj=131, nk=127), None
    dev = DevBlock(wl, q=q, scheme=scheme)
    try:
        mask = ALL_INV if "Euler" in case else B.CFD_ALL
        got = dev.rhs(mask).copy()
        B.cfd_block_set_tiles(dev.h, B.cfd_block_tiles(dev.h))
        err = normwise(got, dev.rhs(mask))
    finally:
        dev.close()
    print(case, err)
    assert np.all(err < 1e-12), err
