"""Scratch of blocks whose rows and columns are those of a much larger array: a small one keeps one
set of partial sums, like a large block, and gives the bits that the same block gives in a tight
layout."""
import numpy as np
import pytest

from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [B.CFD_FP64, B.CFD_MIXED])
def test_small_block_in_a_large_array(precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = W.vortex_wavy(24, nj=20, nk=16)
    tight = DevBlock(wl, precision=precision)
    wide = DevBlock(wl, precision=precision, ld_i=512, ld_j=400)
    near = DevBlock(wl, precision=precision, ld_i=128, ld_j=64)
    try:
        plane = 512 * 400 * 22
        # 10 metric planes in FP64; 12 fluxes and 5 sums, and in mixed precision 19 metric planes
        want = plane * (80 + (17 * 8 if precision == B.CFD_FP64 else 36 * 4))
        assert B.cfd_block_bytes(wide.h) == want
        assert B.CFD_SWEEP_ONE_LAUNCH not in B.cfd_block_sweep_forms(wide.h)
        for d in (tight, near):
            assert B.cfd_block_sweep_forms(d.h) == [B.CFD_SWEEP_ONE_LAUNCH] * 3
        for d in (tight, wide, near):
            B.cfd_block_set_tiles(d.h, [5, 6, 6] if precision == B.CFD_FP64 else [5, 2, 2])
        want = tight.rhs().copy()
        np.testing.assert_array_equal(wide.rhs(), want)
        np.testing.assert_array_equal(near.rhs(), want)
        B.cfd_block_reset_tiles(near.h)
        np.testing.assert_array_equal(near.rhs(), want)
    finally:
        for d in (tight, wide, near):
            d.close()
