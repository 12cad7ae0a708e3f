"""The viscous prepass at the edges of its two tile shapes (32 x 8 and 64 x 16 columns), of
its chunks along k and on both sides of the block sizes where the shape changes, against the
oracle's viscous right-hand side.

Tolerances: FP64 as for every right-hand side (5e-11).  FP32: the velocity enters rounded to
6e-8 of |u| ~ 0.7 and passes two sixth-order differences (absolute weights sum to 1.83 each,
together < 4), while the terms come from perturbations of 1e-3 per node: 6e-8 * 0.7 * 4 / 1e-3
= 1.7e-4 of the largest value, times 3 for the other roundings of the chain = 5e-4.
"""
import pytest

import oracle as O
from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock, vector_norm_err

pytestmark = pytest.mark.gpu

VIS = 7 | B.CFD_TERM_VIS


@pytest.mark.parametrize("size,precision", [
    # one node more or less than a tile across, chunks of one plane and uneven last chunks
    ((33, 7, 9), B.CFD_FP64), ((31, 9, 7), B.CFD_FP64), ((65, 17, 61), B.CFD_FP64),
    ((33, 7, 9), B.CFD_MIXED), ((65, 17, 61), B.CFD_MIXED),
    # just below and above the sizes at which the wide tile takes over
    ((189, 179, 177), B.CFD_FP64), ((190, 181, 177), B.CFD_FP64),
    ((101, 100, 99), B.CFD_MIXED), ((101, 101, 99), B.CFD_MIXED),
    # between: the shape with the cheaper rounds, the narrow tile's and the wide tile's
    ((96, 100, 98), B.CFD_FP64), ((101, 94, 99), B.CFD_FP64),
    ((96, 100, 98), B.CFD_MIXED), ((101, 94, 99), B.CFD_MIXED)])
def test_viscous_rhs_at_tile_edges(size, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = W.vortex_wavy(size[0], nj=size[1], nk=size[2])
    c = O.cfg_from_workload(wl)
    met = O.metrics(c, wl.blocks[0].xyz)
    dev = DevBlock(wl, precision=precision)
    try:
        err = vector_norm_err(dev.rhs(VIS), O.rhs(c, met, wl.blocks[0].q, VIS))
    finally:
        dev.close()
    print(size, precision, err)
    assert err < (5e-11 if precision == B.CFD_FP64 else 5e-4)
