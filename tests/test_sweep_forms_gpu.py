"""Which form the sweeps of a block run in, and the marching form where it is at its edges: fewer
lines than a workgroup has threads, a last chunk of one output, lines of one short chunk.  The
results are compared with the tile kernels at the tolerance of the marching form's other tests:
the two differ by roundings of the fluxes, about ten of 1.1e-16 on fluxes whose differences
between nodes are 1e-3 of them, 1e-12 of the largest value."""
import numpy as np
import pytest

from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock, normwise

pytestmark = pytest.mark.gpu

TILES, ROWS, MARCH, ONE = B.CFD_SWEEP_TILES, B.CFD_SWEEP_ROWS, B.CFD_SWEEP_MARCH, B.CFD_SWEEP_ONE_LAUNCH


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield


@pytest.mark.parametrize("size,over,forms", [
    ((32, 32, 32), {}, [ONE] * 3), ((67, 67, 66), {}, [ONE] * 3), ((85, 84, 84), {}, [ROWS, TILES, TILES]),
    ((85, 84, 83), dict(precision=B.CFD_MIXED), [ONE] * 3), ((86, 84, 84), dict(precision=B.CFD_MIXED), [TILES] * 3),
    ((32, 32, 32), dict(scheme=B.CFD_AFWENO_ORIGINAL), [ROWS, TILES, TILES]),
    ((129, 131, 127), dict(precision=B.CFD_MIXED), [TILES] * 3),
    ((129, 131, 127), dict(weights=B.CFD_WENO_LINEAR), [ROWS, TILES, TILES]),
    # the sizes of the other tests of the marching form
    ((129, 131, 127), {}, [ROWS, MARCH, MARCH]), ((67, 257, 129), {}, [ROWS, MARCH, MARCH]),
    ((1203, 150, 13), {}, [ROWS, MARCH, MARCH]), ((150, 11, 1203), {}, [ROWS, TILES, MARCH]),
    ((161, 160, 128), {}, [ROWS, MARCH, MARCH]), ((163, 137, 97), {}, [ROWS, MARCH, MARCH]),
    ((131, 127, 139), {}, [ROWS, MARCH, MARCH])])
def test_form_of_each_sweep(size, over, forms):
    import torch
    h = B.cfd_block_create(B.make_desc(*size, **over), torch.cuda.current_stream())
    try:
        assert B.cfd_block_sweep_forms(h) == forms
        tiles = B.cfd_block_tiles(h)
        B.cfd_block_set_tiles(h, tiles)
        assert B.cfd_block_sweep_forms(h) == [TILES] * 3
        B.cfd_block_set_tiles(h, [1, 2, 3])
        B.cfd_block_reset_tiles(h)
        assert B.cfd_block_sweep_forms(h) == forms and B.cfd_block_tiles(h) == tiles
    finally:
        B.cfd_block_destroy(h)


@pytest.mark.parametrize("size,forms", [
    ((15, 9901, 17), [ROWS, MARCH, TILES]),   # eta: 255 lines, a last chunk of one output
    ((15, 17, 9901), [ROWS, TILES, MARCH]),   # zeta: the same
    ((18, 14, 9999), [ROWS, MARCH, MARCH]),   # eta: lines of one chunk
    ((1000, 1000, 8), [ROWS, MARCH, MARCH])])  # zeta: lines of one chunk, the shortest that march
def test_march_at_its_edges(size, forms):
    wl = W.vortex_wavy(size[0], nj=size[1], nk=size[2])
    dev = DevBlock(wl)
    try:
        assert B.cfd_block_sweep_forms(dev.h) == forms
        got = dev.rhs().copy()
        B.cfd_block_set_tiles(dev.h, B.cfd_block_tiles(dev.h))
        err = normwise(got, dev.rhs())
        B.cfd_block_reset_tiles(dev.h)
        np.testing.assert_array_equal(dev.rhs(), got)
    finally:
        dev.close()
    print(size, err)
    assert np.all(err < 1e-12), err
