"""Residual norms on both sides of the block sizes where the reduction changes its workgroups,
and over blocks that take different ones, against numpy's norms.

Tolerance: a sum of n positive squares in any order is off by at most log2-like depth times
1.1e-16 in a tree, here by under (passes + 30) roundings, passes < 100: 130 * 1.1e-16 / 2 for the
square root, below 1e-14.  Maxima are exact.
"""
import numpy as np
import pytest

from paper_2006_07964_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [(64, 64, 64)], [(65, 64, 64)],           # three and six passes saved
    [(40, 48, 64)], [(128, 64, 48)], [(2000, 7, 7)], [(7, 130, 127)],
    [(9, 8, 7), (80, 81, 83), (300, 20, 20), (16, 70, 66)]])
def test_residual_norms_of_small_and_large_blocks(sizes):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(3)
    hs, a, b = [], [], []
    try:
        for n in sizes:
            desc = B.make_desc(*n, ld_i=B.aligned_pitch(n[0]))
            hs.append(B.cfd_block_create(desc, torch.cuda.current_stream()))
            for to in (a, b):
                t = B.state_tensor(desc)
                t.copy_(torch.randn(t.shape, dtype=t.dtype, device="cuda", generator=g))
                to.append(t)
        d = [7.0 * (x - y)[:, 3:-3, 3:3 + n[1], 3:3 + n[0]].cpu().numpy().reshape(5, -1) for x, y, n in zip(a, b, sizes)]
        d = np.concatenate(d, axis=1)
        rms, top = B.cfd_residual(hs, a, b, 7.0)
        want = np.sqrt(np.mean(np.square(d, dtype=np.longdouble), axis=1)).astype(float)
        assert np.all(np.abs(np.array(rms) - want) <= 1e-14 * want), (rms, want)
        assert np.all(np.array(top) == np.max(np.abs(d), axis=1))
        assert (rms, top) == B.cfd_residual_noalloc(hs, a, b, 7.0)
    finally:
        for h in hs:
            B.cfd_block_destroy(h)
