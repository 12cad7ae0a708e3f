"""What a call costs the host does not grow with the length of the block: launch plans are made
once, with the block."""
import time

import pytest

from paper_2006_07964_amd import binding as B

pytestmark = pytest.mark.gpu


def _enqueue_seconds(torch, n):
    """Least host time of one right-hand side in separate sweeps (nothing else enqueued)."""
    desc = B.make_desc(*n)
    h = B.cfd_block_create(desc, torch.cuda.current_stream())
    try:
        k, j, i = (torch.arange(-6, m + 6, dtype=torch.float64, device="cuda") for m in (n[2], n[1], n[0]))
        shape = (n[2] + 12, n[1] + 12, n[0] + 12)
        xyz = torch.stack([i.view(1, 1, -1).expand(shape), j.view(1, -1, 1).expand(shape), k.view(-1, 1, 1).expand(shape)])
        B.cfd_metrics(h, xyz.contiguous(), n[0] + 12, n[1] + 12)
        q, r = B.state_tensor(desc), B.state_tensor(desc)
        q[0], q[4] = 1.0, 2.0
        best = 1.0
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            B.cfd_rhs_sweeps(h, q, r)
            best = min(best, time.perf_counter() - t)
        torch.cuda.synchronize()
        return best
    finally:
        B.cfd_block_destroy(h)


def test_host_cost_of_a_call_on_a_long_block():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    short, lengthy = _enqueue_seconds(torch, (96, 80, 72)), _enqueue_seconds(torch, (8, 8, 60000))
    print(f"{short * 1e6:.1f} us, {lengthy * 1e6:.1f} us")
    assert lengthy < 4.0 * short
