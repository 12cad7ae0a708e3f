"""The numbers that blocks return to the host (time step, residual norms, finiteness) when many
blocks exist at once, blocks come and go between the calls, and several threads use their own
blocks on their own streams: each block gets its own results."""
import threading

import pytest

from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevBlock

pytestmark = pytest.mark.gpu


def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_results_of_blocks_that_come_and_go():
    torch = _gpu()
    dev = DevBlock(W.vortex_wavy(9, nj=8, nk=7))
    others = []

    def check():
        for h, r in others:
            a = torch.full_like(dev.q, r)
            assert B.cfd_residual([h], [a])[1] == [r] * 5
            assert B.cfd_check_finite(h, a)
            a[4, 5, 5, 5] = float("inf")
            assert not B.cfd_check_finite(h, a)

    try:
        want = B.cfd_dt_cfl([dev.h], [dev.q], 0.5)
        # more blocks than one page of result slots, then gaps of every kind
        for n in range(70):
            others.append((B.cfd_block_create(dev.desc, torch.cuda.current_stream()), 1.0 + n))
        check()
        for n in sorted({0, 1, 31, 32, 33, 63, 64, 69}, reverse=True):
            B.cfd_block_destroy(others.pop(n)[0])
        check()
        for n in range(10):
            others.append((B.cfd_block_create(dev.desc, torch.cuda.current_stream()), 100.0 + n))
        check()
        assert B.cfd_dt_cfl([dev.h], [dev.q], 0.5) == want
    finally:
        for h, _ in others:
            B.cfd_block_destroy(h)
        dev.close()


def test_results_of_blocks_on_several_threads():
    torch = _gpu()
    errors = []

    def work(seed):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for turn in range(6):
                    wl = W.vortex_wavy(10 + seed, nj=9, nk=8, amp=0.02 * seed, seed=seed)
                    dev = DevBlock(wl)
                    try:
                        dt = B.cfd_dt_cfl([dev.h], [dev.q], 0.5)
                        a = torch.full_like(dev.q, float(seed))
                        for _ in range(20):
                            assert B.cfd_dt_cfl([dev.h], [dev.q], 0.5) == dt
                            assert B.cfd_residual([dev.h], [a])[1] == [float(seed)] * 5
                            assert B.cfd_check_finite(dev.h, a)
                        steps.setdefault(seed, set()).add(dt)
                    finally:
                        dev.close()
        except Exception as e:  # reported by the main thread
            errors.append((seed, e))

    steps = {}
    threads = [threading.Thread(target=work, args=(n,)) for n in (1, 2, 3, 4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert all(len(v) == 1 for v in steps.values()) and len(steps) == 4, steps
