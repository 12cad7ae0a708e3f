"""The CFL step on the device under stream capture: what a capture records is complete by
itself, and a capture leaves nothing behind that a later call relies on, whether the graph has
run, runs later or is thrown away."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from paper_2006_07964_amd import binding as B
from paper_2006_07964_amd import workloads as W
from tests._gpu import DevMulti, hip, oracle_multi

pytestmark = pytest.mark.gpu

THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal


def _ok(rc):
    assert rc == 0, f"HIP error {rc}"


def _dirty_small_allocations():
    """Leaves the pattern of a huge double in device memory that the next small allocations may take."""
    L = hip()
    L.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    L.hipFree.argtypes = [C.c_void_p]
    host = np.full(4096, 1e250)
    ptrs = []
    for n in (8, 64, 4096, 16384, 32768) * 16:
        p = C.c_void_p()
        _ok(L.hipMalloc(C.byref(p), n))
        _ok(L.hipMemcpy(p, host.ctypes.data, n, 1))
        ptrs.append(p)
    for p in ptrs:
        _ok(L.hipFree(p))


def _capture(stream, call):
    """(graph, kernel nodes) of what call() enqueues on stream."""
    L = hip()
    graph, nodes = C.c_void_p(), C.c_size_t()
    _ok(L.hipStreamBeginCapture(C.c_void_p(stream.cuda_stream), THREAD_LOCAL))
    try:
        call()
    finally:
        _ok(L.hipStreamEndCapture(C.c_void_p(stream.cuda_stream), C.byref(graph)))
    _ok(L.hipGraphGetNodes(graph, None, C.byref(nodes)))
    return graph, nodes.value


def test_capture_of_the_device_step_keeps_no_state():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L = hip()
    wl = W.split_block(W.vortex_wavy(24, nj=20, nk=16, amp=0.06), [[10, 14], [20], [16]])
    _dirty_small_allocations()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        dev = DevMulti(wl)
        want = 0.5 / max(0.5 / O.dt_cfl(c, m, q, 0.5) for c, m, q in zip(*oracle_multi(wl)))
        out = torch.zeros(1, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        graphs, execs = [], []
        try:
            # the first use of the block's scratch is recorded, not run
            first, n_first = _capture(stream, lambda: B.cfd_dt_cfl_dev(dev.h, dev.q, 0.5, out))
            graphs.append(first)
            host = B.cfd_dt_cfl(dev.h, dev.q, 0.5)
            B.cfd_dt_cfl_dev(dev.h, dev.q, 0.5, out)
            assert abs(host - want) <= 1e-13 * want, (host, want)
            assert float(out.item()) == host
            # a later capture records the same work as the first
            second, n_second = _capture(stream, lambda: B.cfd_dt_cfl_dev(dev.h, dev.q, 0.5, out))
            graphs.append(second)
            assert n_first == n_second, (n_first, n_second)
            for g in graphs:
                e = C.c_void_p()
                _ok(L.hipGraphInstantiate(C.byref(e), g, None, None, 0))
                execs.append(e)
            # replays of both with eager calls on another state in between
            last = host
            for n in range(6):
                for q in dev.q:
                    q[4].mul_(1.01)  # a faster sound, a smaller step
                eager = B.cfd_dt_cfl(dev.h, dev.q, 0.5)
                out.zero_()
                _ok(L.hipGraphLaunch(execs[n % 2], C.c_void_p(stream.cuda_stream)))
                torch.cuda.synchronize()
                assert float(out.item()) == eager < last, n
                last = eager
        finally:
            torch.cuda.synchronize()
            for e in execs:
                _ok(L.hipGraphExecDestroy(e))
            for g in graphs:
                _ok(L.hipGraphDestroy(g))
            dev.close()
