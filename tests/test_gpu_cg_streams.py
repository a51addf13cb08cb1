"""A solve on the default stream beside work on a blocking stream of the process.

Launches on the default (null) stream wait for the work that blocking streams
have been given, and hold up what they are given next.  A solve must not: its
kernels run on a stream of their own.  While a solve of some 0.3 s runs, another
thread puts 1 s of waiting on a blocking stream; the solve's own time must not
take that second in.

The measurement is a program of its own: the device has four hardware queues, and
in a process with many streams two that have nothing to do with each other may
share one.
"""
import ctypes
import os
import subprocess
import sys
import threading
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DIMS = [(8, 8, 8, 8), (32, 32, 32, 8)]  # replayed graphs; launched kernel by kernel


def measure(dims):
    import torch

    import paper_2502_03249_amd as lqs
    import synth
    from gpu_util import field, gauge

    hip, handle = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    ctx = lqs.Context(0)
    g = gauge(ctx, dims, synth.gauge(dims, "smooth", seed=91, eps=0.3))
    bf = field(ctx, dims, synth.source(dims, 0, seed=92), 0)
    x = bf.like()

    def solve(iters):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        s = lqs.cg_solve(ctx, [(g, 0.02, bf, x)], tol=1e-30, max_iter=iters)[0]  # (out of reach)
        assert s["iters"] >= 0.9 * iters
        return time.perf_counter() - t0

    solve(200)
    iters = int(0.3 / (solve(2000) / 2000))
    alone = solve(iters)
    assert hip.hipStreamCreate(ctypes.byref(handle)) == 0
    other = torch.cuda.ExternalStream(handle.value)
    n = 10_000_000
    with torch.cuda.stream(other):  # cycles of torch's waiting kernel that take about 1 s
        t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        torch.cuda._sleep(n)
        t[0].record()
        torch.cuda._sleep(n)
        t[1].record()
    t[1].synchronize()
    cycles = int(n * 1000.0 / max(t[0].elapsed_time(t[1]), 1e-3))

    def wait_there():
        time.sleep(alone / 4)
        with torch.cuda.stream(other):
            torch.cuda._sleep(cycles)

    thread = threading.Thread(target=wait_there)
    thread.start()
    beside = solve(iters)
    thread.join()
    torch.cuda.synchronize()
    assert hip.hipStreamDestroy(handle) == 0
    g.close()
    ctx.close()
    print("dims", dims, "alone", alone, "beside", beside, flush=True)
    assert beside <= alone + 0.5


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(DIMS)))
def test_solve_does_not_wait_for_a_blocking_stream(case):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(case)], capture_output=True, text=True, timeout=90)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-2000:]


if __name__ == "__main__":
    sys.path[:0] = [ROOT, os.path.dirname(os.path.abspath(__file__))]
    measure(DIMS[int(sys.argv[1])])
