"""Two processes that solve on one card.  Alone a solve takes a few
milliseconds; with the other process beside it, it may take the sum of both
and what little each then waits for the other, and not the tens of
milliseconds for which the device keeps one process's cooperative queue (a
factor of 15 on one of the two)."""
import os
import subprocess
import sys

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

SOLVE = """
import sys, time
sys.path[:0] = [%r, %r]
import numpy as np, torch
import paper_1602_03643_amd as oa
import synth
from gpu_util import T
from test_gpu_coop import _system
A, H, b = _system(oa, synth.channel(33, 33, 25), 3)
b = T(b)
x, B = torch.zeros_like(b), torch.stack([b, b.flip(0), b * b])
X = torch.zeros_like(B)

def median(seconds):
    times, end = [], time.time() + seconds
    while time.time() < end or len(times) < 5:
        x.zero_(), X.zero_()
        t = time.perf_counter()
        st = [oa.pcg(A, b, x, rtol=1e-8)] + oa.bicgstab(A, B, X, rtol=1e-8, maxit=4000)
        times.append(time.perf_counter() - t)
        assert all(s["status"] == 0 and s["coop_runs"] + s["coop_lost"] > 0 for s in st), st
    return sorted(times)[len(times) // 2]

median(0.2)
for line in sys.stdin:
    print(median(float(line)), flush=True)
""" % (os.path.dirname(HERE), HERE)


def test_two_processes_on_one_card():
    ps = [subprocess.Popen([sys.executable, "-u", "-c", SOLVE], stdin=subprocess.PIPE, stdout=subprocess.PIPE,
                           text=True) for _ in range(2)]
    try:
        def ask(p, seconds):
            p.stdin.write("%g\n" % seconds)
            p.stdin.flush()

        alone = []
        for p in ps:
            ask(p, 0.5)
            alone.append(float(p.stdout.readline()))
        say("alone", alone)
        for p in ps:
            ask(p, 3.0)
        both = [float(p.stdout.readline()) for p in ps]
        say("together", both)
        assert max(both) <= 5 * max(alone)
    finally:
        for p in ps:
            p.stdin.close()
            p.wait(timeout=30)


def test_two_threads_with_full_grids():
    """Two threads on two streams, both solvers on systems that take every CU:
    grids that hold each other up are launched again, so the results are those
    of the same solves alone, bit for bit."""
    import threading

    import numpy as np
    import torch

    import paper_1602_03643_amd as oa
    import synth
    from gpu_util import T
    from test_gpu_coop import _system

    jobs = []
    for seed, mesh in ((3, synth.channel(61, 65, 65)), (4, synth.channel(65, 64, 65))):
        A, _, b = _system(oa, mesh, seed)
        jobs.append((A, T(b), torch.stack([T(b), T(np.roll(b, 7))])))
    torch.cuda.synchronize()

    def solve(job, stream):
        A, b, B = job
        out, lost = [], 0
        with torch.cuda.stream(stream):
            for _ in range(30):
                x, y = torch.zeros_like(b), torch.zeros_like(B)
                st = [oa.pcg(A, b, x, rtol=1e-6, stream=stream)]
                st += oa.bicgstab(A, B, y, rtol=1e-6, maxit=4000, stream=stream)
                assert all(s["status"] == 0 and s["coop_runs"] > 0 for s in st), st
                lost += sum(s["coop_lost"] for s in st[:2])
                out.append((x, y))
            stream.synchronize()
        return out, lost

    alone = [solve(job, torch.cuda.Stream())[0] for job in jobs]
    got, err = [None, None], []

    def work(k):
        try:
            got[k] = solve(jobs[k], torch.cuda.Stream())
        except Exception as e:                                  # noqa: BLE001
            err.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
    assert not err, err
    say("launched again:", got[0][1], got[1][1])
    for a, (g, _) in zip(alone, got):
        assert all(torch.equal(x, u) and torch.equal(y, v) for (x, y), (u, v) in zip(a, g))
