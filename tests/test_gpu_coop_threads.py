"""Cooperative solves from two host threads on two streams at once: every wait
inside the kernels needs all their blocks on the chip, so two of them must
never hold half of it each.  Results are those of the same solves alone, bit
for bit."""
import threading

import numpy as np
import pytest
import torch

import synth
from gpu_util import T, say
from test_gpu_coop import _system

pytestmark = pytest.mark.gpu


def test_two_threads_two_streams():
    import paper_1602_03643_amd as oa
    jobs = []
    for seed, mesh in ((3, synth.channel(41, 41, 41)), (4, synth.channel(65, 49, 49))):
        A, H, b = _system(oa, mesh, seed)
        B = torch.stack([T(b), T(np.roll(b, 7)), T(np.roll(b, 99))])
        jobs.append((A, T(b), B))
    torch.cuda.synchronize()

    def solve(job, stream):
        A, b, B = job
        out = []
        with torch.cuda.stream(stream):
            for _ in range(6):
                x, y = torch.zeros_like(b), torch.zeros_like(B)
                st = [oa.pcg(A, b, x, rtol=1e-9, stream=stream)] + oa.bicgstab(A, B, y, rtol=1e-9, stream=stream)
                assert all(s["status"] == 0 for s in st), st
                out.append((x, y))
            stream.synchronize()
        return out

    alone = [solve(job, torch.cuda.Stream()) for job in jobs]
    say("alone done")
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
    for a, g in zip(alone, got):
        assert all(torch.equal(x, u) and torch.equal(y, v) for (x, y), (u, v) in zip(a, g))
