"""Reverse Cuthill-McKee on meshes in pieces whose depths differ: batches of
levels that are sized by the piece before.  Bit for bit against the oracle,
and many small pieces of a kind in less time a piece than one alone."""
import time

import numpy as np
import pytest
import torch

import synth
from gpu_util import device_mesh, say
from oracle import graph
from test_gpu_graph import _mesh

pytestmark = pytest.mark.gpu


def _pieces(strips, seed=None):
    """Strips of k squares each, one after the other (k = 0: one triangle)."""
    xs, cells, n = [], [], 0
    for q, k in enumerate(strips):
        if k == 0:
            xs.append(np.array([[0, 0], [1, 0], [0, 1]], dtype=float) + [0, 3 * q])
            cells.append(np.array([[0, 1, 2]]) + n)
        else:
            xs.append(np.array([[i, 3 * q + j] for i in range(k + 1) for j in range(2)], dtype=float))
            cells.append(np.array([[2 * i, 2 * i + 2, 2 * i + 3] for i in range(k)] +
                                  [[2 * i, 2 * i + 3, 2 * i + 1] for i in range(k)]) + n)
        n += len(xs[-1])
    m = _mesh(np.concatenate(xs), np.concatenate(cells), "pieces_%s" % "_".join(map(str, strips[:6])))
    return m if seed is None else synth.permute_mesh(m, seed)[0]


@pytest.mark.parametrize("strips", [[40, 0, 0, 1, 16, 17, 15, 31, 0, 33, 2], [0, 0, 70, 0, 14, 3, 16], [15], [16], [0]])
@pytest.mark.parametrize("seed", [None, 4])
def test_rcm_of_pieces_matches_oracle(strips, seed):
    import paper_1602_03643_amd as oa
    mesh = _pieces(strips, seed)
    say("rcm", mesh.name)
    _, pat, _ = device_mesh(mesh, color=False)
    rp, ci = graph.csr_pattern(mesh)
    perm, order = oa.rcm(pat)
    o_ref, p_ref = graph.rcm(rp, ci)
    assert np.array_equal(order.cpu().numpy(), o_ref) and np.array_equal(perm.cpu().numpy(), p_ref)


def test_rcm_of_many_small_pieces_takes_few_launches():
    """One piece has to find out how deep it is (16 levels before the first
    look); the others profit: 203 us a piece against 282 for one alone, and 595
    against 529 in whole batches."""
    import paper_1602_03643_amd as oa

    def median(pieces):
        _, pat, _ = device_mesh(_pieces([0] * pieces), color=False)
        oa.rcm(pat)
        times = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            oa.rcm(pat)
            times.append(time.perf_counter() - t)
        return sorted(times)[4]

    one, many = median(1), median(200) / 200
    say("us a piece: one %.0f, of many %.0f" % (1e6 * one, 1e6 * many))
    assert many <= 0.9 * one
