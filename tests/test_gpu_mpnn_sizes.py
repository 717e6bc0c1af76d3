"""Backward pass of the warm-start network at the edges of its tiles.

The gradient kernels work on tiles of 128 nodes over 512 blocks: fewer nodes
than one tile, a tile and a remainder, a second tile for some of the blocks
only.  The oracle's backward pass runs on a forward pass whose stored
activations are rounded to bfloat16 as the network stores them: on a mesh of
45 nodes the FP64 activations take a few nodes to the other side of a ReLU,
7% of a gradient, which says nothing about the backward pass.  The gradients
that it stores are bfloat16 too (8 bits, 4e-3 a value), hence 5e-2 per
tensor; the K-norm gradient of the output bias is zero but for rounding and
is bounded against the decoder's other gradient.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import T, dev, rel, say
from oracle import ipcs, mpnn
from test_gpu_mpnn import _flat, _gpu_graph, _params, _unflat

pytestmark = pytest.mark.gpu


def _bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a)).float().bfloat16().double().numpy()


def _forward_as_stored(P, X, W):
    """The oracle's forward pass with bfloat16 activations and weights."""
    Q = dict(P, Ws=_bf16(P["Ws"]), Wn=_bf16(P["Wn"]))
    z0 = _bf16(X @ Q["We"].T + Q["ce"])
    h = np.maximum(z0, 0.0)
    cache = {"X": X, "z0": z0, "z": [], "h": [h], "a": []}
    for l in range(mpnn.LAYERS):
        a = _bf16(W @ h)
        z = h @ Q["Ws"][l].T + a @ Q["Wn"][l].T + Q["c"][l]
        h = _bf16(h + np.maximum(z, 0.0))
        cache["a"].append(a)
        cache["z"].append(_bf16(z))
        cache["h"].append(h)
    return Q, h @ Q["wd"] + Q["cd"][0], cache


@pytest.mark.parametrize("kind", ["mse", "knorm"])
@pytest.mark.parametrize("size", [(4, 5, 4), (5, 9, 5), (9, 11, 7), (41, 43, 41)])
def test_backward_at_tile_edges(size, kind):
    import paper_1602_03643_amd as oa
    pr = synth.channel_flow(size, seed=4)
    n = pr.mesh.n_dof
    say("mpnn backward", size, n, kind)
    S = ipcs.setup(pr.mesh, pr.nu, pr.dt, pr.f)
    rng = np.random.default_rng(5)
    prev, phi, b = rng.normal(size=n), rng.normal(size=n), rng.normal(size=n)
    Ks, s = _gpu_graph(oa, pr, S)
    P = _params(6)
    net = oa.MPNN(Ks, s, T(pr.mesh.dof_coords))
    pt = T(_flat(P), torch.float32)
    net.forward(pt, T(b), T(prev))
    grad = torch.full((oa.MPNN.NPARAM,), float("nan"), dtype=torch.float32, device=dev())
    loss = net.backward(pt, T(phi), T(prev), grad, oa.MPNN_LOSS_KNORM if kind == "knorm" else oa.MPNN_LOSS_MSE)
    X, sigma = mpnn.features(S.K, b, prev, pr.mesh.dof_coords)
    W = mpnn.edge_weights(S.K)
    Q, d_ref, cache = _forward_as_stored(P, X, W)
    target = (phi - prev) / sigma
    G = mpnn.backward(Q, cache, d_ref, target, W, kind, S.K)
    assert abs(loss / mpnn.loss(d_ref, target, kind, S.K) - 1.0) < 3e-2
    g = _unflat(grad.cpu().numpy())
    for k, _ in mpnn.PARAM_SHAPES:
        if kind == "knorm" and k == "cd":
            assert abs(g["cd"][0]) < 1e-5 * np.linalg.norm(G["wd"])
            continue
        assert rel(g[k], G[k]) < 5e-2, (k, rel(g[k], G[k]))
