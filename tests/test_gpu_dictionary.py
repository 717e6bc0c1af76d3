"""The offset dictionary of the ELL products is built on the device: its size
must be the number of distinct offset lists counted on the host, or the
per-entry offsets stay when there are more than a dictionary may hold
(n / 8)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import T, device_mesh, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


def _lists(pat):
    rp, ci = pat.row_ptr.cpu().numpy(), pat.col_idx.cpu().numpy()
    n = rp.size - 1
    half = n // 2
    rows = np.repeat(np.arange(n), np.diff(rp))
    d = ci.astype(np.int64) - rows
    d = np.where(d >= half, d - n, d)
    d = np.where(d < -half, d + n, d)
    out = np.zeros((n, 16), np.int64)
    out[rows, np.arange(ci.size) - rp[rows]] = d
    return len(np.unique(out, axis=0))


@pytest.mark.parametrize("mesh", [synth.unit_square(6), synth.unit_square(33), synth.channel(6, 6, 6),
                                  synth.channel(17, 17, 13), synth.channel(34, 21, 18, displace_seed=1),
                                  synth.permute_mesh(synth.channel(9, 9, 7), 1)[0]], ids=lambda m: m.name)
def test_dictionary_size(oa, mesh):
    say("dictionary", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    A = pat.with_values(oa.assemble_p1(dm, pat, oa.FORM_STIFF, base=oa.assemble_p1(dm, pat, oa.FORM_MASS, alpha=10.0)))
    b = T(np.random.default_rng(1).normal(size=mesh.n_dof))
    x = torch.zeros_like(b)
    out = oa.pcg(A, b, x, rtol=1e-8)
    want = _lists(pat)
    assert out["rc"] == 0
    assert out["ell_patterns"] == (want if want <= min(4096, mesh.n_dof // 8) else -1)


def test_far_more_lists_than_slots(oa):
    """Nearly every one of 49,920 rows has a list of its own, and the table has
    8192 slots: the search gives up, and the per-entry offsets stay."""
    mesh = synth.permute_mesh(synth.channel(41, 39, 33), 3)[0]
    say("dictionary", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    assert _lists(pat) > 40000
    A = pat.with_values(oa.assemble_p1(dm, pat, oa.FORM_STIFF, base=oa.assemble_p1(dm, pat, oa.FORM_MASS, alpha=10.0)))
    b = T(np.random.default_rng(1).normal(size=mesh.n_dof))
    for _ in range(3):
        out = oa.pcg(A, b, torch.zeros_like(b), rtol=1e-3)
        assert out["rc"] == 0 and out["ell_patterns"] == -1
