"""CG runs by one block (systems of up to 2048 rows), at the edges of its
shapes: one and two rows a thread, full and not, rows of 7 entries and of
15, and the first size that takes several blocks.  As the runs by several
blocks: the tolerance in a residual computed on the host in FP64, the
two-kernel form's iteration count, the same bits however often interrupted."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import T, say
from test_gpu_coop import _system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("mesh", [lambda: synth.unit_square(1), lambda: synth.unit_square(31),      # 4, 1024 rows
                                  lambda: synth.unit_square(32), lambda: synth.unit_square(44),     # 1089, 2025
                                  lambda: synth.unit_square(45), lambda: synth.channel(9, 16, 9),   # 2116, 1024
                                  lambda: synth.channel(17, 8, 17), lambda: synth.channel(12, 13, 13)])  # 2048, 1716
def test_one_block_cg(mesh, precision):
    import paper_1602_03643_amd as oa
    mesh = mesh()
    say("one block cg", mesh.name, mesh.n_dof, precision)
    A, H, b = _system(oa, mesh, 3)
    outs, xs = [], []
    for kw in (dict(), dict(check_every=7), dict(cg_form=oa.CG_FORM_TWO)):
        x = torch.zeros(mesh.n_dof, dtype=torch.float64, device="cuda")
        outs.append(oa.pcg(A, T(b), x, rtol=1e-9, precision=oa.F64 if precision == "f64" else oa.F32, **kw))
        xs.append(x)
        assert outs[-1]["rc"] == 0
        assert np.linalg.norm(b - H @ x.cpu().numpy()) <= 1.001e-9 * np.linalg.norm(b)
    assert torch.equal(xs[0], xs[1]) and outs[0]["iters"] == outs[1]["iters"]
    assert abs(outs[0]["iters"] - outs[2]["iters"]) <= max(3, outs[2]["iters"] // 50)
