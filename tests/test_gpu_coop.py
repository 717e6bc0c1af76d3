"""CG runs in one cooperative launch (systems of up to 1024 rows per CU).

The sizes sit at the edges of the kernel's shapes: less than one block, one
row more than a block, the three block sizes (up to 256, 512 and 1024 rows
per block), the largest system that fits and the first that does not, and a
randomly numbered mesh whose blocks reference too many foreign columns, for
which the solver must go on with its other kernels.  Every solve must meet
the tolerance in a residual computed on the host in FP64, take as many
iterations as the two-kernel form (both are the same recurrences; partial
sums differ in order), and give the same bits however often it is
interrupted.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import T, csr_host, device_mesh, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


def _system(oa, mesh, seed):
    """K + 10 M: positive definite, conditioned as the pressure matrix is at
    its upper end."""
    dm, pat, _ = device_mesh(mesh)
    A = pat.with_values(oa.assemble_p1(dm, pat, oa.FORM_STIFF, base=oa.assemble_p1(dm, pat, oa.FORM_MASS, alpha=10.0)))
    b = np.random.default_rng(seed).normal(size=mesh.n_dof)
    return A, csr_host(pat, A.val), b


MESHES = {
    "below one block": lambda: synth.channel(6, 6, 6),                    # 150 rows
    "two blocks": lambda: synth.unit_square(16),                          # 289
    "13 blocks": lambda: synth.channel(17, 17, 13),                       # 3264
    "512 threads": lambda: synth.channel(49, 45, 41),                     # 86,400: 338 per block
    "displaced, 512 threads": lambda: synth.channel(45, 43, 37, displace_seed=3),
    "1024 threads, full": lambda: synth.channel(65, 64, 65),              # 262,144: every thread has a row
    "too large": lambda: synth.channel(65, 65, 65),                       # 266,240
    "halo too wide": lambda: synth.permute_mesh(synth.channel(17, 17, 13), 9)[0],
}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name", list(MESHES))
def test_coop_cg(oa, name, precision):
    mesh = MESHES[name]()
    say("coop cg", name, mesh.name, precision)
    A, H, b = _system(oa, mesh, 3)
    prec = oa.F64 if precision == "f64" else oa.F32
    outs, xs = [], []
    for kw in (dict(), dict(check_every=37), dict(cg_form=oa.CG_FORM_TWO)):
        x = torch.zeros(mesh.n_dof, dtype=torch.float64, device="cuda")
        outs.append(oa.pcg(A, T(b), x, rtol=1e-9, precision=prec, **kw))
        xs.append(x)
        assert outs[-1]["rc"] == 0
        # 1e-9 on the device's own residual; the host's differs by rounding
        assert np.linalg.norm(b - H @ x.cpu().numpy()) <= 1.001e-9 * np.linalg.norm(b)
    assert torch.equal(xs[0], xs[1]) and outs[0]["iters"] == outs[1]["iters"]
    assert abs(outs[0]["iters"] - outs[2]["iters"]) <= max(3, outs[2]["iters"] // 50)


def test_coop_cg_stops_at_maxit_and_on_nan(oa):
    mesh = synth.channel(17, 17, 13)
    say("coop cg maxit, nan", mesh.name)
    A, H, b = _system(oa, mesh, 4)
    x = torch.zeros(mesh.n_dof, dtype=torch.float64, device="cuda")
    out = oa.pcg(A, T(b), x, rtol=1e-9, maxit=7, raise_on=False)
    assert out["rc"] == oa.ENOTCONV and out["iters"] == 7
    two = torch.zeros_like(x)
    oa.pcg(A, T(b), two, rtol=1e-9, maxit=7, raise_on=False, cg_form=oa.CG_FORM_TWO)
    assert float((x - two).norm()) <= 1e-12 * float(two.norm())
    bad = b.copy()
    bad[1234] = np.nan
    x = torch.zeros_like(x)
    assert oa.pcg(A, T(bad), x, rtol=1e-9, raise_on=False)["rc"] == oa.ENAN
