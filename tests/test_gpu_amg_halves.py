"""The cycle on levels where its two halves are multiplied out, and on a
hierarchy where the first coarse level is too large for that, against the
oracle's smoothing, restriction, prolongation and smoothing on the same
levels.  The same linear maps in another order of operations: the tolerances
are those of the two-level cycle's parity test, 1e-12 and 2e-5 relative for
FP64 and FP32 (a few hundred roundings of 1e-16 and 6e-8)."""
import time

import numpy as np
import pytest

import synth
from gpu_util import T, device_mesh, rel, say
from oracle import amg
from test_gpu_amg import _device_amg, _oracle_hierarchy

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("storage", ["auto", "csr"])
@pytest.mark.parametrize("coarse", [4, 40])
@pytest.mark.parametrize("mesh", [lambda: synth.channel(17, 17, 13), lambda: synth.unit_square(48),
                                  lambda: synth.permute_mesh(synth.channel(17, 17, 13), 2000)[0]])
def test_multiplied_out_levels(oa, mesh, coarse, storage, precision):
    mesh = mesh()
    say("amg halves", mesh.name, coarse, storage, precision)
    h, _, _, keep = _device_amg(oa, mesh, oa.F64 if precision == "f64" else oa.F32, coarse_size=coarse,
                                storage=oa.STORAGE_AUTO if storage == "auto" else oa.STORAGE_CSR)
    assert h.n_levels() > 2
    H = _oracle_hierarchy([h.level(l) for l in range(h.n_levels())])
    rng = np.random.default_rng(9)
    for _ in range(2):
        r = rng.normal(size=mesh.n_dof)
        assert rel(h.vcycle(T(r)).cpu().numpy(), amg.vcycle(H, r)) <= (1e-12 if precision == "f64" else 2e-5)


def test_large_first_coarse_level(oa):
    t = time.time()
    mesh = synth.channel(113, 113, 97)
    dm, pat, _ = device_mesh(mesh)
    A = pat.with_values(oa.assemble_p1(dm, pat, oa.FORM_STIFF, base=oa.assemble_p1(dm, pat, oa.FORM_MASS, alpha=0.1)))
    h = oa.AMG(A, None, precision=oa.F32)
    H = _oracle_hierarchy([h.level(l) for l in range(h.n_levels())])
    say("amg large", mesh.n_dof, h.n_levels(), "%.1f s" % (time.time() - t))
    r = np.random.default_rng(3).normal(size=mesh.n_dof)
    assert rel(h.vcycle(T(r)).cpu().numpy(), amg.vcycle(H, r)) <= 2e-5
