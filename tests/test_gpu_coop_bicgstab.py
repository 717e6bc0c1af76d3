"""BiCGStab solves in one cooperative launch against the three-kernel form.

The meshes sit at the edges of the kernel's shapes (less than one block, one
row more than a block, the three block sizes, a full grid, one row too many,
a halo that does not fit), with one to three right-hand sides that stop at
different iterations: a rough one, one whose start is nearly the solution, a
zero one, one with a NaN.  A grid that the caller asks for selects the other
form.  Both are the same recurrences with partial sums in another order, so
the counts may differ by the few iterations that rounding moves a stopping
test; every solution meets the tolerance in a residual computed on the host
in FP64, with 0.1% for the rounding of the device's own.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import T, csr_host, device_mesh, say
from test_gpu_coop import MESHES

pytestmark = pytest.mark.gpu
RTOL = 1e-9


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


def _system(oa, mesh, seed):
    """The velocity matrix of a time step: mass, diffusion and convection."""
    dm, pat, _ = device_mesh(mesh)
    rng = np.random.default_rng(seed)
    base = oa.assemble_p1(dm, pat, oa.FORM_MASS, alpha=100.0)
    base = oa.assemble_p1(dm, pat, oa.FORM_STIFF, alpha=0.05, base=base)
    u = [T(rng.normal(size=mesh.n_dof)) for _ in range(dm.dim)]
    A = pat.with_values(oa.assemble_p1(dm, pat, oa.FORM_CONV, uab=u, alpha=0.5, base=base))
    return A, csr_host(pat, A.val), rng


def _both(oa, A, b, x0, **kw):
    res = []
    for cap in (0, 512):
        x = x0.clone()
        st = oa.bicgstab(A, b, x, rtol=RTOL, grid_cap=cap, raise_on=False, **kw)
        res.append((x, st))
    return res


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("nrhs", [1, 2, 3])
@pytest.mark.parametrize("name", list(MESHES))
def test_coop_bicgstab(oa, name, nrhs, precision):
    mesh = MESHES[name]()
    n = mesh.n_dof
    say("coop bicgstab", name, mesh.name, nrhs, precision)
    A, H, rng = _system(oa, mesh, 3)
    prec = oa.F64 if precision == "f64" else oa.F32
    b, x0 = rng.normal(size=(nrhs, n)), np.zeros((nrhs, n))
    if nrhs > 1:      # a start one part in a million from the solution: stops early
        sol = rng.normal(size=n)
        b[1], x0[1] = H @ sol, sol * (1 + 1e-6 * rng.normal(size=n))
    if nrhs > 2:
        b[2] = 0.0
    (x, st), (y, gen) = _both(oa, A, T(b), T(x0), precision=prec)
    for k in range(nrhs):
        assert st[k]["rc"] == gen[k]["rc"] == 0 and st[k]["status"] == gen[k]["status"] == 0
        assert np.linalg.norm(b[k] - H @ x[k].cpu().numpy()) <= 1.001 * RTOL * np.linalg.norm(b[k])
        assert abs(st[k]["iters"] - gen[k]["iters"]) <= max(2, gen[k]["iters"] // 10)
    if nrhs > 2:
        assert torch.count_nonzero(x[2]) == 0


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_coop_bicgstab_iteration_cap_and_nan(oa, precision):
    mesh = synth.channel(17, 17, 13)
    n = mesh.n_dof
    say("coop bicgstab maxit, nan", mesh.name, precision)
    prec = oa.F64 if precision == "f64" else oa.F32
    A, H, rng = _system(oa, mesh, 5)
    b, x0 = rng.normal(size=(3, n)), np.zeros((3, n))
    (x, st), (y, gen) = _both(oa, A, T(b), T(x0), precision=prec, maxit=3)
    assert [s["status"] for s in st] == [g["status"] for g in gen] == [oa.ENOTCONV] * 3
    assert [s["iters"] for s in st] == [g["iters"] for g in gen]
    if precision == "f64":
        assert float((x - y).norm()) <= 1e-11 * float(y.norm())
    b[1, 77] = np.nan
    (x, st), (y, gen) = _both(oa, A, T(b), T(x0), precision=prec)
    assert [s["status"] for s in st] == [g["status"] for g in gen]
    assert st[1]["status"] == oa.ENAN
    for k in (0, 2):
        if gen[k]["status"] == 0:
            assert np.linalg.norm(b[k] - H @ x[k].cpu().numpy()) <= 1.001 * RTOL * np.linalg.norm(b[k])
