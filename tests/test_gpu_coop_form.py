"""Which kernels a solve took (coop_runs, coop_lost), and BiCGStab solves in
one cooperative launch through every part of that kernel.

The meshes are those at the edges of the cooperative kernels' shapes; a
randomly numbered one of 25,600 rows (a halo of about 3,500 entries where
2,048 fit) stands for those that do not fit, which is known before the solve:
no launch of theirs is lost.  BiCGStab solves take the
cooperative form up to an iteration cap of 4096, which the calls therefore
lower from the default.  Both forms are the same recurrences with partial
sums in another order, so the counts may differ by the few iterations that
rounding moves a stopping test; every solution meets the tolerance in a
residual computed on the host in FP64, with 0.1% for the rounding of the
device's own.
"""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import synth
from gpu_util import T, say
from test_gpu_coop import MESHES, _system as _spd
from test_gpu_coop_bicgstab import _system

pytestmark = pytest.mark.gpu
RTOL = 1e-9
FORMS = {name: (make, name not in ("too large", "halo too wide")) for name, make in MESHES.items()}
FORMS["halo too wide"] = (lambda: synth.permute_mesh(synth.channel(33, 33, 25), 9)[0], False)


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name", list(FORMS))
def test_cg_form_is_the_expected_one(oa, name, precision):
    make, coop = FORMS[name]
    mesh = make()
    say("cg form", name, mesh.name, precision)
    A, H, b = _spd(oa, mesh, 3)
    prec = oa.F64 if precision == "f64" else oa.F32
    for kw, want in ((dict(), coop), (dict(cg_form=oa.CG_FORM_TWO), False), (dict(grid_cap=512), False)):
        x = torch.zeros(mesh.n_dof, dtype=torch.float64, device="cuda")
        st = oa.pcg(A, T(b), x, rtol=RTOL, precision=prec, **kw)
        assert (st["coop_runs"] > 0) == want and st["coop_lost"] == 0, (kw, st)
        assert np.linalg.norm(b - H @ x.cpu().numpy()) <= 1.001 * RTOL * np.linalg.norm(b)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("nrhs", [1, 2, 3])
@pytest.mark.parametrize("name", list(FORMS))
def test_bicgstab_coop_against_launched(oa, name, nrhs, precision):
    make, coop = FORMS[name]
    mesh = make()
    n = mesh.n_dof
    say("bicgstab form", name, mesh.name, nrhs, precision)
    A, H, rng = _system(oa, mesh, 3)
    prec = oa.F64 if precision == "f64" else oa.F32
    b, x0 = rng.normal(size=(nrhs, n)), np.zeros((nrhs, n))
    if nrhs > 1:      # a start one part in a million from the solution: stops early
        sol = rng.normal(size=n)
        b[1], x0[1] = H @ sol, sol * (1 + 1e-6 * rng.normal(size=n))
    if nrhs > 2:
        b[2] = 0.0
    res = []
    for cap in (0, 512):
        x = T(x0)
        st = oa.bicgstab(A, T(b), x, rtol=RTOL, precision=prec, maxit=4000, grid_cap=cap, raise_on=False)
        res.append((x.cpu().numpy(), st))
        want = coop and cap == 0
        assert all((s["coop_runs"] > 0) == want for s in st if s["iters"] > 0), (cap, st)
        assert st[0]["coop_lost"] == 0, (cap, st)
    (x, st), (y, gen) = res
    for k in range(nrhs):
        assert st[k]["rc"] == gen[k]["rc"] == 0 and st[k]["status"] == gen[k]["status"] == 0
        assert np.linalg.norm(b[k] - H @ x[k]) <= 1.001 * RTOL * np.linalg.norm(b[k])
        assert abs(st[k]["iters"] - gen[k]["iters"]) <= max(2, gen[k]["iters"] // 10)
    if nrhs > 2:
        assert not np.any(x[2])


def test_bicgstab_coop_breakdown_and_nan(oa):
    """Two-by-two blocks [[1, -5/4], [-5/4, 1]] and b = (1, 2, 1, 2, ...):
    r_hat . A r is exactly zero at the start and again after the restart;
    beside it a right-hand side that converges and one with a NaN.  Both
    forms must say the same."""
    n = 3000
    say("bicgstab coop breakdown, nan")
    H = sp.block_diag([np.array([[1.0, -1.25], [-1.25, 1.0]])] * (n // 2), format="csr")
    H.sort_indices()
    A = oa.DeviceCSR(T(H.indptr, torch.int32), T(H.indices, torch.int32), T(H.data))
    rng = np.random.default_rng(4)
    b = np.stack([np.tile([1.0, 2.0], n // 2), rng.normal(size=n), rng.normal(size=n)])
    for nan in (False, True):
        if nan:
            b[2, 777] = np.nan
        got = []
        for cap in (0, 512):
            x = torch.zeros((3, n), dtype=torch.float64, device="cuda")
            st = oa.bicgstab(A, T(b), x, rtol=RTOL, maxit=50, grid_cap=cap, raise_on=False)
            got.append([(s["status"], s["iters"], s["restarts"]) for s in st])
            assert all(s["coop_runs"] == (1 if cap == 0 else 0) for s in st)
            assert np.linalg.norm(b[1] - H @ x[1].cpu().numpy()) <= 1.001 * RTOL * np.linalg.norm(b[1])
        assert got[0] == got[1], got
        assert got[0][0][0] == oa.EBREAKDOWN and got[0][0][2] == 1 and got[0][1][0] == oa.OK
        assert got[0][2][0] == (oa.ENAN if nan else oa.OK)


def test_step_counts_its_runs(oa):
    """A step with a scalar and an iteration cap that both solvers' cooperative
    forms take: one run for the velocity, at least one for the pressure, one
    for the scalar; none where the caller gives the grid."""
    from gpu_util import device_mesh
    mesh = synth.channel(9, 9, 7)
    say("step form", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    n = mesh.n_dof
    for cap, runs in ((0, 3), (512, 0)):
        h = oa.IPCS(dm, pat, 0.01, 0.01, (1.0, 0.0, 0.0), T(mesh.bc_dofs, torch.int32), maxit=4000, diffusivity=[0.02],
                    grid_cap=cap)
        z = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")     # noqa: E731
        c = T(np.random.default_rng(1).normal(size=(1, n)))
        st = h.step(z(3, n), z(3, n), z(3, n), z(n), z(n), bc_values=z(3, mesh.bc_dofs.size), C1=c, Cn=z(1, n),
                    C_bc=z(1, mesh.bc_dofs.size))
        assert st["status"] == 0 and st["coop_lost"] == 0
        assert st["coop_runs"] >= runs if runs else st["coop_runs"] == 0, st


def _bicgstab(oa, A, b, x0, prec, flags=0, **kw):
    """oa.bicgstab with flags of its own."""
    import ctypes as C
    from paper_1602_03643_amd import _lib as L
    x = x0.clone()
    o = L.KrylovOpts(RTOL, kw.get("maxit", 4000), prec, 1e-4, 50, 0, flags, L.Tuning(0, kw.get("grid_cap", 0), 0))
    nb = C.c_size_t()
    assert L.load().oasis_krylov_workspace_size(A.n, A.nnz, b.shape[0], C.byref(o), C.byref(nb)) == 0
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    st = (L.KrylovStats * b.shape[0])()
    ptr = lambda t: C.c_void_p(t.data_ptr())                            # noqa: E731
    rc = L.load().oasis_bicgstab(None, C.byref(A.c()), b.shape[0], ptr(b), ptr(x), C.byref(o), ptr(ws), ws.numel(), st)
    return rc, x, st


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("mesh", [lambda: synth.channel(17, 17, 13), lambda: synth.channel(49, 45, 41),
                                  lambda: synth.channel(65, 64, 65)])
def test_bicgstab_after_a_lost_wait(oa, mesh, precision):
    """A wait lost in the first sum, in products, in sums and late in the solve.
    The repeat, and after too many of them the launched form, must start from
    the caller's iterate: results are those of an undisturbed solve, bit for
    bit, whatever the lost launches had done to x."""
    mesh = mesh()
    say("bicgstab lost wait", mesh.name, precision)
    prec = oa.F64 if precision == "f64" else oa.F32
    A, H, rng = _system(oa, mesh, 6)
    b, x0 = T(rng.normal(size=(2, mesh.n_dof))), T(rng.normal(size=(2, mesh.n_dof)))
    torch.cuda.synchronize()
    refs = []
    for always, cap in ((0, 0), (1, 512)):
        rc, x, st = _bicgstab(oa, A, b, x0, prec, grid_cap=cap)
        assert rc == 0 and (st[0].coop_runs == 0) == (always == 1) and st[0].coop_lost == 0
        refs.append((x, [s.iters for s in st]))
    for k in (1, 2, 3, 4, 5, 6, 7, 16, 17, 18):
        for always, (ref, iters) in enumerate(refs):
            rc, x, st = _bicgstab(oa, A, b, x0, prec, flags=(k + (always << 14)) << 16)
            # once for each solve (the refinement steps of FP32), or every time:
            # six launches that do not come together, two that lose a later wait
            lost = [6 if k == 1 else 2] if always else range(1, 1 + max(1, st[0].outer_iters))
            assert rc == 0 and all(s.coop_lost in lost and (s.coop_runs > 0) == (not always) for s in st), (k, always)
            assert torch.equal(x, ref) and [s.iters for s in st] == iters, (k, always)


def _pcg(oa, A, b, prec, flags=0):
    """oa.pcg from zero with flags of its own."""
    import ctypes as C
    from paper_1602_03643_amd import _lib as L
    x = torch.zeros_like(b)
    o = L.KrylovOpts(RTOL, 4000, prec, 0.1, 50, 0, flags, L.Tuning(0, 0, 0))
    nb = C.c_size_t()
    assert L.load().oasis_krylov_workspace_size(A.n, A.nnz, 1, C.byref(o), C.byref(nb)) == 0
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    st = L.KrylovStats()
    ptr = lambda t: C.c_void_p(t.data_ptr())                            # noqa: E731
    rc = L.load().oasis_pcg(None, C.byref(A.c()), ptr(b), ptr(x), C.byref(o), ptr(ws), ws.numel(), C.byref(st))
    return rc, x, st


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("mesh", [lambda: synth.channel(17, 17, 13), lambda: synth.channel(49, 45, 41),
                                  lambda: synth.channel(65, 64, 65)])
def test_cg_after_a_lost_wait(oa, mesh, precision):
    """Waits lost in the first exchanges, later, and in the one in which the
    others see convergence: the launch must not count, and the solve still
    meets its tolerance."""
    mesh = mesh()
    say("cg lost wait", mesh.name, precision)
    prec = oa.F64 if precision == "f64" else oa.F32
    A, H, b = _spd(oa, mesh, 6)
    B = T(b)
    torch.cuda.synchronize()
    rc, first, ref = _pcg(oa, A, B, prec)
    assert rc == 0 and ref.coop_runs > 0 and ref.coop_lost == 0
    # a mixed solve's first launch ends when the residual has fallen tenfold
    last = [2 * ref.iters + 1] * 4 if precision == "f64" else []
    for k in [2, 3, 4, 9, 10, (1 << 14) + 1] + last:
        rc, x, st = _pcg(oa, A, B, prec, flags=k << 16)
        assert rc == 0 and st.coop_lost == (6 if k >> 14 else 1) and st.coop_runs == 0, (k, st.coop_lost, st.coop_runs)
        assert np.linalg.norm(b - H @ x.cpu().numpy()) <= 1.001 * RTOL * np.linalg.norm(b), k
        assert abs(st.iters - ref.iters) <= max(3, ref.iters // 10) + (k & 0x3fff) // 2
    # a grid that does not come together has changed nothing and is launched again
    rc, y, st = _pcg(oa, A, B, prec, flags=1 << 16)
    assert rc == 0 and st.coop_runs == ref.coop_runs and st.coop_lost == (1 if precision == "f64" else ref.coop_runs)
    assert torch.equal(y, first) and st.iters == ref.iters


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_timed_launches_are_those_of_the_header(oa, precision):
    """OASIS_KRYLOV_TIME repeats the single-reduction pass in FP32 and the
    product of the two-kernel form in FP64, also after cooperative runs (of
    which it leaves the iterates alone): the times are those of the calls that
    ask for that form, within a fifth.  The other form's launch takes under
    three quarters or over five quarters of it."""
    mesh = synth.channel(65, 64, 65)
    say("timed launches", mesh.name, precision)
    A, H, b = _spd(oa, mesh, 8)
    b = T(b)
    prec = oa.F64 if precision == "f64" else oa.F32

    def timed(**kw):
        x, best = torch.zeros_like(b), []
        for _ in range(5):
            x.zero_()
            st = oa.pcg(A, b, x, rtol=1e-30, maxit=200, precision=prec, time_kernel=True, raise_on=False, **kw)
            assert st["status"] == oa.ENOTCONV and st["kernel_count"] == 200
            best.append(st["kernel_ms"] / 200)
        return sorted(best)[2], st["coop_runs"], x

    us, runs, x = timed()
    two, single = timed(cg_form=oa.CG_FORM_TWO), timed(cg_form=oa.CG_FORM_SINGLE)
    say("us: here %.2f, two %.2f, single %.2f" % (1e3 * us, 1e3 * two[0], 1e3 * single[0]))
    want, other = (two[0], single[0]) if precision == "f64" else (single[0], two[0])
    assert runs > 0 and two[1] == single[1] == 0
    assert not 0.75 <= other / want <= 1.25
    assert abs(us / want - 1) <= 0.2


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("check", [1, 4, 16, 40])
def test_polls_of_cooperative_runs(oa, check, precision):
    """However often the caller asks for polls, a run is not cut into pieces of
    fewer than 16 iterations, and the result is that without polls, bit for
    bit."""
    mesh = synth.channel(17, 17, 13)
    say("polls", mesh.name, check, precision)
    A, H, b = _spd(oa, mesh, 9)
    prec = oa.F64 if precision == "f64" else oa.F32
    x, y = (torch.zeros(mesh.n_dof, dtype=torch.float64, device="cuda") for _ in range(2))
    one = oa.pcg(A, T(b), x, rtol=RTOL, precision=prec)
    st = oa.pcg(A, T(b), y, rtol=RTOL, precision=prec, check_every=check)
    assert torch.equal(x, y) and st["iters"] == one["iters"] and st["coop_lost"] == 0
    assert one["coop_runs"] <= st["coop_runs"] <= one["coop_runs"] + st["iters"] // max(check, 16)
