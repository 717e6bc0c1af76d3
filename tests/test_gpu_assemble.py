"""The row-wise assembly (oasis_assemble_p1_ws, what the binding calls)
against the colour-wise one and the oracle: every form, in 2D and 3D, with
rows longer than the kernel's register slots, with a base matrix, in place,
and with an entry missing from the pattern (skipped by both)."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from gpu_util import T, csr_host, device_mesh, say
from oracle import p1
from test_gpu_graph import _fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


def _colour_wise(oa, dm, pat, form, uab, alpha, base):
    from paper_1602_03643_amd import _lib as L
    val = torch.empty(pat.nnz, dtype=torch.float64, device=pat.row_ptr.device)
    arr = (C.c_void_p * 3)(*[u.data_ptr() for u in uab] + [None] * (3 - len(uab)))
    A = pat.with_values(val).c()
    B = None if base is None else C.byref(pat.with_values(base).c())
    rc = L.load().oasis_assemble_p1(None, C.byref(dm.c()), form, arr, float(alpha), B, C.byref(A))
    assert rc == 0
    torch.cuda.synchronize()
    return val


@pytest.mark.parametrize("mesh", [_fan(5), _fan(15), _fan(16), _fan(40), synth.unit_square(7),
                                  synth.channel(9, 9, 7), synth.channel(18, 15, 12, displace_seed=2),
                                  synth.permute_mesh(synth.channel(17, 17, 13), 4)[0]], ids=lambda m: m.name)
def test_rows_match_colours_and_oracle(oa, mesh):
    say("assembly by rows", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    rng = np.random.default_rng(5)
    u = rng.normal(size=(mesh.dim, mesh.n_dof))
    uab = [T(v) for v in u]
    base = T(rng.normal(size=pat.nnz))
    geo = p1.element_geometry(mesh)
    H = csr_host(pat)
    K, Cm = p1.on_pattern(p1.stiffness_matrix(mesh, geo), H), p1.on_pattern(p1.convection_matrix(mesh, u, geo), H)
    forms = [oa.FORM_MASS, oa.FORM_STIFF, oa.FORM_GRAD_X, oa.FORM_GRAD_Y, oa.FORM_CONV]
    if mesh.dim == 3:
        forms.append(oa.FORM_GRAD_Z)
    for form in forms:
        for b in (None, base):
            ref = _colour_wise(oa, dm, pat, form, uab, -0.75, b).cpu().numpy()
            out = None if b is None else b.clone()
            val = oa.assemble_p1(dm, pat, form, uab=uab, alpha=-0.75, base=out, out=out).cpu().numpy()
            # sums of at most some 50 terms per entry
            assert np.abs(val - ref).max() <= 1e-14 * max(1.0, np.abs(ref).max())
        if form in (oa.FORM_STIFF, oa.FORM_CONV):
            want = base.cpu().numpy() - 0.75 * (K if form == oa.FORM_STIFF else Cm)
            assert np.linalg.norm(val - want) <= 1e-13 * np.linalg.norm(want)


def test_entries_outside_the_pattern_are_skipped(oa):
    mesh = synth.channel(9, 9, 7)
    say("assembly on a pattern with holes", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    full = oa.assemble_p1(dm, pat, oa.FORM_STIFF)
    rows = np.repeat(np.arange(mesh.n_dof), np.diff(pat.row_ptr.cpu().numpy()))
    keep = rows != pat.col_idx.cpu().numpy()                      # no diagonal
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=mesh.n_dof))])
    cut = oa.DeviceCSR(T(rp, torch.int32), pat.col_idx[torch.as_tensor(keep, device=full.device)].contiguous())
    assert torch.equal(oa.assemble_p1(dm, cut, oa.FORM_STIFF), full[torch.as_tensor(keep, device=full.device)])


def test_rows_out_of_column_order(oa):
    """A matrix whose rows list their columns backwards: the rows' entries are
    found one by one, and are those of the sorted matrix."""
    mesh = synth.channel(9, 9, 7)
    say("assembly on reversed rows", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    rp = pat.row_ptr.cpu().numpy()
    back = np.concatenate([np.arange(rp[i + 1] - 1, rp[i] - 1, -1) for i in range(mesh.n_dof)])
    rev = oa.DeviceCSR(pat.row_ptr, pat.col_idx[torch.as_tensor(back, device=pat.col_idx.device)].contiguous())
    u = [T(v) for v in np.random.default_rng(5).normal(size=(3, mesh.n_dof))]
    for form in (oa.FORM_MASS, oa.FORM_CONV):
        want = oa.assemble_p1(dm, pat, form, uab=u)[torch.as_tensor(back, device=pat.col_idx.device)]
        assert torch.equal(oa.assemble_p1(dm, rev, form, uab=u), want)


def test_cells_that_no_class_lists_are_left_out(oa):
    """A list that names one cell twice and another not at all: the first is
    added once, the second not, and no slot beside the table is written."""
    mesh = synth.channel(9, 9, 7)
    say("assembly with a cell missing", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    ref_mesh, _, _ = device_mesh(mesh)
    two = dm.color_cells[:2].cpu().numpy()
    dm.color_cells = dm.color_cells.clone()
    dm.color_cells[0] = dm.color_cells[1]
    one = oa.DeviceMesh(dm.dim, dm.coords, dm.cells[int(two[0])][None].contiguous(), dm.vert2dof, dm.n_dof,
                        np.array([0, 1], np.int32), T([0], torch.int32))
    uab = [T(v) for v in np.random.default_rng(7).normal(size=(3, mesh.n_dof))]
    for form in (oa.FORM_MASS, oa.FORM_STIFF, oa.FORM_CONV):
        whole = oa.assemble_p1(ref_mesh, pat, form, uab=uab).cpu().numpy()
        lost = _colour_wise(oa, one, pat, form, uab, 1.0, None).cpu().numpy()
        for _ in range(3):
            got = oa.assemble_p1(dm, pat, form, uab=uab).cpu().numpy()
            assert np.abs(got - (whole - lost)).max() <= 1e-14 * max(1.0, np.abs(whole).max())


def test_without_room_for_the_workspace(oa, monkeypatch):
    """The call that had needed no memory still succeeds when there is none for
    the rows' workspace: the colours one by one, bit for bit."""
    from paper_1602_03643_amd import api
    mesh = synth.channel(9, 9, 7)
    say("assembly without memory", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    uab = [T(v) for v in np.random.default_rng(7).normal(size=(3, mesh.n_dof))]
    ref = _colour_wise(oa, dm, pat, oa.FORM_CONV, uab, 0.5, None)

    def none(nbytes, device=None):
        raise torch.cuda.OutOfMemoryError("none left")

    monkeypatch.setattr(api, "_workspace", none)
    assert torch.equal(oa.assemble_p1(dm, pat, oa.FORM_CONV, uab=uab, alpha=0.5), ref)


def test_streams_of_other_kinds(oa):
    """Any object with a cuda_stream is a stream, as in the other calls."""
    mesh = synth.channel(9, 9, 7)
    say("assembly on streams", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    ref = oa.assemble_p1(dm, pat, oa.FORM_STIFF)
    s = torch.cuda.Stream()

    class Other:
        def __init__(self, p):
            self.cuda_stream = p

    torch.cuda.synchronize()
    for stream in (s, Other(s.cuda_stream), Other(0), torch.cuda.ExternalStream(s.cuda_stream), torch.cuda.default_stream()):
        out = torch.zeros(pat.nnz, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        oa.assemble_p1(dm, pat, oa.FORM_STIFF, out=out, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_captured(oa):
    """Under capture the workspace is the graph's; every replay gives the eager
    bits on the velocity of its time, with eager work and synchronisations
    between the replays."""
    mesh = synth.channel(9, 9, 7)
    say("assembly captured", mesh.name)
    dm, pat, _ = device_mesh(mesh)
    rng = np.random.default_rng(8)
    uab = [T(v) for v in rng.normal(size=(3, mesh.n_dof))]
    out = torch.zeros(pat.nnz, dtype=torch.float64, device="cuda")
    oa.assemble_p1(dm, pat, oa.FORM_CONV, uab=uab, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        oa.assemble_p1(dm, pat, oa.FORM_CONV, uab=uab, out=out)
    for _ in range(4):
        for u in uab:
            u.copy_(T(rng.normal(size=mesh.n_dof)))
        ref = oa.assemble_p1(dm, pat, oa.FORM_CONV, uab=uab)
        junk = [torch.full((50000,), 7, dtype=torch.int32, device="cuda") for _ in range(8)]
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and all(bool((j == 7).all()) for j in junk)
