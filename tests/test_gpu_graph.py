"""Graph set-up at the edges of its kernels' shapes, bit for bit against the
oracle: rows with more neighbours than the row kernel keeps in LDS, colours
in both halves of the 128-colour mask and one too many, several components
(with one-cell ones), more levels than a batch holds, and priorities that
are not distinct."""
import numpy as np
import pytest

import synth
from gpu_util import T, dev, device_mesh, say
from oracle import graph
from synth.meshes import Mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_1602_03643_amd as m
    return m


def _mesh(coords, cells, name):
    n = len(coords)
    coords = np.asarray(coords, dtype=np.float64)
    return Mesh(2, coords, np.asarray(cells, dtype=np.int32), np.arange(n, dtype=np.int32), n,
                np.zeros(0, np.int32), coords.copy(), name=name)


def _fan(k):
    """k triangles around one vertex: a row of k + 1 entries, k colours."""
    a = 2 * np.pi * np.arange(k) / k
    return _mesh(np.concatenate([[[0, 0]], np.stack([np.cos(a), np.sin(a)], 1)]),
                 [[0, 1 + i, 1 + (i + 1) % k] for i in range(k)], "fan_%d" % k)


def _parts():
    """A square, a long strip (more levels than a batch of 16) and three
    triangles of their own, renumbered at random."""
    a = synth.unit_square(6)
    xs, cells, n = [a.coords], [a.cells], a.n_vert
    strip = np.array([[i, j] for i in range(60) for j in range(2)], dtype=float)
    quads = [[2 * i, 2 * i + 2, 2 * i + 3] for i in range(59)] + [[2 * i, 2 * i + 3, 2 * i + 1] for i in range(59)]
    xs.append(strip + 100)
    cells.append(np.array(quads) + n)
    n += len(strip)
    for q in range(3):
        xs.append(np.array([[0, 0], [1, 0], [0, 1]], dtype=float) + 200 + 10 * q)
        cells.append(np.array([[n, n + 1, n + 2]]))
        n += 3
    return synth.permute_mesh(_mesh(np.concatenate(xs), np.concatenate(cells), "parts"), 5)[0]


@pytest.mark.parametrize("mesh", [_fan(31), _fan(32), _fan(64), _fan(65), _fan(128), _parts(),
                                  synth.permute_mesh(synth.channel(9, 9, 7), 2)[0]], ids=lambda m: m.name)
def test_graph_set_up_matches_oracle(oa, mesh):
    say("graph set-up", mesh.name)
    dm, pat, color = device_mesh(mesh)
    rp, ci = graph.csr_pattern(mesh)
    assert np.array_equal(pat.row_ptr.cpu().numpy(), rp) and np.array_equal(pat.col_idx.cpu().numpy(), ci)
    ref = graph.greedy_coloring(mesh, synth.cell_priorities(mesh.n_cell, 7))
    assert np.array_equal(color.cpu().numpy(), ref)
    cptr, cells = graph.color_classes(ref)
    assert np.array_equal(dm.color_ptr, cptr) and np.array_equal(dm.color_cells.cpu().numpy(), cells)
    perm, order = oa.rcm(pat)
    o_ref, p_ref = graph.rcm(rp, ci)
    assert np.array_equal(order.cpu().numpy(), o_ref) and np.array_equal(perm.cpu().numpy(), p_ref)


def test_too_many_colours_and_equal_priorities_are_refused(oa):
    import torch
    for mesh, pri in ((_fan(129), np.arange(129)), (_fan(40), np.zeros(40))):
        say("colouring refused", mesh.name)
        dm = oa.DeviceMesh.from_arrays(2, mesh.coords, mesh.cells, mesh.vert2dof, mesh.n_dof, dev())
        with pytest.raises(oa.OasisError):
            oa.color_cells(dm, T(pri, torch.int32))


def test_pattern_in_one_call_and_in_two(oa):
    """oasis_p1_pattern with col_idx against the binding's count and columns."""
    import ctypes as C
    import torch
    from paper_1602_03643_amd import _lib as L
    mesh = synth.permute_mesh(synth.channel(9, 9, 7), 2)[0]
    say("pattern in one call", mesh.name)
    dm = oa.DeviceMesh.from_arrays(mesh.dim, mesh.coords, mesh.cells, mesh.vert2dof, mesh.n_dof, dev())
    pat, cm, nb, nnz = oa.p1_pattern(dm), dm.c(), C.c_size_t(), C.c_int32()
    assert L.load().oasis_graph_workspace_size(C.byref(cm), C.byref(nb)) == 0
    ws = torch.empty(nb.value, dtype=torch.uint8, device=dev())
    rp, ci = torch.empty_like(pat.row_ptr), torch.empty_like(pat.col_idx)
    ptr = lambda t: C.c_void_p(t.data_ptr())                            # noqa: E731
    assert L.load().oasis_p1_pattern(None, C.byref(cm), ptr(rp), ptr(ci), ci.numel(), C.byref(nnz), ptr(ws),
                                     ws.numel()) == 0
    assert torch.equal(rp, pat.row_ptr) and torch.equal(ci, pat.col_idx) and nnz.value == ci.numel()


def test_cells_with_a_dof_twice_are_refused(oa):
    """The kernels count on distinct dofs within a cell: pattern and colouring
    refuse a mesh where two vertices of one share theirs, or an index is out of
    range."""
    import torch
    mesh = synth.unit_square(3)
    for v2d, code in ((np.minimum(mesh.vert2dof, mesh.n_dof - 5), oa.EUNSUPPORTED),
                      (mesh.vert2dof + 1, oa.EINVAL), (mesh.vert2dof - 1, oa.EINVAL)):
        dm = oa.DeviceMesh.from_arrays(2, mesh.coords, mesh.cells, v2d.astype(np.int32), mesh.n_dof, dev())
        for call in (lambda: oa.p1_pattern(dm),
                     lambda: oa.color_cells(dm, T(np.arange(mesh.n_cell), torch.int32))):
            with pytest.raises(oa.OasisError) as e:
                call()
            assert e.value.code == code
    dm = oa.DeviceMesh.from_arrays(2, mesh.coords, mesh.cells, mesh.vert2dof, mesh.n_dof, dev())
    assert oa.p1_pattern(dm).n == mesh.n_dof
