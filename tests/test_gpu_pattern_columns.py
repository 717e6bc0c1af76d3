"""oasis_p1_pattern_columns checks what it is given: the room for the columns,
whose lists the workspace holds, and that row_ptr is theirs.  Wrong ones get
EINVAL, and no column beyond the room is written.  Rows that fit the row
kernel's LDS (a box) and one that does not (40 triangles around a vertex)."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from gpu_util import T, dev, say
from test_gpu_graph import _fan

pytestmark = pytest.mark.gpu
GUARD = -77


class _Calls:
    """The two calls of a mesh on one workspace."""

    def __init__(self, mesh):
        import paper_1602_03643_amd as oa
        from paper_1602_03643_amd import _lib as L
        self.L, self.lib = L, L.load()
        self.dm = oa.DeviceMesh.from_arrays(mesh.dim, mesh.coords, mesh.cells, mesh.vert2dof, mesh.n_dof, dev())
        self.c, nb = self.dm.c(), C.c_size_t()
        assert self.lib.oasis_graph_workspace_size(C.byref(self.c), C.byref(nb)) == 0
        self.ws = torch.zeros(nb.value, dtype=torch.uint8, device=dev())
        self.rp = torch.empty(mesh.n_dof + 1, dtype=torch.int32, device=dev())
        self.pat = oa.p1_pattern(self.dm)
        torch.cuda.synchronize()

    def count(self):
        nnz = C.c_int32()
        assert self.lib.oasis_p1_pattern(None, C.byref(self.c), self.rp.data_ptr(), None, 0, C.byref(nnz),
                                         self.ws.data_ptr(), self.ws.numel()) == 0
        return nnz.value

    def columns(self, room, rp=None):
        """The status, and the columns in a buffer longer than `room` says."""
        col = torch.full((self.pat.nnz + 64,), GUARD, dtype=torch.int32, device=dev())
        torch.cuda.synchronize()
        rc = self.lib.oasis_p1_pattern_columns(None, C.byref(self.c), (self.rp if rp is None else rp).data_ptr(),
                                               col.data_ptr(), room, self.ws.data_ptr(), self.ws.numel())
        return rc, col.cpu().numpy()


@pytest.mark.parametrize("mesh", [synth.permute_mesh(synth.channel(9, 9, 7), 2)[0], _fan(40)], ids=lambda m: m.name)
def test_columns_are_checked(mesh):
    say("pattern columns", mesh.name)
    k = _Calls(mesh)
    bad, ref = k.L.EINVAL, k.pat.col_idx.cpu().numpy()
    assert k.columns(ref.size, k.pat.row_ptr)[0] == bad           # no lists yet
    nnz = k.count()
    assert nnz == ref.size
    for room in (0, nnz - 1, nnz // 2):
        rc, col = k.columns(room)
        assert rc == bad and np.all(col[room:] == GUARD), room
    rc, col = k.columns(nnz)                                      # the refusals took nothing away
    assert rc == 0 and np.array_equal(col[:nnz], ref) and np.all(col[nnz:] == GUARD)
    for wrong in (torch.zeros_like(k.rp), k.rp.flip(0), k.rp + 3, torch.clamp(k.rp - 1, min=0)):
        rc, col = k.columns(nnz, wrong.contiguous())
        assert rc == bad and np.all(col[nnz:] == GUARD)
    # the workspace after something else used it
    pri = T(synth.cell_priorities(mesh.n_cell, 7), torch.int32)
    color, nc = torch.empty(mesh.n_cell, dtype=torch.int32, device=dev()), C.c_int32()
    torch.cuda.synchronize()
    assert k.lib.oasis_color_cells(None, C.byref(k.c), pri.data_ptr(), color.data_ptr(), C.byref(nc), k.ws.data_ptr(),
                                   k.ws.numel()) == 0
    assert k.columns(nnz)[0] == bad
    k.count()
    cptr, cells = (C.c_int32 * (nc.value + 1))(), torch.empty_like(color)
    assert k.lib.oasis_color_classes(None, mesh.n_cell, color.data_ptr(), nc.value, cptr, cells.data_ptr(),
                                     k.ws.data_ptr(), k.ws.numel()) == 0
    assert k.columns(nnz)[0] == bad
    assert k.count() == nnz and k.columns(nnz)[0] == 0
