"""The work that users of this framework have it do, as timed cases.

A case is one call sequence through the package's public entry points, on
synthetic inputs made on the device from a seed:

  step      one IPCS time step (IPCS.step), from given velocity, pressure and
            correction fields: what a simulation runs all the time
  pcg       a stand-alone pressure-type solve (pcg, or AMG.pcg on a kept handle)
  bicgstab  a stand-alone solve of the convection-diffusion matrix for up to
            three right-hand sides
  assemble  one convection matrix on a kept pattern (assemble_p1)
  spmv      one sparse product
  graph     what every new mesh needs once: pattern, reverse Cuthill-McKee
            reordering, pattern of the reordered mesh, cell colouring
  mpnn      one training step of the warm-start network (forward, backward, Adam)

The meshes are those of the tests and of bench.py: the Taylor-Green square
(right triangles, Dirichlet all round) and the wall-stretched channel box
(Kuhn-split hexahedra, periodic in x and z, no-slip walls); `order` is
"grid" for the structured numbering, "local" for one that a reordered
unstructured mesh has (dofs shuffled among near neighbours, cells and
vertices in random order, nodes displaced) and "random" for a raw
unstructured one.  Solves run to tolerances (`_rtol`) at which two correct
solvers' fields agree to about ten digits.

`exact` solves the same discrete equations in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

NU, DT = 1.0 / 180.0, 0.01
MAXIT = 4000


def _rtol(case):
    """Tight, and still above what rounding leaves reachable at that size."""
    if case["mesh"] == "square":
        return 1e-13 if case["nx"] <= 40 else 3e-13
    return 1e-12 if case["nx"] * case["ny"] * case["nz"] <= 60000 else 1e-11


def listed():
    step = dict(kind="step", order="grid", mixed=False, amg=False, inner=1, update="lumped", scalars=0,
                convection="abcn")
    return [
        # the verification problem of every scheme change: 1089 nodes, thousands of steps, latency only
        dict(step, name="step_tg32_f64", mesh="square", nx=32, ny=32, nz=0),
        # a unit-test or parameter-study channel with the scheme's options on
        dict(step, name="step_ch17_f64_options", mesh="channel", nx=17, ny=17, nz=13, inner=2, update="consistent",
             scalars=1),
        # a coarse run in mixed precision, Jacobi preconditioning, explicit convection
        dict(step, name="step_ch33_mixed_abe", mesh="channel", nx=33, ny=33, nz=25, mixed=True, convection="abe"),
        # the plain FP64 channel run that others are judged by
        dict(step, name="step_ch65_f64", mesh="channel", nx=65, ny=65, nz=49),
        # an unstructured-like mesh of odd size with a scalar, all in FP64
        dict(step, name="step_local57_f64_amg", mesh="channel", order="local", nx=57, ny=47, nz=41, amg=True,
             scalars=1, update="gradient"),
        # the production run: 1.6 million nodes, mixed precision, multigrid
        dict(step, name="step_ch129_mixed_amg", mesh="channel", nx=129, ny=129, nz=97, mixed=True, amg=True),
        # a caller with a pressure matrix and right-hand sides of its own
        dict(kind="pcg", name="pcg_ch65_mixed", mesh="channel", order="grid", nx=65, ny=65, nz=49, mixed=True,
             amg=False),
        # the velocity systems of another time integrator, three components at once
        dict(kind="bicgstab", name="bicgstab_ch81_f64x3", mesh="channel", order="grid", nx=81, ny=71, nz=61,
             mixed=False, nrhs=3),
        # a caller's own time integrator: the convection matrix of each step
        dict(kind="assemble", name="assemble_ch97_conv", mesh="channel", order="grid", nx=97, ny=97, nz=73),
        # the product alone, as in any outer iteration written in Python
        dict(kind="spmv", name="spmv_local101_f32", mesh="channel", order="local", nx=101, ny=87, nz=73, dtype="f32"),
        # a new unstructured mesh arrives in random order
        dict(kind="graph", name="graph_random57", mesh="channel", order="random", nx=57, ny=51, nz=45),
        # training the warm-start network on its usual mesh
        dict(kind="mpnn", name="mpnn_train_ch65", mesh="channel", order="grid", nx=65, ny=65, nz=49, loss="knorm"),
    ]


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm, odd ones
    among them; slow solver choices (FP64 or Jacobi) on meshes up to 200,000
    nodes, the production choices on all."""
    kind = rng.choice(["step"] * 6 + ["pcg", "pcg", "bicgstab", "assemble", "spmv", "graph", "mpnn"])
    if kind == "step" and rng.random() < 0.2:
        n = int(round(math.exp(rng.uniform(math.log(8), math.log(64)))))
        return dict(kind="step", mesh="square", order="grid", nx=n, ny=n, nz=0, mixed=rng.random() < 0.5, amg=False,
                    inner=rng.choice([1, 1, 2]), update=rng.choice(["lumped", "consistent"]), scalars=rng.choice([0, 1]),
                    convection=rng.choice(["abcn", "abe"]))
    mixed, amg = rng.random() < 0.6, rng.random() < 0.6
    production = kind in ("assemble", "spmv") or (kind == "step" and mixed and amg)
    top = 1.2e6 if production else 2.0e5
    n = math.exp(rng.uniform(math.log(700.0), math.log(top)))
    h = (n / (1.0 * 1.0 * 0.75)) ** (1.0 / 3.0)
    nx, ny, nz = (max(6, int(round(h * f * rng.uniform(0.85, 1.15)))) for f in (1.0, 1.0, 0.75))
    case = dict(kind=kind, mesh="channel", order=rng.choice(["grid", "grid", "local"]), nx=nx, ny=ny, nz=nz)
    if kind == "step":
        case.update(mixed=mixed, amg=amg, inner=rng.choice([1, 1, 1, 2]),
                    update=rng.choice(["lumped", "lumped", "consistent", "gradient"]),
                    scalars=rng.choice([0, 0, 1]), convection=rng.choice(["abcn", "abcn", "abe"]))
    elif kind == "pcg":
        case.update(mixed=mixed, amg=amg)
    elif kind == "bicgstab":
        case.update(mixed=mixed, nrhs=rng.choice([1, 2, 3]))
    elif kind == "spmv":
        case.update(dtype=rng.choice(["f32", "f64"]))
    elif kind == "graph":
        case.update(order=rng.choice(["grid", "random"]))
    elif kind == "mpnn":
        case.update(loss=rng.choice(["mse", "knorm"]))
    return case


# ---------------------------------------------------------------------------
# meshes and fields (plain torch, on the device)

def _device():
    return torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")


def _gen(seed):
    return torch.Generator().manual_seed(int(seed))


class _Mesh:
    pass


def _square(n, dev):
    m = _Mesh()
    m.dim = 2
    g = torch.arange(n + 1, dtype=torch.float64, device=dev) / n
    m.coords = torch.stack([g.repeat(n + 1), g.repeat_interleave(n + 1)], 1).contiguous()
    i = torch.arange(n, device=dev).repeat(n)
    j = torch.arange(n, device=dev).repeat_interleave(n)

    def v(a, b):
        return a + (n + 1) * b
    m.cells = torch.cat([torch.stack([v(i, j), v(i + 1, j), v(i + 1, j + 1)], 1),
                         torch.stack([v(i, j), v(i + 1, j + 1), v(i, j + 1)], 1)]).to(torch.int32).contiguous()
    m.n = (n + 1) ** 2
    m.v2d = torch.arange(m.n, dtype=torch.int32, device=dev)
    k = torch.arange(m.n, device=dev)
    kx, ky = k % (n + 1), k // (n + 1)
    m.bc = torch.nonzero((kx == 0) | (kx == n) | (ky == 0) | (ky == n))[:, 0].to(torch.int32)
    m.xyz = m.coords.clone()
    return m


def _channel(nx, ny, nz, order, seed, dev):
    m = _Mesh()
    m.dim = 3
    x = torch.linspace(0, 4 * math.pi, nx, dtype=torch.float64, device=dev)
    eta = torch.linspace(-1, 1, ny, dtype=torch.float64, device=dev)
    y = torch.tanh(2.0 * eta) / math.tanh(2.0)
    z = torch.linspace(0, 4 * math.pi / 3, nz, dtype=torch.float64, device=dev)
    nv = nx * ny * nz
    k = torch.arange(nv, device=dev)
    ix, iy, iz = k % nx, (k // nx) % ny, k // (nx * ny)
    m.coords = torch.stack([x[ix], y[iy], z[iz]], 1).contiguous()
    if order != "grid":
        # interior nodes moved by up to 0.15 of the nearer spacing: every cell keeps its orientation
        dy = torch.zeros(ny, dtype=torch.float64, device=dev)
        dy[1:-1] = torch.minimum(y[2:] - y[1:-1], y[1:-1] - y[:-2])
        space = torch.stack([(x[1] - x[0]).expand(nv), dy[iy], (z[1] - z[0]).expand(nv)], 1)
        move = (2 * torch.rand((nv, 3), dtype=torch.float64, generator=_gen(seed + 11)) - 1).to(dev)
        inside = (ix > 0) & (ix < nx - 1) & (iy > 0) & (iy < ny - 1) & (iz > 0) & (iz < nz - 1)
        m.coords += 0.15 * space * move * inside[:, None]
    c = torch.arange((nx - 1) * (ny - 1) * (nz - 1), device=dev)
    c0 = c % (nx - 1) + nx * ((c // (nx - 1)) % (ny - 1) + ny * (c // ((nx - 1) * (ny - 1))))
    ax = [1, nx, nx * ny]
    tets = []
    for p, odd in (((0, 1, 2), 0), ((0, 2, 1), 1), ((1, 0, 2), 1), ((1, 2, 0), 0), ((2, 0, 1), 0), ((2, 1, 0), 1)):
        v = [c0, c0 + ax[p[0]], c0 + ax[p[0]] + ax[p[1]], c0 + sum(ax)]
        if odd:
            v[2], v[3] = v[3], v[2]
        tets.append(torch.stack(v, 1))
    m.cells = torch.stack(tets, 1).reshape(-1, 4).to(torch.int32).contiguous()
    mx, mz = nx - 1, nz - 1
    m.n = mx * ny * mz
    m.v2d = (ix % mx + mx * (iy + ny * (iz % mz))).to(torch.int32)
    d = torch.arange(m.n, device=dev)
    dix, diy, diz = d % mx, (d // mx) % ny, d // (mx * ny)
    m.xyz = m.coords[dix + nx * (diy + ny * diz)].contiguous()
    bc = torch.nonzero((diy == 0) | (diy == ny - 1))[:, 0]
    if order != "grid":
        g = _gen(seed + 12)
        if order == "local":
            # dofs change places with near neighbours only, as a bandwidth-reducing ordering leaves them
            at = torch.argsort(torch.arange(m.n, dtype=torch.float64) + 48 * torch.rand(m.n, dtype=torch.float64,
                                                                                       generator=g))
        else:
            at = torch.randperm(m.n, generator=g)
        at = at.to(dev)
        new = torch.empty_like(at)
        new[at] = torch.arange(m.n, device=dev)
        m.v2d = new[m.v2d.long()].to(torch.int32)
        m.xyz = m.xyz[at].contiguous()
        bc = torch.sort(new[bc])[0]
        vp = torch.randperm(nv, generator=g).to(dev)
        vn = torch.empty_like(vp)
        vn[vp] = torch.arange(nv, device=dev)
        m.coords, m.v2d = m.coords[vp].contiguous(), m.v2d[vp].contiguous()
        m.cells = vn[m.cells.long()][torch.randperm(m.cells.shape[0], generator=g).to(dev)].to(torch.int32).contiguous()
    m.bc = bc.to(torch.int32)
    return m


def _mesh(case, seed, dev):
    if case["mesh"] == "square":
        return _square(case["nx"], dev)
    return _channel(case["nx"], case["ny"], case["nz"], case["order"], seed, dev)


def _waves(m, g, count, amp):
    """A smooth field: a few random waves that fit the channel's periods."""
    x = m.xyz
    f = torch.zeros(m.n, dtype=torch.float64, device=x.device)
    for _ in range(count):
        r = torch.rand(4, dtype=torch.float64, generator=g).tolist()
        kx, kz = 0.5 * (1 + int(3 * r[0])), 1.5 * (1 + int(2 * r[1]))
        s = kx * x[:, 0] + 6.283 * r[2]
        if m.dim == 3:
            s = s + kz * x[:, 2]
        f += amp * torch.sin(s) * torch.cos(2.0 * r[3] * x[:, 1] + r[2])
    return f


def _fields(m, seed):
    """Velocity history, pressure and last correction, as they are in the
    middle of a run."""
    g = _gen(seed + 21)
    x = m.xyz
    if m.dim == 2:
        a, b = torch.rand(2, dtype=torch.float64, generator=g).tolist()

        def tg(t):
            e = math.exp(-2 * math.pi ** 2 * 0.01 * t)
            return torch.stack([-torch.sin(math.pi * (x[:, 1] - b)) * torch.cos(math.pi * (x[:, 0] - a)) * e,
                                torch.sin(math.pi * (x[:, 0] - a)) * torch.cos(math.pi * (x[:, 1] - b)) * e])
        e4 = math.exp(4 * math.pi ** 2 * 0.01 * 0.5e-3)
        p = -0.25 * (torch.cos(2 * math.pi * (x[:, 0] - a)) + torch.cos(2 * math.pi * (x[:, 1] - b))) * e4
        phi = 1e-3 * p
        bc = tg(1e-3)[:, m.bc.long()].contiguous()
        return tg(0.0).contiguous(), tg(-1e-3).contiguous(), p, phi, bc
    wall = 1.0 - x[:, 1] ** 2
    U1 = torch.stack([_waves(m, g, 4, 0.05) for _ in range(3)]) * wall
    U1[0] += wall
    noise = (2 * torch.rand((3, m.n), dtype=torch.float64, generator=g) - 1).to(x.device)
    U1 += 0.02 * noise * wall
    U2 = U1 - DT * torch.stack([_waves(m, g, 2, 0.1) for _ in range(3)]) * wall
    p, phi = _waves(m, g, 4, 0.05), _waves(m, g, 4, 1e-3)
    U1[:, m.bc.long()] = 0
    U2[:, m.bc.long()] = 0
    return U1.contiguous(), U2.contiguous(), p, phi, torch.zeros((3, m.bc.numel()), dtype=torch.float64, device=x.device)


def _scalars(m, seed, count):
    g = _gen(seed + 31)
    y = m.xyz[:, 1]
    c1 = torch.stack([y + 0.05 * _waves(m, g, 3, 1.0) for _ in range(count)])
    cb = y[m.bc.long()].repeat(count, 1).contiguous()
    c1[:, m.bc.long()] = cb
    return c1.contiguous(), cb


def _rhs(m, seed, count):
    g = _gen(seed + 41)
    b = torch.stack([_waves(m, g, 4, 1.0) for _ in range(count)])
    return b + (0.1 * (2 * torch.rand((count, m.n), dtype=torch.float64, generator=g) - 1)).to(b.device)


def _net(m, seed):
    """Network weights as training leaves them, and a right-hand side, the
    correction it belongs to and the previous one."""
    g = _gen(seed + 51)
    p = 0.1 * torch.randn(6497, dtype=torch.float64, generator=g)
    return p.to(torch.float32).to(m.xyz.device), _rhs(m, seed, 1)[0], _waves(m, g, 4, 1e-3), _waves(m, g, 4, 1e-3)


def _params(case):
    """dt, nu and body force of a case's mesh."""
    return (1e-3, 0.01, (0.0, 0.0)) if case["mesh"] == "square" else (DT, NU, (1.0, 0.0, 0.0))


# ---------------------------------------------------------------------------
# the framework's side

def _device_mesh(oa, m, seed, color=True):
    dm = oa.DeviceMesh(m.dim, m.coords, m.cells, m.v2d, m.n)
    pri = torch.randperm(m.cells.shape[0], generator=_gen(seed + 61)).to(torch.int32).to(m.coords.device)
    if not color:
        return dm, None, pri
    pat = oa.p1_pattern(dm)
    oa.colorize(dm, pri)
    return dm, pat, pri


def prepare(case, seed):
    import paper_1602_03643_amd as oa
    dev = _device()
    m = _mesh(case, seed, dev)
    kind = case["kind"]
    st = {"oa": oa, "case": case, "kind": kind}
    if kind == "graph":
        st["dm"], _, st["pri"] = _device_mesh(oa, m, seed, color=False)
        return st
    dm, pat, _ = _device_mesh(oa, m, seed)
    st.update(dm=dm, pat=pat)
    dt, nu, f = _params(case)
    if kind == "step":
        up = {"lumped": oa.UPDATE_LUMPED, "consistent": oa.UPDATE_CONSISTENT, "gradient": oa.UPDATE_GRADIENT}
        st["h"] = oa.IPCS(dm, pat, dt, nu, f, m.bc, rtol_u=_rtol(case), rtol_p=_rtol(case),
                          maxit=MAXIT, precision=oa.F32 if case["mixed"] else oa.F64, inner_iters=case["inner"],
                          velocity_update=up[case["update"]], diffusivity=[nu / 0.71] * case["scalars"],
                          convection=oa.CONV_ABE if case["convection"] == "abe" else oa.CONV_ABCN)
        if case["amg"]:
            st["amg"] = st["h"].pressure_amg(precision=oa.F32 if case["mixed"] else oa.F64, half_level0=case["mixed"])
        U1, U2, p, phi, bc = _fields(m, seed)
        st.update(U1=U1, U2=U2, Un=torch.empty_like(U1), p0=p, phi0=phi, p=p.clone(), phi=phi.clone(), bc=bc)
        if case["scalars"]:
            st["C1"], st["Cb"] = _scalars(m, seed, case["scalars"])
            st["Cn"] = torch.empty_like(st["C1"])
    elif kind in ("pcg", "mpnn"):
        val = oa.assemble_p1(dm, pat, oa.FORM_STIFF)
        if kind == "pcg":
            st["A"] = pat.with_values(val)
            b = _rhs(m, seed, 1)[0]
            st["b"] = b - b.mean()
            if case["amg"]:
                st["amg"] = oa.AMG(st["A"], None, precision=oa.F32 if case["mixed"] else oa.F64, singular=True)
            st["x"] = torch.empty_like(b)
            return st
        rows = torch.repeat_interleave(torch.arange(m.n, device=dev), torch.diff(pat.row_ptr).long())
        cols = pat.col_idx.long()
        s = torch.sqrt(val[rows == cols])
        st["net"] = oa.MPNN(pat.with_values((val / (s[rows] * s[cols])).contiguous()), s.contiguous(), m.xyz)
        st["params"], st["b"], st["phi"], st["prev"] = _net(m, seed)
        st["guess"] = torch.empty(m.n, dtype=torch.float64, device=dev)
        st["delta"] = torch.empty(m.n, dtype=torch.float32, device=dev)
        st["grad"] = torch.empty_like(st["params"])
        st["loss"] = oa.MPNN_LOSS_KNORM if case["loss"] == "knorm" else oa.MPNN_LOSS_MSE
    elif kind == "spmv":
        dt_ = torch.float32 if case["dtype"] == "f32" else torch.float64
        st["A"] = pat.with_values(oa.assemble_p1(dm, pat, oa.FORM_STIFF).to(dt_))
        st["x"] = _rhs(m, seed, 1)[0].to(dt_).contiguous()
        st["y"] = torch.empty_like(st["x"])
    else:
        base = oa.assemble_p1(dm, pat, oa.FORM_MASS, alpha=1.0 / dt)
        st["base"] = oa.assemble_p1(dm, pat, oa.FORM_STIFF, alpha=0.5 * nu, base=base)
        U1, U2 = _fields(m, seed)[:2]
        st["ub"] = [u.contiguous() for u in 1.5 * U1 - 0.5 * U2]
        st["val"] = torch.empty_like(base)
        if kind == "bicgstab":
            oa.assemble_p1(dm, pat, oa.FORM_CONV, uab=st["ub"], alpha=0.5, base=st["base"], out=st["val"])
            st["A"] = pat.with_values(st["val"])
            st["b"] = _rhs(m, seed, case["nrhs"]).contiguous()
            st["x"] = torch.empty_like(st["b"])
    return st


def run(st):
    oa, case, kind = st["oa"], st["case"], st["kind"]
    if kind == "step":
        st["p"].copy_(st["p0"])
        st["phi"].copy_(st["phi0"])
        if case["scalars"]:
            st["h"].step(st["U1"], st["U2"], st["Un"], st["p"], st["phi"], bc_values=st["bc"], C1=st["C1"],
                         Cn=st["Cn"], C_bc=st["Cb"])
            return st["Un"], st["p"], st["phi"], st["Cn"]
        st["h"].step(st["U1"], st["U2"], st["Un"], st["p"], st["phi"], bc_values=st["bc"])
        return st["Un"], st["p"], st["phi"]
    if kind == "pcg":
        x = st["x"].zero_()
        if case["amg"]:
            st["amg"].pcg(st["b"], x, rtol=_rtol(case))
        else:
            oa.pcg(st["A"], st["b"], x, rtol=_rtol(case), maxit=MAXIT, precision=oa.F32 if case["mixed"] else oa.F64,
                   nullspace_const=True)
        return x - x.mean()          # a pressure is fixed up to a constant
    if kind == "bicgstab":
        x = st["x"].zero_()
        oa.bicgstab(st["A"], st["b"], x, rtol=_rtol(case), precision=oa.F32 if case["mixed"] else oa.F64)
        return x
    if kind == "assemble":
        return oa.assemble_p1(st["dm"], st["pat"], oa.FORM_CONV, uab=st["ub"], alpha=0.5, base=st["base"],
                              out=st["val"])
    if kind == "spmv":
        return oa.spmv(st["A"], st["x"], st["y"])
    if kind == "graph":
        dm = st["dm"]
        perm, order = oa.rcm(oa.p1_pattern(dm))
        new = oa.DeviceMesh(dm.dim, dm.coords, dm.cells, oa.relabel(dm.vert2dof, perm), dm.n_dof)
        pat = oa.p1_pattern(new)
        color = oa.colorize(new, st["pri"])
        return pat.row_ptr, pat.col_idx, perm, order, color, new.color_ptr, new.color_cells
    net = st["net"]
    net.forward(st["params"], st["b"], st["prev"], st["guess"], st["delta"])
    loss = net.backward(st["params"], st["phi"], st["prev"], st["grad"], st["loss"])
    new = st["params"].clone()
    net.adam(new, st["grad"], torch.zeros_like(new), torch.zeros_like(new), 1)
    return st["guess"], st["delta"], st["grad"], new, loss


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["mesh"] == "square":
        d, n, nc, per = 2, (nx + 1) ** 2, 2 * nx * nx, 7
        nv = n
    else:
        d, n, nc, per = 3, (nx - 1) * ny * (nz - 1), 6 * (nx - 1) * (ny - 1) * (nz - 1), 15
        nv = nx * ny * nz
    nnz = per * n
    mesh = 4 * (d + 1) * nc + (8 * d + 4) * nv
    kind, vb = case["kind"], 4 if case.get("mixed") else 8
    span = max(nx, ny, nz)

    def krylov(iters, products, vectors, nrhs):
        """Iterations at the matrix once a product and the method's own vectors."""
        return (iters * (products * (vb + 4) * nnz + vectors * nrhs * vb * n),
                iters * nrhs * (products * 2 * nnz + 2 * vectors * n))
    # iterations that these solves take to 1e-12 at the least: a multigrid one 18, Jacobi ones by the mesh width
    pressure = krylov(18, 3, 12, 1) if case.get("amg") else krylov(10 * span, 1, 8, 1)
    if kind == "step":
        u = krylov(20, 2, 12, d)
        rhs = (8 * nnz * (d + 2) + 4 * nnz + mesh + 8 * n * (4 * d + 6), 2 * nnz * (3 * d + 3) + 150 * nc)
        by = [rhs] + [u, pressure] * case["inner"] + [krylov(15, 2, 12, 1)] * case["scalars"]
        if case["update"] == "consistent":
            by += [krylov(10, 1, 8, 1)] * d
    elif kind == "pcg":
        by = [(12 * nnz + 16 * n, 0), pressure]
    elif kind == "bicgstab":
        by = [(12 * nnz + 16 * n * case["nrhs"], 0), krylov(20, 2, 12, case["nrhs"])]
    elif kind == "assemble":
        by = [(16 * nnz + 4 * nnz + mesh + 8 * d * n, 150 * nc)]
    elif kind == "spmv":
        vb = 4 if case["dtype"] == "f32" else 8
        by = [((vb + 4) * nnz + 4 * n + 2 * vb * n, 2 * nnz)]
    elif kind == "graph":
        by = [(2 * mesh + 12 * nnz + 8 * n + 12 * nc, 0)]
    else:
        by = [(6 * 12 * nnz + 64 * 25 * n, n * (3 * 6 * 2 * 32 * 32 * 2) + 6 * 2 * 32 * nnz)]
    return {"bytes": sum(b for b, _ in by), "flops": sum(f for _, f in by)}


# ---------------------------------------------------------------------------
# the same equations in 64 bits, plain torch

class _Discrete:
    """P1 matrices on the mesh's pattern, rows padded to one width."""

    def __init__(self, m):
        self.m, self.n, self.d = m, m.n, m.dim
        self.dof = m.v2d.long()[m.cells.long()]
        x = m.coords[m.cells.long()]
        J = (x[:, 1:] - x[:, :1]).transpose(1, 2)
        inv = torch.linalg.inv(J)
        self.vol = torch.linalg.det(J).abs() / math.factorial(self.d)
        self.g = torch.cat([-inv.sum(1, keepdim=True), inv], 1)
        key = self.dof[:, :, None] * self.n + self.dof[:, None, :]
        key, self.slot = torch.unique(key.reshape(-1), return_inverse=True)
        self.nnz = key.numel()
        self.row, self.col = key // self.n, key % self.n
        count = torch.bincount(self.row, minlength=self.n)
        first = torch.cumsum(count, 0) - count
        self.at = self.row * int(count.max()) + (torch.arange(self.nnz, device=key.device) - first[self.row])
        self.shape = (self.n, int(count.max()))
        self.cols = self.pad(self.col)

    def pad(self, v):
        out = torch.zeros(self.shape[0] * self.shape[1], dtype=v.dtype, device=v.device)
        out[self.at] = v
        return out.view(self.shape)

    def gather(self, local):
        out = torch.zeros(self.nnz, dtype=torch.float64, device=local.device)
        return out.index_add_(0, self.slot, local.reshape(-1))

    def mass(self):
        k = self.d + 1
        w = (torch.ones(k, k, dtype=torch.float64, device=self.vol.device) +
             torch.eye(k, dtype=torch.float64, device=self.vol.device)) / (k * (k + 1))
        return self.gather(self.vol[:, None, None] * w)

    def stiff(self):
        return self.gather(self.vol[:, None, None] * (self.g @ self.g.transpose(1, 2)))

    def grad(self, k):
        return self.gather((self.vol[:, None] * self.g[:, :, k] / (self.d + 1))[:, None, :].expand(
            -1, self.d + 1, -1))

    def conv(self, u):
        w = u.T[self.dof]                                      # [cell, vertex, component]
        w = w + w.sum(1, keepdim=True)
        return self.gather((self.vol / ((self.d + 1) * (self.d + 2)))[:, None, None] * (w @ self.g.transpose(1, 2)))

    def mul(self, val):
        v, c = self.pad(val), self.cols

        def f(x):
            return (v * x[c]).sum(1)
        return f

    def diag(self, val):
        out = torch.zeros(self.n, dtype=torch.float64, device=val.device)
        on = self.row == self.col
        out[self.row[on]] = val[on]
        return out

    def identity_rows(self, val, bc):
        hit = torch.zeros(self.n, dtype=torch.bool, device=val.device)
        hit[bc.long()] = True
        return torch.where(hit[self.row], (self.row == self.col).to(torch.float64), val)


def _cg(A, diag, b, mean_free=False):
    x = torch.zeros_like(b)
    for _ in range(4):                                         # refinement on the true residual
        r = b - A(x)
        if mean_free:
            r = r - r.mean()
        e, z = torch.zeros_like(b), r / diag
        p, rz, stop = z.clone(), r @ z, 1e-6 * float(r.norm())
        if stop <= 1e-22 * float(b.norm()):
            break
        for it in range(3000):
            q = A(p)
            a = rz / (p @ q)
            e += a * p
            r = r - a * q
            z = r / diag
            new = r @ z
            p = z + (new / rz) * p
            rz = new
            if it % 10 == 9 and float(r.norm()) <= stop:
                break
        x = x + (e - e.mean() if mean_free else e)
    return x


def _bicgstab(A, diag, b, x):
    for _ in range(6):                                         # restarts from the true residual
        r = b - A(x)
        rh, p, rho, stop = r.clone(), r.clone(), r @ r, 1e-16 * float(b.norm())
        if float(r.norm()) <= 1e-15 * float(b.norm()):
            break
        for _ in range(60):
            y = p / diag
            v = A(y)
            a = rho / (rh @ v)
            s = r - a * v
            z = s / diag
            t = A(z)
            tt = t @ t
            if float(tt) == 0.0:
                x = x + a * y
                break
            w = (t @ s) / tt
            x = x + a * y + w * z
            r = s - w * t
            new = rh @ r
            if float(r.norm()) <= stop or float(new) == 0.0:
                break
            p = r + (new / rho) * (a / w) * (p - w * v)
            rho = new
    return x


def _exact_step(case, m, seed):
    D = _Discrete(m)
    dt, nu, f = _params(case)
    U1, U2, p, phi, bcv = _fields(m, seed)
    M, K = D.mass(), D.stiff()
    ML, Kd = torch.zeros(m.n, dtype=torch.float64, device=M.device).index_add_(0, D.row, M), D.diag(K)
    dP = [D.mul(D.grad(k)) for k in range(D.d)]
    Km = D.mul(K)
    ub = 1.5 * U1 - 0.5 * U2
    bc = m.bc.long()
    A = M / dt + 0.5 * nu * K
    if case["convection"] == "abcn":
        A = A + 0.5 * D.conv(ub)
    Ex = D.mul(2.0 / dt * M - A)
    b = torch.stack([f[k] * ML + Ex(U1[k]) - dP[k](p) for k in range(D.d)])
    if case["convection"] == "abe":
        C1, C2 = D.mul(D.conv(U1)), D.mul(D.conv(U2))
        b -= torch.stack([1.5 * C1(U1[k]) - 0.5 * C2(U2[k]) for k in range(D.d)])
    b[:, bc] = bcv
    A = D.identity_rows(A, m.bc)
    Am, Ad = D.mul(A), D.diag(A)
    UI = U1.clone()
    for it in range(case["inner"]):
        if it:
            more = torch.stack([dP[k](phi) for k in range(D.d)])
            more[:, bc] = 0
            b = b - more
        UI = torch.stack([_bicgstab(Am, Ad, b[k], UI[k]) for k in range(D.d)])
        bp = sum(dP[k](UI[k]) for k in range(D.d)) * (-1.0 / dt)
        phi = _cg(Km, Kd, bp - bp.mean(), mean_free=True)
        p = p + phi
        p = p - p.mean()
    g = torch.stack([dP[k](phi) for k in range(D.d)])
    if case["update"] == "consistent":
        hit = torch.zeros(m.n, dtype=torch.float64, device=M.device)
        hit[bc] = 1
        keep = M * (1 - hit[D.row]) * (1 - hit[D.col]) + hit[D.row] * (D.row == D.col)
        Mm, Mk = D.mul(M), D.mul(keep)
        Un = []
        for k in range(D.d):
            wall = torch.zeros_like(p)
            wall[bc] = bcv[k]
            r = Mm(UI[k]) - dt * g[k] - Mm(wall)
            r[bc] = bcv[k]
            Un.append(_cg(Mk, D.diag(keep), r))
        Un = torch.stack(Un)
    else:
        Un = UI - dt * g / ML
    Un[:, bc] = bcv
    if not case["scalars"]:
        return Un, p, phi
    c1, cb = _scalars(m, seed, case["scalars"])
    Ac = M / dt + 0.5 * nu / 0.71 * K + 0.5 * D.conv(ub)
    Ec = D.mul(2.0 / dt * M - Ac)
    Ac = D.identity_rows(Ac, m.bc)
    Cn = []
    for a in range(case["scalars"]):
        r = Ec(c1[a])
        r[bc] = cb[a]
        Cn.append(_bicgstab(D.mul(Ac), D.diag(Ac), r, c1[a].clone()))
    return Un, p, phi, torch.stack(Cn)


def _exact_mpnn(case, m, seed):
    D = _Discrete(m)
    K = D.stiff()
    Km, d = D.mul(K), D.diag(K)
    w = torch.where(D.row == D.col, torch.zeros_like(K), -K / d[D.row])
    wv, cols = D.pad(w), D.cols
    params, b, phi, prev = _net(m, seed)

    def rms(v):
        return float(v.square().mean().sqrt())
    s, bd = (b - Km(prev)) / d, b / d
    sigma = rms(s)
    lo, hi = m.xyz.min(0)[0], m.xyz.max(0)[0]
    X = torch.cat([torch.stack([s / sigma, bd / rms(bd), prev / rms(prev)], 1), 2 * (m.xyz - lo) / (hi - lo) - 1], 1)
    P = params.double().requires_grad_(True)
    sizes = (192, 32, 3072, 3072, 96, 32, 1)
    We, ce, Ws, Wn, c, wd, cd = torch.split(P, sizes)
    We, Ws, Wn, c = We.view(32, 6), Ws.view(3, 32, 32), Wn.view(3, 32, 32), c.view(3, 32)
    h = torch.relu(X @ We.T + ce)
    for l in range(3):
        agg = sum(wv[:, k, None] * h[cols[:, k]] for k in range(cols.shape[1]))
        h = h + torch.relu(h @ Ws[l].T + agg @ Wn[l].T + c[l])
    delta = h @ wd + cd
    t = (phi - prev) / sigma
    e = delta - t
    loss = (e @ Km(e)) / (t @ Km(t)) if case["loss"] == "knorm" else (e * e).mean()
    loss.backward()
    delta = delta.detach()
    # the first Adam step moves every weight by lr in its gradient's direction: it has no smooth exact value
    return prev + sigma * delta, delta, P.grad, None, float(loss.detach())


def exact(case, seed):
    m = _mesh(case, seed, _device())
    kind = case["kind"]
    if kind == "graph":
        return None
    if kind == "step":
        return _exact_step(case, m, seed)
    if kind == "mpnn":
        return _exact_mpnn(case, m, seed)
    D = _Discrete(m)
    dt, nu, _ = _params(case)
    if kind == "pcg":
        K = D.stiff()
        b = _rhs(m, seed, 1)[0]
        return _cg(D.mul(K), D.diag(K), b - b.mean(), mean_free=True)
    if kind == "spmv":
        # the operands as the call gets them, in its type
        dt_ = torch.float32 if case["dtype"] == "f32" else torch.float64
        return D.mul(D.stiff().to(dt_).double())(_rhs(m, seed, 1)[0].to(dt_).double())
    U1, U2 = _fields(m, seed)[:2]
    A = D.mass() / dt + 0.5 * nu * D.stiff() + 0.5 * D.conv(1.5 * U1 - 0.5 * U2)
    if kind == "assemble":
        return A
    return torch.stack([_bicgstab(D.mul(A), D.diag(A), b, torch.zeros_like(b)) for b in _rhs(m, seed, case["nrhs"])])
