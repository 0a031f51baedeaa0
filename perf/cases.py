"""The measured cases of the FTLE library: what a user's program has it do.

Every case goes through the package's public Python calls.  The listed cases
stand for the ranges that draw() samples:

  forward   one FTLE field of a flow map on a prepared mesh, 2D and 3D, float32
            and float64, the one-ring and the axis stencil, points numbered row
            by row or in random order, and the binary16 flow map (2D)
  gradient  the differentiable FTLE: field and dL/dphi by autograd
  batched   one call over many meshes (a sweep of time windows)
  build     a mesh that is new in every frame: built on the GPU, then one field
  list      the paper's pipeline without a mesh object: one-ring stencil,
            fixed-width axis list, FTLE from the list
  flowmap   RK4 flow maps: the analytic double gyre (2D) and ABC flow (3D)
  gridmap   RK4 flow maps in a velocity field sampled on a grid

Meshes are the jittered triangulated grids and Kuhn-split grids of the
repository's workloads, made here with torch on the GPU; flow maps are RK4 maps
of the double gyre and the ABC flow.
"""
from __future__ import annotations

import itertools
import math

import torch

import paper_2408_02758_amd as F

_DEV = "cuda"
_OMEGA = 2.0 * math.pi / 10.0
_DGYRE_BOX = (2.0, 1.0)
_TORCH = {"f32": torch.float32, "f64": torch.float64, "f16": torch.float32}


# -- the cases -----------------------------------------------------------------
def listed():
    return [
        # the smallest call: one 64 x 64 field in float64 (the paper's precision)
        dict(name="forward2d_small_f64", kind="forward", dim=2, nx=64, ny=64, dtype="f64", stencil="ring1",
             shuffle=False, T=15.0),
        # the largest 2D field: 2048 x 2048, float32
        dict(name="forward2d_large_f32", kind="forward", dim=2, nx=2048, ny=2048, dtype="f32", stencil="ring1",
             shuffle=False, T=15.0),
        # an unstructured mesh: odd size, points numbered at random, float64
        dict(name="forward2d_shuffled_f64", kind="forward", dim=2, nx=701, ny=503, dtype="f64", stencil="ring1",
             shuffle=True, T=15.0),
        # the largest 3D field: 160^3 tetrahedral mesh, float32
        dict(name="forward3d_large_f32", kind="forward", dim=3, nx=160, ny=160, nz=160, dtype="f32",
             stencil="ring1", shuffle=False, T=10.0),
        # optimisation through a 2D field, odd size, float64
        dict(name="gradient2d_odd_f64", kind="gradient", dim=2, nx=613, ny=409, dtype="f64", stencil="ring1",
             shuffle=False, T=15.0),
        # optimisation through a 3D field, float32
        dict(name="gradient3d_f32", kind="gradient", dim=3, nx=96, ny=96, nz=96, dtype="f32", stencil="ring1",
             shuffle=False, T=10.0),
        # a sweep: 48 meshes of 64..1024 points a side in one call, float32
        dict(name="batched2d_48_f32", kind="batched", dim=2, count=48, lo=64, hi=1024, pick=3, dtype="f32"),
        # a moving tetrahedral mesh: rebuilt in every frame, ragged sides
        dict(name="build3d_f32", kind="build", dim=3, nx=127, ny=113, nz=101, dtype="f32", stencil="ring1",
             shuffle=False, T=10.0),
        # the paper's list, made and read on the GPU
        dict(name="list2d_f32", kind="list", dim=2, nx=1023, ny=769, dtype="f32", shuffle=False, T=15.0),
        # the flow map before the field: the double gyre over 1500 steps
        dict(name="flowmap2d_f32", kind="flowmap", dim=2, nx=1024, ny=512, dtype="f32", T=15.0, dt=0.01),
        # the ABC flow over 500 steps, ragged sides, float64
        dict(name="flowmap3d_f64", kind="flowmap", dim=3, nx=81, ny=67, nz=59, dtype="f64", T=10.0, dt=0.02),
        # particles in simulation output: 61 slices of a sampled double gyre
        dict(name="gridmap2d_f32", kind="gridmap", dim=2, nx=1024, ny=512, dtype="f32", gx=513, gy=257, slices=61,
             T=15.0, dt=0.01),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, dim, lo, hi):
    s = _log_int(rng, lo, hi)
    side = lambda: max(8, min(hi, int(round(s * rng.uniform(0.6, 1.0)))))   # noqa: E731
    c = dict(nx=side(), ny=side())
    if dim == 3:
        c["nz"] = side()
    return c


def draw(rng):
    kind = rng.choice(["forward", "forward", "gradient", "batched", "build", "list", "flowmap", "gridmap"])
    dim = rng.choice([2, 3])
    c = dict(kind=kind, dim=dim)
    if kind == "batched":
        c.update(count=rng.randint(2, 48), lo=24, hi=_log_int(rng, 64, 640), pick=rng.randint(0, 10 ** 6), dtype="f32")
        c["dim"] = 2
        return c
    lo, hi = {("forward", 2): (32, 2048), ("forward", 3): (10, 160), ("gradient", 2): (32, 1024),
              ("gradient", 3): (10, 112), ("build", 2): (32, 1024), ("build", 3): (10, 112),
              ("list", 2): (32, 1024), ("list", 3): (10, 112), ("flowmap", 2): (32, 720), ("flowmap", 3): (10, 80),
              ("gridmap", 2): (32, 720), ("gridmap", 3): (10, 72)}[(kind, dim)]
    c.update(_sides(rng, dim, lo, hi))
    c["dtype"] = rng.choice(["f32", "f64"])
    if kind in ("forward", "gradient", "build", "list"):
        c.update(shuffle=rng.random() < 0.3, T=15.0 if dim == 2 else 10.0)
        if kind != "list":
            c["stencil"] = rng.choice(["ring1", "ring1", "axis"])
        if kind == "forward" and dim == 2 and c["nx"] * c["ny"] <= 2 ** 18 and rng.random() < 0.25:
            c["dtype"] = "f16"
    else:
        c["T"] = round(rng.uniform(2.0, 15.0 if dim == 2 else 10.0), 3)
        c["dt"] = 0.01 if dim == 2 else 0.02
        if kind == "gridmap":
            g = _log_int(rng, 32, 256) if dim == 2 else _log_int(rng, 16, 96)
            c.update(gx=(2 if dim == 2 else 1) * g + 1, gy=g + 1, slices=rng.choice([1, 21, 61]))
            if dim == 3:
                c["gz"] = g
    return c


# -- inputs --------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=_DEV).manual_seed(int(seed) * 7919 + 17)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=_DEV, dtype=torch.float64)


def _tri_grid(nx, ny, g):
    """Jittered cell-centred grid on [0,2] x [0,1], each quad split on its shorter diagonal."""
    lx, ly = _DGYRE_BOX
    jit = _rand(g, ny, nx, 2) * 0.6 - 0.3
    x = (torch.arange(nx, device=_DEV, dtype=torch.float64)[None, :] + 0.5 + jit[..., 0]) * (lx / nx)
    y = (torch.arange(ny, device=_DEV, dtype=torch.float64)[:, None] + 0.5 + jit[..., 1]) * (ly / ny)
    xy = torch.stack([x.reshape(-1), y.reshape(-1)], 1)
    p00 = (torch.arange(ny - 1, device=_DEV)[:, None] * nx + torch.arange(nx - 1, device=_DEV)[None, :]).reshape(-1)
    p10, p01, p11 = p00 + 1, p00 + nx, p00 + nx + 1
    main = ((xy[p11] - xy[p00]).square().sum(1) <= (xy[p01] - xy[p10]).square().sum(1))[:, None]
    t1 = torch.where(main, torch.stack([p00, p10, p11], 1), torch.stack([p00, p10, p01], 1))
    t2 = torch.where(main, torch.stack([p00, p11, p01], 1), torch.stack([p10, p11, p01], 1))
    return xy, torch.stack([t1, t2], 1).reshape(-1, 3).to(torch.int32).contiguous()


def _box_points(nx, ny, nz, g):
    """Points of a regular grid over a period of the ABC flow, at a random offset."""
    org = _rand(g, 3)
    ax = [torch.arange(n, device=_DEV, dtype=torch.float64) * (2.0 * math.pi / max(n - 1, 1)) + org[d]
          for d, n in enumerate((nx, ny, nz))]
    zz, yy, xx = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return torch.stack([xx.reshape(-1), yy.reshape(-1), zz.reshape(-1)], 1)


def _kuhn_cells(nx, ny, nz):
    """Six tetrahedra per cube, one per order of the three unit steps."""
    r = lambda n: torch.arange(n - 1, device=_DEV)   # noqa: E731
    base = ((r(nz)[:, None, None] * ny + r(ny)[None, :, None]) * nx + r(nx)[None, None, :]).reshape(-1)
    steps = (1, nx, nx * ny)
    tets = []
    for perm in itertools.permutations(range(3)):
        v = [base]
        for axis in perm:
            v.append(v[-1] + steps[axis])
        tets.append(torch.stack(v, 1))
    return torch.stack(tets, 1).reshape(-1, 4).to(torch.int32).contiguous()


def _mesh_arrays(case, g):
    """(coords float64, cells int32) of a case, in the caller's numbering."""
    if case["dim"] == 2:
        x, cells = _tri_grid(case["nx"], case["ny"], g)
    else:
        x, cells = _box_points(case["nx"], case["ny"], case["nz"], g), _kuhn_cells(case["nx"], case["ny"], case["nz"])
    if case.get("shuffle"):
        p = torch.randperm(x.shape[0], generator=g, device=_DEV)
        y = torch.empty_like(x)
        y[p] = x
        order = torch.randperm(cells.shape[0], generator=g, device=_DEV)
        x, cells = y, p.to(torch.int32)[cells.long()][order].contiguous()
    return x, cells


def _gyre(p, t):
    s = torch.sin(_OMEGA * t)
    a, b = 0.25 * s, 1.0 - 0.5 * s
    f = (a * p[:, 0] + b) * p[:, 0]
    return torch.stack([-math.pi * 0.1 * torch.sin(math.pi * f) * torch.cos(math.pi * p[:, 1]),
                        math.pi * 0.1 * torch.cos(math.pi * f) * torch.sin(math.pi * p[:, 1]) * (2 * a * p[:, 0] + b)],
                       1)


def _abc(p, t):
    s, c = torch.sin(p), torch.cos(p)
    A, B, C = math.sqrt(3.0), math.sqrt(2.0), 1.0
    return torch.stack([A * s[:, 2] + C * c[:, 1], B * s[:, 0] + A * c[:, 2], C * s[:, 1] + B * c[:, 0]], 1)


def _rk4(vel, p, t0, T, steps):
    """x(t0 + T) by classical RK4; t0 and T numbers or (N,) tensors."""
    h = T / steps
    col = (lambda v: v[:, None]) if isinstance(h, torch.Tensor) else (lambda v: v)
    for s in range(steps):
        t = t0 + s * h
        k1 = vel(p, t)
        k2 = vel(p + col(0.5 * h) * k1, t + 0.5 * h)
        k3 = vel(p + col(0.5 * h) * k2, t + 0.5 * h)
        k4 = vel(p + col(h) * k3, t + h)
        p = p + col(h / 6.0) * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
    return p


def _velocity(dim):
    if dim == 2:
        return lambda p, t: _gyre(p, t if isinstance(t, torch.Tensor) else torch.tensor(t, dtype=torch.float64, device=_DEV))
    return _abc


def _field_inputs(case, seed):
    """Stored coordinates, cells and flow map of a mesh case."""
    g = _gen(seed)
    x, cells = _mesh_arrays(case, g)
    t0 = float(torch.rand((), generator=g, device=_DEV)) * 10.0
    phi = _rk4(_velocity(case["dim"]), x, t0, case["T"], 48)
    dt = _TORCH[case["dtype"]]
    return x.to(dt).contiguous(), cells, phi.to(dt).contiguous(), g


def _batched_inputs(case, seed):
    sides_rng = torch.Generator().manual_seed(case["pick"])      # the set of meshes is the case's
    u = torch.rand(case["count"], generator=sides_rng, dtype=torch.float64)
    sides = [int(round(math.exp(math.log(case["lo"]) + float(v) * math.log(case["hi"] / case["lo"])))) for v in u]
    g = _gen(seed)
    geo = [_tri_grid(s, s, g) for s in sides]
    t0 = (_rand(g, len(sides)) * 10.0).tolist()
    Ts = (_rand(g, len(sides)) * 15.0 + 5.0).tolist()
    n = torch.tensor([x.shape[0] for x, _ in geo], device=_DEV)
    per = lambda v: torch.repeat_interleave(torch.tensor(v, dtype=torch.float64, device=_DEV), n)   # noqa: E731
    phi = _rk4(_gyre, torch.cat([x for x, _ in geo]), per(t0), per(Ts), 48)
    flows = [f.float().contiguous() for f in torch.split(phi, n.tolist())]
    return [(x.float().contiguous(), cells) for x, cells in geo], flows, Ts


def _particle_inputs(case, seed):
    g = _gen(seed)
    if case["dim"] == 2:
        x = _rand(g, case["nx"] * case["ny"], 2) * 0.6 - 0.3
        i = torch.arange(case["nx"] * case["ny"], device=_DEV)
        x[:, 0] = (x[:, 0] + (i % case["nx"]) + 0.5) * (2.0 / case["nx"])
        x[:, 1] = (x[:, 1] + torch.div(i, case["nx"], rounding_mode="floor") + 0.5) * (1.0 / case["ny"])
    else:
        x = _box_points(case["nx"], case["ny"], case["nz"], g)
    t0 = float(torch.rand((), generator=g, device=_DEV)) * 10.0 if case["kind"] == "flowmap" else 0.0
    return x.to(_TORCH[case["dtype"]]).contiguous(), t0, g


def _sampled(case, g):
    """A velocity field as simulation output holds it: float32 values at the nodes and slices."""
    vel = _velocity(case["dim"])
    phase = float(torch.rand((), generator=g, device=_DEV)) * 10.0
    if case["dim"] == 2:
        shape, top = (case["gx"], case["gy"]), _DGYRE_BOX
    else:
        shape, top = (case["gx"], case["gy"], case["gz"]), (2.0 * math.pi + 1.0,) * 3
    spacing = [t / (n - 1) for t, n in zip(top, shape)]
    axes = [torch.arange(n, device=_DEV, dtype=torch.float64) * h for n, h in zip(shape, spacing)]
    grids = torch.meshgrid(*axes[::-1], indexing="ij")
    pts = torch.stack([m.reshape(-1) for m in grids[::-1]], 1)
    t_step = case["T"] / max(1, case["slices"] - 1)
    field = [(vel(pts, phase + k * t_step) * (1.0 + 0.2 * math.sin(phase + k * t_step))).float()
             for k in range(case["slices"])]
    return torch.stack(field).reshape(case["slices"], *shape[::-1], case["dim"]).contiguous(), spacing, t_step


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batched":
        geo, flows, Ts = _batched_inputs(case, seed)
        meshes = [F.Mesh.on_device(x, cells) for x, cells in geo]
        return dict(kind=kind, call=F.BatchedCall(meshes, flows, Ts))
    if kind in ("flowmap", "gridmap"):
        x, t0, g = _particle_inputs(case, seed)
        s = dict(kind=kind, dim=case["dim"], x=x, t0=t0, T=case["T"], dt=case["dt"])
        if kind == "gridmap":
            s["field"], s["spacing"], s["t_step"] = _sampled(case, g)
        return s
    x, cells, phi, g = _field_inputs(case, seed)
    s = dict(kind=kind, dim=case["dim"], x=x, cells=cells, phi=phi, T=case["T"], stencil=case.get("stencil"))
    if kind in ("forward", "gradient"):
        s["mesh"] = F.Mesh.on_device(x, cells, stencil=case["stencil"])
        if case["dtype"] == "f16":
            s["kind"], s["delta"] = "forward16", s["mesh"].encode_flow_f16(phi)
        if kind == "gradient":
            s["phi"] = phi.requires_grad_(True)
            s["g"] = torch.randn(x.shape[0], generator=g, device=_DEV, dtype=torch.float64).to(x.dtype)
        del s["x"], s["cells"]
    return s


# -- one pass ------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "forward":
        return s["mesh"].forward(s["phi"], s["T"])
    if kind == "forward16":
        return s["mesh"].forward_f16(s["delta"], s["T"])
    if kind == "gradient":
        f = F.ftle(s["mesh"], s["phi"], s["T"])
        (grad,) = torch.autograd.grad(f, s["phi"], s["g"])
        return f.detach(), grad
    if kind == "batched":
        return s["call"]()
    if kind == "build":
        return F.Mesh.on_device(s["x"], s["cells"], stencil=s["stencil"]).forward(s["phi"], s["T"])
    if kind == "list":
        row_ptr, col = F.ring1_csr(s["dim"], s["x"].shape[0], s["cells"])
        ell = F.axis_ell(s["x"], row_ptr, col)
        return row_ptr, col, ell, F.forward_ell(s["x"], ell, s["phi"], s["T"])
    if kind == "flowmap":
        return F.advect_rk4("double_gyre" if s["dim"] == 2 else "abc", s["x"], s["t0"], s["T"], s["dt"])
    return F.advect_rk4_grid(s["field"], [0.0] * s["dim"], s["spacing"], 0.0, s["t_step"], s["x"], s["t0"], s["T"],
                             s["dt"])


# -- what a pass cannot do without -----------------------------------------------
def _points(case):
    return case["nx"] * case["ny"] * case.get("nz", 1)


def _n_cells(case):
    if case["dim"] == 2:
        return 2 * (case["nx"] - 1) * (case["ny"] - 1)
    return 6 * (case["nx"] - 1) * (case["ny"] - 1) * (case["nz"] - 1)


def work(case):
    """Coordinates, flow map, results (and, where the pass makes or reads them,
    cells, lists, gradients and fields) once each; the arithmetic of the least
    squares per stencil entry and of the solve and eigenvalue per point, of the
    velocity per RK4 stage."""
    kind, d = case["kind"], case["dim"]
    e = 8 if case["dtype"] == "f64" else 4
    per_entry, per_point, degree = (18, 45, 6) if d == 2 else (36, 150, 14)
    if kind == "batched":
        sides_rng = torch.Generator().manual_seed(case["pick"])
        u = torch.rand(case["count"], generator=sides_rng, dtype=torch.float64)
        n = sum(int(round(math.exp(math.log(case["lo"]) + float(v) * math.log(case["hi"] / case["lo"])))) ** 2
                for v in u)
        return {"bytes": n * (2 * d + 1) * e, "flops": n * (degree * per_entry + per_point)}
    n = _points(case)
    if kind in ("flowmap", "gridmap"):
        steps = max(1, math.ceil(abs(case["T"]) / case["dt"] - 1e-9))
        stage = (50 if d == 2 else 100) if kind == "flowmap" else (24 if d == 2 else 60)
        field = case["slices"] * case["gx"] * case["gy"] * case.get("gz", 1) * d * 4 if kind == "gridmap" else 0
        return {"bytes": 2 * n * d * e + field, "flops": n * steps * 4 * (stage + 4 * d)}
    if case.get("stencil") == "axis" or kind == "list":
        degree_used = 2 * d
    else:
        degree_used = degree
    flops = n * (degree_used * per_entry + per_point)
    bytes_ = n * (2 * d + 1) * e
    if case["dtype"] == "f16":
        bytes_ = n * (8 + 4 + 4)
    if kind == "gradient":      # the cotangent read, the gradient written; the adjoint's arithmetic
        bytes_ += n * (d + 1) * e
        flops += n * degree_used * (4 * d + 4)
    elif kind == "build":
        bytes_ += _n_cells(case) * (d + 1) * 4
    elif kind == "list":
        bytes_ += _n_cells(case) * (d + 1) * 4 + 8 * (n + 1) + 4 * degree * n + 4 * 2 * d * n
    return {"bytes": bytes_, "flops": flops}


# -- the same in 64 bits, by plain torch -----------------------------------------
def _ring1(n, cells):
    """Directed edges (i, j) of the one-ring stencil, sorted by i then j."""
    k = cells.shape[1]
    c = cells.long()
    keys = [torch.minimum(c[:, a], c[:, b]) * n + torch.maximum(c[:, a], c[:, b])
            for a in range(k) for b in range(a)]
    u = torch.unique(torch.cat(keys))
    i, j = torch.div(u, n, rounding_mode="floor"), u % n
    both = torch.sort(torch.cat([u, j * n + i])).values
    return torch.div(both, n, rounding_mode="floor"), both % n


def _axis(x, i, j):
    """The fixed-width list (N, 2 dim): per signed axis the neighbour with the largest cosine, ties to the smaller index."""
    n, d = x.shape
    dx = x[j] - x[i]
    nrm = dx.square().sum(1).sqrt()
    out = torch.full((n, 2 * d), -1, dtype=torch.int64, device=x.device)
    for k in range(2 * d):
        along = dx[:, k // 2] * (1.0 if k % 2 else -1.0)
        side = along > 0
        cos = (along / nrm)[side]
        at, to = i[side], j[side]
        best = torch.full((n,), -1.0, dtype=torch.float64, device=x.device).scatter_reduce_(0, at, cos, "amax")
        win = cos == best[at]
        first = torch.full((n,), n, dtype=torch.int64, device=x.device)
        first.scatter_reduce_(0, at[win], to[win], "amin")
        out[:, k] = torch.where(first < n, first, -1)
    return out


def _edges_of(ell):
    at, k = torch.nonzero(ell >= 0, as_tuple=True)
    return at, ell[at, k]


def _top_eigen(C):
    """Largest eigenvalue and its unit eigenvector of symmetric (N, D, D), by cyclic Jacobi rotations."""
    D = C.shape[1]
    C, V = C.clone(), torch.eye(D, dtype=C.dtype, device=C.device).expand(C.shape[0], D, D).clone()
    for _ in range(1 if D == 2 else 7):
        for p, q in ([(0, 1)] if D == 2 else [(0, 1), (0, 2), (1, 2)]):
            off = C[:, p, q]
            theta = (C[:, q, q] - C[:, p, p]) / (2.0 * torch.where(off == 0, torch.ones_like(off), off))
            t = torch.where(theta >= 0, 1.0, -1.0) / (theta.abs() + torch.sqrt(theta * theta + 1.0))
            t = torch.where(off == 0, torch.zeros_like(t), t)
            c = 1.0 / torch.sqrt(t * t + 1.0)
            s = t * c
            for M, rows in ((C, False), (C, True), (V, False)):
                a, b = (M[:, p, :], M[:, q, :]) if rows else (M[:, :, p], M[:, :, q])
                a, b = c[:, None] * a - s[:, None] * b, s[:, None] * a + c[:, None] * b
                if rows:
                    M[:, p, :], M[:, q, :] = a, b
                else:
                    M[:, :, p], M[:, :, q] = a, b
    lam = torch.diagonal(C, dim1=1, dim2=2)
    k = lam.argmax(1)
    return lam.gather(1, k[:, None])[:, 0], V.gather(2, k[:, None, None].expand(-1, D, 1))[:, :, 0]


def _inverse(M):
    """Inverses of symmetric (N, D, D) by the adjugate."""
    if M.shape[1] == 2:
        det = M[:, 0, 0] * M[:, 1, 1] - M[:, 0, 1] ** 2
        A = torch.stack([M[:, 1, 1], -M[:, 0, 1], -M[:, 0, 1], M[:, 0, 0]], 1)
        return A.reshape(-1, 2, 2) / det[:, None, None]
    a, b, c = M[:, 0], M[:, 1], M[:, 2]
    A = torch.stack([torch.cross(b, c, dim=1), torch.cross(c, a, dim=1), torch.cross(a, b, dim=1)], 2)
    return A / (a * torch.cross(b, c, dim=1)).sum(1)[:, None, None]


def _exact_field(x, phi, i, j, T, weights=None):
    """FTLE, and with weights dL/dphi of sum(weights * FTLE), over directed edges i -> j."""
    n, d = x.shape
    dx, df = x[j] - x[i], phi[j] - phi[i]
    M = torch.zeros(n, d * d, dtype=torch.float64, device=x.device)
    B = torch.zeros_like(M)
    for r in range(d):
        for c in range(d):
            M[:, r * d + c].index_add_(0, i, dx[:, r] * dx[:, c])
            B[:, r * d + c].index_add_(0, i, df[:, r] * dx[:, c])
    Mi = _inverse(M.reshape(n, d, d))
    mul = lambda P, Q: (P[:, :, :, None] * Q[:, None, :, :]).sum(2)   # noqa: E731
    J = mul(B.reshape(n, d, d), Mi)
    lam, v = _top_eigen(mul(J.transpose(1, 2), J))
    f = 0.5 * torch.log(lam) / abs(T)
    if weights is None:
        return f
    p = (J * v[:, None, :]).sum(2) * (weights / (abs(T) * lam))[:, None]
    h = (Mi * v[:, None, :]).sum(2)
    grad = torch.zeros_like(x)
    w = (h[i] * dx).sum(1)
    for r in range(d):
        add = p[:, r][i] * w
        grad[:, r].index_add_(0, j, add)
        grad[:, r].index_add_(0, i, -add)
    return f, grad


def _interpolated(field, spacing, t_step):
    """The sampled field's velocity: multilinear in space, linear in time, the nearest value outside."""
    D = field.shape[-1]
    nt, shape = field.shape[0], field.shape[1:-1][::-1]
    flat = field.double().reshape(nt, -1, D)

    def vel(p, t):
        s = min(max(t / t_step, 0.0), nt - 1.0) if nt > 1 else 0.0
        k = min(int(s), max(nt - 2, 0))
        here = flat[k] if nt == 1 else flat[k] * (1.0 - (s - k)) + flat[k + 1] * (s - k)
        base, fr, stride = 0, [], []
        step = 1
        for d in range(D):
            u = (p[:, d] / spacing[d]).clamp(0.0, shape[d] - 1.0)
            c = u.long().clamp(max=shape[d] - 2)
            fr.append(u - c)
            base = base + c * step
            stride.append(step)
            step *= shape[d]
        v = torch.zeros_like(p)
        for m in range(1 << D):
            w, o = 1.0, 0
            for d in range(D):
                w = w * (fr[d] if m >> d & 1 else 1.0 - fr[d])
                o += stride[d] if m >> d & 1 else 0
            v += here[base + o] * w[:, None]
        return v

    return vel


def exact(case, seed):
    kind = case["kind"]
    if kind == "batched":
        geo, flows, Ts = _batched_inputs(case, seed)
        return [_exact_field(x.double(), f.double(), *_ring1(x.shape[0], cells), T)
                for (x, cells), f, T in zip(geo, flows, Ts)]
    if kind in ("flowmap", "gridmap"):
        x, t0, g = _particle_inputs(case, seed)
        steps = max(1, math.ceil(abs(case["T"]) / case["dt"] - 1e-9))
        vel = _velocity(case["dim"]) if kind == "flowmap" else _interpolated(*_sampled(case, g))
        return _rk4(vel, x.double(), t0, case["T"], steps)
    x, cells, phi, g = _field_inputs(case, seed)
    n = x.shape[0]
    xd, pd = x.double(), phi.double()
    i, j = _ring1(n, cells)
    if kind == "list":
        row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=_DEV)
        row_ptr[1:] = torch.bincount(i, minlength=n).cumsum(0)
        ell = _axis(xd, i, j)
        return row_ptr, j.int(), ell.int(), _exact_field(xd, pd, *_edges_of(ell), case["T"])
    if case.get("stencil") == "axis":
        i, j = _edges_of(_axis(xd, i, j))
    if case["dtype"] == "f16":
        pd = (x + (phi - x).half().float()).double()
    if kind == "gradient":
        w = torch.randn(n, generator=g, device=_DEV, dtype=torch.float64).to(x.dtype)
        return _exact_field(xd, pd, i, j, case["T"], w.double())
    return _exact_field(xd, pd, i, j, case["T"])
