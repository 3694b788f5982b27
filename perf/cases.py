"""The work that users of this framework have it do, as cases that can be timed.

A case is a dict of plain values; `kind` names the entry points that it goes
through:

  pass     fem.residual_tangent into the buffers that a Newton loop keeps
  vjp      fem.residual_vjp, the parameter gradient of one load step
  batch    many uneven specimens in one forward call and one VJP call
  adjoint  one backward step of the time-history adjoint (adjoint.gradient):
           mu -> ubar, K^T (F-bar only), then (lam, mu) -> g, hbar
  pattern  fem.csr_pattern, once per mesh
  newton   newton.solve_step, one load increment from the undeformed state
  solve    fem.Solver.solve with the drivers' defaults (flexible GMRES, the
           aggregation multigrid's K-cycle), a tangent kept in float

Meshes are grids of nx x ny x nz hexahedra, jittered, with elements knocked
out and nodes and elements numbered out of order where `voids` asks for it.  Every input is made on the device from the
seed.  exact() computes the same quantities in 64 bits with plain torch: a
series for the logarithmic strain, Newton on the closest-point equations with
derivatives by automatic differentiation, and conjugate gradients or a dense
factorization for the linear systems.
"""
import math
import random

import torch

from paper_2606_17390_amd import fem, newton

F64 = torch.float64
_HEX = ((0, 0, 0), (1, 0, 0), (1, 1, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1))
_PREC = {"fp64": fem.FP64, "mixed": fem.FP32_MIXED, "k32": fem.FP64_K32}
_GRAD = (2, 3, 4, 7, 8, 9, 10)  # the differentiated parameters among the eleven
_R2 = math.sqrt(2.0)
# Yld2004-18p coefficients of AA6111-T4: c' 12 13 21 23 31 32 44 55 66, c'' likewise, m
_AA6111 = (-0.069888, 0.936408, 0.079143, 1.003060, 0.524741, 1.363180, 1.023770, 1.069060, 0.954322,
           0.981171, 0.476741, 0.575316, 0.866827, 1.145010, -0.079294, 1.051660, 1.147100, 1.404620, 8.0)


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _case(kind, nx, ny, nz, **more):
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "voids": 0.0, "law": "swift", "yield": "hill", "fbar": False,
         "orient": "none", "fields": "one", "prec": "fp64"}
    c.update(more)
    return c


def listed():
    cases = [
        # one Newton iteration's pass on a verification cube: launches and latency
        ("pass_tiny", _case("pass", 4, 4, 4)),
        # an anisotropic sheet, reduced precision
        ("pass_sheet_mixed", _case("pass", 40, 40, 4, prec="mixed")),
        # the large heterogeneous cube (3.09M dofs): the headline pass and its reduced-precision form
        ("pass_cube_fp64", _case("pass", 100, 100, 100, fields="fgh")),
        ("pass_cube_mixed", _case("pass", 100, 100, 100, fields="fgh", prec="mixed")),
        # the pass of the load-path driver with the paper's element: exact residual, float tangent, textured sheet
        ("pass_fbar_newton", _case("pass", 61, 47, 53, law="voce", fbar=True, orient="elem", prec="k32")),
        # the 18-parameter yield function on a rolled sheet with one rolling direction
        ("pass_barlat", _case("pass", 67, 61, 31, **{"yield": "barlat"}, law="voce", orient="one")),
        # per-element parameter identification on a specimen with voids
        ("vjp_voids", _case("vjp", 200, 200, 2, voids=0.25, fields="all")),
        # forward and gradient of many uneven specimens, each with parameters of its own
        ("batch_mixed", _case("batch", 0, 0, 0, specimens=64, least=2000, most=60000, mix=4, prec="mixed",
                              fields="spec")),
        # one backward step of an inverse study with the paper's element
        ("adjoint_fbar", _case("adjoint", 75, 60, 45, law="voce", fbar=True, orient="one")),
        # a new specimen's matrix pattern
        ("pattern_voids", _case("pattern", 97, 83, 71, voids=0.15)),
        # one increment of the tensile specimen of the inverse study, start to converged state
        ("newton_specimen", _case("newton", 35, 30, 5, law="voce", orient="one")),
        # the linear system of one Newton iteration of the forward simulation
        ("solve_cube", _case("solve", 100, 100, 100, rtol=1e-8)),
    ]
    return [dict(c, name=n) for n, c in cases]


def _grid(rng, lo, hi, sheets=True):
    """Grid sizes with lo to hi elements (log-uniform), of any aspect: cubes, blocks, sheets a few elements thick."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if sheets and rng.random() < 0.4 and n > 300:
        nz = rng.randint(2, 6)
        nx = max(3, round(math.sqrt(n / nz) * rng.uniform(0.6, 1.6)))
    else:
        nz = max(3, round(n ** (1 / 3) * rng.uniform(0.7, 1.4)))
        nx = max(3, round(math.sqrt(n / nz) * rng.uniform(0.8, 1.25)))
    return nx, max(3, round(n / nz / nx)), nz


def draw(rng):
    kind = rng.choice(("pass", "pass", "pass", "pass", "vjp", "vjp", "batch", "adjoint", "pattern", "newton", "solve",
                       "solve"))
    model = {"law": rng.choice(("swift", "voce")), "fbar": rng.random() < 0.4,
             "orient": rng.choice(("none", "one", "elem")), "fields": rng.choice(("one", "fgh", "all"))}
    voids = rng.choice((0.0, 0.0, 0.2))
    if kind == "pass":
        if rng.random() < 0.2:
            return _case(kind, *_grid(rng, 64, 120e3), voids=voids, **{"yield": "barlat"},
                         prec=rng.choice(("fp64", "k32")), **model)
        return _case(kind, *_grid(rng, 64, 900e3), voids=voids, prec=rng.choice(("fp64", "mixed", "k32")), **model)
    if kind == "vjp":
        return _case(kind, *_grid(rng, 64, 500e3), voids=voids, prec=rng.choice(("fp64", "mixed")), **model)
    if kind == "batch":
        n = rng.randint(3, 60)
        return _case(kind, 0, 0, 0, specimens=n, least=rng.randint(200, 2000), most=rng.randint(4000, 55000),
                     mix=rng.randint(0, 10 ** 6), prec=rng.choice(("fp64", "mixed")), fields="spec")
    if kind == "adjoint":
        return _case(kind, *_grid(rng, 64, 200e3), voids=voids, **model)
    if kind == "pattern":
        return _case(kind, *_grid(rng, 64, 550e3), voids=rng.uniform(0.0, 0.3))
    if kind == "newton":
        return _case(kind, *_grid(rng, 200, 5000), **{**model, "fields": "one"})
    return _case(kind, *_grid(rng, 1000, 900e3, sheets=False), rtol=rng.choice((1e-6, 1e-8)))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sizes(c):
    """Grids of a batch: element counts log-uniform, sheets of two to four layers."""
    r = random.Random(c["mix"])
    out = []
    for _ in range(c["specimens"]):
        n, nz, aspect = math.exp(r.uniform(math.log(c["least"]), math.log(c["most"]))), r.randint(2, 4), \
            math.exp(r.uniform(0.0, math.log(4.0)))
        nx = max(1, round(math.sqrt(n * aspect / nz)))
        out.append((nx, max(1, round(n / nz / nx)), nz))
    return out


def _smooth(gen, pts, box):
    """A smooth random field of unit deviation at pts [n, 3]."""
    dev = pts.device
    k = torch.randint(-3, 4, (12, 3), generator=gen, device=dev).to(F64) * (2 * math.pi) / box
    phase = torch.rand(12, generator=gen, device=dev, dtype=F64) * 2 * math.pi
    f = torch.zeros(pts.shape[0], dtype=F64, device=dev)
    for m in range(12):
        f += torch.cos((pts * k[m]).sum(1) + phase[m])
    return f / math.sqrt(6.0)


def _displacement(gen, X, box, strain):
    """Three smooth isochoric waves (to first order), strains of the order of `strain`."""
    dev = X.device
    u = torch.zeros_like(X)
    for _ in range(3):
        k = torch.randint(-1, 2, (3,), generator=gen, device=dev).to(F64)
        k = torch.where((k == 0).all(), torch.ones_like(k), k) * (2 * math.pi) / box
        a = torch.randn(3, generator=gen, device=dev, dtype=F64)
        a = a - k * (a * k).sum() / (k * k).sum()
        a = a / a.norm() * strain / k.norm()
        phase = torch.rand(1, generator=gen, device=dev, dtype=F64) * 2 * math.pi
        u += a * torch.cos((X * k).sum(1) + phase)[:, None]
    return u


def _mesh(c, size, gen):
    """Jittered grid with knocked-out element columns: X, conn (VTK order), box."""
    nx, ny, nz = size
    dev = _dev()
    box = torch.tensor([float(nx), float(ny), float(nz)], dtype=F64, device=dev)
    z, y, x = torch.meshgrid(*(torch.arange(n + 1, device=dev) for n in (nz, ny, nx)), indexing="ij")
    X = torch.stack((x, y, z), -1).reshape(-1, 3).to(F64)
    inner = (X > 0) & (X < box)  # faces stay flat
    X = X + 0.1 * (torch.rand(X.shape, generator=gen, device=dev, dtype=F64) - 0.5) * inner
    ids = torch.arange(X.shape[0], device=dev).reshape(nz + 1, ny + 1, nx + 1)
    conn = torch.stack([ids[k:k + nz, j:j + ny, i:i + nx] for i, j, k in _HEX], -1).reshape(-1, 8)
    if c["voids"]:
        # the specimen's shape belongs to the case, not to the seed
        own = torch.Generator(device=dev)
        own.manual_seed(nx + 1000 * ny + 1000000 * nz)
        ey, ex = torch.meshgrid(torch.arange(ny, device=dev), torch.arange(nx, device=dev), indexing="ij")
        f = _smooth(own, torch.stack((ex, ey, 0 * ex), -1).reshape(-1, 3).to(F64), box)
        at = torch.sort(f, stable=True)[1][int(c["voids"] * f.numel()):]
        keep = torch.zeros(f.numel(), dtype=torch.bool, device=dev)
        keep[at] = True
        conn = conn[keep.repeat(nz)]
        used = torch.zeros(X.shape[0], dtype=torch.bool, device=dev)
        used[conn.reshape(-1)] = True
        X, conn = X[used], (torch.cumsum(used, 0) - 1)[conn]
    if c["voids"] or c["kind"] == "pattern":
        # a mesher's numbering: neighbours are near each other, in no order
        def order(n):
            return torch.sort(torch.arange(n, device=dev)
                              + 200 * torch.rand(n, generator=gen, device=dev, dtype=F64), stable=True)[1]
        o = order(X.shape[0])
        place = torch.empty_like(o)
        place[o] = torch.arange(o.numel(), device=dev)
        X, conn = X[o], place[conn][order(conn.shape[0])]
    return X.contiguous(), conn.contiguous(), box


def _angles(t):
    """Rotations about z."""
    o = torch.zeros(t.shape[0], 9, dtype=F64, device=t.device)
    o[:, 0], o[:, 1], o[:, 3], o[:, 4], o[:, 8] = torch.cos(t), -torch.sin(t), torch.sin(t), torch.cos(t), 1.0
    return o


def _parameters(c, gen, n, centers, box):
    """[n, 11] or [11]: E, nu, F, G, H, L, M, N and the three of the hardening law."""
    dev = _dev()
    prm = torch.tensor([200000.0, 0.3, 0.5, 0.5, 0.5, 1.5, 1.5, 1.5]
                       + ([200.0, 150.0, 20.0] if c["law"] == "voce" else [500.0, 0.01, 0.2]), dtype=F64, device=dev)
    if c["fields"] in ("one", "spec"):
        u = torch.rand(11, generator=gen, device=dev, dtype=F64) - 0.5
        prm[2:5] += 0.6 * u[2:5]
        prm[8:] *= 1 + 0.2 * u[8:]
        return prm
    prm = prm.repeat(n, 1)
    for k in (2, 3, 4) + ((7, 8, 9, 10) if c["fields"] == "all" else ()):
        f = torch.clamp(0.15 * _smooth(gen, centers, box), -0.3, 0.3)
        prm[:, k] = prm[:, k] + f if k < 5 else prm[:, k] * (1 + 0.7 * f)
    return prm


def _problem(c, seed):
    """One mesh or one batch of meshes, with the state of a converged earlier increment and the next one's trial."""
    dev = _dev()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    parts = []
    for size in (_sizes(c) if c["kind"] == "batch" else [(c["nx"], c["ny"], c["nz"])]):
        X, conn, box = _mesh(c, size, gen)
        before = _displacement(gen, X, box, 0.01)
        d = before + _displacement(gen, X, box, 0.0017)
        hist = torch.empty(7, 8 * conn.shape[0], dtype=F64, device=dev)
        for a in range(0, conn.shape[0], 1 << 16):
            e = _log_strain(_gradient(before[conn[a:a + (1 << 16)]], _shape(X[conn[a:a + (1 << 16)]])[0]))
            tr = (e[..., 0, 0] + e[..., 1, 1] + e[..., 2, 2]) / 3
            b = slice(8 * a, 8 * a + e.shape[0] * 8)
            for k, (i, j) in enumerate(((0, 0), (1, 1), (2, 2), (1, 2), (0, 2), (0, 1))):
                hist[k, b] = (e[..., i, j] - (tr if i == j else 0.0)).reshape(-1)
        hist[6] = math.sqrt(2 / 3) * ((hist[:3] ** 2).sum(0) + 2 * (hist[3:6] ** 2).sum(0)).sqrt() \
            + 0.05 * torch.rand(hist.shape[1], generator=gen, device=dev, dtype=F64)
        centers = X[conn].mean(1)
        prm = _parameters(c, gen, conn.shape[0], centers, box)
        bc = torch.zeros(X.shape, dtype=torch.uint8, device=dev)
        bc[X[:, 0] == 0] = 1
        lam = torch.randn(X.shape, generator=gen, device=dev, dtype=F64) * (1 - bc.to(F64))
        parts.append((X, conn, d, hist, prm, bc, lam / lam.norm()))
    off_n, off_e = [0], [0]
    for p in parts:
        off_n.append(off_n[-1] + p[0].shape[0])
        off_e.append(off_e[-1] + p[1].shape[0])
    cat = [torch.cat(v, 1) if v[0].shape[0] == 7 and v[0].shape[1] != 3 else torch.cat(v) for v in
           ([p[k] for p in parts] for k in (0, 2, 3, 5, 6))] if len(parts) > 1 else [parts[0][k] for k in (0, 2, 3, 5, 6)]
    conn = torch.cat([p[1] + n for p, n in zip(parts, off_n)])
    ne = conn.shape[0]
    orient = None
    if c["orient"] != "none":
        t = torch.rand(ne if c["orient"] == "elem" else 1, generator=gen, device=dev, dtype=F64) * math.pi
        orient = _angles(t)
    return {"X": cat[0], "conn": conn, "d": cat[1], "hist": cat[2], "bc": cat[3], "lam": cat[4],
            "prm": torch.stack([p[4] for p in parts]) if c["kind"] == "batch" else parts[0][4],
            "orient": orient, "off": off_e,
            "mu": torch.randn(cat[2].shape, generator=gen, device=dev, dtype=F64)}


def _handles(c, p):
    mesh = fem.Mesh(p["X"].cpu().numpy(), p["conn"].to(torch.int32).cpu().numpy(), _dev())
    orient = p["orient"] if p["orient"] is None or p["orient"].shape[0] > 1 else p["orient"].reshape(9)
    params = fem.Params(p["prm"], mesh.n_elems, _dev(), per_spec=c["kind"] == "batch", hardening=c["law"],
                        fbar=c["fbar"], orient=orient, barlat=_AA6111 if c["yield"] == "barlat" else None)
    return mesh, params


def _load(c, seed):
    """The increment of the tensile specimen: y = 0 fixed, the other end gripped and moved."""
    dev = _dev()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    X, conn, box = _mesh(c, (c["nx"], c["ny"], c["nz"]), gen)
    prm = _parameters(c, gen, conn.shape[0], None, box)
    u = torch.rand(3, generator=gen, device=dev, dtype=F64)
    bc = torch.zeros(X.shape, dtype=torch.uint8, device=dev)
    ends = (X[:, 1] == 0) | (X[:, 1] == box[1])
    bc[ends] = 1
    d = torch.zeros_like(X)
    d[:, 1] = X[:, 1] * (0.002 + 0.002 * u[0])
    orient = None if c["orient"] == "none" else \
        _angles(math.pi * torch.rand(conn.shape[0] if c["orient"] == "elem" else 1, generator=gen, device=dev,
                                     dtype=F64))
    return {"X": X, "conn": conn, "d": d, "hist": torch.zeros(7, 8 * conn.shape[0], dtype=F64, device=dev),
            "prm": prm, "bc": bc, "orient": orient}


def _system(c, seed):
    """The tangent of a partly yielded cube on its grid of nodes: elements with
    their own stiffness, softer in shear where they flow; x = 0 clamped, the
    far face moved in x and y, its z motion free.  Returns the 27 blocks of
    every node [n, 27, 3, 3] (float), which of them exist, the right-hand side
    of the face's motion and the constrained dofs."""
    dev = _dev()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    box = torch.tensor([float(nx), float(ny), float(nz)], dtype=F64, device=dev)
    Xe = torch.tensor(_HEX, dtype=F64, device=dev)[None]
    G, dv = _shape(Xe)
    G, dv = G[0], dv[0]
    eye = torch.eye(3, dtype=F64, device=dev)
    vol = (dv[:, None, None, None, None] * G[:, :, None, :, None] * G[:, None, :, None, :]).sum(0)  # I J a b
    lap = (dv[:, None, None, None] * G[:, :, None, :] * G[:, None, :, :]).sum((0, 3))
    dev_part = lap[:, :, None, None] * eye + vol.transpose(2, 3) - (2 / 3) * vol
    z, y, x = torch.meshgrid(*(torch.arange(n, device=dev) for n in (nz, ny, nx)), indexing="ij")
    at = torch.stack((x, y, z), -1).reshape(-1, 3).to(F64) + 0.5
    bulk = (166667.0 * (1 + 0.05 * _smooth(gen, at, box))).reshape(nz, ny, nx)
    flow = _smooth(gen, at, box) > 0.5
    shear = (76923.0 * torch.where(flow, 0.1, 1.0)).reshape(nz, ny, nx)
    D = torch.zeros(nz + 1, ny + 1, nx + 1, 27, 3, 3, dtype=F64, device=dev)
    for I, (i, j, k) in enumerate(_HEX):
        for J, (p, q, r) in enumerate(_HEX):
            n = (r - k + 1) * 9 + (q - j + 1) * 3 + (p - i + 1)
            D[k:k + nz, j:j + ny, i:i + nx, n] += bulk[..., None, None] * vol[I, J] \
                + shear[..., None, None] * dev_part[I, J]
    D = D.reshape(-1, 27, 3, 3)
    zz, yy, xx = torch.meshgrid(*(torch.arange(n + 1, device=dev) for n in (nz, ny, nx)), indexing="ij")
    P = torch.stack((xx, yy, zz), -1).reshape(-1, 3)
    step = torch.tensor([[p - 1, q - 1, r - 1] for r in range(3) for q in range(3) for p in range(3)], device=dev)
    to = P[:, None, :] + step
    there = ((to >= 0) & (to <= box.long())).all(-1)
    col = torch.where(there, (to[..., 2] * (ny + 1) + to[..., 1]) * (nx + 1) + to[..., 0], 0)
    bc = torch.zeros(P.shape, dtype=torch.bool, device=dev)
    bc[P[:, 0] == 0] = True
    bc[P[:, 0] == nx] = torch.tensor([True, True, False], device=dev)
    move = torch.zeros(P.shape, dtype=F64, device=dev)
    u = torch.rand(2, generator=gen, device=dev, dtype=F64)
    move[P[:, 0] == nx] = torch.stack((0.01 * (1 + u[0]), 0.005 * (1 + u[1]), 0 * u[0])) * box[0] / 20
    b = -_blocks_times(D, col, move)
    b[bc] = 0.0
    D[bc.nonzero()[:, 0], :, bc.nonzero()[:, 1], :] = 0.0
    rows = bc.nonzero()
    D[rows[:, 0], 13, rows[:, 1], rows[:, 1]] = 1.0
    return D.float(), there, col, b, bc


def _blocks_times(D, col, x):
    y = torch.empty_like(x)
    for a in range(0, x.shape[0], 1 << 18):  # slices of the rows: bounded scratch memory
        b = slice(a, a + (1 << 18))
        y[b] = (D[b].to(F64) * x[col[b]][:, :, None, :]).sum((1, 3))
    return y


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "solve":
        D, there, _, b, bc = _system(c, seed)
        nx, ny, nz = c["nx"], c["ny"], c["nz"]
        dev = _dev()
        ids = torch.arange((nx + 1) * (ny + 1) * (nz + 1), device=dev).reshape(nz + 1, ny + 1, nx + 1)
        conn = torch.stack([ids[k:k + nz, j:j + ny, i:i + nx] for i, j, k in _HEX], -1).reshape(-1, 8)
        n = ids.reshape(-1)
        X = torch.stack((n % (nx + 1), n // (nx + 1) % (ny + 1), n // ((nx + 1) * (ny + 1))), -1).to(F64)
        mesh = fem.Mesh(X.cpu().numpy(), conn.to(torch.int32).cpu().numpy(), dev)
        csr = fem.csr_pattern(mesh)
        deg = there.sum(1)
        K = torch.empty(csr.nnz, dtype=torch.float32, device=dev)
        # rows 3I + a, then the blocks that exist in ascending node order, then b
        at = torch.cumsum(deg, 0) - deg
        rank = torch.cumsum(there, 1) - 1
        for a in range(3):
            base = 9 * at[:, None] + a * 3 * deg[:, None] + 3 * rank
            for q in range(3):
                K[(base + q)[there]] = D[:, :, a, q][there]
        del D
        solver = fem.Solver(csr, dev, precond=fem.PC_AMG, method="fgmres", bc_mask=bc.to(torch.uint8).reshape(-1))
        solver.solve(K, b.reshape(-1), rtol=0.5, max_iter=1, check=False)  # the hierarchy, once per pattern
        return {"c": c, "solver": solver, "K": K, "b": b.reshape(-1).contiguous()}
    if c["kind"] == "newton":
        p = _load(c, seed)
        mesh, params = _handles(c, p)
        csr = fem.csr_pattern(mesh)
        bc = p["bc"].reshape(-1).contiguous()
        solver = fem.Solver(csr, _dev(), precond=fem.PC_AMG, method="fgmres", bc_mask=bc)
        out = fem.Forward(mesh, csr, fem.FP64)
        fem.residual_tangent(mesh, csr, params, p["d"], p["hist"], bc_mask=bc, out=out)
        solver.solve(out.K, -out.R, rtol=0.5, max_iter=1, check=False)
        return {"c": c, "mesh": mesh, "csr": csr, "params": params, "start": p["d"], "d": p["d"].clone(),
                "hist": p["hist"], "bc": bc, "solver": solver, "out": out}
    p = _problem(c, seed)
    mesh, params = _handles(c, p)
    s = {"c": c, "mesh": mesh, "params": params, "d": p["d"], "hist": p["hist"], "lam": p["lam"], "mu": p["mu"],
         "bc": p["bc"].reshape(-1).contiguous(), "prec": _PREC[c["prec"]], "batch": None}
    if c["kind"] == "pattern":
        return s
    if c["kind"] == "batch":
        s["batch"] = fem.Batch(p["off"], _dev())
    if c["kind"] in ("vjp", "batch"):
        s["vjp"] = fem.Vjp(mesh, len(p["off"]) - 1)
    if c["kind"] == "vjp":
        return s
    s["csr"] = fem.csr_pattern(mesh)
    s["out"] = fem.Forward(mesh, s["csr"], s["prec"])
    if c["kind"] == "adjoint":
        s["adj"] = fem.HistoryAdjoint(mesh)
        fem.residual_tangent(mesh, s["csr"], params, s["d"], s["hist"], bc_mask=s["bc"], out=s["out"])
        # what the backward step is given: the tangent of the converged state, and its transpose's buffer
        s["K"], s["KT"] = s["out"].K, torch.empty_like(s["out"].K)
        s["out"] = None
    return s


def run(s):
    kind = s["c"]["kind"]
    if kind == "solve":
        x, its, _ = s["solver"].solve(s["K"], s["b"], rtol=s["c"]["rtol"], max_iter=2000)
        return {"x": x, "iterations": its}
    if kind == "newton":
        s["d"].copy_(s["start"])
        hist, its, _ = newton.solve_step(s["mesh"], s["csr"], s["params"], s["d"], s["hist"], s["bc"],
                                         solver=s["solver"], out=s["out"])
        return {"d": s["d"], "hist": hist, "iterations": its}
    if kind == "pattern":
        m = fem.csr_pattern(s["mesh"])
        return {"row_ptr": m.row_ptr, "col_idx": m.col_idx, "elem_rank": m.elem_rank, "node_ptr": m.node_elem_ptr,
                "node_elem": m.node_elem}
    if kind == "adjoint":
        a = fem.history_adjoint(s["mesh"], s["csr"], s["params"], s["d"], s["hist"], lam=None, mu=s["mu"],
                                out=s["adj"], want_hbar=False)
        r = {"ubar": a.ubar}
        if s["c"]["fbar"]:
            r["KT"] = fem.csr_transpose(s["csr"], s["K"], bc_mask=s["bc"], out=s["KT"])
        a = fem.history_adjoint(s["mesh"], s["csr"], s["params"], s["d"], s["hist"], lam=s["lam"], mu=s["mu"],
                                out=s["adj"], want_ubar=False)
        return dict(r, g=a.g_uniform, g_elem=a.g_elem, hbar=a.hbar)
    r = {}
    if kind in ("pass", "batch"):
        o = fem.residual_tangent(s["mesh"], s["csr"], s["params"], s["d"], s["hist"], bc_mask=s["bc"], out=s["out"],
                                 batch=s["batch"])
        r = {"R": o.R, "K": o.K, "hist": o.hist, "rnorm2": o.rnorm2}
    if kind in ("vjp", "batch"):
        v = fem.residual_vjp(s["mesh"], s["params"], s["d"], s["hist"], s["lam"], prec=s["prec"], out=s["vjp"],
                             batch=s["batch"])
        r = dict(r, g=v.g_uniform, g_elem=v.g_elem)
    return r


def work(case):
    """Bytes: every input read once, every output written once (the matrix from
    the pattern's block count; a solve reads it three times per iteration, for
    the product and the finest level of the cycle, at some 20 iterations).
    Operations: what the constitutive update, the residual and the tangent
    contraction take per Gauss point."""
    c = case
    grids = _sizes(c) if c["kind"] == "batch" else [(c["nx"], c["ny"], c["nz"])]
    ne = sum(x * y * z for x, y, z in grids) * (1 - c["voids"])
    nn = sum((x + 1) * (y + 1) * (z + 1) for x, y, z in grids)
    blocks = sum((3 * x + 1) * (3 * y + 1) * (3 * z + 1) for x, y, z in grids) * (1 - c["voids"])
    kb = 9 * blocks * (8 if c["prec"] == "fp64" else 4)
    gp = 8 * ne
    per_elem = {"one": 0, "spec": 0, "fgh": 3, "all": 7}[c["fields"]] + (9 if c["orient"] == "elem" else 0)
    state = 48 * nn + ne * (32 + 8 * per_elem) + 56 * gp  # X, d, conn, parameters, history
    fpass = {"bytes": state + kb + 64 * ne + 36 * nn + 56 * gp, "flops": gp * (25000 if c["yield"] == "barlat" else 6000)}
    fvjp = {"bytes": state + 24 * nn + 56 * ne, "flops": gp * 2500}
    if c["kind"] == "pass":
        return fpass
    if c["kind"] == "vjp":
        return fvjp
    if c["kind"] == "batch":
        return {k: fpass[k] + fvjp[k] for k in fpass}
    if c["kind"] == "adjoint":
        return {"bytes": 2 * state + 2 * 56 * gp + 48 * nn + 56 * ne + 56 * gp
                + (2 * 72 * blocks + 4 * blocks if c["fbar"] else 0), "flops": gp * 6000}
    if c["kind"] == "pattern":
        return {"bytes": 32 * ne + 36 * blocks + 64 * ne + 32 * ne + 16 * nn, "flops": 0}
    if c["kind"] == "newton":
        return {"bytes": 7 * (fpass["bytes"] + 40 * 3 * 72 * blocks), "flops": 7 * (fpass["flops"] + 40 * 6 * 9 * blocks)}
    return {"bytes": 20 * 3 * 40 * blocks, "flops": 20 * 3 * 18 * blocks}


# ---------------------------------------------------------------------------
# the same quantities in 64 bits, plain torch
# ---------------------------------------------------------------------------

def _mm(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _t(a):
    return a.transpose(-1, -2)


def _det(a):
    return a[..., 0, 0] * (a[..., 1, 1] * a[..., 2, 2] - a[..., 1, 2] * a[..., 2, 1]) \
        - a[..., 0, 1] * (a[..., 1, 0] * a[..., 2, 2] - a[..., 1, 2] * a[..., 2, 0]) \
        + a[..., 0, 2] * (a[..., 1, 0] * a[..., 2, 1] - a[..., 1, 1] * a[..., 2, 0])


def _inv(a):
    r = [torch.cross(a[..., (i + 1) % 3, :], a[..., (i + 2) % 3, :], dim=-1) for i in range(3)]
    return torch.stack(r, -1) / _det(a)[..., None, None]


def _shape(Xe):
    """Shape-function gradients [e, g, node, 3] and volumes [e, g] at the eight Gauss points."""
    s = torch.tensor([[2 * i - 1.0 for i in h] for h in _HEX], dtype=F64, device=Xe.device)
    g = torch.tensor([[2.0 * (n >> k & 1) - 1 for k in range(3)] for n in range(8)], dtype=F64, device=Xe.device) \
        / math.sqrt(3.0)
    f = 1 + g[:, None, :] * s  # gp, node, direction
    dN = torch.stack([s[:, 0] * f[..., 1] * f[..., 2], f[..., 0] * s[:, 1] * f[..., 2],
                      f[..., 0] * f[..., 1] * s[:, 2]], -1) / 8
    J = (Xe[:, None, :, :, None] * dN[None, :, :, None, :]).sum(2)
    return _mm(dN[None].expand(Xe.shape[0], -1, -1, -1), _inv(J)), _det(J)


def _gradient(de, G):
    return (de[:, None, :, :, None] * G[:, :, :, None, :]).sum(2)


def _log_strain(H):
    """Half the logarithm of F^T F as atanh((C - I)(C + I)^-1): no eigenvectors, smooth where stretches coincide."""
    A = H + _t(H) + _mm(_t(H), H)
    eye = torch.eye(3, dtype=F64, device=H.device)
    Z = _mm(A, _inv(A + 2 * eye))
    W = _mm(Z, Z)
    S = eye / 31.0 + 0 * W
    for n in range(29, 0, -2):
        S = eye / n + _mm(W, S)
    return _mm(Z, S)


def _mandel(a):
    return torch.stack((a[..., 0, 0], a[..., 1, 1], a[..., 2, 2], _R2 * a[..., 1, 2], _R2 * a[..., 0, 2],
                        _R2 * a[..., 0, 1]), -1)


def _matrix(v):
    r = v / _R2
    return torch.stack((torch.stack((v[..., 0], r[..., 5], r[..., 4]), -1),
                        torch.stack((r[..., 5], v[..., 1], r[..., 3]), -1),
                        torch.stack((r[..., 4], r[..., 3], v[..., 2]), -1)), -2)


def _phi(c, v, prm, Q):
    """Equivalent stress of Mandel stresses [n, 6]."""
    if Q is not None:
        v = _mandel(_mm(_mm(_t(Q), _matrix(v)), Q))
    if c["yield"] == "hill":
        F, G, H, L, M, N = (prm[:, k] for k in range(2, 8))
        return (F * (v[:, 1] - v[:, 2]) ** 2 + G * (v[:, 2] - v[:, 0]) ** 2 + H * (v[:, 0] - v[:, 1]) ** 2
                + L * v[:, 3] ** 2 + M * v[:, 4] ** 2 + N * v[:, 5] ** 2).sqrt()
    m = (v[:, 0] + v[:, 1] + v[:, 2])[:, None] / 3
    s = torch.cat((v[:, :3] - m, v[:, 3:]), 1)
    sums = []
    for k in (0, 9):
        a = _AA6111[k:k + 9]
        w = _matrix(torch.stack((-a[0] * s[:, 1] - a[1] * s[:, 2], -a[2] * s[:, 0] - a[3] * s[:, 2],
                                 -a[4] * s[:, 0] - a[5] * s[:, 1], a[6] * s[:, 3], a[7] * s[:, 4],
                                 a[8] * s[:, 5]), -1))
        scale = (w.detach() ** 2).sum((-1, -2)).sqrt()
        sums.append((w, scale))
    scale = torch.maximum(sums[0][1], sums[1][1])
    tr = []
    for w, _ in sums:  # power sums of the principal values: tr w^k
        w1 = w / scale[:, None, None]
        w2 = _mm(w1, w1)
        w4 = _mm(w2, w2)
        dot = lambda a, b: (a * b).sum((-1, -2))  # noqa: E731
        w3 = _mm(w2, w1)
        eye = torch.eye(3, dtype=F64, device=v.device)
        tr.append((3.0, dot(w1, eye), dot(w1, w1), dot(w2, w1), dot(w2, w2), dot(w3, w2), dot(w3, w3), dot(w4, w3),
                   dot(w4, w4)))
    total = sum(math.comb(8, k) * (-1) ** k * tr[0][8 - k] * tr[1][k] for k in range(9))
    return scale * (total / 4) ** 0.125


def _sigma_y(c, alpha, prm):
    if c["law"] == "voce":
        return prm[:, 8] + prm[:, 9] * (1 - torch.exp(-prm[:, 10] * alpha))
    return prm[:, 8] * (prm[:, 9] + alpha) ** prm[:, 10]


def _elastic(v, prm, inverse=False):
    k3, m2 = prm[:, 0] / (1 - 2 * prm[:, 1]), prm[:, 0] / (1 + prm[:, 1])
    tr = (v[:, 0] + v[:, 1] + v[:, 2])[:, None] / 3
    i = torch.cat((tr.expand(-1, 3), torch.zeros_like(v[:, 3:])), 1)
    return i / k3[:, None] + (v - i) / m2[:, None] if inverse else i * k3[:, None] + (v - i) * m2[:, None]


def _flow(c, T, prm, Q):
    with torch.enable_grad():
        T = T if T.requires_grad else T.requires_grad_(True)
        f = _phi(c, T, prm, Q)
        return f, torch.autograd.grad(f.sum(), T, create_graph=True)[0]


def _corrector(c, trial, alpha_n, prm, Q):
    """Stress and plastic multiplier of the closest-point projection; a last
    Newton step outside no_grad carries the derivatives by every input."""
    def system(T, g, prm, trial, alpha_n, Q):
        f, N = _flow(c, T, prm, Q)
        return T - trial + g[:, None] * _elastic(N, prm), f - _sigma_y(c, alpha_n + g, prm), N

    T0, p0, a0, Q0 = trial.detach(), prm.detach(), alpha_n.detach(), None if Q is None else Q.detach()
    f, _ = _flow(c, T0.clone(), p0, Q0)
    s = (_sigma_y(c, a0, p0) / f.detach())[:, None]
    mean = torch.zeros_like(T0)
    mean[:, :3] = T0[:, :3].mean(1, keepdim=True)
    T = mean + (T0 - mean) * s
    N = _flow(c, T.clone(), p0, Q0)[1].detach()
    D = _elastic(N, p0)
    g = ((T0 - T) * D).sum(1) / (D * D).sum(1)

    def jacobian(T, g):
        T, g = T.clone().requires_grad_(True), g.clone().requires_grad_(True)
        G1, G3, N = system(T, g, p0, T0, a0, Q0)
        J = torch.empty(T.shape[0], 7, 7, dtype=F64, device=T.device)
        for r in range(7):
            out = torch.autograd.grad((G1[:, r] if r < 6 else G3).sum(), (T, g), retain_graph=True)
            J[:, r, :6], J[:, r, 6] = out
        return J, G1.detach(), G3.detach()

    def merit(G1, G3):
        return (G1 ** 2).sum(1) + G3 ** 2

    for _ in range(60):
        J, G1, G3 = jacobian(T, g)
        step = torch.linalg.solve(J, -torch.cat((G1, G3[:, None]), 1))
        z, m0 = torch.ones_like(g), merit(G1, G3)
        for _ in range(12):
            H1, H3, _ = system(T + z[:, None] * step[:, :6], g + z * step[:, 6], p0, T0, a0, Q0)
            worse = ~(merit(H1.detach(), H3.detach()) < m0) & (m0 > 1e-16 * (T0 ** 2).sum(1))
            if not bool(worse.any()):
                break
            z = torch.where(worse, 0.5 * z, z)
        T, g = (T + z[:, None] * step[:, :6]).detach(), (g + z * step[:, 6]).detach()
        if float((step[:, :6].abs().amax(1) / T0.abs().amax(1)).max()) < 1e-13:
            break
    J, _, _ = jacobian(T, g)
    G1, G3, _ = system(T.clone(), g, prm, trial, alpha_n, Q)
    y = torch.linalg.solve(J, -torch.cat((G1, G3[:, None]), 1))
    return T + y[:, :6], g + y[:, 6]


def _elements(c, Xe, de, hist, prm, orient):
    """Element forces [e, 8, 3] and updated history [e, 8, 7], differentiable by displacements, history and parameters."""
    G, dv = _shape(Xe)
    H = _gradient(de, G)
    Hb = H
    if c["fbar"]:
        eye = torch.eye(3, dtype=F64, device=H.device)
        J = _det(eye + H)
        Jb = (dv * J).sum(1, keepdim=True) / dv.sum(1, keepdim=True)
        b = torch.exp(torch.log(Jb / J) / 3)[..., None, None]
        Hb = b * H + (b - 1) * eye
    eps = _log_strain(Hb)
    n = eps.shape[0] * 8
    per = prm[:, None, :].expand(-1, 8, -1).reshape(n, 11)
    Q = None if orient is None else orient.reshape(-1, 1, 3, 3).expand(Hb.shape[0], 8, 3, 3).reshape(n, 3, 3)
    h = hist.reshape(n, 7)
    ep_n = torch.cat((h[:, :3], _R2 * h[:, 3:6]), 1)
    e = _mandel(eps).reshape(n, 6)
    trial = _elastic(e - ep_n, per)
    with torch.no_grad():
        at = torch.nonzero(_phi(c, trial, per, Q) > _sigma_y(c, h[:, 6], per))[:, 0]
    T, ep, al = trial, ep_n, h[:, 6]
    if at.numel():
        Tp, g = _corrector(c, trial[at], h[at, 6], per[at], None if Q is None else Q[at])
        T = T.index_copy(0, at, Tp)
        ep = ep.index_copy(0, at, e[at] - _elastic(Tp, per[at], inverse=True))
        al = al.index_copy(0, at, h[at, 6] + g)
    P = torch.autograd.grad(eps, Hb, grad_outputs=_matrix(T).reshape(eps.shape), create_graph=True)[0]
    force = (dv[:, :, None, None] * (P[:, :, None, :, :] * G[:, :, :, None, :]).sum(-1)).sum(1)
    new = torch.cat((ep[:, :3], ep[:, 3:] / _R2, al[:, None]), 1)
    return force, new.reshape(-1, 8, 7)


def _spread(c, p):
    ne = p["conn"].shape[0]
    prm = p["prm"]
    if c["kind"] == "batch":
        n = torch.tensor([b - a for a, b in zip(p["off"], p["off"][1:])], device=prm.device)
        return prm.repeat_interleave(n, 0)
    return prm.expand(ne, 11) if prm.dim() == 1 else prm


def _chunks(c, p, d, size=4096):
    """Element slices with their differentiable leaves: displacements, history, parameters."""
    prm = _spread(c, p)
    for a in range(0, p["conn"].shape[0], size):
        cn = p["conn"][a:a + size]
        de = d[cn].clone().requires_grad_(True)
        h = p["hist"][:, 8 * a:8 * (a + cn.shape[0])].t().reshape(-1, 8, 7).clone().requires_grad_(True)
        th = prm[a:a + size].clone().requires_grad_(True)
        o = p["orient"]
        yield a, cn, de, h, th, _elements(c, p["X"][cn], de, h, th, o if o is None or o.shape[0] == 1 else
                                          o[a:a + size])


def _tangents(force, de):
    K = torch.empty(de.shape[0], 24, 24, dtype=F64, device=de.device)
    f = force.reshape(-1, 24)
    for i in range(24):
        K[:, i] = torch.autograd.grad(f[:, i].sum(), de, retain_graph=True)[0].reshape(-1, 24)
    return K


def _exact_pass(c, p, want_K):
    nn, ne = p["X"].shape[0], p["conn"].shape[0]
    R = torch.zeros(nn, 3, dtype=F64, device=p["X"].device)
    hist = torch.empty_like(p["hist"])
    blk = None
    if want_K:
        key = p["conn"][:, :, None] * nn + p["conn"][:, None, :]
        uniq, inv = torch.unique(key.reshape(-1), return_inverse=True)
        inv = inv.reshape(ne, 64)
        blk = torch.zeros(uniq.numel(), 9, dtype=F64, device=R.device)
    for a, cn, de, _, _, (force, new) in _chunks(c, p, p["d"], 4096 if want_K else 16384):
        R.index_add_(0, cn.reshape(-1), force.detach().reshape(-1, 3))
        hist[:, 8 * a:8 * (a + cn.shape[0])] = new.detach().reshape(-1, 7).t()
        if want_K:
            K = _tangents(force, de).reshape(-1, 8, 3, 8, 3).permute(0, 1, 3, 2, 4).reshape(-1, 9)
            blk.index_add_(0, inv[a:a + cn.shape[0]].reshape(-1), K)
    bc = p["bc"].bool().reshape(-1, 3)
    R[bc] = 0.0
    vals = None
    if want_K:
        I, J = uniq // nn, uniq % nn
        blk = blk.reshape(-1, 3, 3)
        eye = (I == J)[:, None, None] * torch.eye(3, dtype=F64, device=R.device)
        blk = torch.where(bc[I][:, :, None], eye, blk)
        vals = _csr_values(I, blk, nn)
    return R, vals, hist


def _csr_values(I, blk, nn):
    deg = torch.bincount(I, minlength=nn)
    first = torch.cumsum(deg, 0) - deg
    vals = torch.empty(9 * I.numel(), dtype=F64, device=blk.device)
    base = 9 * first[I] + 3 * (torch.arange(I.numel(), device=blk.device) - first[I])
    for a in range(3):
        for b in range(3):
            vals[base + a * 3 * deg[I] + b] = blk[:, a, b]
    return vals


def _exact_gradients(c, p, lam, mu):
    """lam.R + mu.H by parameters and history, and mu.H by displacements."""
    ne = p["conn"].shape[0]
    g = torch.zeros(7, ne, dtype=F64, device=p["X"].device)
    hbar, ubar = torch.zeros_like(p["hist"]), torch.zeros_like(p["X"])
    for a, cn, de, h, th, (force, new) in _chunks(c, p, p["d"], 16384):
        n = cn.shape[0]
        L = (force * lam[cn]).sum()
        if mu is not None:
            M = (new * mu[:, 8 * a:8 * (a + n)].t().reshape(-1, 8, 7)).sum()
            u = torch.autograd.grad(M, de, retain_graph=True)[0]
            ubar.index_add_(0, cn.reshape(-1), u.reshape(-1, 3))
            L = L + M
        t, k = torch.autograd.grad(L, (th, h))
        g[:, a:a + n] = t[:, list(_GRAD)].t()
        hbar[:, 8 * a:8 * (a + n)] = k.reshape(-1, 7).t()
    return g, hbar, ubar


def _exact_newton(c, p):
    free = ~p["bc"].bool().reshape(-1)
    d = p["d"].clone()
    q = dict(p)
    n = d.numel()
    for it in range(25):
        R = torch.zeros_like(d)
        K = torch.zeros(n, n, dtype=F64, device=d.device)
        hist = torch.empty_like(p["hist"])
        for a, cn, de, _, _, (force, new) in _chunks(c, q, d):
            R.index_add_(0, cn.reshape(-1), force.detach().reshape(-1, 3))
            hist[:, 8 * a:8 * (a + cn.shape[0])] = new.detach().reshape(-1, 7).t()
            dof = (3 * cn[:, :, None] + torch.arange(3, device=d.device)).reshape(-1, 24)
            K.view(-1).index_add_(0, (dof[:, :, None] * n + dof[:, None, :]).reshape(-1), _tangents(force, de).reshape(-1))
        du = torch.zeros(n, dtype=F64, device=d.device)
        r = R.reshape(-1)
        du[free] = torch.linalg.solve(K[free][:, free], -r[free])
        if float(du.abs().max()) < 1e-14 * float(d.abs().max()):
            return d, hist
        t, rn = 1.0, float(r[free].norm())
        for _ in range(8):
            trial = d + t * du.view(-1, 3)
            R2 = torch.zeros_like(d)
            for a, cn, _, _, _, (force, _) in _chunks(c, q, trial, 16384):
                R2.index_add_(0, cn.reshape(-1), force.detach().reshape(-1, 3))
            if float(R2.reshape(-1)[free].norm()) < rn or rn < 1e-9:
                break
            t *= 0.5
        d = trial
        if it > 5 and rn < 1e-9:
            break
    return d, hist


def _exact_solve(c, seed):
    """Conjugate gradients with the node blocks to the rounding level."""
    D, _, col, b, bc = _system(c, seed)
    M = torch.linalg.inv(D[:, 13].to(F64))

    def apply(x):
        y = _blocks_times(D, col, x)
        y[bc] = 0.0
        return y

    def precondition(r):
        z = (M * r[:, None, :]).sum(2)
        z[bc] = 0.0
        return z

    x, stop = torch.zeros_like(b), 1e-13 * float(b.norm())
    r = b.clone()
    z = precondition(r)
    q, rz = z.clone(), (r * z).sum()
    for it in range(8000):
        v = apply(q)
        a = rz / (q * v).sum()
        x += a * q
        r -= a * v
        z = precondition(r)
        rz, old = (r * z).sum(), rz
        q = z + (rz / old) * q
        if it % 50 == 49 and float(r.norm()) < stop:
            return x.reshape(-1)
    return None


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "pattern":
        return None
    if c["kind"] == "solve":
        if c["nx"] * c["ny"] * c["nz"] > 300000:
            return None
        x = _exact_solve(c, seed)
        return None if x is None else {"x": x, "iterations": None}
    if c["kind"] == "newton":
        if (c["nx"] + 1) * (c["ny"] + 1) * (c["nz"] + 1) > 7000:
            return None
        d, hist = _exact_newton(c, _load(c, seed))
        return {"d": d, "hist": hist, "iterations": None}
    p = _problem(c, seed)
    ne = p["conn"].shape[0]
    if c["yield"] == "barlat" and ne > 150000:
        return None
    r = {}
    if c["kind"] in ("pass", "batch"):
        R, K, hist = _exact_pass(c, p, ne <= 160000)
        r = {"R": R.reshape(-1), "K": K, "hist": hist, "rnorm2": (R ** 2).sum().reshape(1)}
    if c["kind"] in ("vjp", "batch"):
        g, _, _ = _exact_gradients(c, p, p["lam"], None)
        r = dict(r, g=torch.stack([g[:, a:b].sum(1) for a, b in zip(p["off"], p["off"][1:])]), g_elem=g)
    if c["kind"] == "adjoint":
        g, hbar, ubar = _exact_gradients(c, p, p["lam"], p["mu"])
        r = {"ubar": ubar, "g": g.sum(1), "g_elem": g, "hbar": hbar}
        if c["fbar"]:
            r["KT"] = None
    return r
