"""Aggregation multigrid preconditioner on the GPU (through the C ABI):
  - a hierarchy of one dense level is the exact inverse;
  - the aggregates partition each level into connected groups of at most
    eight nodes, and the level sizes agree with them;
  - one V-cycle equals a numpy V-cycle built from the documented definitions
    (masked piecewise-constant prolongation, FP32 Galerkin operators, damped
    block-Jacobi sweeps, dense coarsest inverse) on the same aggregates and
    damping factors, and the damping times the exact spectral radius of
    D^-1 A lies in [1.2, 1.6] (4/3 for an exact estimate);
  - the preconditioned CG (plain tangent) and BiCGSTAB (F-bar tangent) solves
    match a dense solve, and repeat bitwise;
  - fewer iterations than node-block Jacobi on a 16^3 plastic state, and a
    symmetric operator for a symmetric tangent.
The matrices are tangents of the unit-cube forward problem of Sec. 3.1.3 at
a trial state (x = 1 face moved by t (0.2, 0.1), t = 0.05, zero history):
every Gauss point plastic, the tangent positive definite on the free dofs."""
import dataclasses
import sys

import numpy as np
import pytest

from helpers import gpu_problem
from paper_2606_17390_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fem():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2606_17390_amd import fem as F
    F.lib()
    return F


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def cube_state(n, t=0.05, fbar=False, ny=None, nz=None):
    p = synth.unit_cube_forward(n, ny, nz)
    d = np.zeros_like(p.X)
    d[:, 0] = 0.2 * t * p.X[:, 0]
    d[:, 1] = 0.1 * t * p.X[:, 0]
    return dataclasses.replace(p, d=d, fbar=fbar)


def tangent(fem, p, prec):
    mesh, params, d, h, bc, _ = gpu_problem(p, fem)
    csr = fem.csr_pattern(mesh)
    out = fem.residual_tangent(mesh, csr, params, d, h, bc_mask=bc, prec=prec)
    torch.cuda.synchronize()
    return csr, out.K, bc


def host_csr(csr, K):
    import scipy.sparse as sp
    n = csr.n_rows
    return sp.csr_matrix((K.double().cpu().numpy(), csr.col_idx.cpu().numpy(), csr.row_ptr.cpu().numpy()),
                         shape=(n, n))


def bj_blocks(A, omega=1.0):
    """omega times the inverses of the 3x3 diagonal blocks of A (scipy)"""
    import scipy.sparse as sp
    n = A.shape[0] // 3
    coo = A.tocoo()
    inb = (coo.row // 3) == (coo.col // 3)
    D = np.zeros((n, 3, 3))
    np.add.at(D, (coo.row[inb] // 3, coo.row[inb] % 3, coo.col[inb] % 3), coo.data[inb])
    Minv = omega * np.linalg.inv(D)
    rows = np.repeat(np.arange(3 * n), 3)
    cols = (3 * (np.arange(3 * n) // 3))[:, None] + np.arange(3)[None, :]
    return sp.csr_matrix((Minv.reshape(-1), (rows, cols.reshape(-1))), shape=A.shape)


def ref_vcycle(A0, free0, aggs, omegas, r, dense=True, klevels=()):
    """V(1,1)-cycle from the definitions (host, FP64 vectors): A0 the finest
    operator (scipy CSR), free0 its free-dof mask, aggs the aggregate map of
    each level transition, omegas the smoother damping per level; the
    coarsest level inverted exactly (dense) or smoothed twice.  On the
    levels in klevels the coarse correction is the K-cycle's: two GCR steps
    with the cycle below as preconditioner (the minimal-residual combination
    of c1 = B rc and c2 = B r2)."""
    import scipy.sparse as sp

    As, Ms, Ps, masks = [A0], [], [], [free0]
    for agg in aggs:
        nf, nc = agg.size, int(agg.max()) + 1
        m = masks[-1].astype(float)
        P = sp.csr_matrix((m, (np.arange(3 * nf), 3 * np.repeat(agg, 3) + np.tile(np.arange(3), nf))),
                          shape=(3 * nf, 3 * nc))
        Ac = (P.T @ As[-1] @ P).tocsr()
        mc = np.zeros(3 * nc, dtype=bool)
        np.logical_or.at(mc, 3 * np.repeat(agg, 3) + np.tile(np.arange(3), nf), masks[-1])
        Ac = Ac + sp.diags((~mc).astype(float))
        Ac.data = Ac.data.astype(np.float32).astype(np.float64)
        Ps.append(P)
        As.append(Ac.tocsr())
        masks.append(mc)
    for A, om in zip(As, omegas):
        Ms.append(bj_blocks(A, om))
    Cinv = np.linalg.inv(As[-1].toarray()) if dense else None

    def cycle(l, b):
        if l == len(As) - 1:
            if dense:
                return Cinv @ b
            x = Ms[l] @ b
            return x + Ms[l] @ (b - As[l] @ x)
        x = Ms[l] @ b
        rc = Ps[l].T @ (b - As[l] @ x)
        c = l + 1
        if c in klevels:
            Ac = As[c]
            c1 = cycle(c, rc)
            v1 = Ac @ c1
            vv = v1 @ v1
            a1 = (v1 @ rc) / vv if vv > 0 else 0.0
            r2 = rc - a1 * v1
            c2 = cycle(c, r2)
            v2 = Ac @ c2
            g = (v2 @ v1) / vv if vv > 0 else 0.0
            den = v2 @ v2 - g * (v2 @ v1)  # |v2 - g v1|^2
            a2 = (v2 @ r2) / den if den > 0 else 0.0
            e = (a1 - a2 * g) * c1 + a2 * c2
        else:
            e = cycle(c, rc)
        x = x + Ps[l] @ e
        return x + Ms[l] @ (b - As[l] @ x)

    return cycle(0, r)


@pytest.mark.parametrize("prec_name", ["FP64", "FP32_MIXED"])
def test_single_dense_level_is_the_inverse(fem, prec_name):
    p = synth.small_slab(61, 3, 2, 1)
    assert p.n_nodes <= 32
    csr, K, bc = tangent(fem, p, getattr(fem, prec_name))
    amg = fem.AMG(csr, K, bc)
    amg.update(K)
    levels, dense = amg.info()
    say(f"dense level {prec_name}: {levels}")
    assert len(levels) == 1 and dense and levels[0][0] == p.n_nodes
    A = host_csr(csr, K).toarray()
    r = np.random.default_rng(7).standard_normal(csr.n_rows)
    z = amg.apply(torch.as_tensor(r).cuda())
    torch.cuda.synchronize()
    ref = np.linalg.solve(A, r)
    assert np.abs(z.cpu().numpy() - ref).max() <= 1e-9 * np.abs(ref).max()


def check_aggregates(G, agg):
    """agg partitions the nodes of the node graph G (scipy CSR pattern) into
    connected groups of at most eight nodes; returns their number."""
    import scipy.sparse as sp
    import scipy.sparse.csgraph as cg
    n = G.shape[0]
    assert agg.shape == (n,) and agg.min() == 0
    nc = int(agg.max()) + 1
    sizes = np.bincount(agg, minlength=nc)
    assert sizes.min() >= 1 and sizes.max() <= 8
    coo = G.tocoo()
    same = agg[coo.row] == agg[coo.col]
    Gin = sp.csr_matrix((np.ones(same.sum()), (coo.row[same], coo.col[same])), shape=(n, n))
    ncomp, _ = cg.connected_components(Gin, directed=False)
    assert ncomp == nc  # one component per aggregate
    return nc


@pytest.mark.parametrize("prec_name", ["FP64", "FP32_MIXED"])
def test_hierarchy_and_vcycle_match_the_definitions(fem, prec_name):
    import scipy.sparse as sp
    p = cube_state(10, ny=9, nz=7)
    csr, K, bc = tangent(fem, p, getattr(fem, prec_name))
    amg = fem.AMG(csr, K, bc)
    amg.update(K)
    levels, dense, omegas = amg.info(omega=True)
    say(f"hierarchy {prec_name}: {levels} dense {dense} omega {omegas}")
    assert len(levels) >= 3 and dense and levels[0] == (p.n_nodes, csr.nnz // 9)
    assert levels[-1][0] <= fem.AMG_DENSE_NODES and omegas[-1] == 1.0
    A0 = host_csr(csr, K)
    free0 = p.bc_mask == 0
    coo = A0.tocoo()
    G = sp.csr_matrix((np.ones(coo.nnz), (coo.row // 3, coo.col // 3)), shape=(p.n_nodes, p.n_nodes))
    aggs = []
    for l in range(1, len(levels)):
        agg = amg.aggregates(l)
        nc = check_aggregates(G, agg)
        assert nc == levels[l][0]
        # the coarse pattern: one block per pair of aggregates joined by a fine block
        Pn = sp.csr_matrix((np.ones(agg.size), (np.arange(agg.size), agg)), shape=(agg.size, nc))
        G = (Pn.T @ G @ Pn).tocsr()
        assert G.nnz == levels[l][1]
        aggs.append(agg)
    # the damping against the spectral radius of D^-1 A on the free dofs
    Dinv = bj_blocks(A0).toarray()
    rho = np.abs(np.linalg.eigvals((Dinv @ A0.toarray())[np.ix_(free0, free0)])).max()
    say(f"  level 0: omega {omegas[0]:.4f}, rho {rho:.4f}, omega rho {omegas[0] * rho:.3f}")
    assert 1.2 <= omegas[0] * rho <= 1.6
    rng = np.random.default_rng(11)
    for trial in range(2):
        r = rng.standard_normal(csr.n_rows) * free0
        z = amg.apply(torch.as_tensor(r).cuda())
        torch.cuda.synchronize()
        ref = ref_vcycle(A0, free0, aggs, omegas, r)
        err = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
        say(f"  V-cycle {trial}: rel err {err:.2e}")
        assert err <= 2e-6
        assert np.all(z.cpu().numpy()[~free0] == 0.0)


@pytest.mark.parametrize("prec_name", ["FP64", "FP32_MIXED"])
@pytest.mark.parametrize("fbar,method", [(False, "cg"), (True, "bicgstab"), (True, "gmres"), (False, "gmres")])
def test_preconditioned_solve_matches_dense_solve(fem, prec_name, fbar, method):
    """CG on the plain (symmetric) tangent, BiCGSTAB and GMRES on the F-bar
    one, GMRES on both; the right-hand side is zero on the constrained dofs
    (a Newton correction)."""
    p = cube_state(7, fbar=fbar, ny=6, nz=5)
    csr, K, bc = tangent(fem, p, getattr(fem, prec_name))
    A = host_csr(csr, K).toarray()
    b = np.random.default_rng(5).standard_normal(csr.n_rows)
    b[p.bc_mask.astype(bool)] = 0.0
    s = fem.Solver(csr, precond=fem.PC_AMG, method=method, bc_mask=bc)
    x, its, res = s.solve(K, torch.as_tensor(b).cuda(), rtol=1e-12)
    torch.cuda.synchronize()
    say(f"AMG {method} {prec_name}: {its} iterations, res {res:.2e}, levels {s.amg.info()}")
    ref = np.linalg.solve(A, b)
    assert res <= 1e-12 and its > 0
    assert np.abs(x.cpu().numpy() - ref).max() <= 1e-8 * np.abs(ref).max()
    assert np.linalg.norm(b - A @ x.cpu().numpy()) <= 1e-9 * np.linalg.norm(b)
    x2, its2, _ = s.solve(K, torch.as_tensor(b).cuda(), rtol=1e-12)
    assert its2 == its and torch.equal(x, x2)


def test_fewer_iterations_than_block_jacobi_and_symmetric(fem):
    p = cube_state(16)
    csr, K, bc = tangent(fem, p, fem.FP64_K32)
    b = np.random.default_rng(9).standard_normal(csr.n_rows)
    b[p.bc_mask.astype(bool)] = 0.0
    bt = torch.as_tensor(b).cuda()
    s = fem.Solver(csr, precond=fem.PC_AMG, method="cg", bc_mask=bc)
    x, its_amg, res = s.solve(K, bt, rtol=1e-8, max_iter=20000)
    _, its_bj, res_bj = s.solve(K, bt, rtol=1e-8, max_iter=20000, precond=fem.PC_BLOCK_JACOBI)
    torch.cuda.synchronize()
    say(f"16^3 CG to 1e-8: AMG {its_amg} ({res:.1e}), block Jacobi {its_bj} ({res_bj:.1e}), levels {s.amg.info()}")
    assert res <= 1e-8 and res_bj <= 1e-8
    assert its_amg * 3 < its_bj
    # M symmetric for the symmetric free-free block
    free = torch.as_tensor(p.bc_mask == 0).cuda()
    rng = np.random.default_rng(10)
    u = torch.as_tensor(rng.standard_normal(csr.n_rows)).cuda() * free
    v = torch.as_tensor(rng.standard_normal(csr.n_rows)).cuda() * free
    Mu, Mv = s.amg.apply(u), s.amg.apply(v)
    a, c = float(torch.dot(v, Mu)), float(torch.dot(u, Mv))
    say(f"  v.Mu {a:.12e} u.Mv {c:.12e}")
    assert abs(a - c) <= 1e-6 * max(abs(a), abs(c))
    assert float(torch.dot(u, Mu)) > 0.0


@pytest.mark.parametrize("case", ["all_decoupled", "half_decoupled"])
def test_stalled_coarsening_paths(fem, case):
    """Coupling blocks of some nodes zeroed (rows and columns, the pattern
    kept), so the matching finds no partner for them and the coarsening
    stalls: with every node decoupled the hierarchy is one level that is not
    inverted exactly (two damped block-Jacobi sweeps); with half of them the
    coarsest level keeps more than 512 nodes (no single-workgroup tail, no
    dense inverse).  The cycle equals the numpy cycle on the same
    aggregates and damping."""
    import scipy.sparse as sp
    p = cube_state(14, ny=12, nz=10)
    csr, K, bc = tangent(fem, p, fem.FP64)
    A = host_csr(csr, K).tocoo()
    n = p.n_nodes
    dec = np.ones(n, bool) if case == "all_decoupled" else (np.arange(n) < n // 2)
    bi, bj = A.row // 3, A.col // 3
    keep = (bi == bj) | ~(dec[bi] | dec[bj])
    vals = np.where(keep, A.data, 0.0)
    # back into the CSR order of csr (coo of a csr keeps the order)
    K2 = torch.as_tensor(vals).cuda()
    amg = fem.AMG(csr, K2, bc)
    amg.update(K2)
    levels, dense, omegas = amg.info(omega=True)
    say(f"{case}: levels {levels} dense {dense} omega {omegas}")
    if case == "all_decoupled":
        assert len(levels) == 1 and not dense
    else:
        assert not dense and levels[-1][0] > 512
    A0 = sp.csr_matrix((vals, (A.row, A.col)), shape=A.shape)
    free0 = p.bc_mask == 0
    aggs = [amg.aggregates(l) for l in range(1, len(levels))]
    r = np.random.default_rng(12).standard_normal(csr.n_rows) * free0
    z = amg.apply(torch.as_tensor(r).cuda())
    torch.cuda.synchronize()
    ref = ref_vcycle(A0, free0, aggs, omegas, r, dense=False)
    err = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
    say(f"  rel err {err:.2e}")
    assert err <= 2e-6


@pytest.mark.parametrize("method", ["cg", "bicgstab"])
def test_voided_sheet_solve_matches_dense_solve(fem, method):
    """An irregular mesh: a 24 x 24 x 2 sheet with a quarter of its element
    columns removed along a random field (holes and narrow ligaments, the
    bottom face clamped), its plain Hill-48 tangent at a plastic state.  The
    aggregates stay connected and the multigrid-preconditioned solve matches
    a dense solve."""
    import scipy.sparse as sp
    p = synth.void_specimen(seed=21, nx=24, ny=24, nz=2)
    csr, K, bc = tangent(fem, p, fem.FP64)
    A = host_csr(csr, K)
    b = np.random.default_rng(8).standard_normal(csr.n_rows)
    b[p.bc_mask.astype(bool)] = 0.0
    s = fem.Solver(csr, precond=fem.PC_AMG, method=method, bc_mask=bc)
    x, its, res = s.solve(K, torch.as_tensor(b).cuda(), rtol=1e-12, max_iter=5000)
    torch.cuda.synchronize()
    levels, dense = s.amg.info()
    say(f"voided sheet {method}: {p.n_nodes} nodes, {its} iterations, levels {levels}")
    ref = np.linalg.solve(A.toarray(), b)
    assert res <= 1e-12
    assert np.abs(x.cpu().numpy() - ref).max() <= 1e-8 * np.abs(ref).max()
    coo = A.tocoo()
    G = sp.csr_matrix((np.ones(coo.nnz), (coo.row // 3, coo.col // 3)), shape=(p.n_nodes, p.n_nodes))
    agg = s.amg.aggregates(1)
    check_aggregates(G, agg)


def k_levels(levels, k_min_nodes):
    """Levels that take the K-cycle's two Krylov steps: above the first
    level of at most 512 nodes, not the coarsest, at least k_min_nodes nodes."""
    nl = len(levels)
    t = next((l for l in range(1, nl) if levels[l][0] <= 512), nl)
    return {c for c in range(1, nl) if c < t and c < nl - 1 and levels[c][0] >= k_min_nodes}


@pytest.mark.parametrize("n,fbar,k_min", [(24, False, 0), (32, True, 0), (24, False, 10 ** 9)])
def test_kcycle_matches_the_definition(fem, n, fbar, k_min):
    """The K-cycle against the numpy cycle on the same aggregates and damping
    (the plain tangent and the nonsymmetric F-bar one; with k_min above every
    level it is the V-cycle), and two applications agree bitwise (the
    device-side sums restart cleanly)."""
    p = cube_state(n, fbar=fbar)
    csr, K, bc = tangent(fem, p, fem.FP64)
    amg = fem.AMG(csr, K, bc)
    amg.update(K)
    amg.set_cycle("k", k_min)
    levels, dense, omegas = amg.info(omega=True)
    kl = k_levels(levels, k_min)
    say(f"K-cycle {n}^3 fbar={fbar} k_min={k_min}: levels {levels}, Krylov levels {sorted(kl)}")
    assert dense and (len(kl) >= (2 if n == 32 else 1) or k_min > 0)
    A0 = host_csr(csr, K)
    free0 = p.bc_mask == 0
    aggs = [amg.aggregates(l) for l in range(1, len(levels))]
    r = np.random.default_rng(13).standard_normal(csr.n_rows) * free0
    rt = torch.as_tensor(r).cuda()
    z = amg.apply(rt)
    z2 = amg.apply(rt)
    torch.cuda.synchronize()
    ref = ref_vcycle(A0, free0, aggs, omegas, r, klevels=kl)
    err = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
    say(f"  rel err {err:.2e}")
    assert err <= 2e-6
    assert torch.equal(z, z2)
    assert np.all(z.cpu().numpy()[~free0] == 0.0)
    if k_min > 0:
        amg.set_cycle("v")
        assert torch.equal(amg.apply(rt), z)


@pytest.mark.parametrize("prec_name", ["FP64", "FP32_MIXED"])
@pytest.mark.parametrize("fbar", [False, True])
def test_flexible_gmres_with_kcycle_matches_sparse_solve(fem, prec_name, fbar):
    """FGMRES preconditioned by the K-cycle solves the 24^3 tangent (plain and
    F-bar) to the sparse direct solution, in fewer iterations than FGMRES
    with the V-cycle; FGMRES with block Jacobi (a fixed preconditioner)
    forms the GMRES iterate; a K-cycle with a method that is not
    flexible is rejected."""
    import ctypes
    import scipy.sparse.linalg as spla
    p = cube_state(24, fbar=fbar)
    csr, K, bc = tangent(fem, p, getattr(fem, prec_name))
    A = host_csr(csr, K).tocsc()
    b = np.random.default_rng(6).standard_normal(csr.n_rows)
    b[p.bc_mask.astype(bool)] = 0.0
    bt = torch.as_tensor(b).cuda()
    ref = spla.spsolve(A, b)
    s = fem.Solver(csr, precond=fem.PC_AMG, method="fgmres", bc_mask=bc)
    x, its_k, res = s.solve(K, bt, rtol=1e-10, max_iter=2000)
    x2, its_k2, _ = s.solve(K, bt, rtol=1e-10, max_iter=2000)
    sv = fem.Solver(csr, precond=fem.PC_AMG, method="fgmres", bc_mask=bc, cycle="v")
    xv, its_v, res_v = sv.solve(K, bt, rtol=1e-10, max_iter=2000)
    torch.cuda.synchronize()
    say(f"24^3 fbar={fbar} {prec_name}: FGMRES K-cycle {its_k} ({res:.1e}), V-cycle {its_v} ({res_v:.1e}), "
        f"levels {s.amg.info()}")
    assert res <= 1e-10 and res_v <= 1e-10
    for xs in (x, xv):
        assert np.abs(xs.cpu().numpy() - ref).max() <= 1e-7 * np.abs(ref).max()
    assert its_k < its_v
    assert its_k2 == its_k and torch.equal(x, x2)
    # within one restart cycle FGMRES with a fixed preconditioner forms the
    # GMRES iterate (x0 + Z y = x0 + M V y)
    sb = fem.Solver(csr, precond=fem.PC_BLOCK_JACOBI, method="fgmres")
    xb, its_b, res_b = sb.solve(K, bt, rtol=1e-14, max_iter=25, check=False)
    xg, its_g, res_g = sb.solve(K, bt, rtol=1e-14, max_iter=25, method="gmres", check=False)
    torch.cuda.synchronize()
    dx = float((xb - xg).abs().max() / xg.abs().max())
    say(f"  block Jacobi, 25 steps: FGMRES res {res_b:.3e}, GMRES res {res_g:.3e}, rel diff {dx:.1e}")
    assert its_b == its_g == 25 and dx <= 1e-9 and abs(res_b - res_g) <= 1e-9 * res_g
    # the K-cycle with CG is refused (the cycle is not a fixed linear operator)
    s.amg.set_cycle("k")
    it, rr = ctypes.c_int32(0), ctypes.c_double(0.0)
    rc = fem.lib().fem_solve_amg(ctypes.byref(csr.c()), fem._ptr(K), fem._kprec(K), fem.KRYLOV["cg"], s.amg.h,
                                 fem._ptr(bt), fem._ptr(torch.zeros_like(bt)), 10, 1e-8, ctypes.byref(it),
                                 ctypes.byref(rr), fem._ptr(s.ws), s.ws_bytes, None)
    assert rc == fem.FEM_EINVAL and b"flexible" in fem.lib().fem_last_error()
    # the cycle setter checks its arguments on a live handle
    assert fem.lib().fem_amg_set_cycle(s.amg.h, 7, 0) == fem.FEM_EINVAL
    assert fem.lib().fem_amg_set_cycle(s.amg.h, fem.AMG_CYCLE["k"], -1) == fem.FEM_EINVAL


def test_fgmres_kcycle_full_size_true_residual(fem):
    """The 100^3 unit cube (3,090,903 dofs): FGMRES with the K-cycle on the
    elastic tangent of the undeformed cube with the first load increment's
    right-hand side reaches rtol 1e-8 by the true residual b - K x (the CSR
    product, itself checked against scipy), with the hierarchy's Krylov
    levels in use, and repeats bitwise."""
    p = synth.unit_cube_forward(100)
    mesh, params, d, h, bc, _ = gpu_problem(p, fem)
    csr = fem.csr_pattern(mesh)
    params = fem.Params(p.prm, p.n_elems, hardening="voce")
    h0 = torch.zeros((7, 8 * p.n_elems), dtype=torch.float64, device="cuda")
    u = torch.as_tensor(p.meta["bc_at"](1e-3)).cuda()
    K = fem.residual_tangent(mesh, csr, params, torch.zeros_like(u), h0, bc_mask=bc, prec=fem.FP64_K32).K
    b = -fem.residual_tangent(mesh, csr, params, u, h0, bc_mask=bc, prec=fem.FP64, want_K=False).R
    s = fem.Solver(csr, precond=fem.PC_AMG, method="fgmres", bc_mask=bc)
    x, its, res = s.solve(K, b, rtol=1e-8, max_iter=500)
    x2, its2, _ = s.solve(K, b, rtol=1e-8, max_iter=500)
    r = b - fem.csr_spmv(csr, K, x)
    true = float(r.norm() / b.norm())
    levels, _ = s.amg.info()
    kl = k_levels(levels, 0)
    torch.cuda.synchronize()
    say(f"100^3 FGMRES K-cycle: {its} iterations, recursive {res:.2e}, true {true:.2e}, levels {levels}, "
        f"Krylov levels {sorted(kl)}")
    assert len(kl) >= 2 and its <= 60
    assert res <= 1e-8 and true <= 1.5e-8
    assert its2 == its and torch.equal(x, x2)


def test_a_body_that_is_not_finite_stays_by_itself(fem):
    """Forty disjoint cubes, whose hierarchy ends in forty nodes without
    couplings (no dense inverse): a right-hand side that is not a number in one
    body leaves the cycle's result on the others as it is."""
    n = 40
    Xc, cc = synth.hex_grid(1, 1, 1, 1.0, 1.0, 1.0)
    X = np.concatenate([Xc + np.array([2.0 * i, 0.0, 0.0]) for i in range(n)])
    conn = np.concatenate([cc + 8 * i for i in range(n)]).astype(np.int32)
    bc = np.zeros(24 * n, np.uint8)
    bc.reshape(n, 8, 3)[:, :2] = 1
    p = synth.Problem("bodies", X, conn, np.zeros_like(X), np.zeros((7, 8 * n)), synth.params(), bc, None)
    csr, K, bcm = tangent(fem, p, fem.FP64)
    amg = fem.AMG(csr, K, bcm)
    amg.update(K)
    levels, dense = amg.info()
    say(f"disjoint bodies: levels {levels} dense {dense}")
    assert [l[0] for l in levels] == [8 * n, n] and not dense
    r = np.random.default_rng(15).standard_normal(csr.n_rows) * (bc == 0)
    z = amg.apply(torch.as_tensor(r).cuda())
    r[23] = np.nan  # a free dof of the first body
    zn = amg.apply(torch.as_tensor(r).cuda())
    torch.cuda.synchronize()
    assert torch.isfinite(z).all() and torch.isnan(zn[23])
    assert torch.equal(zn[24:], z[24:])


def tail_segments(csr, aggs, t):
    """Segments of four blocks of level t's rows, from the pattern of K and the
    aggregates."""
    import scipy.sparse as sp
    rp, ci = csr.row_ptr.cpu().numpy(), csr.col_idx.cpu().numpy()
    n = csr.n_rows // 3
    deg = np.diff(rp)[::3] // 3
    first = np.repeat(rp[:-1:3], deg) + 3 * (np.arange(deg.sum()) - np.repeat(np.cumsum(deg) - deg, deg))
    G = sp.csr_matrix((np.ones(deg.sum()), ci[first] // 3, np.concatenate([[0], np.cumsum(deg)])), shape=(n, n))
    for agg in aggs[:t]:
        P = sp.csr_matrix((np.ones(agg.size), (np.arange(agg.size), agg)))
        G = (P.T @ G @ P).tocsr()
    return int((-(-np.diff(G.indptr) // 4)).sum())


@pytest.mark.parametrize("cycle", ["v", "k"])
def test_tail_too_large_to_be_packed_matches_the_definition(fem, cycle):
    """A 30^3 cube, whose first level of at most 512 nodes has more than the
    2,048 segments of four blocks that the packed single-workgroup tail holds:
    the cycle through the unpacked one equals the numpy cycle."""
    p = cube_state(30)
    csr, K, bc = tangent(fem, p, fem.FP64)
    amg = fem.AMG(csr, K, bc)
    amg.update(K)
    amg.set_cycle(cycle, 0 if cycle == "k" else None)
    levels, dense, omegas = amg.info(omega=True)
    aggs = [amg.aggregates(l) for l in range(1, len(levels))]
    t = next(l for l in range(1, len(levels)) if levels[l][0] <= 512)
    seg = tail_segments(csr, aggs, t)
    say(f"unpacked tail, {cycle}-cycle: levels {levels}, tail from level {t}, {seg} segments")
    assert dense and seg > 2048
    A0 = host_csr(csr, K)
    free0 = p.bc_mask == 0
    r = np.random.default_rng(16).standard_normal(csr.n_rows) * free0
    rt = torch.as_tensor(r).cuda()
    z, z2 = amg.apply(rt), amg.apply(rt)
    torch.cuda.synchronize()
    ref = ref_vcycle(A0, free0, aggs, omegas, r, klevels=k_levels(levels, 0) if cycle == "k" else ())
    err = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
    say(f"  rel err {err:.2e}")
    assert err <= 2e-6
    assert torch.equal(z, z2)


def device_cycle(row_ptr, col, val, free, aggs, omegas, r, klevels):
    """ref_vcycle on the device (torch, FP64), for systems too large for the
    host: the finest operator in CSR form, node blocks of coarse operators
    summed by key."""
    def operator(I, J, B, n):
        # CSR of node blocks B [nb, 3, 3] sorted by (I, J)
        deg = torch.bincount(I, minlength=n)
        bp = torch.cat([deg.new_zeros(1), torch.cumsum(deg, 0)])
        k = torch.arange(I.numel(), device=I.device) - bp[I]
        at = 9 * bp[I] + 3 * k
        v = torch.empty(9 * I.numel(), dtype=torch.float64, device=I.device)
        c = torch.empty(9 * I.numel(), dtype=torch.int64, device=I.device)
        for a in range(3):
            for b in range(3):
                v[at + a * 3 * deg[I] + b] = B[:, a, b]
                c[at + a * 3 * deg[I] + b] = 3 * J + b
        rp = (9 * bp[:-1, None] + 3 * deg[:, None] * torch.arange(3, device=I.device)).reshape(-1)
        return torch.sparse_csr_tensor(torch.cat([rp, 9 * bp[-1:]]), c, v, size=(3 * n, 3 * n))

    def smoother(I, J, B, omega):
        M = omega * torch.linalg.inv(B[I == J])
        return lambda x: (M @ x.view(-1, 3, 1)).view(-1)

    n = row_ptr.numel() // 3
    row_ptr, col = row_ptr.long(), col.long()
    deg = (row_ptr[1::3] - row_ptr[:-1:3]) // 3
    I = torch.repeat_interleave(torch.arange(n, device=col.device), deg)
    base = row_ptr[3 * I] + 3 * (torch.arange(I.numel(), device=col.device) - (row_ptr[:-1:3] // 9)[I])
    J = col[base] // 3
    B = torch.stack([val[base + a * 3 * deg[I] + b].double() for a in range(3) for b in range(3)], 1).view(-1, 3, 3)
    As = [torch.sparse_csr_tensor(row_ptr, col, val.double(), size=(3 * n, 3 * n))]
    Ms, masks = [smoother(I, J, B, omegas[0])], [free]
    for l, agg in enumerate(aggs, start=1):
        nc, m = int(agg.max()) + 1, masks[-1].view(-1, 3).double()
        B *= m[I][:, :, None] * m[J][:, None, :]
        key, inv = torch.unique(agg[I] * nc + agg[J], return_inverse=True)
        B = torch.zeros((key.numel(), 9), dtype=torch.float64, device=B.device).index_add_(0, inv, B.reshape(-1, 9))
        B = B.view(-1, 3, 3)
        I, J = key // nc, key % nc
        mc = torch.zeros((nc, 3), device=B.device).index_add_(0, agg, m.float()) > 0
        B[I == J] += torch.diag_embed((~mc).double())
        B = B.float().double()
        As.append(operator(I, J, B, nc))
        Ms.append(smoother(I, J, B, omegas[l]))
        masks.append(mc.view(-1))
    C = torch.linalg.inv(As[-1].to_dense())

    def cycle(l, b):
        if l == len(As) - 1:
            return C @ b
        x = Ms[l](b)
        agg, m, nc = aggs[l], masks[l].double(), masks[l + 1].numel() // 3
        rc = torch.zeros((nc, 3), dtype=torch.float64, device=b.device)
        rc = rc.index_add_(0, agg, (m * (b - As[l] @ x)).view(-1, 3)).view(-1)
        if l + 1 in klevels:
            A = As[l + 1]
            c1 = cycle(l + 1, rc)
            v1 = A @ c1
            vv = v1 @ v1
            a1 = (v1 @ rc) / vv
            r2 = rc - a1 * v1
            c2 = cycle(l + 1, r2)
            v2 = A @ c2
            g = (v2 @ v1) / vv
            a2 = (v2 @ r2) / (v2 @ v2 - g * (v2 @ v1))
            e = (a1 - a2 * g) * c1 + a2 * c2
        else:
            e = cycle(l + 1, rc)
        x = x + m * e.view(-1, 3)[agg].reshape(-1)
        return x + Ms[l](b - As[l] @ x)

    return cycle(0, r)


@pytest.mark.parametrize("n", [24, 105])
def test_kcycle_on_the_device_matches_the_definition(fem, n):
    """The K-cycle against its definition evaluated with torch: on 105^3
    elements, where the finest level and the first coarse one are so large (more
    than 131,072 nodes) that the coefficients of their Krylov steps come from
    kernels of their own, and on 24^3, where every consumer forms them."""
    p = cube_state(n)
    csr, K, bc = tangent(fem, p, fem.FP64_K32)
    amg = fem.AMG(csr, K, bc)
    amg.update(K)
    amg.set_cycle("k", 0)
    levels, dense, omegas = amg.info(omega=True)
    kl = k_levels(levels, 0)
    say(f"K-cycle {n}^3 on the device: levels {levels}, Krylov levels {sorted(kl)}")
    assert dense and 1 in kl and (levels[1][0] > 131072) == (n == 105)
    aggs = [torch.as_tensor(amg.aggregates(l)).cuda().long() for l in range(1, len(levels))]
    free = bc == 0
    r = torch.randn(csr.n_rows, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(17))
    r *= free
    z = amg.apply(r)
    ref = device_cycle(csr.row_ptr, csr.col_idx, K, free, aggs, omegas, r, kl)
    err = float((z - ref).abs().max() / ref.abs().max())
    say(f"  rel err {err:.2e}")
    assert err <= 2e-6
    assert torch.equal(amg.apply(r), z) and bool((z[~free] == 0).all())
