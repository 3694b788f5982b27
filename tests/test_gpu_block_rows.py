"""The node-block products of the Krylov solve on both sides of the line
between the direct and the staged form (32,768 nodes), with ragged last chunks
and with rows too long for the staging buffer: BiCGSTAB on a diagonally
dominant matrix of that pattern reaches its tolerance by the true residual."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fem():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2606_17390_amd import fem as F
    F.lib()
    return F


def _system(n, degrees, dtype):
    """Node blocks I -> I, I + 1, ..., (cyclic), degrees[I] of them per node."""
    deg = np.asarray(degrees)
    first = np.concatenate([[0], np.cumsum(deg)])
    node = np.repeat(np.arange(n), deg)
    col = (node + np.arange(first[-1]) - first[node]) % n
    order = np.lexsort((col, node))
    col = col[order]
    rng = np.random.default_rng(11)
    blk = rng.standard_normal((first[-1], 3, 3))
    blk[col == node] += 4.0 * np.sqrt(deg.max()) * 3 * np.eye(3)
    vals = np.empty(9 * first[-1])
    base = 9 * first[node] + 3 * (np.arange(first[-1]) - first[node])
    for a in range(3):
        for b in range(3):
            vals[base + a * 3 * deg[node] + b] = blk[:, a, b]
    cols = np.empty(9 * first[-1], dtype=np.int32)
    for a in range(3):
        for b in range(3):
            cols[base + a * 3 * deg[node] + b] = 3 * col + b
    row_ptr = np.append((9 * first[:-1, None] + 3 * deg[:, None] * np.arange(3)).ravel(), 9 * first[-1])
    to = lambda v: torch.as_tensor(v).to("cuda")  # noqa: E731
    return to(row_ptr.astype(np.int32)), to(cols), to(vals).to(dtype)


CASES = {
    "direct_edge": (32768, lambda n: np.full(n, 9)),
    "staged_one_more": (32769, lambda n: np.full(n, 9)),
    "staged_ragged": (33003, lambda n: 1 + np.arange(n) % 27),
    "staged_full_27": (32800, lambda n: np.full(n, 27)),
    "rows_too_long": (32801, lambda n: np.full(n, 41)),
    "some_too_long": (32817, lambda n: np.where(np.arange(n) % 4000 < 1500, 45, 3)),
}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", list(CASES))
def test_product_inside_a_solve(fem, name, dtype):
    n, degrees = CASES[name]
    print(name, dtype, flush=True)
    row_ptr, col, K = _system(n, degrees(n), dtype)
    csr = fem.Csr(row_ptr, col, None, int(col.numel()), 3 * n, row_ptr, col)
    b = torch.randn(3 * n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    solver = fem.Solver(csr, "cuda", precond=fem.PC_BLOCK_JACOBI, method="bicgstab")
    x, its, res = solver.solve(K, b, rtol=1e-10, max_iter=200)
    A = torch.sparse_csr_tensor(row_ptr.long(), col.long(), K.double(), size=(3 * n, 3 * n))
    true = float((b - A @ x).norm() / b.norm())
    assert its > 1 and res <= 1e-10 and true <= 1e-9
    # the standalone product over the same rows
    if name in ("staged_ragged", "some_too_long"):
        y = fem.csr_spmv(csr, K, x)
        assert float((y - A @ x).norm() / y.norm()) <= 1e-13


@pytest.mark.parametrize("method", ["gmres", "fgmres"])
@pytest.mark.parametrize("n", [1, 85, 10922, 10923, 21845, 21846, 349526])
def test_gram_schmidt_sizes(fem, n, method):
    """GMRES around the lines of its vector kernels (one entry per thread up to
    65,536 unknowns; the partial products summed by the update up to 128
    workgroups; several pieces per workgroup past 1,048,576)."""
    print(n, method, flush=True)
    row_ptr, col, K = _system(n, np.full(n, min(n, 3)), torch.float64)
    csr = fem.Csr(row_ptr, col, None, int(col.numel()), 3 * n, row_ptr, col)
    b = torch.randn(3 * n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    solver = fem.Solver(csr, "cuda", precond=fem.PC_JACOBI, method=method)
    x, its, res = solver.solve(K, b, rtol=1e-10, max_iter=400)
    y, _, _ = solver.solve(K, b, rtol=1e-10, max_iter=400)
    A = torch.sparse_csr_tensor(row_ptr.long(), col.long(), K, size=(3 * n, 3 * n))
    assert its > 1 and float((b - A @ x).norm() / b.norm()) <= 1e-9
    assert torch.equal(x, y)
