"""Which Gauss-Seidel levels invert their blocks, and the inverted blocks after an
update and on sliced rows.

Levels with long rows whose blocks are small, or whose rows couple outside
their block, keep the substitution: their inverses would be many times the
matrix (32 KB a block of any size below 64 rows).
"""
import numpy as np
import pytest
import scipy.sparse as sp

import paper_2210_16660_amd as pamg
from workloads import CSR, q1_stretched, uniform_rhs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def laplacian(M):
    """A symmetric weight matrix as the CSR of an M-matrix, 1 % more on the diagonal."""
    M = M.tocsr()
    M.setdiag(0)
    M.eliminate_zeros()
    M = (sp.diags(np.asarray(M.sum(1)).ravel() * 1.01) - M).tocsr()
    M.sort_indices()
    return CSR(M.shape[0], M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data)


def stencil125(n, seed):
    """All neighbours within two steps in each direction of an n^3 grid, random weights."""
    T = sp.diags([1.0] * 5, [-2, -1, 0, 1, 2], shape=(n, n))
    w = sp.diags(1.0 + np.random.default_rng(seed).random(n ** 3))
    return laplacian(w @ sp.kron(sp.kron(T, T), T) @ w)


def scattered(n, seed):
    """80 couplings a row to anywhere."""
    rng = np.random.default_rng(seed)
    i, j = np.repeat(np.arange(n), 40), rng.integers(0, n, 40 * n)
    M = sp.csr_matrix((1.0 + rng.random(40 * n), (i, j)), shape=(n, n))
    return laplacian(M + M.T)


def wide_band(n, reach, seed):
    """Rows of 2 reach + 1 consecutive columns, built row by row without a sparse product."""
    rng = np.random.default_rng(seed)
    v = np.zeros((n, 2 * reach + 1))
    for d in range(1, reach + 1):
        w = -1.0 - rng.random(n - d)
        v[:n - d, reach + d] = w
        v[d:, reach - d] = w
    v[:, reach] = -1.01 * v.sum(1)
    c = np.arange(n, dtype=np.int32)[:, None] + np.arange(-reach, reach + 1, dtype=np.int32)
    inside = (c >= 0) & (c < n)
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(inside.sum(1), out=rp[1:])
    return CSR(n, rp, c[inside], v[inside])


@pytest.mark.parametrize("device", [0, 1])
def test_blocks_that_do_not_pay_are_not_inverted(device):
    """Device bytes beyond the block schedule (8 bytes a block) do not grow as blocks shrink, but
    for small inverses (16 MB a level at five entries before a row)."""
    for A, kw in ((stencil125(22, 5), {}), (q1_stretched(16, 1.05), dict(agg_steps=3, smooth_prolongator=1))):
        size = {}
        for nb in (1, 8, 16, 256):
            H = pamg.Hierarchy(A, smoother="hgs", gs_block=nb, build_f32=1, device_setup=device, **kw)
            rows = sum(H.level_sizes()[0])
            size[nb] = H.info().device_bytes
        assert max(size[1], size[8], size[16]) <= size[256] + 16 * rows + (20 << 20), size
    B = scattered(12000, 6)                       # half a coupling in the block on average
    size = {nb: pamg.Hierarchy(B, smoother="hgs", gs_block=nb, max_levels=2, device_setup=device).info().device_bytes
            for nb in (1, 64, 256)}
    assert max(size.values()) <= min(size.values()) + 16 * 18000, size


@pytest.mark.parametrize("n", [12, 22])           # built on the host and on the device
@pytest.mark.parametrize("nb", [16, 40, 256])
def test_inverted_blocks_follow_new_coefficients(n, nb):
    # four times the matrix: the same aggregates, every value four times
    A = stencil125(n, 7)
    A4 = CSR(A.n, A.row_ptr, A.col, 4.0 * A.val)
    kw = dict(smoother="hgs", gs_block=nb, sweeps=2, build_f32=1)
    U, F, O = pamg.Hierarchy(A, **kw), pamg.Hierarchy(A4, **kw), pamg.Hierarchy(A, **kw)
    U.update_values(dev(A4.val))
    r, x0 = dev(uniform_rhs(A.n, 1)), dev(uniform_rhs(A.n, 2))
    for prec in (pamg.PREC_F64, pamg.PREC_F32):
        for start in (None, x0):
            got = []
            for H in (U, F, O):
                y = torch.empty_like(r)
                H.debug_apply(pamg.OP_SMOOTH, 0, r, y, in1=start, precision=prec)
                got.append(y.cpu().numpy().view(np.uint64))
            assert np.array_equal(got[0], got[1])
            assert not np.array_equal(got[0], got[2])
    b, xs = dev(uniform_rhs(A.n, 3)), []
    for H in (U, F):
        x = torch.zeros_like(b)
        H.solve(b, x, tol=1e-8)
        xs.append(x.cpu().numpy().view(np.uint64))
    assert np.array_equal(*xs)


@pytest.mark.parametrize("nb,strips", [(8, 0), (40, 1), (256, 4)])
def test_a_timed_sweep_counts_the_bytes_of_its_kernel(nb, strips):
    # strips: 64-row strips of an inverted block (0: substitution)
    A = stencil125(12, 7)
    H = pamg.Hierarchy(A, smoother="hgs", gs_block=nb, build_f32=1)
    n, nnz, blocks = A.n, len(A.col), -(-A.n // nb)
    for prec, sz in ((pamg.PREC_F64, 8), (pamg.PREC_F32, 4)):
        matrix = H.time_op(pamg.OP_SPMV, 0, 1, prec)[1] - n * (sz + 8)
        if strips:
            want = matrix + blocks * strips * (strips + 1) // 2 * 64 * 64 * sz + n * (8 + 5 * sz)
        else:
            want = nnz * (4 + sz) + 4 * (n + 1) + n * (8 + 3 * sz + 1) + 8 * blocks
        assert H.time_op(pamg.OP_SMOOTH, 0, 1, prec)[1] == want


def hierarchical_order(H):
    """Position of every level-0 row in nested-aggregate order."""
    sizes = H.level_sizes()[0]
    pos = np.arange(sizes[-1])
    for l in range(len(sizes) - 2, -1, -1):
        order = np.lexsort((np.arange(sizes[l]), pos[H.aggregates(l)]))
        pos = np.empty(sizes[l], np.int64)
        pos[order] = np.arange(sizes[l])
    return pos


def test_inverted_blocks_on_sliced_rows():
    """One sweep each way on 900,001 rows of 65, blocks of 256: the sweep's
    correction d solves (L_pp + D_pp) d = r in every block, (U_pp + D_pp) d =
    r - A x back.  Tolerance: as the sweeps' comparison with the oracle, 1e-11 and
    2e-5 normwise (the triangles are diagonally dominant)."""
    A = wide_band(900_001, 32, 8)
    H = pamg.Hierarchy(A, smoother="hgs", gs_block=256, sweeps=1, omega=1.25, agg_steps=4, build_f32=1)
    assert (H.info().spmv_bytes - 16 * A.n) / 10.0 / A.nnz >= 1.15, "not in sliced rows: the case tests nothing"
    pos = hierarchical_order(H)
    rows = pos[np.repeat(np.arange(A.n), np.diff(A.row_ptr))]
    cols = pos[A.col]
    block = rows // 256 == cols // 256
    M = A.to_scipy()
    lower, upper = (sp.csr_matrix((np.where(block & side, A.val, 0.0), A.col, A.row_ptr), shape=M.shape)
                    for side in (cols <= rows, cols >= rows))
    assert (block & (cols < rows)).sum() >= 8 * A.n
    r, x = uniform_rhs(A.n, 11), uniform_rhs(A.n, 12)
    out = torch.empty(A.n, dtype=torch.float64, device="cuda:0")
    for prec, tol in ((pamg.PREC_F64, 1e-11), (pamg.PREC_F32, 2e-5)):
        H.debug_apply(pamg.OP_SMOOTH, 0, dev(r), out, precision=prec)
        d = 1.25 * out.cpu().numpy()
        assert np.linalg.norm(lower @ d - r) <= tol * np.linalg.norm(abs(lower) @ np.abs(d) + np.abs(r)), prec
        H.debug_apply(pamg.OP_SMOOTH, 0, dev(r), out, in1=dev(x), precision=prec)
        d = 1.25 * (out.cpu().numpy() - x)
        t = r - M @ x
        scale = abs(upper) @ np.abs(d) + np.abs(r) + abs(M) @ np.abs(x)
        assert np.linalg.norm(upper @ d - t) <= tol * np.linalg.norm(scale), prec
