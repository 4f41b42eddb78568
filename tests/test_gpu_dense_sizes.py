"""The coarsest level's factorization and inverse at the sizes where its
64 x 64 tiles end: one row, one row short of a tile, one tile, one row more,
several tiles and a ragged one.

Tolerance: Cholesky and the explicit inverse are backward stable, so
A^-1 r is within c n u cond(A) of the exact product; measured against numpy's
solve (same bound), with c n u cond(A) <= 64 cond(A) u for these sizes and
the 1e-13 floor used for the operator's other checks.
"""
import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import CSR, uniform_rhs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _spd(n, seed):
    """A dense-pattern diagonally dominant symmetric matrix as CSR."""
    M = uniform_rhs(n * n, seed).reshape(n, n)
    M = 0.5 * (M + M.T)
    M[np.arange(n), np.arange(n)] = 1.0 + np.abs(M).sum(1)
    rp = np.arange(n + 1, dtype=np.int32) * n
    ci = np.tile(np.arange(n, dtype=np.int32), n)
    return M, CSR(n, rp, ci, np.ascontiguousarray(M.reshape(-1)))


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 200, 449])
def test_coarse_inverse_at_tile_edges(n):
    M, A = _spd(n, 40 + n)
    H = pamg.Hierarchy(A, max_coarse=512, build_f32=1)
    assert H.levels == 1
    r = uniform_rhs(n, 7)
    out = torch.empty(n, dtype=torch.float64, device="cuda:0")
    x = np.linalg.solve(M, r)
    cond = np.linalg.cond(M)
    for prec, u in ((pamg.PREC_F64, 1.2e-16), (pamg.PREC_F32, 6e-8)):
        H.debug_apply(pamg.OP_COARSE, 0, torch.from_numpy(r).cuda(), out, precision=prec)
        err = np.linalg.norm(out.cpu().numpy() - x) / np.linalg.norm(x)
        assert err <= max(1e-13, 64 * cond * u), (n, prec, err, cond)


@pytest.mark.parametrize("bad", [0, 63, 64, 140])
def test_a_negative_pivot_is_refused_wherever_it_is(bad):
    M, A = _spd(150, 3)
    v = A.val.copy()
    # a 2 x 2 indefinite block: positive diagonal entries, negative determinant
    j = bad + 1
    v[bad * 150 + j] = v[j * 150 + bad] = 10.0 * max(v[bad * 150 + bad], v[j * 150 + j])
    with pytest.raises(pamg.PamgError) as e:
        pamg.Hierarchy(CSR(150, A.row_ptr, A.col, v), max_coarse=512)
    assert e.value.code == pamg.E_NOT_SPD
