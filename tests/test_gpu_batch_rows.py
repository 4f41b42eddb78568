"""Rows of every length through the batch kernels: the fifteen variants (unroll
depth, columns per lane) sum a row's entries in the same order, so a column's
bits may not depend on which runs.  Rows of 1 to 40 entries put every remainder
against every unroll depth; the sliced rows of the largest levels are taken two
at a time where they are long, with aggregates of one to eight rows (odd ones
leave a single row), and one at a time where they are short."""
import numpy as np
import pytest
import scipy.sparse as sp

import paper_2210_16660_amd as pamg
from workloads import CSR, lap7, q1_stretched, uniform_rhs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def ragged(n, seed):
    """Graph Laplacian plus identity, rows of 1 to about 40 entries."""
    rng = np.random.default_rng(seed)
    deg = np.arange(n) % 20
    lo = np.repeat(np.arange(n), deg)
    hi = rng.integers(0, n, len(lo))
    keep = lo != hi
    U = sp.coo_matrix((rng.uniform(0.1, 1.0, keep.sum()), (lo[keep], hi[keep])), shape=(n, n)).tocsr()
    S = (U + U.T).tocsr()
    A = (sp.diags(np.asarray(S.sum(axis=1)).ravel() + 1.0) - S).tocsr()
    A.sort_indices()
    return CSR(n, A.indptr.astype(np.int32), A.indices.astype(np.int32), np.ascontiguousarray(A.data))


CASES = {
    "ragged_3000": (lambda: ragged(3000, 8), {}, [(u, c) for c in (1, 2, 4) for u in (1, 2, 4, 8, 16)]),
    "sliced_q1_92": (lambda: q1_stretched(92, 1.05), {}, [(1, 4), (2, 1), (4, 2), (8, 4), (16, 4)]),
    "sliced_q1_92_composed3": (lambda: q1_stretched(92, 1.05), {"agg_steps": 3}, [(1, 4), (2, 4), (16, 2)]),
    "sliced_lap7_93": (lambda: lap7(93), {}, [(1, 4), (4, 4), (16, 1)]),
}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("prec", [pamg.PREC_F64, pamg.PREC_F32])
def test_variants_sum_rows_alike(case, prec):
    make, kw, variants = CASES[case]
    A = make()
    H = pamg.Hierarchy(A, build_f32=1, **kw)
    full = None
    for nrhs in (16, 3, 7):
        B = torch.from_numpy(np.stack([uniform_rhs(A.n, 80 + c) for c in range(nrhs)])).cuda()
        ref = None
        for v in variants:
            H.set_batch_config([v + v] * (H.levels - 1), precision=prec)
            X = torch.zeros_like(B)
            H.solve_batch(B, X, tol=0.0, fixed_iters=3, precision=prec)
            assert bool(torch.isfinite(X).all())
            if ref is None:
                ref = X
            assert torch.equal(X.view(torch.int64), ref.view(torch.int64)), (v, nrhs)
        full = ref if full is None else full
        assert torch.equal(ref.view(torch.int64), full[:nrhs].view(torch.int64)), nrhs
