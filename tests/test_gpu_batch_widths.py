"""Batches run at the width (4, 8 or 16 columns) that holds their right-hand
sides: at every count around the width changes a column is bitwise what it is in
a full batch of 16, in both precisions and for both recurrences, after batches
of other widths on the same hierarchy, with a zero right-hand side among the
columns; operators: an ordinary one, a coarsest level of hundreds of rows (the
product split over waves), two levels and a single level."""
import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import lap7, q1_stretched, uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "q1_17": (lambda: q1_stretched(17, 1.05), {}),
    "stalled_varcoef_40": (lambda: varcoef7(40, seed=5000), {"max_coarse": 300}),
    "two_levels": (lambda: lap7(11), {"max_levels": 2, "max_coarse": 300}),
    "single_level": (lambda: lap7(5), {"max_coarse": 1000}),
}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_columns_do_not_depend_on_the_width(case, precision):
    mk, kw = CASES[case]
    A = mk()
    H = pamg.Hierarchy(A, build_f32=1, **kw)
    B = np.stack([uniform_rhs(A.n, 60 + c) for c in range(16)])
    B[2] = 0.0
    B = torch.from_numpy(B).cuda()
    for krylov in ("fcg", "cg"):
        full = torch.full_like(B, 7.0)
        infos = H.solve_batch(B, full, tol=1e-8, precision=precision, krylov=krylov, true_residual=1)
        assert all(i.status == pamg.OK and i.relres_true <= 1e-8 for i in infos)
        assert not full[2].any()
        for nrhs in (9, 5, 4, 1, 8, 3, 16):
            X = torch.full((nrhs, A.n), 7.0, dtype=torch.float64, device="cuda:0")
            got = H.solve_batch(B[:nrhs].contiguous(), X, tol=1e-8, precision=precision, krylov=krylov)
            assert [i.iterations for i in got] == [i.iterations for i in infos[:nrhs]]
            assert torch.equal(X.view(torch.int64), full[:nrhs].view(torch.int64)), (nrhs, krylov)
