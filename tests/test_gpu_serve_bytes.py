"""What a server holds for an operator, against its budget."""
import time

import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import CSR, lap7, uniform_rhs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def serve(A, count, **kw):
    """Statuses of `count` requests at once, and the server's statistics after them."""
    B = torch.from_numpy(np.stack([uniform_rhs(A.n, 40 + c) for c in range(count)])).cuda()
    X = torch.zeros_like(B)
    torch.cuda.synchronize()
    S = pamg.Server(**kw)
    for c in range(count):
        S.submit(1, A, B[c], X[c], tol=1e-6, tag=c)
    done, t0 = {}, time.time()
    while len(done) < count and time.time() - t0 < 60:
        done.update({int(d.tag): d.status for d in S.poll()})
    st = S.stats()
    S.close()
    assert len(done) == count
    return set(done.values()), st


@pytest.mark.parametrize("device_setup", [0, 1])
@pytest.mark.parametrize("precision,value", [(pamg.PREC_F64, 8), (pamg.PREC_F32, 12)])
def test_batches_alone_hold_no_dense_operator_of_the_last_levels(precision, value, device_setup):
    # 93,312 entries: the cycle's levels from 432 rows on are one dense product
    # (5 x the entries reach 683 rows) in the single-right-hand-side solver
    A = lap7(24)
    kw = dict(precision=precision, device_setup=device_setup)
    status, batch = serve(A, 8, **kw)
    assert status == {pamg.OK} and batch.engines_built == 1
    status, single = serve(A, 8, single_path=1, **kw)
    assert status == {pamg.OK} and single.engines_built == 1
    assert single.bytes_in_use - batch.bytes_in_use == 432 * 432 * value
    # a budget that holds the hierarchy and the engine serves the operator
    status, st = serve(A, 8, hbm_budget_bytes=batch.bytes_in_use, **kw)
    assert status == {pamg.OK} and st.bytes_in_use == batch.bytes_in_use


def with_isolated_rows(A, extra):
    """A and `extra` uncoupled unknowns, which coarsening keeps on every level."""
    rp = np.concatenate([A.row_ptr, A.row_ptr[-1] + np.arange(1, extra + 1, dtype=np.int32)]).astype(np.int32)
    col = np.concatenate([A.col, A.n + np.arange(extra, dtype=np.int32)]).astype(np.int32)
    return CSR(A.n + extra, rp, col, np.concatenate([A.val, np.full(extra, 6.0)]))


@pytest.mark.parametrize("precision,value", [(pamg.PREC_F64, 8), (pamg.PREC_F32, 12)])
def test_a_large_coarsest_inverse_is_charged_before_it_is_built(precision, value):
    A = with_isolated_rows(lap7(24), 6000)
    n_coarsest = pamg.Hierarchy(A, host_only=1).level_sizes()[0][-1]
    inverse = n_coarsest ** 2 * value
    assert inverse >= 6000 ** 2 * value
    # built on the device its scratch (some 7 MB) does not cover the inverse
    status, st = serve(A, 1, precision=precision, hbm_budget_bytes=inverse - 1)
    assert status == {pamg.E_BUSY} and st.setups == 0 and st.bytes_in_use == 0
    status, st = serve(A, 1, precision=precision, hbm_budget_bytes=2 * inverse)
    assert status == {pamg.OK} and inverse < st.bytes_in_use <= 2 * inverse
