"""The cycle's last levels as one dense product: the whole V-cycle against the
oracle where the dense operator starts at exactly 1024 rows (32^3), at a ragged
size, above aggregates of up to 16 rows, directly below level 0 (two levels),
at the coarsest level itself (nothing collapsed), and after new coefficients.

Tolerance: the dense operator is built in FP64 from the same levels (sums of a
few thousand products, each of relative size u), so the cycle keeps the 1e-12
of the level-by-level one; the FP32 cycle is within a few hundred FP32
roundings of the FP64 cycle, 5e-5.
"""
import numpy as np
import pytest

import oracle
import paper_2210_16660_amd as pamg
from workloads import lap7, q1_stretched, uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "lap7_32": (lambda: lap7(32), {}),
    "lap7_31": (lambda: lap7(31), {}),
    "varcoef_29": (lambda: varcoef7(29, seed=6), {}),
    "q1_22_agg4": (lambda: q1_stretched(22, 1.05), {"agg_steps": 4, "max_coarse": 20}),
    "q1_18_agg3": (lambda: q1_stretched(18, 1.05), {"agg_steps": 3, "max_coarse": 30}),
    "two_levels": (lambda: lap7(12), {"max_levels": 2, "max_coarse": 300}),
    "three_levels": (lambda: lap7(12), {"max_levels": 3}),
    "coarsest_large": (lambda: lap7(20), {"max_coarse": 2500}),
}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def cycle(H, r, prec):
    out = torch.empty(r.size, dtype=torch.float64, device="cuda:0")
    H.debug_apply(pamg.OP_VCYCLE, 0, dev(r), out, precision=prec)
    return out.cpu().numpy()


@pytest.mark.parametrize("case", sorted(CASES))
def test_vcycle_with_a_dense_tail(case):
    mk, kw = CASES[case]
    A = mk()
    H = pamg.Hierarchy(A, build_f32=1, **kw)
    O = oracle.Hierarchy(A, **kw)
    assert H.levels == O.nlevels
    r = uniform_rhs(A.n, 17)
    zo = O.vcycle(r)
    for prec, tol in ((pamg.PREC_F64, 1e-12), (pamg.PREC_F32, 5e-5)):
        assert np.linalg.norm(cycle(H, r, prec) - zo) <= tol * np.linalg.norm(zo), prec


def test_dense_tail_follows_new_coefficients():
    A = varcoef7(26, seed=7)
    H = pamg.Hierarchy(A, build_f32=1)
    r = uniform_rhs(A.n, 18)
    before = cycle(H, r, pamg.PREC_F64)
    H.update_values(4.0 * A.val)
    for prec, tol in ((pamg.PREC_F64, 1e-14), (pamg.PREC_F32, 5e-5)):
        # B(4 A) = B(A) / 4: the same aggregates, and a power of two rounds nothing
        assert np.linalg.norm(4.0 * cycle(H, r, prec) - before) <= tol * np.linalg.norm(before), prec
