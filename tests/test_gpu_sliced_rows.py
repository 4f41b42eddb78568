"""The sliced-row layout of the largest levels (from 786,432 rows): every kernel
that reads it, on operators just above that size, with pairs and with
aggregates of up to 16 rows, built on the device and on the host, in both
precisions, against scipy products of the same matrix.

The sizes are ragged on purpose (the last tile is not full, aggregates end
tiles early, and boundary rows are shorter than the rest, so rows are reordered
inside their tiles).  Tolerances as for the operators' other checks: a row sums
at most 27 products, normwise 1e-13 (FP64) and 2e-6 (FP32, against the matrix
rounded to FP32) of |A| |x|.
"""
import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import CSR, lap7, q1_stretched, uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

OPERATORS = {
    "lap7_93": lambda: lap7(93),                     # 804,357 rows of 4 to 7 entries
    "q1_92": lambda: q1_stretched(92, 1.05),         # 795,707 rows of 7 to 27 entries
}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


@pytest.fixture(scope="module")
def matrices():
    return {k: f() for k, f in OPERATORS.items()}


@pytest.mark.parametrize("name,steps,device", [("lap7_93", 1, 1), ("lap7_93", 4, 0), ("q1_92", 1, 0), ("q1_92", 3, 1)])
def test_level0_operators(matrices, name, steps, device):
    A = matrices[name]
    M = A.to_scipy()
    H = pamg.Hierarchy(A, agg_steps=steps, device_setup=device, build_f32=1)
    n, nc = A.n, H.level_sizes()[0][1]
    agg = H.aggregates(0)
    out, outc = (torch.empty(k, dtype=torch.float64, device="cuda:0") for k in (n, nc))
    H.debug_apply(pamg.OP_PROLONG, 0, dev(np.zeros(n)), out, in1=dev(np.ones(nc)))
    p = out.cpu().numpy()
    x, r = uniform_rhs(n, 5), uniform_rhs(n, 6)
    for prec, tol in ((pamg.PREC_F64, 1e-13), (pamg.PREC_F32, 2e-6)):
        B = M if prec == pamg.PREC_F64 else M.astype(np.float32).astype(np.float64)
        absB = abs(B)
        dinv = 1.0 / np.asarray(abs(M).sum(1)).ravel()
        H.debug_apply(pamg.OP_SPMV, 0, dev(x), out, precision=prec)
        assert np.linalg.norm(out.cpu().numpy() - B @ x) <= tol * np.linalg.norm(absB @ np.abs(x))
        H.debug_apply(pamg.OP_UP, 0, dev(r), out, in1=dev(x), precision=prec)
        ref = x + dinv * (r - B @ x)
        scale = np.linalg.norm(np.abs(x) + dinv * (np.abs(r) + absB @ np.abs(x)))
        assert np.linalg.norm(out.cpu().numpy() - ref) <= tol * scale
        H.debug_apply(pamg.OP_DOWN, 0, dev(r), outc, precision=prec)
        t = r - B @ (dinv * r)
        ref = np.bincount(agg, weights=p * t, minlength=nc)
        scale = np.linalg.norm(np.bincount(agg, weights=np.abs(p) * (np.abs(r) + absB @ (dinv * np.abs(r))), minlength=nc))
        assert np.linalg.norm(outc.cpu().numpy() - ref) <= tol * scale


def test_host_and_device_layouts_give_the_same_bits(matrices):
    A = matrices["q1_92"]
    b = dev(uniform_rhs(A.n, 8))
    B3 = torch.stack([b, dev(uniform_rhs(A.n, 9)), dev(uniform_rhs(A.n, 10))])
    xs = []
    for device in (1, 0):
        H = pamg.Hierarchy(A, device_setup=device, build_f32=1)
        for prec in ("f64", "f32"):
            x = torch.zeros_like(b)
            assert H.solve(b, x, tol=1e-6, precision=prec, true_residual=1).relres_true <= 1e-6
            xs.append(x.cpu().numpy().view(np.uint64))
        X = torch.zeros_like(B3)
        for i in H.solve_batch(B3, X, tol=1e-6, precision="f32"):
            assert i.relres_true <= 1e-6
        xs.append(X.cpu().numpy().view(np.uint64))
        assert np.array_equal(H.level_csr(0)[2], A.val)
    for a, c in zip(xs[:3], xs[3:]):
        assert np.array_equal(a, c)


def test_new_coefficients_on_sliced_rows():
    A, B = varcoef7(93, seed=3), varcoef7(93, seed=4)
    b = dev(uniform_rhs(A.n, 2))
    G = pamg.Hierarchy(A, build_f32=1)
    G.update_values(dev(B.val))
    assert np.array_equal(G.level_csr(0)[2], B.val)
    Bs = B.to_scipy()
    for prec in ("f64", "f32"):
        x = torch.zeros_like(b)
        G.solve(b, x, tol=1e-6, precision=prec)
        xs = x.cpu().numpy()
        assert np.linalg.norm(b.cpu().numpy() - Bs @ xs) <= 1.001e-6 * float(b.norm())
    # four times the matrix: bitwise the solve of a fresh setup of it
    A4 = CSR(A.n, A.row_ptr, A.col, 4.0 * A.val)
    G.update_values(A4.val)
    F = pamg.Hierarchy(A4)
    xs = []
    for K in (F, pamg.Hierarchy(A)):
        if K is not F:
            K.update_values(A4.val)
        x = torch.zeros_like(b)
        K.solve(b, x, tol=1e-6)
        xs.append(x.cpu().numpy().view(np.uint64))
    assert np.array_equal(*xs)


@pytest.mark.parametrize("name", sorted(OPERATORS))
@pytest.mark.parametrize("prec", [pamg.PREC_F32, pamg.PREC_F64])
def test_admission_estimate_covers_the_slices(matrices, name, prec):
    # just above the least size the tiles' unused room is largest
    A = matrices[name]
    S = pamg.Server(precision=prec, single_path=1)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda:0")
    S.submit(1, A, dev(np.zeros(A.n)), x, tag=1)
    done = []
    while not done:
        done = S.poll()
    st = S.stats()
    S.close()
    assert done[0].status == pamg.OK and st.setups == 1
    est = pamg.server_estimate_bytes(A, prec)
    assert est // 16 <= st.bytes_in_use <= est
