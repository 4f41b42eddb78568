"""Hybrid Gauss-Seidel levels with long rows run a product with the inverted
blocks: the sweeps at the block sizes where its 64 x 64 tiles and 16-column
groups end (one row, one tile, one tile and a row, ragged, full), with a last
block that is not full, in both precisions, against the oracle.

Tolerance: W = (L + D)^-1 is computed by substitution, so W t and the
substitution on t differ by a few u |W| |L + D| |W| |t|; the blocks are
diagonally dominant triangles (|W| (|L| + D) is O(1) per row), so the normwise
1e-11 of the smoother's other checks holds with margin in FP64 and 2e-5 in
FP32 (some 100 roundings of 6e-8 per value, four sweeps each way).
"""
import numpy as np
import pytest

import oracle
import paper_2210_16660_amd as pamg
from workloads import q1_stretched, uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("nb", [1, 16, 37, 63, 64, 65, 130, 255, 256])
@pytest.mark.parametrize("name", ["varcoef_13", "q1_14_agg3"])
def test_sweeps_on_long_rows_match_oracle(name, nb):
    A, steps = (varcoef7(13, seed=31), 1) if name == "varcoef_13" else (q1_stretched(14, 1.05), 3)
    kw = dict(agg_steps=steps, smooth_prolongator=1)
    H = pamg.Hierarchy(A, smoother="hgs", sweeps=2, gs_block=nb, omega=1.3, build_f32=1, max_coarse=40, **kw)
    O = oracle.Hierarchy(A, max_coarse=40, agg_steps=steps, smooth_prolongator=True).set_smoother("hgs", nu=2, nb=nb, omega=1.3)
    assert H.levels == O.nlevels
    n, nnz = H.level_sizes()
    long_rows = [l for l in range(H.levels - 1) if nnz[l] >= 64 * n[l]]
    assert long_rows, "no level with long rows: the case tests nothing"
    for l in long_rows:
        r = uniform_rhs(n[l], 200 + l)
        out = torch.empty(n[l], dtype=torch.float64, device="cuda:0")
        fwd = O.hgs_smooth(l, r)
        bwd = O.hgs_smooth(l, r, x=fwd, backward=True)
        for prec, tol in ((pamg.PREC_F64, 1e-11), (pamg.PREC_F32, 2e-5)):
            H.debug_apply(pamg.OP_SMOOTH, l, dev(r), out, precision=prec)
            assert np.linalg.norm(host(out) - fwd) <= tol * np.linalg.norm(fwd), (l, prec, "forward")
            H.debug_apply(pamg.OP_SMOOTH, l, dev(r), out, in1=dev(fwd), precision=prec)
            assert np.linalg.norm(host(out) - bwd) <= tol * np.linalg.norm(bwd), (l, prec, "backward")
