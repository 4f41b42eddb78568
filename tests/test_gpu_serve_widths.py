"""Batches of the server are as wide as the columns in use need and are widened
while columns run: requests that arrive 1, 3, 4 and 8 at a time, with pauses
shorter than a solve between them, get bitwise the results and iteration counts
of one full batch, with direct launches and with replayed graphs; a batch that
starts after the operator was idle is narrow again."""
import time

import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", [pamg.PREC_F64, pamg.PREC_F32])
@pytest.mark.parametrize("graph", [0, 1])
def test_joining_columns_keep_their_bits(precision, graph):
    A = varcoef7(26, seed=9)
    B = torch.from_numpy(np.stack([uniform_rhs(A.n, 300 + c) for c in range(16)])).cuda()
    H = pamg.Hierarchy(A, build_f32=1)
    full = torch.zeros_like(B)
    infos = H.solve_batch(B, full, tol=1e-8, precision=precision)
    S = pamg.Server(precision=precision, use_graph=graph)
    for pause in (0.0, 3e-4, 1e-3):
        X = torch.full_like(B, 3.0)
        torch.cuda.synchronize()
        done, at = {}, 0
        for count in (1, 3, 4, 8):
            for c in range(at, at + count):
                S.submit(1, A, B[c], X[c], tol=1e-8, tag=c)
            at += count
            time.sleep(pause)
        t0 = time.time()
        while len(done) < 16 and time.time() - t0 < 60:
            done.update({int(d.tag): d for d in S.poll()})
        assert len(done) == 16
        for c in range(16):
            assert done[c].status == pamg.OK and done[c].iterations == infos[c].iterations, (pause, c)
        assert torch.equal(X.view(torch.int64), full.view(torch.int64)), pause
    S.close()
