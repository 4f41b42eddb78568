"""The width of a server's batches, read off the bytes it accounts for (an
iteration of W columns is charged the matrices and W columns of the vectors): a
request alone runs 4 wide, is widened to 16 while it runs when eight more join,
keeps its bits through that, and the next one alone is narrow again."""
import time

import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LONG = 300          # iterations of the request that the others join (FP64: its residual stays far from underflow)


def iteration_bytes(H, width):
    n, nnz = H.level_sizes()
    cycle = sum(2 * (nnz[l] * 12 + 4 * (n[l] + 1)) + (10 * n[l] + 2 * n[l + 1]) * width * 8 for l in range(len(n) - 1))
    return cycle + nnz[0] * 12 + 4 * (n[0] + 1) + 12 * n[0] * width * 8


@pytest.mark.parametrize("graph", [0, 1])
def test_running_batch_is_widened_and_the_next_is_narrow(graph):
    A = varcoef7(26, seed=9)
    B = torch.from_numpy(np.stack([uniform_rhs(A.n, 300 + c) for c in range(9)])).cuda()
    H = pamg.Hierarchy(A)
    four, sixteen = iteration_bytes(H, 4), iteration_bytes(H, 16)
    ref, alone = torch.zeros_like(B), torch.zeros_like(B[:1])
    infos = H.solve_batch(B, ref, tol=1e-8)
    assert H.solve_batch(B[:1], alone, tol=1e-300, maxit=LONG)[0].iterations == LONG
    S = pamg.Server(precision=pamg.PREC_F64, use_graph=graph)
    X = torch.zeros_like(B)
    torch.cuda.synchronize()

    def wait(tags):
        done, t0 = {}, time.time()
        while len(done) < len(tags) and time.time() - t0 < 60:
            done.update({int(d.tag): d for d in S.poll()})
        assert sorted(done) == sorted(tags)
        return done

    def moved():
        # the last block is accounted before its requests complete, published at the tick's end
        time.sleep(0.02)
        return S.stats().algorithmic_bytes

    S.submit(1, A, B[0], X[0], tol=1e-8, tag=0)
    first = wait([0])[0].iterations
    assert first == infos[0].iterations and moved() == first * four
    before, blocks = moved(), S.stats().blocks
    S.submit(1, None, B[0], X[0], tol=1e-300, tag=100, maxit=LONG)
    while S.stats().blocks < blocks + 3:
        pass
    for c in range(1, 9):
        S.submit(1, None, B[c], X[c], tol=1e-8, tag=c)
    done = wait([100] + list(range(1, 9)))
    assert done[100].iterations == LONG and done[100].status == pamg.NOT_CONVERGED
    # 16 wide from the eighth's joining (it takes the ninth column) to the end, not before the third block;
    # a joining that falls between two blocks may pass through 8
    wide, rest = divmod(moved() - before - LONG * four, (sixteen - four) // 3)
    assert rest == 0 and 3 * infos[8].iterations <= wide <= 3 * (LONG - 8)
    assert torch.equal(X[0].view(torch.int64), alone[0].view(torch.int64))
    assert torch.equal(X[1:].view(torch.int64), ref[1:].view(torch.int64))
    before = moved()
    S.submit(1, None, B[0], X[0], tol=1e-8, tag=7)
    assert wait([7])[7].iterations == first and moved() == before + first * four
    S.close()
