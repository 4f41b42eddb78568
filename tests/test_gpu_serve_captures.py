"""With graph replay an operator's graphs are captured when its batch engine is
built, at every width: while later requests come and go at other widths, no
capture runs, so device-wide calls of the application succeed (they fail while
the scheduler captures)."""
import threading
import time

import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import uniform_rhs, varcoef7

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", [pamg.PREC_F32, pamg.PREC_F64])
def test_no_capture_once_an_engine_exists(precision):
    A = varcoef7(26, seed=9)
    B = torch.from_numpy(np.stack([uniform_rhs(A.n, 300 + c) for c in range(16)])).cuda()
    X = torch.zeros_like(B)
    torch.cuda.synchronize()
    S = pamg.Server(precision=precision, use_graph=1)

    def wait(tags):
        left, t0 = set(tags), time.time()
        while left and time.time() - t0 < 60:
            for d in S.poll():
                assert d.status == pamg.OK
                left.discard(int(d.tag))
        assert not left

    S.submit(1, A, B[0], X[0], tol=1e-8, tag=0)          # the engine, one column wide
    wait([0])
    assert S.stats().engines_built == 1
    stop, calls, errors = threading.Event(), [0], []

    def synchronize():
        while not stop.is_set():
            try:
                torch.cuda.synchronize()
                calls[0] += 1
            except Exception as e:                        # noqa: BLE001
                errors.append(str(e))
                return

    t = threading.Thread(target=synchronize)
    t.start()
    for count in (5, 16, 2):                              # 8, 16 and 4 columns wide
        for c in range(count):
            S.submit(1, A, B[c], X[c], tol=1e-8, tag=c)
        wait(range(count))
    stop.set()
    t.join()
    S.close()
    assert not errors and calls[0] > 0
