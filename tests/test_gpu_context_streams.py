"""Temporaries go back to a caller's allocator on the stream they were taken on: a
stream-ordered allocator may hand them out again in that order only."""
import numpy as np
import pytest

import paper_2210_16660_amd as pamg
from workloads import q1_stretched

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("steps", [1, 2])
def test_temporaries_are_freed_on_their_stream(steps):
    taken, freed = {}, []

    def alloc(nbytes, stream):
        p = torch.cuda.caching_allocator_alloc(nbytes, torch.cuda.current_device(), stream)
        taken[p] = stream
        return p

    def free(ptr, stream):
        freed.append((taken.pop(ptr), stream))
        torch.cuda.caching_allocator_delete(ptr)

    A = q1_stretched(32, 1.05)
    ctx = pamg.Context(allocator=(alloc, free))
    side = torch.cuda.Stream()
    for device_setup in (1, 0):
        H = pamg.Hierarchy(A, stream=side, context=ctx, build_f32=1, agg_steps=steps, device_setup=device_setup)
        assert (H.info().device_levels > 0) == bool(device_setup)
        assert len(freed) >= 4 and all(s == t == side.cuda_stream for t, s in freed)
        freed.clear()
        H.update_values(A.val * 2.0, stream=side)
        assert freed and all(s == t == side.cuda_stream for t, s in freed)
        H.close()
        freed.clear()
    assert not taken
    ctx.close()
