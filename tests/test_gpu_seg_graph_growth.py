"""A segmented sort's own graph is not replayed after its queues have grown.

The explicit forms always replay a graph (MELD_AUTO may sort in registers, which has
none): a call at 100 segments captures one over the context's queues, a call over more
segments replaces them, and the first call again, with the same pointers, must not replay
the graph of the old ones.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


@pytest.mark.parametrize("variant", ["divergent", "melded"])
def test_graph_is_dropped_when_the_queues_grow(variant):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = meld.new_context(0)
    try:
        runs = []
        for nseg, seed in ((100, 21), (5000, 22)):
            off = workloads.segment_offsets(seed, nseg)
            off = np.minimum(off, 1 << 21).astype(np.uint32)  # the rest are empty
            keys = workloads.keys_u32(seed, int(off[-1]))
            runs.append((keys, off, *(torch.from_numpy(a.view(np.int32)).cuda()
                                      for a in (off, keys))))
        for k in (0, 1, 0, 1, 0):
            keys, off, od, kd = runs[k]
            kd.copy_(torch.from_numpy(keys.view(np.int32)))
            meld.segmented_sort(kd, od, variant=variant, ctx=ctx)
            torch.cuda.synchronize()
            junk = torch.full((1 << 20,), -1, dtype=torch.int32, device="cuda:0")
            assert np.array_equal(kd.cpu().numpy().view(np.uint32),
                                  oracle.segmented_sort_u32(keys, off))
            assert bool((junk == -1).all())
        meld.segmented_sort_check(0, ctx=ctx)
    finally:
        torch.cuda.synchronize()
        meld.destroy_context(ctx)
