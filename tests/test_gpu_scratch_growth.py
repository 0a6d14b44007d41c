"""Sorts of slowly growing n allocate once per power of two, not on every call.

Bar: after the first call of a size class the device's free memory stays as it is for
every larger n up to the power of two (the inputs are allocated before), and the results
are the oracle's.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")

TOP = 1 << 21
SIZES = [(1 << 20) + 1, (1 << 20) + 77_777, (1 << 20) + 400_000, TOP - 1, TOP]


@pytest.mark.parametrize("call", ["keys", "pairs", "merge", "merge_melded"])
def test_one_allocation_per_power_of_two(call):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = meld.new_context(0)
    try:
        keys = workloads.keys_u32(7, TOP)
        src = torch.from_numpy(keys.view(np.int32)).cuda()
        work = torch.empty_like(src)
        index = torch.arange(TOP, dtype=torch.int32, device="cuda:0")
        payload = torch.empty_like(index)
        free = None
        for n in SIZES:
            k, v = work[:n], payload[:n] if call == "pairs" else None
            k.copy_(src[:n])
            payload.copy_(index)
            torch.cuda.synchronize()
            if call == "merge":
                meld.merge_sort(k, ctx=ctx)
            elif call == "merge_melded":
                meld.merge_sort(k, variant="melded", ctx=ctx)
            else:
                meld.sort(k, v, ctx=ctx)
            torch.cuda.synchronize()
            after = torch.cuda.mem_get_info(0)[0]
            assert free is None or after == free, n
            free = after
            assert np.array_equal(k.cpu().numpy().view(np.uint32), oracle.sort_u32(keys[:n]))
    finally:
        torch.cuda.synchronize()
        meld.destroy_context(ctx)
