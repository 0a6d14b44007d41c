"""The network's tile under MELD_AUTO without a decision of the tuner's (capture, and
meld_sort_u32_noalloc): the one that its trials choose on the hardware.

The GPU part checks those calls at both ends of every class bit-exact against the oracle.
"""
import numpy as np
import pytest

import oracle
import workloads

meld = pytest.importorskip("paper_2107_05681_amd")

# log2 of the size class -> log2 of the fastest tile, timed on one MI355X.
KEYS = {**{k: 12 for k in range(12, 18)}, **{k: 13 for k in range(18, 22)},
        **{k: 14 for k in range(22, 29)}}
PAIRS = {12: 12, **{k: 11 for k in range(13, 20)}, 20: 12, 21: 13, 22: 13, 23: 12,
         **{k: 13 for k in range(24, 29)}}


@pytest.mark.parametrize("pairs", [False, True])
def test_untuned_plan_takes_the_fastest_tile(pairs):
    for log_n, tile in (PAIRS if pairs else KEYS).items():
        for n in ((1 << log_n - 1) + 1, 1 << log_n):
            d = meld.sort_plan(n, pairs, "auto")
            assert d["log_tile"] == tile and d["tuned"] is False, (n, pairs)
            assert d["low"] == d["high"] == "melded"


@pytest.mark.gpu
@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("log_n", [3, 8, 11, 12, 13, 17, 18, 20, 21, 22])
def test_untuned_sorts_match_the_oracle(log_n, pairs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = meld.new_context(0)
    try:
        for n in ((1 << log_n - 1) + 1, 1 << log_n):
            keys, vals = workloads.keys_u32(n, n), workloads.iota_u32(n)
            rk, rv = oracle.sort_pairs_u32(keys, vals)
            kd, vd = (torch.from_numpy(a.view(np.int32)).cuda() for a in (keys, vals))
            k, v = kd.clone(), vd.clone() if pairs else None

            def check():
                torch.cuda.synchronize()
                assert np.array_equal(k.cpu().numpy().view(np.uint32), rk), n
                assert v is None or np.array_equal(v.cpu().numpy().view(np.uint32), rv), n

            def restore():
                k.copy_(kd)
                if pairs:
                    v.copy_(vd)

            meld.sort(k, v, variant="auto", ctx=ctx, noalloc=True)
            check()
            restore()
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                meld.sort(k, v, variant="auto", ctx=ctx)
            for _ in range(3):
                restore()
                torch.cuda.synchronize()
                graph.replay()
                check()
    finally:
        torch.cuda.synchronize()
        meld.destroy_context(ctx)
