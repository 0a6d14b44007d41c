"""Host threads that share one context and stream: their calls use the same scratch, so
each call's launches have to reach the stream together.

Bar: bit-exact against the oracle for every call of every thread.
"""
import threading

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")

THREADS, REPS = 6, 12


def _to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.uint32).view(np.int32)).cuda()


def _case(kind, seed):
    """(run(), expected) of one thread: the call returns its sorted keys on the device."""
    n = (1 << 12, 5000, 70_001, 1 << 17, 300_007, 1 << 18)[seed % 6] + seed
    if kind == "segments":
        off = workloads.segment_offsets(seed, 40 + 60 * seed)
        keys = workloads.keys_u32(seed, int(off[-1]))
        od = _to_dev(off)
        call, ref = (lambda k: meld.segmented_sort(k, od)), oracle.segmented_sort_u32(keys, off)
    else:
        keys = workloads.keys_u32(seed, n)
        ref = oracle.sort_u32(keys)
        call = meld.merge_sort if kind == "merge" else meld.sort
        if kind == "pairs":
            vd = _to_dev(workloads.keys_u32(seed + 100, n))
            call = lambda k: meld.sort(k, vd.clone())
    kd = _to_dev(keys)

    def run():
        k = kd.clone()
        call(k)
        return k
    return run, ref


@pytest.mark.parametrize("kinds", [("keys",), ("pairs",), ("merge",), ("segments",),
                                   ("keys", "pairs", "merge", "segments")])
def test_threads_on_one_stream(kinds):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cases = [_case(kinds[t % len(kinds)], t) for t in range(THREADS)]
    torch.cuda.synchronize()
    got = [[] for _ in cases]
    start = threading.Barrier(THREADS)

    def work(t):
        start.wait()
        for _ in range(REPS):
            got[t].append(cases[t][0]())

    threads = [threading.Thread(target=work, args=(t,)) for t in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for t, (_, ref) in enumerate(cases):
        assert len(got[t]) == REPS
        for r, k in enumerate(got[t]):
            assert np.array_equal(k.cpu().numpy().view(np.uint32), ref), (kinds, t, r)
