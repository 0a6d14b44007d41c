"""Captured merge and segmented sorts: their graphs stay valid whatever the context runs
later.

Bar: bit-exact against the oracle at every replay, with eager work of the same context
(a larger sort by radix passes, a larger merge sort, more segments) and synchronisations
in between.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


@pytest.fixture
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = meld.new_context(0)
    yield c
    torch.cuda.synchronize()
    meld.destroy_context(c)


def _to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.uint32).view(np.int32)).cuda()


def _capture(ctx, work, variant):
    """A graph of one merge sort of ``work``; the calls of the context go to its stream."""
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        meld.merge_sort(work, variant=variant, ctx=ctx)
    return graph


def _replay(graph, work, keys, times=1):
    for _ in range(times):
        work.copy_(_to_dev(keys))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(work.cpu().numpy().view(np.uint32), oracle.sort_u32(keys))


@pytest.mark.parametrize("variant", ["divergent", "melded"])
def test_later_calls_leave_a_captured_merge_sort_its_buffers(ctx, variant):
    n = (1 << 15) + 5
    keys = workloads.keys_u32(1, n)
    work = _to_dev(keys)
    meld.merge_sort(work, variant=variant, ctx=ctx)  # allocates outside the capture
    torch.cuda.synchronize()
    graph = _capture(ctx, work, variant)
    _replay(graph, work, keys, 2)
    # A sort whose scratch is larger than the merge buffer, then a larger merge sort.
    for run, m in ((lambda k: meld.sort(k, variant="auto", ctx=ctx), (1 << 18) + 9),
                   (lambda k: meld.merge_sort(k, variant=variant, ctx=ctx), (1 << 17) + 3)):
        other = workloads.keys_u32(2, m)
        kd = _to_dev(other)
        run(kd)
        torch.cuda.synchronize()
        junk = torch.full((4 << 20,), -1, dtype=torch.int32, device="cuda:0")  # takes freed memory
        _replay(graph, work, workloads.keys_u32(3, n), 2)
        assert np.array_equal(kd.cpu().numpy().view(np.uint32), oracle.sort_u32(other))
        assert bool((junk == -1).all())


@pytest.mark.parametrize("variant", ["auto", "melded", "divergent"])
@pytest.mark.parametrize("n", [5000, (1 << 14) + 1, 70_001, 1 << 18])
def test_an_eager_auto_call_is_the_warm_up_of_a_capture(ctx, n, variant):
    keys = workloads.keys_u32(4, n)
    work = _to_dev(keys)
    meld.merge_sort(work, variant="auto", ctx=ctx)
    torch.cuda.synchronize()
    assert np.array_equal(work.cpu().numpy().view(np.uint32), oracle.sort_u32(keys))
    graph = _capture(ctx, work, variant)
    for seed in (4, 5, 6):
        _replay(graph, work, workloads.keys_u32(seed, n))


@pytest.mark.parametrize("variant", ["auto", "melded"])
def test_later_calls_leave_a_captured_segmented_sort_its_queues(ctx, variant):
    off = workloads.segment_offsets(8, 100)
    n = int(off[-1])
    work, od = _to_dev(workloads.keys_u32(8, n)), _to_dev(off)
    meld.segmented_sort(work, od, variant=variant, ctx=ctx)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        meld.segmented_sort(work, od, variant=variant, ctx=ctx)
    for seed, nseg in ((9, 0), (10, 3000), (11, 70_000)):
        if nseg:
            more = torch.arange(nseg + 1, dtype=torch.int32, device="cuda:0") * 3
            kd = _to_dev(workloads.keys_u32(seed, 3 * nseg))
            ref = (kd.view(-1, 3).cpu().numpy().view(np.uint32)).copy()
            meld.segmented_sort(kd, more, variant=variant, ctx=ctx)
            torch.cuda.synchronize()
            assert np.array_equal(kd.cpu().numpy().view(np.uint32).reshape(-1, 3),
                                  np.sort(ref, axis=1))
            junk = torch.full((4 << 20,), -1, dtype=torch.int32, device="cuda:0")
        keys = workloads.keys_u32(seed, n)
        for _ in range(2):
            work.copy_(_to_dev(keys))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(work.cpu().numpy().view(np.uint32),
                                  oracle.segmented_sort_u32(keys, off))
        assert not nseg or bool((junk == -1).all())
    meld.segmented_sort_check(0, ctx=ctx)
