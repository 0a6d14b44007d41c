"""MELD_AUTO sorts of up to 2^14 keys (one workgroup, 8 or 16 keys per lane) against the oracle.

Bar: bit-exact. Sizes around every power of two, arrays that are not 16-byte aligned,
ties and the padding's value, sorted and reversed input, 0/1 inputs; above 2^13 keys
inside a graph, where the sort may take no scratch.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


def _sort(keys, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    guard = np.arange(80, dtype=np.uint32)
    buf = torch.from_numpy(np.concatenate([guard[:offset], keys, guard]).view(np.int32)).to("cuda:0")
    meld.sort(buf[offset:offset + len(keys)], variant="auto")
    got = buf.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:offset], guard[:offset])
    assert np.array_equal(got[offset + len(keys):], guard)
    return got[offset:offset + len(keys)]


@pytest.mark.parametrize("log", range(1, 14))
def test_around_powers_of_two(log):
    for n in sorted({2, (1 << log) - 3, (1 << log) - 1, 1 << log, (1 << log) + 1,
                     3 << (log - 1)}):
        if n < 2:
            continue
        keys = workloads.keys_u32(n, n)
        ends = keys.copy()
        ends[::3] = 0xFFFFFFFF
        for k in (keys, keys % np.uint32(3), ends, np.sort(keys), np.sort(keys)[::-1],
                  (np.arange(n) * 7 % n).astype(np.uint32)):
            k = np.ascontiguousarray(k)
            for offset in (0, 1):
                assert np.array_equal(_sort(k, offset), oracle.sort_u32(k)), n


def test_zero_one():
    # every split point, in several orders, at the sizes with waves that exchange
    rng = np.random.RandomState(2)
    for n in (600, 1024, 1500, 4096, 8192):
        for ones in range(0, n + 1, n // 25):
            k = np.zeros(n, np.uint32)
            k[:ones] = 1
            for order in (k, k[::-1], rng.permutation(k)):
                order = np.ascontiguousarray(order)
                assert np.array_equal(_sort(order, 0), np.sort(order)), (n, ones)


@pytest.mark.parametrize("n", [(1 << 13) + 1, 12000, 1 << 14])
def test_captured(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    buf = torch.zeros(n, dtype=torch.int32, device="cuda:0")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        meld.sort(buf, variant="auto")
    for seed in range(3):
        keys = workloads.keys_u32(seed, n)
        buf.copy_(torch.from_numpy(keys.view(np.int32)))
        graph.replay()
        assert np.array_equal(buf.cpu().numpy().view(np.uint32), oracle.sort_u32(keys))


@pytest.mark.parametrize("n", [(1 << 11) + 1, 3000, 1 << 12])
def test_captured_pairs(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    key, val = (torch.zeros(n, dtype=torch.int32, device="cuda:0") for _ in range(2))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        meld.sort(key, val, variant="auto")
    for seed in range(3):
        k, v = workloads.keys_u32(seed, n) % np.uint32(64), workloads.keys_u32(seed + 9, n)
        key.copy_(torch.from_numpy(k.view(np.int32)))
        val.copy_(torch.from_numpy(v.view(np.int32)))
        graph.replay()
        rk, rv = oracle.sort_pairs_u32(k, v)
        assert np.array_equal(key.cpu().numpy().view(np.uint32), rk)
        assert np.array_equal(val.cpu().numpy().view(np.uint32), rv)
