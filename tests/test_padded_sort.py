"""Sorts of sizes that are no power of two: padding without memory.

CPU: Figure 1's network with the direction bit taken from i ^ (n - 1), run on the
padded array with every comparator, equals the sorted array and never moves an element
past n; a last block whose second half is padding is ascending before its phase.
GPU: the explicit forms against the oracle at the edges of tiles and blocks. Bit-exact.
"""
import numpy as np
import pytest

import oracle
import workloads

PAD = np.uint32(0xFFFFFFFF)


def _network(keys, log_t):
    """The padded network; phases above 2^log_t as the library runs them."""
    n = len(keys)
    log_n = max(1, (n - 1).bit_length())
    a = np.concatenate([keys, np.full((1 << log_n) - n, PAD, np.uint32)])
    i = np.arange(1 << log_n)
    for m in range(1, log_n + 1):
        end = len(a)
        if m > log_t:
            start = (n - 1) >> m << m
            if start and n <= start + (1 << (m - 1)):
                end = start
                assert (np.diff(a[start:].astype(np.int64)) >= 0).all()
        # inside a tile the directions are Figure 1's; only its last phase looks above
        d = (n - 1) >> log_t << log_t
        for b in range(m - 1, -1, -1):
            j = 1 << b
            lo = i[(i & j == 0) & (i < end)]
            up = ((lo ^ d) >> m) & 1 == 0
            x, y = a[lo], a[lo + j]
            swap = np.where(up, y < x, y > x)
            a[lo], a[lo + j] = np.where(swap, y, x), np.where(swap, x, y)
        if m >= log_t:
            assert (a[n:] == PAD).all()
    return a[:n]


@pytest.mark.parametrize("log_t", [1, 3, 4])
def test_direction_rule(log_t):
    rng = np.random.RandomState(1)
    for n in range((1 << log_t) + 1, 150):
        if n & (n - 1):
            keys = rng.randint(0, 40, n).astype(np.uint32)
            keys[rng.randint(n)] = PAD
            assert np.array_equal(_network(keys, log_t), np.sort(keys)), n


SIZES = [(1 << 11) + 1, (1 << 11) + 256, 3 << 10, (3 << 10) + 1, (1 << 12) - 1, (5 << 10) + 2,
         (1 << 14) + 3, (1 << 16) + (1 << 13) + 5, (1 << 17) - 300, (9 << 15) + 77]


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["divergent", "melded"])
@pytest.mark.parametrize("log_t", [0, 8, 11])
@pytest.mark.parametrize("n", SIZES)
def test_padded_sizes(n, log_t, variant):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05681_amd as meld

    meld.set_option(0, meld.OPT_SORT_LOG_TILE, log_t)
    try:
        for pairs in (False, True):
            for offset in (0, 1):  # 16-byte groups, and arrays that are not aligned
                keys = workloads.keys_u32(n, n) % np.uint32(n)
                keys[n // 2] = PAD
                vals = workloads.keys_u32(n + 1, n)
                guard = np.arange(64, dtype=np.uint32)
                bufs = [torch.from_numpy(np.concatenate([guard[:offset], a, guard])
                                         .view(np.int32)).to("cuda:0") for a in (keys, vals)]
                views = [b[offset:offset + n] for b in bufs]
                if pairs:
                    meld.sort(*views, variant=variant)
                    want = oracle.sort_pairs_u32(keys, vals)
                else:
                    meld.sort(views[0], variant=variant)
                    want = (oracle.sort_u32(keys), vals)
                for b, w in zip(bufs, want):
                    got = b.cpu().numpy().view(np.uint32)
                    assert np.array_equal(got[offset:offset + n], w)
                    assert np.array_equal(got[offset + n:], guard)
    finally:
        meld.set_option(0, meld.OPT_SORT_LOG_TILE, 0)
