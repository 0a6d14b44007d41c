"""MELD_AUTO on fixed buckets (the ascending register network) against the oracle.

Bar: bit-exact (a bucket's sorted order is unique). Every bucket size, array ends at
the edges of a wave's 2048 keys, of a bucket and of a workgroup; arrays that are not
16-byte aligned; all 0/1 patterns of a small bucket; ties and the padding's value.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


def _sorted(keys, log_b, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    guard = np.arange(40, dtype=np.uint32)
    buf = torch.from_numpy(np.concatenate([guard[:offset], keys, guard]).view(np.int32)).to("cuda:0")
    meld.oddeven_sort_buckets(buf[offset:offset + len(keys)], log_b, variant="auto")
    got = buf.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:offset], guard[:offset])
    assert np.array_equal(got[offset + len(keys):], guard)
    return got[offset:offset + len(keys)]


def _oracle(keys, log_b):
    n = len(keys)
    bounds = np.array(list(range(0, n, 1 << log_b)) + [n], dtype=np.uint32)
    return oracle.segmented_sort_u32(keys, bounds)


@pytest.mark.parametrize("offset", [0, 3])
@pytest.mark.parametrize("log_b", range(6, 15))
def test_array_ends(log_b, offset):
    for n in sorted({1, 2, 63, (1 << log_b) - 1, (1 << log_b) + 1, 2047, 2048, 2049, 8191,
                     3 * (1 << log_b) + 5, (1 << 15) + 2048, (1 << 16) - 1}):
        keys = workloads.keys_u32(n, n)
        if n % 2:
            keys = keys % np.uint32(50)  # ties
            keys[::7] = 0xFFFFFFFF       # the padding's value
        assert np.array_equal(_sorted(keys, log_b, offset), _oracle(keys, log_b)), n


@pytest.mark.parametrize("log_b", [6, 11, 12, 14])
def test_zero_one_thresholds(log_b):
    # Rotations and random placements of k ones, k = 0 .. 2^b over 256 buckets.
    rng = np.random.RandomState(log_b)
    size = 1 << log_b
    rows = np.zeros((256, size), np.uint32)
    for i, k in enumerate(np.linspace(0, size, 256).astype(int)):
        rows[i, :k] = 1
        rows[i] = np.roll(rows[i], rng.randint(size)) if i % 2 else rng.permutation(rows[i])
    want = np.sort(rows, axis=1).ravel()
    assert np.array_equal(_sorted(rows.ravel(), log_b, 0), want)


@pytest.mark.parametrize("n", [2, 64, 2048, 2049, 5000, 1 << 14, (1 << 14) + 1, 1 << 15,
                               (1 << 15) + 1, (1 << 19) + 1])
def test_whole_arrays(n):
    # The edges of the rules that send MELD_AUTO sorts and merge sorts to one
    # workgroup, to the network and to radix passes.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    keys = workloads.keys_u32(n, n)
    want = oracle.sort_u32(keys)
    for sort in (meld.sort, meld.merge_sort):
        k = torch.from_numpy(keys.view(np.int32)).to("cuda:0")
        sort(k, variant="auto")
        assert np.array_equal(k.cpu().numpy().view(np.uint32), want), sort.__name__
