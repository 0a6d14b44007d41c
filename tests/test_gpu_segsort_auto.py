"""MELD_AUTO segmented sorts in registers against the oracle.

Bar: bit-exact. Every size class at its edges, chunk counts 1 to 4 of the segments
above 2^14 keys, few and many segments of a class (partly filled work items), calls in
a row on one context, a refused call between two good ones.
"""
import json

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


@pytest.fixture
def ctx(tmp_path):
    """A context whose tuner always picks the sort in registers."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = meld.new_context(0)
    head = json.loads(meld.plan_describe(ctx=c))
    lines = ['{"op": "segsort", "key": "nseg=%d keys=%d r", "lo": 1, "hi": 1, "log_t": 0, '
             '"xch": 2, "form": 1, "ms": 1.0, "mixed_lo": 0.0, "mixed_hi": 0.0, "trials": 9}'
             % (s, k) for s in range(0, 20) for k in range(0, 32)]
    path = tmp_path / "tune.json"
    path.write_text('{"version": %d, "arch": "%s", "runtime": %d, "entries": [\n'
                    % (head["version"], head["arch"], head["runtime"])
                    + ",\n".join(lines) + "\n]}\n")
    assert meld.load_library().meld_tune(c, str(path).encode()) == meld.OK
    yield c
    meld.destroy_context(c)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.uint32).view(np.int32)).to("cuda:0")


def _check(ctx, lengths, seed, kind="uniform"):
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.uint32)
    n = int(off[-1])
    guard = np.arange(99, dtype=np.uint32)
    keys = workloads.keys_u32(seed, n)
    if kind == "ties":
        keys = keys % np.uint32(5)
        keys[::11] = 0xFFFFFFFF
    buf = _dev(np.concatenate([keys, guard]))
    meld.segmented_sort(buf[:n], _dev(off), variant="auto", ctx=ctx)
    got = buf.cpu().numpy().view(np.uint32)
    meld.segmented_sort_check(0, ctx=ctx)
    assert np.array_equal(got[n:], guard)
    assert np.array_equal(got[:n], oracle.segmented_sort_u32(keys, off))


@pytest.mark.parametrize("kind", ["uniform", "ties"])
def test_class_edges(ctx, kind):
    lengths = [0, 1]
    for c in range(1, 17):
        lengths += [(1 << c) - 1, 1 << c, min((1 << c) + 1, 65536)]
    lengths += [3 << 14, (3 << 14) + 1, (3 << 14) - 1, (1 << 15) + (1 << 14) - 5, 65535, 40000]
    _check(ctx, lengths, 3, kind)
    _check(ctx, lengths[::-1], 4, kind)


@pytest.mark.parametrize("length,count", [(5, 3000), (33, 1), (64, 65), (100, 17), (700, 300),
                                          (2048, 9), (3000, 5), (5000, 3), (9000, 2),
                                          (16384, 3), (20000, 2), (65536, 2)])
def test_counts_of_one_class(ctx, length, count):
    _check(ctx, [length] * count, length)


def test_zero_one_and_orders(ctx):
    n = 50_000
    i = np.arange(n)
    rows = [i, i[::-1], i % 2, (i < 20_000), (i >= 20_000), (i // 16384) % 2, np.zeros(n),
            i ^ 0x5555]
    keys = np.concatenate(rows).astype(np.uint32)
    off = (np.arange(len(rows) + 1) * n).astype(np.uint32)
    buf = _dev(keys)
    meld.segmented_sort(buf, _dev(off), variant="auto", ctx=ctx)
    want = np.concatenate([np.sort(r) for r in rows]).astype(np.uint32)
    assert np.array_equal(buf.cpu().numpy().view(np.uint32), want)


def test_refused_calls_leave_the_context_usable(ctx):
    _check(ctx, [100, 20000, 7], 1)
    keys = workloads.keys_u32(2, 200)
    for off in ([0, 100, 300], [0, 150, 120, 200], [4, 100, 200], [0, 70000]):
        kd = _dev(keys if off[-1] != 70000 else np.zeros(70000, np.uint32))
        before = kd.clone()
        if off[-1] == 300:  # beyond the keys: refused at once, nothing recorded
            with pytest.raises(meld.MeldError) as err:
                meld.segmented_sort(kd, _dev(off), variant="auto", ctx=ctx)
            assert err.value.status == meld.EINVAL
            meld.segmented_sort_check(0, ctx=ctx)
        else:
            meld.segmented_sort(kd, _dev(off), variant="auto", ctx=ctx)
            with pytest.raises(meld.MeldError):
                meld.segmented_sort_check(0, ctx=ctx)
        assert torch.equal(kd, before)
        _check(ctx, [3000, 40000, 64, 0, 9], 5)
