"""MELD_AUTO sorts above the network's sizes (radix passes) against the oracle.

Bar: bit-exact; the order of the keys, and of the (key, payload) pairs, is unique.
Sizes at the edges of the rule and of the tiles (2048 up to 2^19 elements, 4096 up to
12 2^20, 8192 above; no scan up to 64 tiles), inputs that leave passes out.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.uint32).view(np.int32)).to(_dev())


def _to_host(t):
    return t.cpu().numpy().view(np.uint32)


def _check(keys, vals, offset=0):
    """Sorts views that start `offset` elements into their buffers."""
    kb = _to_dev(np.concatenate([np.full(offset, 7, np.uint32), keys]))
    if vals is None:
        meld.sort(kb[offset:], variant="auto")
        got, ref = _to_host(kb)[offset:], oracle.sort_u32(keys)
        assert np.array_equal(got, ref)
    else:
        vb = _to_dev(np.concatenate([np.full(offset, 9, np.uint32), vals]))
        meld.sort(kb[offset:], vb[offset:], variant="auto")
        rk, rv = oracle.sort_pairs_u32(keys, vals)
        assert np.array_equal(_to_host(kb)[offset:], rk)
        assert np.array_equal(_to_host(vb)[offset:], rv)
        assert (_to_host(vb)[:offset] == 9).all()
    assert (_to_host(kb)[:offset] == 7).all()


SIZES = [(1 << 15) + 1, (1 << 17) - 1, 1 << 17, (1 << 17) + 1, (1 << 18) + 2047, 1 << 19,
         (1 << 19) + 1, (1 << 20) + 4095]


@pytest.mark.parametrize("n", SIZES)
def test_sizes(n):
    _dev()
    keys = workloads.keys_u32(n, n)
    _check(keys, None)
    _check(keys, workloads.iota_u32(n))
    _check(keys % np.uint32(1000), workloads.keys_u32(n + 1, n))


def _patterns(n):
    u = workloads.keys_u32(5, n)
    yield "equal", np.full(n, 0xFFFFFFFF, np.uint32)
    yield "ascending", np.arange(n, dtype=np.uint32)
    yield "descending", np.arange(n, dtype=np.uint32)[::-1].copy()
    yield "one digit", u & np.uint32(0x00FF0000)
    yield "two digits", u & np.uint32(0xFF0000FF)
    yield "three digits", u & np.uint32(0x00FFFFFF)
    yield "extremes", np.where(u & 1, np.uint32(0xFFFFFFFF), np.uint32(0)).astype(np.uint32)


@pytest.mark.parametrize("n", [(1 << 18) + 5, 150_001])
def test_inputs_that_leave_passes_out(n):
    _dev()
    cases = dict(_patterns(n))
    for name, keys in cases.items():
        _check(keys, None)
        for vals in (workloads.iota_u32(n), workloads.iota_u32(n)[::-1].copy(),
                     cases["one digit"], cases["three digits"]):
            _check(keys, vals)


@pytest.mark.parametrize("offset", [1, 3])
def test_unaligned_views(offset):
    _dev()
    n = (1 << 19) + 4099
    _check(workloads.keys_u32(6, n), workloads.keys_u32(7, n), offset)


@pytest.mark.parametrize("n", [12 << 20, (12 << 20) + 1, 4 * 8192 * 400 + 8191])
def test_large_tiles(n):
    dev = _dev()
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    keys = torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int32, device=dev, generator=gen)
    vals = torch.randint(0, 50, (n,), dtype=torch.int32, device=dev, generator=gen)
    keys[::3] = 11
    k64 = keys.to(torch.int64) & 0xFFFFFFFF
    ref = torch.sort(k64).values
    k = keys.clone()
    meld.sort(k, variant="auto")
    assert torch.equal(k.to(torch.int64) & 0xFFFFFFFF, ref)
    comp = torch.sort(k64 * 64 + vals).values
    for v in (vals.clone(), vals[1:].clone()):
        k = keys[:v.numel()].clone()
        ref = comp if v.numel() == n else torch.sort(k64[:-1] * 64 + v).values
        meld.sort(k, v, variant="auto")
        assert torch.equal((k.to(torch.int64) & 0xFFFFFFFF) * 64 + v, ref)


def test_capture_and_fixed_options_run_the_network():
    dev = _dev()
    n = 1 << 18  # a power of two: the network needs no scratch
    keys = _to_dev(workloads.keys_u32(8, n))
    ref = oracle.sort_u32(workloads.keys_u32(8, n))
    work = torch.empty_like(keys)
    ctx = meld.new_context(0)
    try:
        assert meld.sort_plan(n, variant="auto", ctx=ctx)["sorts_by"] == "radix"
        assert meld.sort_plan(1 << 15, variant="auto", ctx=ctx)["sorts_by"] == "ranks"
        assert meld.sort_plan(n, variant="melded", ctx=ctx)["sorts_by"] == "network"
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            meld.sort(work, variant="auto", ctx=ctx)
        for _ in range(3):
            work.copy_(keys)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(_to_host(work), ref)
            eager = keys.clone()  # scratch of the context comes and goes between replays
            meld.sort(eager, variant="auto", ctx=ctx)
            assert np.array_equal(_to_host(eager), ref)
    finally:
        torch.cuda.synchronize()
        meld.destroy_context(ctx)


@pytest.mark.parametrize("n", [(5 << 14) - 1, 5 << 14, (5 << 14) + 1, (3 << 15) + 5])
def test_pairs_at_the_edge_of_the_rule(n):
    _dev()
    by = meld.sort_plan(n, pairs=True, variant="auto", ctx=meld.context(0))["sorts_by"]
    assert by == ("radix" if n > 5 << 14 else "network")
    keys = workloads.keys_u32(n, n)
    _check(keys, workloads.iota_u32(n))
    _check(keys % np.uint32(1000), workloads.keys_u32(n + 1, n))
