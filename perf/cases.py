"""Workloads that stand for the use of this library, for timing one tree against another.

A case is a dict of plain values; ``prepare`` makes its inputs on the GPU from a seed,
``run`` is one pass through the public entry points, ``work`` what a pass cannot do
without, and ``exact`` the floating-point results in 64 bits.

The sorts work in place, so a pass first copies the unsorted arrays into the ones it
sorts: every pass sorts fresh data, as a program does that keeps its input.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2107_05681_amd as meld
from paper_2107_05681_amd import serve

DEVICE = "cuda:0"
GOLDEN = 0x9E3779B97F4A7C15

# The sides of the region calls: multiplier, stride into the table, and the
# part of the table where the side's offset lies.
SIDES = (dict(a=0.5, step=1031, part=0), dict(a=0.625, step=1543, part=1),
         dict(a=0.75, step=2053, part=2))


def listed():
    return [
        # A short list sorted once in a while: one tile, one launch; call latency counts.
        dict(name="sort_keys_1000", op="sort", n=1000, pairs=False, payload="", keys="uniform",
             form="auto"),
        # The single-array sort of 2^16 random keys: launches and latency of a small sort.
        dict(name="sort_keys_2p16", op="sort", n=1 << 16, pairs=False, payload="",
             keys="uniform", form="auto"),
        # A column of ten million keys with the form fixed by the caller, as the serving loop
        # fixes it; no power of two.
        dict(name="sort_keys_10M_melded", op="sort", n=10_000_019, pairs=False, payload="",
             keys="uniform", form="melded"),
        # A table's rows: a million keys with values of their own beside them.
        dict(name="sort_pairs_1M_values", op="sort", n=1_000_003, pairs=True, payload="values",
             keys="uniform", form="auto"),
        # The largest single-array sort: 2^28 keys with their indices (a stable argsort).
        dict(name="sort_pairs_2p28_index", op="sort", n=1 << 28, pairs=True, payload="index",
             keys="uniform", form="auto"),
        # The batched sort: 4096 uneven buckets, lengths log-uniform in [2^6, 2^16].
        dict(name="segments_4096_uneven", op="segments", nseg=4096, lo=6, hi=16, form="auto"),
        # Many short rows, some of them empty: neighbour lists, per-row candidates.
        dict(name="segments_30k_short", op="segments", nseg=30_001, lo=0, hi=8, form="auto"),
        # The two-sided loop region over 2^24 lanes with a 64 MiB table.
        dict(name="region_2p24", op="region", n=1 << 24, tab=24, p=0.5, t0=10, t1=10,
             form="auto"),
        # The three-way region on a ragged million of lanes, one way much longer.
        dict(name="region3_1M", op="region3", n=1_000_003, tab=24, p0=0.333, p1=0.667, t0=10,
             t1=10, t2=28, form="auto"),
        # Fixed buckets through the odd-even merge network, the last bucket ragged.
        dict(name="oddeven_2p26_b13", op="oddeven", n=(1 << 26) - 77, bucket=13, form="auto"),
        # Bottom-up merge sort of a million keys.
        dict(name="merge_sort_2p20", op="mergesort", n=1 << 20, form="auto"),
        # A burst of mixed requests through the serving loop, results read back.
        dict(name="serve_burst_32", op="serve", jobs=32, lo=10, hi=20),
    ]


def _size(rng, lo, hi):
    """A size log-uniform in [2^lo, 2^hi]: mostly odd ones, now and then a power of two."""
    if rng.random() < 0.25:
        return 1 << rng.randint(math.ceil(lo), math.floor(hi))
    return max(1, int(2.0 ** rng.uniform(lo, hi)) | 1)


def draw(rng):
    op = rng.choice(("sort", "sort", "sort", "segments", "segments", "region", "region3",
                     "lanetrips", "oddeven", "mergesort", "serve"))
    form = "melded" if rng.random() < 0.2 else "auto"
    if op == "sort":
        pairs = rng.random() < 0.5
        return dict(op=op, n=_size(rng, 6, 27), pairs=pairs,
                    payload=rng.choice(("index", "values")) if pairs else "",
                    keys=rng.choice(("uniform", "uniform", "uniform", "narrow")), form=form)
    if op == "segments":
        lo = rng.randint(0, 10)
        hi = rng.randint(lo + 2, 16)
        top = 25.0 - hi  # at most about 2^25 keys in all
        return dict(op=op, nseg=_size(rng, 4, min(17.0, top + 3)), lo=lo, hi=hi, form=form)
    if op in ("region", "region3", "lanetrips"):
        c = dict(op=op, n=_size(rng, 10, 24), tab=rng.randint(16, 24),
                 form=form)
        if op == "region":
            c.update(p=round(rng.uniform(0.05, 0.95), 3), t0=rng.randint(8, 32),
                     t1=rng.randint(8, 32))
        elif op == "region3":
            c.update(p0=round(rng.uniform(0.1, 0.5), 3), p1=round(rng.uniform(0.5, 0.95), 3),
                     t0=rng.randint(8, 32), t1=rng.randint(8, 32), t2=rng.randint(8, 32))
        else:
            c.update(p=round(rng.uniform(0.05, 0.95), 3), t0=8, t1=rng.randint(8, 32))
        return c
    if op == "oddeven":
        return dict(op=op, n=_size(rng, 10, 26), bucket=rng.randint(6, 14), form=form)
    if op == "mergesort":
        return dict(op=op, n=_size(rng, 8, 25), form=form)
    return dict(op="serve", jobs=rng.randint(8, 48), lo=10, hi=rng.randint(16, 20))


def _keys(gen, n, kind="uniform"):
    """Random u32 keys in int32 storage; narrow: ids below 2^20, so with many ties."""
    if kind == "narrow":
        return torch.randint(0, 1 << 20, (n,), dtype=torch.int32, device=DEVICE, generator=gen)
    return torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int32, device=DEVICE,
                         generator=gen)


def _region_inputs(gen, case):
    x = torch.rand(case["n"], dtype=torch.float32, device=DEVICE, generator=gen)
    tab = 0.5 + 0.5 * torch.rand(1 << case["tab"], dtype=torch.float32, device=DEVICE,
                                 generator=gen)
    return x, tab


def _sides(case):
    """The sides (ways) of a region case, each with its offset into the table."""
    quarter = 1 << (case["tab"] - 2)
    which = {"region": (0, 2), "lanetrips": (0, 2), "region3": (0, 1, 2)}[case["op"]]
    out = []
    for k, w in enumerate(which):
        s = SIDES[w]
        side = dict(a=s["a"], off=s["part"] * quarter, step=s["step"])
        if case["op"] == "lanetrips":
            side.update(trips_lo=case["t0"], trips_hi=case["t1"])
        else:
            side.update(trips=case["t%d" % k])
        out.append(side)
    return out


def _thr(p):
    return int(p * 2.0 ** 32)


def _segment_offsets(case, seed):
    """Lengths at the quantiles of the log-uniform distribution, in an order of the seed."""
    q = (np.arange(case["nseg"]) + 0.5) / case["nseg"]
    lens = np.floor(2.0 ** (case["lo"] + (case["hi"] - case["lo"]) * q)).astype(np.int64)
    if case["lo"] == 0:
        lens -= 1  # lengths from 0 up
    np.random.RandomState(seed % (1 << 32)).shuffle(lens)
    return np.concatenate([[0], np.cumsum(lens)])


class _Serving:
    """A server and the requests of one burst; the server ends with the state."""

    def __init__(self, case, seed):
        r = np.random.RandomState(seed % (1 << 32))
        st = dict(a=0.5, off=0, step=1031, trips=10)
        sf = dict(a=0.75, off=1 << 21, step=2053, trips=10)
        self.trace = []
        for k in range(case["jobs"]):
            # Sizes at the quantiles of their log-uniform distributions, small and large
            # ones in turn; what the requests hold comes from the seed.
            q = ((k * 7) % case["jobs"] + 0.5) / case["jobs"]
            job = dict(seed=int(r.randint(1 << 30)), arrival_s=0.0, slot=k)
            if k % 2 == 0:
                job.update(kind=serve.JOB_SORT,
                           n=int(2.0 ** (case["lo"] + (case["hi"] - case["lo"]) * q)))
            else:
                job.update(kind=serve.JOB_REGION, n=int(2.0 ** (16 + 4 * q)), thr=1 << 31,
                           side_true=st, side_false=sf)
            self.trace.append(job)
        self.server = serve.Server(budget_bytes=1 << 30, table_log2=22,
                                   table_seed=seed % (1 << 30))

    def __del__(self):
        if hasattr(self, "server"):
            self.server.close()


def prepare(case, seed):
    if case["op"] == "serve":
        return dict(case=case, serving=_Serving(case, seed))
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    s = dict(case=case)
    if case["op"] == "sort":
        s["keys"] = _keys(gen, case["n"], case["keys"])
        s["out"] = torch.empty_like(s["keys"])
        if case["pairs"]:
            s["payload"] = (torch.arange(case["n"], dtype=torch.int32, device=DEVICE)
                            if case["payload"] == "index" else _keys(gen, case["n"]))
            s["payload_out"] = torch.empty_like(s["payload"])
    elif case["op"] == "segments":
        off = _segment_offsets(case, seed)
        s["offsets"] = torch.from_numpy(off.astype(np.int32)).to(DEVICE)
        s["keys"] = _keys(gen, int(off[-1]))
        s["out"] = torch.empty_like(s["keys"])
    elif case["op"] in ("oddeven", "mergesort"):
        s["keys"] = _keys(gen, case["n"])
        s["out"] = torch.empty_like(s["keys"])
    else:
        s["x"], s["tab"] = _region_inputs(gen, case)
        s["y"] = torch.empty_like(s["x"])
        s["sides"] = _sides(case)
        s["seed"] = seed
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "serve":
        return _run_serve(s["serving"])
    form = case["form"]
    if op == "sort":
        keys = s["out"].copy_(s["keys"])
        if not case["pairs"]:
            return meld.sort(keys, variant=form)
        return meld.sort(keys, s["payload_out"].copy_(s["payload"]), variant=form)
    if op == "segments":
        return meld.segmented_sort(s["out"].copy_(s["keys"]), s["offsets"], variant=form)
    if op == "oddeven":
        meld.oddeven_sort_buckets(s["out"].copy_(s["keys"]), case["bucket"], variant=form)
        return s["out"]
    if op == "mergesort":
        meld.merge_sort(s["out"].copy_(s["keys"]), variant=form)
        return s["out"]
    if op == "region3":
        return meld.region3(s["x"], s["tab"], s["seed"], _thr(case["p0"]), _thr(case["p1"]),
                            *s["sides"], variant=form, out=s["y"])
    call = meld.divergent_region if op == "region" else meld.region_lanetrips
    return call(s["x"], s["tab"], s["seed"], _thr(case["p"]), *s["sides"], variant=form,
                out=s["y"])


def _run_serve(serving):
    results = [None] * len(serving.trace)

    def read(completion, job):
        results[job["slot"]] = serving.server.read(
            completion["job_id"], job["n"],
            "int32" if job["kind"] == serve.JOB_SORT else "float32")

    serve.replay(serving.server, serving.trace, on_complete=read, lead_s=0.0)
    return results


def _mean_trips(case):
    """Steps of a lane on average."""
    if case["op"] == "region":
        return case["p"] * case["t0"] + (1 - case["p"]) * case["t1"]
    if case["op"] == "lanetrips":
        return (case["t0"] + case["t1"]) / 2
    return (case["p0"] * case["t0"] + (case["p1"] - case["p0"]) * case["t1"]
            + (1 - case["p1"]) * case["t2"])


def work(case):
    """Every input read once and every output written once; a region's steps are one
    multiply-add each, and it reads each entry of the sides' table windows once."""
    op = case["op"]
    if op in ("sort", "oddeven", "mergesort"):
        return dict(bytes=8 * case["n"] * (2 if case.get("pairs") else 1), flops=0)
    if op == "segments":
        return dict(bytes=8 * int(_segment_offsets(case, 0)[-1]) + 4 * (case["nseg"] + 1),
                    flops=0)
    if op == "serve":
        # The results; sort inputs and region inputs are made on the device from a seed.
        sizes = case["jobs"] / 2
        mean = (2 ** case["hi"] - 2 ** case["lo"]) / math.log(2.0 ** (case["hi"] - case["lo"]))
        mean_region = (2 ** 20 - 2 ** 16) / math.log(2.0 ** 4)
        return dict(bytes=12 * sizes * (mean + mean_region), flops=20 * sizes * mean_region)
    trips = _mean_trips(case)
    longest = [s["trips"] if "trips" in s else s["trips_hi"] for s in _sides(case)]
    entries = min(1 << case["tab"],
                  sum(case["n"] + t * s["step"] for t, s in zip(longest, _sides(case))))
    return dict(bytes=8 * case["n"] + 4 * entries, flops=2 * trips * case["n"])


def _i64(v):
    """The 64-bit pattern of v as a signed integer."""
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _shift(z, s):
    return (z >> s) & ((1 << (64 - s)) - 1)


def _mix64(z):
    """SplitMix64's output mixer on int64 tensors (their products wrap)."""
    z = (z ^ _shift(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shift(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shift(z, 31)


def _lane_bits(seed, tag, lanes):
    """The upper 32 bits of the hash of (seed, tag, lane)."""
    base = _mix64(torch.tensor(_i64(seed + tag * GOLDEN), dtype=torch.int64, device=DEVICE))
    return _shift(_mix64(base + lanes), 32)


def exact(case, seed):
    if case["op"] not in ("region", "region3", "lanetrips"):
        return None  # whole numbers
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    x, tab = _region_inputs(gen, case)
    tab = tab.double()
    sides = _sides(case)
    out = torch.empty(case["n"], dtype=torch.float64, device=DEVICE)
    block = 1 << 22
    for lo in range(0, case["n"], block):
        lanes = torch.arange(lo, min(lo + block, case["n"]), dtype=torch.int64, device=DEVICE)
        h = _lane_bits(seed, 4, lanes)
        if case["op"] == "region3":
            way = (h >= _thr(case["p0"])).long() + (h >= _thr(case["p1"])).long()
        else:
            way = (h >= _thr(case["p"])).long()

        def pick(key):
            vals = torch.tensor([float(s[key]) for s in sides], dtype=torch.float64,
                                device=DEVICE)
            return vals[way]

        a, off, step = pick("a"), pick("off").long(), pick("step").long()
        if case["op"] == "lanetrips":
            span = case["t1"] - case["t0"] + 1
            trips = case["t0"] + _lane_bits(seed, 11, lanes) % span
        else:
            trips = pick("trips").long()
        acc = x[lo:lo + block].double()
        for k in range(int(trips.max())):
            idx = ((lanes + off + k * step) & 0xFFFFFFFF) & ((1 << case["tab"]) - 1)
            acc = torch.where(k < trips, acc * a + tab[idx], acc)
        out[lo:lo + block] = acc
    return out
