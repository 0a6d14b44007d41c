// Segmented sort in registers (wave_network.h): the candidate of MELD_AUTO that
// sorts many uneven buckets with the ascending network. In place, without
// staging memory, in three launches:
//   1. classify — checks, and the size class of every segment: the smallest c
//                 with len <= 2^c, at least 6 (0 for len <= 1: nothing to do);
//   2. scatter  — segment ids into a queue, largest class first;
//   3. sort     — a persistent grid of eight-wave workgroups takes work items
//                 from a counter. An item of a class >= 12 is 2^14 positions (one
//                 segment of more, or 2^(14-c) of class c) and belongs to a
//                 workgroup; below, where no data crosses a wave, it is 2^11
//                 positions (2^(11-c) segments) and belongs to a wave, dealt out
//                 in turn (one counter for 4096 waves took 55 us by itself).
// The counters exist twice: a call's sort clears those of the next call.
//
// A segment of more than 2^14 keys is sorted in chunks of 2^14, then merged in
// phases 2^15 and 2^16: the steps across chunks while loading, the rest of a
// chunk in registers. The direction of a chunk is bit p of i ^ (len - 1), so that
// the segment's end ascends in every phase, its padding stays past len and no
// chunk without keys is ever touched.
#include <type_traits>

#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kSaPad = 0xFFFFFFFFu;
constexpr uint32_t kSaWaves = 8;
constexpr uint32_t kSaThreads = kSaWaves * 64;
constexpr uint32_t kSaMinClass = 6;
constexpr uint32_t kSaLogTile = 14, kSaTile = 1u << kSaLogTile;
constexpr uint32_t kSaTopWaveClass = 11;
constexpr size_t kSaLds = (size_t)wave_lds_words(kSaTile) * sizeof(uint32_t);

__device__ __forceinline__ uint32_t sa_class(uint32_t len) {
    if (len <= 1) return 0;
    const uint32_t c = 32u - (uint32_t)__clz(len - 1);
    return c < kSaMinClass ? kSaMinClass : c;
}

// total: NULL, or host memory that receives offsets[nseg]; the caller then
// refuses a call whose offsets[nseg] lies beyond the keys, which is therefore
// not recorded for meld_segmented_sort_check.
__global__ __launch_bounds__(256) void sa_classify_kernel(const uint32_t *__restrict__ off,
                                                          uint32_t nseg, uint32_t n_keys,
                                                          SegAutoState *st, uint32_t *sticky,
                                                          uint8_t *__restrict__ cls,
                                                          uint32_t *total) {
    __shared__ uint32_t lcnt[kSegClasses];
    if (threadIdx.x < kSegClasses) lcnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t s = blockIdx.x * 256 + threadIdx.x;
    if (s == 0 && total != nullptr) *total = off[nseg];
    if (s < nseg) {
        const uint32_t lo = off[s];
        const uint32_t hi = off[s + 1];
        uint32_t f = 0;
        if (s == 0 && lo != 0) f |= kSegBadFirst;
        if (hi > n_keys) f |= kSegBeyondEnd;
        if (hi < lo)
            f |= kSegDecreasing;
        else if (hi - lo > kSegMaxLen)
            f |= kSegTooLong;
        if (f != 0) {
            atomicOr(&st->flag, f);
            if (total == nullptr || off[nseg] <= n_keys) atomicOr(sticky, f);
        }
        const uint32_t c = f != 0 ? 0u : sa_class(hi - lo);
        cls[s] = (uint8_t)c;
        if (c != 0) atomicAdd(&lcnt[c], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kSegClasses && lcnt[threadIdx.x] != 0)
        atomicAdd(&st->cnt[threadIdx.x], lcnt[threadIdx.x]);
}

__global__ __launch_bounds__(256) void sa_scatter_kernel(uint32_t nseg,
                                                         const uint8_t *__restrict__ cls,
                                                         SegAutoState *st,
                                                         uint32_t *__restrict__ queue) {
    __shared__ uint32_t lcnt[kSegClasses];
    __shared__ uint32_t lbase[kSegClasses];
    if (threadIdx.x < kSegClasses) lcnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t s = blockIdx.x * 256 + threadIdx.x;
    const uint32_t c = s < nseg ? cls[s] : 0u;
    const uint32_t rank = c != 0 ? atomicAdd(&lcnt[c], 1u) : 0u;
    __syncthreads();
    if (threadIdx.x < kSegClasses && lcnt[threadIdx.x] != 0) {
        uint32_t base = 0;
        for (uint32_t k = threadIdx.x + 1; k < kSegClasses; ++k) base += st->cnt[k];
        lbase[threadIdx.x] = base + atomicAdd(&st->fill[threadIdx.x], lcnt[threadIdx.x]);
    }
    __syncthreads();
    if (c != 0) queue[lbase[c] + rank] = s;
}

// Where the queue's classes and their work items start.
struct SaPlan {
    uint32_t cnt[kSegClasses];
    uint32_t base[kSegClasses];
    uint32_t first[kSegClasses];  // first item, of the workgroups' or of the waves'
    uint32_t big, small;          // items of either kind
    uint32_t flag;
    uint32_t item;
};

__device__ __forceinline__ uint32_t sa_items(uint32_t c, uint32_t cnt) {
    const uint32_t top = c > kSaTopWaveClass ? kSaLogTile : kSaTopWaveClass;
    return c >= top ? cnt : (cnt + (1u << (top - c)) - 1) >> (top - c);
}

__device__ __forceinline__ void sa_plan(SegAutoState *st, SaPlan &p) {
    if (threadIdx.x < kSegClasses) p.cnt[threadIdx.x] = st->cnt[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t at = 0, big = 0, small = 0;
        for (uint32_t c = kSegClasses - 1; c >= kSaMinClass; --c) {
            p.base[c] = at;
            at += p.cnt[c];
            uint32_t &items = c > kSaTopWaveClass ? big : small;
            p.first[c] = items;
            items += sa_items(c, p.cnt[c]);
        }
        p.big = big;
        p.small = small;
        p.flag = st->flag;
    }
    __syncthreads();
}

// Hides v's value from the optimiser at this point, so that what is computed
// from it is computed where it is used, not kept in registers from before.
__device__ __forceinline__ void opaque(uint32_t &v) { asm volatile("" : "+v"(v)); }

// Key i of a segment: its start plus a byte offset of 32 bits, which a segment
// that is the workgroup's takes from a scalar register.
__device__ __forceinline__ uint32_t &key_at(uint32_t *k, uint32_t i) {
    return *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(k) + (i << 2));
}

__device__ __forceinline__ uint32_t scalar(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// The class of classes hi .. lo whose items hold `item`.
__device__ __forceinline__ uint32_t sa_class_of(const SaPlan &p, uint32_t item, uint32_t hi,
                                                uint32_t lo) {
    uint32_t c = hi;
    while (c > lo && item >= p.first[c] + sa_items(c, p.cnt[c])) --c;
    return c;
}

// Phases 2^M .. 2^min(c, 11) on keys complemented for phase 2^M.
template <int M>
__device__ __forceinline__ void sa_wave_phases(uint32_t (&e)[kWaveE], const WaveLane &w,
                                               uint32_t high, uint32_t c) {
    wave_steps<M - 1>(e, w);
    if constexpr (M < 11) {
        if (c > M) {
            const uint32_t now = wave_down<M, 16>(high);
            wave_flip(e, c > M + 1 ? now ^ wave_down<M + 1, 16>(high) : now);
            sa_wave_phases<M + 1>(e, w, high, c);
        }
    }
}

// Phases 2^M .. 2^c (M >= 12) on keys complemented for phase 2^(M-1).
template <int M>
__device__ __forceinline__ void sa_cross_phases(uint32_t (&e)[kWaveE], uint32_t *s,
                                                const WaveLane &w, uint32_t high, uint32_t c) {
    if constexpr (M <= (int)kSaLogTile) {
        if (c >= M) {
            const uint32_t now = wave_down<M - 1, 16>(high);
            wave_flip(e, c > M ? now ^ wave_down<M, 16>(high) : now);
            wave_cross_steps<kSaLogTile, M - 1>(e, s, w);
            wave_steps<10>(e, w);
            sa_cross_phases<M + 1>(e, s, w, high, c);
        }
    }
}

// Where the keys of a tile or of a wave's part of one go: a segment of len keys
// at lo, per lane; or, whole, a tile of 2^14 keys that all exist, at an lo that is
// the workgroup's: then no access needs a check, and all of them share one
// scalar base (checked, an access takes three to five VALU operations).
struct SaPlace {
    uint32_t lo, len;
    bool whole;
};

// Writes the wave's sorted rows to the caller's keys: position i of the wave's
// 2^11 is key (first + i) mod 2^c of the segment of the lanes that hold it, if it
// has one. traded: bits 9 and 10 are in each other's place.
__device__ __forceinline__ void sa_store(const uint32_t (&e)[kWaveE], uint32_t *own,
                                         const WaveLane &w, uint32_t *__restrict__ keys,
                                         const SaPlace &at, uint32_t c, uint32_t first,
                                         bool traded, uint32_t flip) {
    if (traded)
        wave_to_lds<true>(e, own, w);
    else
        wave_to_lds<false>(e, own, w);
    __builtin_amdgcn_wave_barrier();
    uint32_t lane = threadIdx.x & 63;
    if (at.whole) {
        uint32_t *k = keys + scalar(at.lo) + scalar(first);
#pragma unroll
        for (int r = 0; r < kWaveE; ++r)
            key_at(k + r * 64, lane) = own[wave_phys(lane) + wave_phys(r * 64)] ^ flip;
    } else {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) {
            opaque(lane);
            const uint32_t i = r * 64;
            // Lanes of the wave by element order, one per 32 positions.
            const uint32_t id = c < kSaTopWaveClass ? i >> c << (c - 5) : 0u;
            const int src = (int)(id ^ ((id & 4) ? 3u : 0u));
            const uint32_t slo = (uint32_t)__builtin_amdgcn_readlane((int)at.lo, src);
            const uint32_t slen = (uint32_t)__builtin_amdgcn_readlane((int)at.len, src);
            const uint32_t p = (first + i + lane) & ((1u << c) - 1);
            if (p < slen) key_at(keys + slo, p) = own[wave_phys(lane) + wave_phys(i)] ^ flip;
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// Keys b + r * 512 + thread of a segment, padding past its end.
__device__ __forceinline__ void sa_load_rows(uint32_t (&e)[kWaveE], uint32_t *__restrict__ k,
                                             uint32_t b, uint32_t len) {
    if (b + kSaTile <= len) {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) e[r] = key_at(k + b + r * kSaThreads, threadIdx.x);
    } else {
        uint32_t p = b + threadIdx.x;
        opaque(p);
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) {
            e[r] = kSaPad;
            if (p < len) e[r] = key_at(k, p);
            p += kSaThreads;
            opaque(p);
        }
    }
}

// The keys of the lane's segment, at most 2^c shared by 2^(c-5) lanes, in any
// order; id as for sa_sort.
__device__ __forceinline__ void sa_load(uint32_t (&e)[kWaveE], uint32_t *__restrict__ keys,
                                        uint32_t lo, uint32_t len, uint32_t c, uint32_t id) {
    const uint32_t log_lanes = c - 5;
    uint32_t p = id & ((1u << log_lanes) - 1);
    uint32_t *k = keys + lo;
#pragma unroll
    for (int r = 0; r < kWaveE; ++r) {
        e[r] = kSaPad;
        if (p < len) e[r] = key_at(k, p);
        p += 1u << log_lanes;
        opaque(p);  // one address at a time
    }
}

// Sorts the keys loaded for the segment of at most 2^c keys of the 2^(c-5) lanes
// that share it (6 <= c <= 14) and stores them; id numbers the lanes by element
// order, in the wave for c <= 11, in the workgroup above, where all eight waves
// take part. With flip = ~0 in descending order (a whole tile).
__device__ __forceinline__ void sa_sort(uint32_t (&e)[kWaveE], uint32_t *__restrict__ keys,
                                        const SaPlace &at, uint32_t c, uint32_t id, uint32_t flip,
                                        uint32_t *s, const WaveLane &w) {
    if (flip != 0) wave_flip(e, ~0u);
    wave_first_phases<1, 0>(e);
    wave_flip(e, wave_down<5, 16>(id));
    sa_wave_phases<5>(e, w, id, c);
    sa_cross_phases<12>(e, s, w, id, c);
    uint32_t *own = s + threadIdx.x / 64 * wave_lds_words(kWaveTile);
    sa_store(e, own, w, keys, at, c, (id & ~63u) * 32, c >= kSaTopWaveClass, flip);
}

// Steps j = 2^13 .. 1 on a chunk held as element r * 512 + thread, then its
// store.
__device__ __forceinline__ void sa_merge(uint32_t (&e)[kWaveE], uint32_t *__restrict__ keys,
                                         const SaPlace &at, uint32_t flip, uint32_t *s,
                                         const WaveLane &w) {
    uint32_t t = threadIdx.x;
    opaque(t);
    wave_reg_steps<4>(e);
    __syncthreads();  // every wave has read its rows of the last tile
#pragma unroll
    for (int r = 0; r < kWaveE; ++r) s[wave_phys(t) + wave_phys(r * kSaThreads)] = e[r];
    __syncthreads();
    uint32_t *own = s + t / 64 * wave_lds_words(kWaveTile);
    wave_from_lds<false>(e, own, w);
    wave_steps<8>(e, w);
    sa_store(e, own, w, keys, at, kSaLogTile, (t & ~63u) * 32, false, flip);
}

// Phase 2^P (15 or 16) on the block of 2^(P-14) chunks at position b of the
// segment of len keys at keys + lo: the first chunk's keys stay in registers, the
// others' go back to memory after the steps across chunks; each is read again
// while the one before it is merged.
template <int P>
__device__ __forceinline__ void sa_phase(uint32_t *__restrict__ keys, uint32_t lo, uint32_t len,
                                         uint32_t b, uint32_t *s, const WaveLane &w) {
    constexpr uint32_t G = 1u << (P - kSaLogTile);
    if (b + G / 2 * kSaTile >= len) return;  // one half alone: ascending already
    const uint32_t flip = (uint32_t)-(int32_t)(((b ^ (len - 1)) >> P) & 1u);
    uint32_t *k = keys + lo;
    uint32_t e[kWaveE];
    __syncthreads();  // the stores of the last phase are visible to the workgroup
    constexpr int R = 32 / G;  // rows in flight
    auto cross = [&](auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        uint32_t p = b + threadIdx.x;
        if (!WHOLE) opaque(p);
#pragma unroll
        for (int r0 = 0; r0 < kWaveE; r0 += R) {
            uint32_t v[R][G];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (uint32_t q = 0; q < G; ++q) {
                    if (WHOLE) {
                        v[r][q] = key_at(k + b + q * kSaTile + (r0 + r) * kSaThreads, threadIdx.x);
                    } else {
                        const uint32_t i = p + r * kSaThreads + q * kSaTile;
                        v[r][q] = kSaPad;
                        if (i < len) v[r][q] = key_at(k, i);
                    }
                }
            if (!WHOLE) opaque(p);
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (uint32_t q = 0; q < G; ++q) v[r][q] ^= flip;
#pragma unroll
                for (uint32_t j = G / 2; j >= 1; j /= 2)
#pragma unroll
                    for (uint32_t q = 0; q < G; ++q)
                        if ((q & j) == 0) {
                            const uint32_t x = v[r][q], y = v[r][q | j];
                            v[r][q] = x < y ? x : y;
                            v[r][q | j] = x < y ? y : x;
                        }
                e[r0 + r] = v[r][0];
#pragma unroll
                for (uint32_t q = 1; q < G; ++q) {
                    if (WHOLE) {
                        key_at(k + b + q * kSaTile + (r0 + r) * kSaThreads, threadIdx.x) = v[r][q];
                    } else {
                        const uint32_t i = p + r * kSaThreads + q * kSaTile;
                        if (i < len) key_at(k, i) = v[r][q];
                    }
                }
            }
            p += R * kSaThreads;
            if (!WHOLE) opaque(p);
        }
    };
    if (b + G * kSaTile <= len)
        cross(std::true_type{});
    else
        cross(std::false_type{});
#pragma unroll 1
    for (uint32_t q = 0;;) {
        const uint32_t at = b + q * kSaTile;
        const bool more = ++q < G && at + kSaTile < len;
        uint32_t f[kWaveE];
        if (more) sa_load_rows(f, k, at + kSaTile, len);
        sa_merge(e, keys, SaPlace{lo + at, len - at, at + kSaTile <= len}, flip, s, w);
        if (!more) break;
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) e[r] = f[r];
    }
}

// A work item of a workgroup: class c >= 12, number k of the class.
__device__ __forceinline__ void sa_big_item(uint32_t *__restrict__ keys,
                                            const uint32_t *__restrict__ off,
                                            const uint32_t *__restrict__ queue, const SaPlan &plan,
                                            uint32_t c, uint32_t k, uint32_t *s,
                                            const WaveLane &w) {
    const uint32_t id = (threadIdx.x & ~63u) | w.id;
    const uint32_t cc = c < kSaLogTile ? c : kSaLogTile;
    const uint32_t q = (k << (kSaLogTile - cc)) + (id >> (cc - 5));
    uint32_t lo = 0, len = 0;  // lanes past the class's last segment idle
    if (q < plan.cnt[c]) {
        const uint32_t seg = queue[plan.base[c] + q];
        lo = off[seg];
        len = off[seg + 1] - lo;
    }
    uint32_t e[kWaveE];
    if (c >= kSaLogTile) {  // one segment
        lo = scalar(lo);
        len = scalar(len);
        sa_load_rows(e, keys + lo, 0, len);
    } else {
        sa_load(e, keys, lo, len, c, id);
    }
    uint32_t b = 0;
#pragma unroll 1
    for (;;) {
        const bool more = c > kSaLogTile && b + kSaTile < len;
        uint32_t f[kWaveE];
        if (more) sa_load_rows(f, keys + lo, b + kSaTile, len);  // while this chunk is sorted
        SaPlace at{lo + b, len - b, false};
        uint32_t flip = 0;
        if (c >= kSaLogTile) {
            at.whole = b + kSaTile <= len;
            flip = (uint32_t)-(int32_t)(((b ^ (len - 1)) >> kSaLogTile) & 1u);
        }
        sa_sort(e, keys, at, cc, id, flip, s, w);
        if (!more) break;
        b += kSaTile;
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) e[r] = f[r];
    }
    if (c <= kSaLogTile) return;
#pragma unroll 1
    for (b = 0; b < len; b += 2 * kSaTile) sa_phase<15>(keys, lo, len, b, s, w);
    if (c > 15) sa_phase<16>(keys, lo, len, 0, s, w);
}

// Two workgroups of eight waves per CU (72 KiB of LDS each). 4096 segments of
// log-uniform length in [2^6, 2^16], 3.9e7 keys: 315 us (the network's kernel: 500).
// 2048 segments of 2^14 keys run at the rate of VALU issue (157 operations a key);
// at 2^16 keys the two phases across chunks, 50 more operations, wait for the
// memory half of their time, and the last segments of 2^15 keys leave the chip
// partly idle.
__global__ __launch_bounds__(kSaThreads, 4) void sa_sort_kernel(uint32_t *__restrict__ keys,
                                                                const uint32_t *__restrict__ off,
                                                                const uint32_t *__restrict__ queue,
                                                                SegAutoState *st,
                                                                SegAutoState *next) {
    extern __shared__ __align__(16) uint32_t s[];
    __shared__ SaPlan plan;
    const WaveLane w = wave_lane();
    const uint32_t tid = threadIdx.x;
    sa_plan(st, plan);
    if (blockIdx.x == 0 && tid < sizeof(SegAutoState) / 4) reinterpret_cast<uint32_t *>(next)[tid] = 0;
    if (plan.flag == 0) {  // otherwise invalid offsets: leave the keys untouched
        // The first item is the workgroup's own number, later ones come from the
        // counter when it is done: largest first, whoever is free.
        for (uint32_t item = blockIdx.x; item < plan.big;) {
            const uint32_t c = sa_class_of(plan, item, kSegClasses - 1, kSaTopWaveClass + 1);
            sa_big_item(keys, off, queue, plan, c, item - plan.first[c], s, w);
            __syncthreads();
            if (tid == 0) plan.item = gridDim.x + atomicAdd(&st->head, 1u);
            __syncthreads();
            item = scalar(plan.item);
        }
        // Neighbouring items go to different CUs.
        for (uint32_t item = scalar(tid / 64 * gridDim.x + blockIdx.x); item < plan.small;
             item += kSaWaves * gridDim.x) {
            const uint32_t c = sa_class_of(plan, item, kSaTopWaveClass, kSaMinClass);
            const uint32_t q = ((item - plan.first[c]) << (kSaTopWaveClass - c)) + (w.id >> (c - 5));
            uint32_t lo = 0, len = 0;
            if (q < plan.cnt[c]) {
                const uint32_t seg = queue[plan.base[c] + q];
                lo = off[seg];
                len = off[seg + 1] - lo;
            }
            uint32_t e[kWaveE];
            sa_load(e, keys, lo, len, c, w.id);
            sa_sort(e, keys, SaPlace{lo, len, false}, c, w.id, 0, s, w);
        }
    }
}

}  // namespace

hipError_t seg_auto_grid(int device, uint32_t *grid) {
    int cus = 0, per_cu = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(sa_sort_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSaLds);
    if (e != hipSuccess) return e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(sa_sort_kernel), kSaThreads, kSaLds);
    if (e != hipSuccess) return e;
    *grid = (uint32_t)(cus * (per_cu < 1 ? 1 : per_cu));
    return hipSuccess;
}

hipError_t launch_segmented_auto_plan(uint32_t n_keys, const uint32_t *off, uint32_t nseg,
                                      SegAutoState *st, uint32_t *sticky, uint8_t *cls,
                                      uint32_t *total, hipStream_t stream) {
    hipLaunchKernelGGL(sa_classify_kernel, dim3(blocks_for(nseg, 256)), dim3(256), 0, stream, off,
                       nseg, n_keys, st, sticky, cls, total);
    return hipGetLastError();
}

hipError_t launch_segmented_auto_sort(uint32_t *keys, const uint32_t *off, uint32_t nseg,
                                      SegAutoState *st, SegAutoState *next, const uint8_t *cls,
                                      uint32_t *queue, uint32_t grid, hipStream_t stream) {
    hipLaunchKernelGGL(sa_scatter_kernel, dim3(blocks_for(nseg, 256)), dim3(256), 0, stream, nseg,
                       cls, st, queue);
    hipLaunchKernelGGL(sa_sort_kernel, dim3(grid), dim3(kSaThreads), kSaLds, stream, keys, off,
                       (const uint32_t *)queue, st, next);
    return hipGetLastError();
}

}  // namespace meld
