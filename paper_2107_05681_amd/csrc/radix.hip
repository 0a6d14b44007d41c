// Least-significant-digit radix sort of u32 keys or (key, payload) pairs, the
// path MELD_AUTO takes for single arrays that outgrow a few tiles.
//
// Eight-bit digits. A word is sorted in up to four passes; pairs sort by the
// payload first and then, stably, by the key, which is the lexicographic
// (key, payload) order. A pass is
//   count    digit counts of every tile (one read of the word),
//   scan     their exclusive prefix over the tiles, digit by digit,
//   scatter  every tile ordered by the digit in LDS and written out.
// Positions come from the counts alone: no workgroup waits for another.
//
// The first count of a word also finds the bits in which its values differ
// and whether they already stand in order. Passes over digits that are the
// same everywhere are left out, and all four where the order is there already
// (a payload that holds the index). The number of passes that run is kept
// even, so that the result ends in the caller's arrays.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace meld {

namespace {

constexpr int kRadixBits = 8;
constexpr uint32_t kDigits = 1u << kRadixBits;
constexpr int kGroupPasses = 32 / kRadixBits;  // passes over one 32-bit word

struct RadixArgs {
    uint32_t *word[2];   // the word to sort by: caller's array, scratch
    uint32_t *other[2];  // the word moved along (NULL for keys alone)
    uint32_t n;
    uint32_t pass;     // 0 .. 3
    uint32_t tiles;    // tiles that cover n
    uint32_t stride;   // row length of counts: tiles, rounded up to 16
    uint32_t *counts;  // [digit][tile]; unscanned [tile][digit], 16 bits each
    uint32_t *totals;  // [digit]
    uint32_t *part;    // [count workgroup]: differing bits, then disorder
    uint32_t parts;    // count workgroups
    uint32_t *ctl;     // mask of the word's passes that run
};

// A wave's 16-bit digit counts, which other lanes clear and add up two to a word
// between barriers of the wave, which order no memory by themselves: a type that may
// alias the words keeps the compiler from moving these accesses past those.
typedef uint16_t __attribute__((may_alias)) Count16;

__device__ __forceinline__ uint32_t digit_of(uint32_t x, uint32_t shift) {
    return (x >> shift) & (kDigits - 1);
}

// Passes that run for a word whose values differ in the bits of diff.
__device__ __forceinline__ uint32_t passes_to_run(uint32_t diff, bool ordered) {
    if (ordered) return 0;
    uint32_t m = 0;
#pragma unroll
    for (int p = 0; p < kGroupPasses; ++p)
        if ((diff >> (p * kRadixBits)) & (kDigits - 1)) m |= 1u << p;
    if (__popc(m) & 1) m |= ~m & (m + 1u);  // the lowest pass left out, so that they are even
    return m;
}

// Which of the two buffers pass `pass` reads.
__device__ __forceinline__ uint32_t source_of(uint32_t run, uint32_t pass) {
    return __popc(run & ((1u << pass) - 1u)) & 1u;
}

__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// Loads with the nontemporal hint where the arrays outgrow the caches.
template <bool NTL>
__device__ __forceinline__ uint32_t load4(const uint32_t *p) {
    if constexpr (NTL) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NTL>
__device__ __forceinline__ uint4 load16(const uint32_t *p) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 *q = reinterpret_cast<const u32x4 *>(p);
    u32x4 v;
    if constexpr (NTL)
        v = __builtin_nontemporal_load(q);
    else
        v = *q;
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x |= (uint32_t)__shfl_xor((int)x, d);
    return x;
}

// Exclusive scan of x over the wave's 64 lanes.
__device__ __forceinline__ uint32_t wave_exclusive_scan(uint32_t x, uint32_t lane) {
    uint32_t v = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)v, d);
        if (lane >= (uint32_t)d) v += y;
    }
    return v - x;
}

// Digit counts of TPB tiles of TILE elements, 256 lanes a tile; every load of
// a tile is issued before the first count. Bound by the read: 184 us per 2^28
// words (5.8 TB/s) with the nontemporal hint, 265 us without it. Groups of
// tiles go to the XCDs in contiguous ranges, so that the short pieces of the
// count rows that neighbours write meet in one L2. FIRST (pass 0): also the bits that
// differ from the array's first value and whether a value exceeds the next.
template <int TILE, int TPB, bool NTL, bool FIRST, bool SCANNED>
__global__ __launch_bounds__(256 * TPB) void radix_count_kernel(RadixArgs a) {
    constexpr int Q = TILE / (256 * 4);  // 16-byte loads per lane
    __shared__ uint32_t hist[TPB][kDigits];
    __shared__ uint32_t red[2][4 * TPB];
    const uint32_t t = threadIdx.x, sub = t / 256, l = t % 256;
    const uint32_t *src = a.word[0];
    if constexpr (!FIRST) {
        const uint32_t run = uniform(*a.ctl);
        if (((run >> a.pass) & 1u) == 0) return;
        src = a.word[source_of(run, a.pass)];
    }
    const uint32_t group = xcd_contiguous_block(blockIdx.x, a.parts);
    const uint32_t tile = group * TPB + sub;
    const uint32_t shift = a.pass * kRadixBits;
    hist[sub][l] = 0;
    __syncthreads();
    uint32_t x0 = 0, diff = 0, bad = 0;
    if constexpr (FIRST) x0 = src[0];
    uint32_t *h = hist[sub];
    const uint64_t base64 = (uint64_t)tile * TILE;
    if (base64 + TILE <= a.n && (((uintptr_t)src) & 15) == 0) {
        const uint32_t *p = src + base64;
        uint4 x[Q];
        uint32_t after[Q];  // the value after the wave's last one (lane 63)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t i = (q * 256 + l) * 4;
            x[q] = load16<NTL>(p + i);
            if constexpr (FIRST) {
                after[q] = 0;
                if ((l & 63) == 63) after[q] = src[min((uint32_t)base64 + i + 4, a.n - 1)];
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            atomicAdd(&h[digit_of(x[q].x, shift)], 1u);
            atomicAdd(&h[digit_of(x[q].y, shift)], 1u);
            atomicAdd(&h[digit_of(x[q].z, shift)], 1u);
            atomicAdd(&h[digit_of(x[q].w, shift)], 1u);
            if constexpr (FIRST) {
                const uint32_t down = (uint32_t)__shfl_down((int)x[q].x, 1);
                const uint32_t next = (l & 63) == 63 ? after[q] : down;
                diff |= (x[q].x ^ x0) | (x[q].y ^ x0) | (x[q].z ^ x0) | (x[q].w ^ x0);
                bad |= (x[q].x > x[q].y) | (x[q].y > x[q].z) | (x[q].z > x[q].w) |
                       (x[q].w > next);
            }
        }
    } else if (base64 < a.n) {
        const uint32_t base = (uint32_t)base64;
        const uint32_t end = min((uint64_t)a.n, base64 + TILE);
        for (uint32_t i = base + l; i < end; i += 256) {
            const uint32_t x = src[i];
            atomicAdd(&h[digit_of(x, shift)], 1u);
            if constexpr (FIRST) {
                diff |= x ^ x0;
                bad |= x > src[min(i + 1, a.n - 1)];
            }
        }
    }
    if constexpr (FIRST) {
        diff = wave_or(diff);
        bad = wave_or(bad);
        if ((t & 63) == 0) {
            red[0][t / 64] = diff;
            red[1][t / 64] = bad;
        }
    }
    __syncthreads();
    if constexpr (!SCANNED) {
        static_assert(TPB == 1 && TILE <= 0xFFFF, "16-bit counts of one tile");
        if (t < kDigits / 2)
            a.counts[(size_t)tile * (kDigits / 2) + t] = h[2 * t] | (h[2 * t + 1] << 16);
    } else if (t < kDigits) {
        uint32_t *row = a.counts + (size_t)t * a.stride + group * TPB;
        if constexpr (TPB == 4) {
            *reinterpret_cast<uint4 *>(row) =
                make_uint4(hist[0][t], hist[1][t], hist[2][t], hist[3][t]);
        } else {
#pragma unroll
            for (int q = 0; q < TPB; ++q) row[q] = hist[q][t];
        }
    }
    if constexpr (FIRST) {
        if (t < 2) {
            uint32_t r = 0;
#pragma unroll
            for (int w = 0; w < 4 * TPB; ++w) r |= red[t][w];
            a.part[t * a.parts + blockIdx.x] = r;
        }
    }
}

// One workgroup per digit: the exclusive prefix of its counts over the tiles,
// in place, and their total. In pass 0 the first workgroup also decides which
// passes of the word run.
template <int NT>
__global__ __launch_bounds__(NT) void radix_scan_kernel(RadixArgs a) {
    constexpr uint32_t W = NT / 64, E = 16;  // counts per lane and round
    __shared__ uint32_t sums[2][W];
    const uint32_t t = threadIdx.x, lane = t & 63, w = t / 64;
    if (a.pass != 0 && ((uniform(*a.ctl) >> a.pass) & 1u) == 0) return;
    uint32_t *row = a.counts + (size_t)blockIdx.x * a.stride;
    uint32_t before = 0;
    for (uint32_t b = 0, k = 0; b < a.tiles; b += NT * E, ++k) {
        const uint32_t i = b + t * E;
        uint32_t c[E];
        uint32_t sum = 0;
        if (i < a.tiles) {  // rows are padded to whole groups of E
#pragma unroll
            for (uint32_t q = 0; q < E; q += 4) {
                const uint4 x = *reinterpret_cast<const uint4 *>(row + i + q);
                c[q] = x.x;
                c[q + 1] = x.y;
                c[q + 2] = x.z;
                c[q + 3] = x.w;
            }
#pragma unroll
            for (uint32_t q = 0; q < E; ++q)
                if (i + q < a.tiles) sum += c[q];
        }
        uint32_t at = wave_exclusive_scan(sum, lane);
        uint32_t all = 0;
        if constexpr (W > 1) {
            if (lane == 63) sums[k & 1][w] = at + sum;
            __syncthreads();
#pragma unroll
            for (uint32_t q = 0; q < W; ++q) {
                if (q < w) at += sums[k & 1][q];
                all += sums[k & 1][q];
            }
        } else {
            all = (uint32_t)__shfl((int)(at + sum), 63);
        }
        if (i < a.tiles) {
            at += before;
#pragma unroll
            for (uint32_t q = 0; q < E; q += 4) {
                uint4 x;
                x.x = at;
                x.y = x.x + c[q];
                x.z = x.y + c[q + 1];
                x.w = x.z + c[q + 2];
                at = x.w + c[q + 3];
                *reinterpret_cast<uint4 *>(row + i + q) = x;
            }
        }
        before += all;
    }
    if (t == 0) a.totals[blockIdx.x] = before;
    if (a.pass == 0 && blockIdx.x == 0) {
        uint32_t diff = 0, bad = 0;
        for (uint32_t b = t; b < a.parts; b += NT) {
            diff |= a.part[b];
            bad |= a.part[a.parts + b];
        }
        diff = wave_or(diff);
        bad = wave_or(bad);
        if constexpr (W > 1) {
            __syncthreads();
            if (lane == 0) {
                sums[0][w] = diff;
                sums[1][w] = bad;
            }
            __syncthreads();
            for (uint32_t q = 0; q < W; ++q) {
                diff |= sums[0][q];
                bad |= sums[1][q];
            }
        }
        if (t == 0) *a.ctl = passes_to_run(diff, bad == 0);
    }
}

// Lanes of the wave whose digit equals this lane's.
__device__ __forceinline__ uint64_t same_digit(uint32_t d) {
    uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
        const uint32_t s = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // ones where bit b is set
        const uint64_t m = __ballot(s != 0);
        lo &= ~((uint32_t)m ^ s);
        hi &= ~((uint32_t)(m >> 32) ^ s);
    }
    return ((uint64_t)hi << 32) | lo;
}

template <int NT, int ITEMS>
constexpr size_t radix_lds_bytes() {
    return (size_t)NT * ITEMS * 4 + (NT / 64) * kDigits * 2 + kDigits * 4;
}

// Sums of the digits' counts over all tiles, to s[0 .. 256), and over the tiles
// before tile_id, to s[NT / 64 * 256 ..): half a wave reads a tile's 512 bytes, 16
// per lane (eight digits), every half wave tiles of its own, eight of them at a
// time. A launch for the scan costs as much at 256 tiles (2^17 keys, 64 tiles: 41 us
// a sort with the scan, 37 so; 2^18 pairs with their index, 128 tiles: 68 and 61;
// 2^19 keys, 256 tiles: 46 and 52).
template <int NT>
__device__ __forceinline__ void radix_add_counts(const RadixArgs &a, uint32_t tile_id,
                                                 uint32_t *s) {
    constexpr uint32_t W = NT / 64, G = NT / 32;
    constexpr int U = 8;  // rows in flight
    const uint32_t t = threadIdx.x, l = t & 31, w = t / 64;
    const uint4 *rows = reinterpret_cast<const uint4 *>(a.counts) + l;
    uint32_t tot[8] = {}, own[8] = {};
    for (uint32_t b0 = t / 32; b0 < a.tiles; b0 += U * G) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t b = b0 + u * G;
            v[u] = make_uint4(0, 0, 0, 0);
            if (b < a.tiles) v[u] = rows[b * 32];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t before = b0 + u * G < tile_id ? ~0u : 0u;
            const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                tot[2 * q] += x[q] & 0xFFFF;
                tot[2 * q + 1] += x[q] >> 16;
                const uint32_t y = x[q] & before;
                own[2 * q] += y & 0xFFFF;
                own[2 * q + 1] += y >> 16;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        tot[q] += (uint32_t)__shfl_xor((int)tot[q], 32);
        own[q] += (uint32_t)__shfl_xor((int)own[q], 32);
    }
    // The wave's lower half stores the totals, the upper one the prefixes.
    const bool upper = (t & 32) != 0;
    uint4 *to = reinterpret_cast<uint4 *>(s + (upper ? W * kDigits : 0) + w * kDigits + 8 * l);
    to[0] = upper ? make_uint4(own[0], own[1], own[2], own[3])
                  : make_uint4(tot[0], tot[1], tot[2], tot[3]);
    to[1] = upper ? make_uint4(own[4], own[5], own[6], own[7])
                  : make_uint4(tot[4], tot[5], tot[6], tot[7]);
    __syncthreads();
    for (uint32_t i = t; i < 2 * kDigits; i += NT) {
        uint32_t *c = s + (i < kDigits ? i : W * kDigits + i - kDigits);
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < W; ++q) sum += c[q * kDigits];
        c[0] = sum;
    }
    __syncthreads();
}

// One tile of NT * ITEMS elements per workgroup: ranks within each wave by
// ballots (the lanes with an equal digit), prefixes over waves and digits, the
// tile brought into digit order in LDS, runs of equal digits written out. Pairs
// move the payload through the same LDS afterwards, along the same positions.
//
// 2^28 pairs take 880 us a pass (4.9 TB/s of the 16 bytes a pair), 2^28 keys
// 480-560 us, there with VALU issue busy for 430 us (63 instructions per 64
// keys). What bounds the pairs are the runs' ends: a run starts and ends inside
// a cache line that the neighbouring tile's run completes, and a line that
// leaves its L2 half written costs memory twice. So tiles go to the XCDs in
// contiguous ranges (neighbours finish their lines in one L2 at about the same
// time): 1940 -> 880 us for pairs, 840 -> 520 us for keys. One workgroup that
// walks through consecutive tiles, whose half lines are evicted between two of
// its tiles, ran 1530 us, and tiles written without the scatter 770 us. 8192
// elements a tile: the counts per tile stay few and the tile's output and its
// neighbours' stay in the L2. SCANNED: the counts hold
// their prefix over the tiles; otherwise (few tiles) every workgroup adds
// them up itself (radix_add_counts), and in pass 0 decides which passes run.
template <bool PAIRS, int NT, int ITEMS, bool NTL, bool SCANNED>
__global__ __launch_bounds__(NT) void radix_scatter_kernel(RadixArgs a) {
    constexpr uint32_t W = NT / 64;
    constexpr uint32_t TILE = NT * ITEMS;
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *exch = reinterpret_cast<uint32_t *>(smem);
    uint32_t *wc32 = exch + TILE;  // [wave][digit]: 16-bit counts, two a word
    uint32_t *goff = wc32 + W * kDigits / 2;
    const uint32_t t = threadIdx.x, lane = t & 63, w = t / 64;
    Count16 *wc = reinterpret_cast<Count16 *>(wc32) + w * kDigits;

    uint32_t run;
    if (!SCANNED && a.pass == 0) {
        uint32_t diff = 0, bad = 0;
        for (uint32_t b = lane; b < a.parts; b += 64) {
            diff |= a.part[b];
            bad |= a.part[a.parts + b];
        }
        run = passes_to_run(wave_or(diff), wave_or(bad) == 0);
        if (blockIdx.x == 0 && t == 0) *a.ctl = run;
    } else {
        run = *a.ctl;
    }
    run = uniform(run);
    if (((run >> a.pass) & 1u) == 0) return;
    const uint32_t from = source_of(run, a.pass);
    const uint32_t shift = a.pass * kRadixBits;
    const uint32_t tile_id = xcd_contiguous_block(blockIdx.x, a.tiles);
    const uint64_t base = (uint64_t)tile_id * TILE;
    const uint32_t *win = a.word[from] + base;
    uint32_t *wout = a.word[from ^ 1];
    const uint32_t *vin = PAIRS ? a.other[from] + base : nullptr;
    uint32_t *vout = PAIRS ? a.other[from ^ 1] : nullptr;

    // The tile, as FULL or as its first `left` elements.
    auto sort_tile = [&](uint32_t left, auto full) {
        constexpr bool FULL = decltype(full)::value;
        const uint32_t first = w * (64 * ITEMS) + lane;
        uint32_t k[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t p = first + i * 64;
            // Past the end: the largest digit, after every element that has it.
            k[i] = FULL || p < left ? load4<NTL>(win + p) : 0xFFFFFFFFu;
        }
        // Output position of digits 4 lane .. 4 lane + 3 (wave 0).
        uint32_t pre[4] = {0, 0, 0, 0};
        if constexpr (SCANNED) {
            if (w == 0) {
                const uint4 tot = reinterpret_cast<const uint4 *>(a.totals)[lane];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    pre[q] = a.counts[(size_t)(4 * lane + q) * a.stride + tile_id];
                const uint32_t at = wave_exclusive_scan(tot.x + tot.y + tot.z + tot.w, lane);
                pre[0] += at;
                pre[1] += at + tot.x;
                pre[2] += at + tot.x + tot.y;
                pre[3] += at + tot.x + tot.y + tot.z;
            }
        } else {
            radix_add_counts<NT>(a, tile_id, exch);
            if (w == 0) {
                const uint4 tot = reinterpret_cast<const uint4 *>(exch)[lane];
                const uint4 own = reinterpret_cast<const uint4 *>(exch + W * kDigits)[lane];
                const uint32_t at = wave_exclusive_scan(tot.x + tot.y + tot.z + tot.w, lane);
                pre[0] = at + own.x;
                pre[1] = at + tot.x + own.y;
                pre[2] = at + tot.x + tot.y + own.z;
                pre[3] = at + tot.x + tot.y + tot.z + own.w;
            }
        }
        // This wave's digit counts; only the wave itself uses them until the barrier.
#pragma unroll
        for (uint32_t i = 0; i < kDigits / 2; i += 64) wc32[w * (kDigits / 2) + i + lane] = 0;
        __builtin_amdgcn_wave_barrier();
        uint32_t pos[ITEMS];
        uint32_t d = digit_of(k[0], shift);
        uint64_t peers = same_digit(d);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            // The next row's peers are found while this row's counts arrive.
            const uint32_t old = wc[d];
            uint32_t dn = 0;
            uint64_t pn = 0;
            if (i + 1 < ITEMS) {
                dn = digit_of(k[i + 1], shift);
                asm volatile("" : "+v"(dn));
                pn = same_digit(dn);
            }
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0));
            __builtin_amdgcn_wave_barrier();
            wc[d] = (Count16)(old + __popcll(peers));  // the same value from every peer
            __builtin_amdgcn_wave_barrier();
            pos[i] = old + below;
            asm volatile("" : "+v"(pos[i]));
            d = dn;
            peers = pn;
        }
        __syncthreads();
        if (w == 0) {
            // Per digit the exclusive prefix over the waves (two digits a word:
            // a tile's counts fit 16 bits), then over the digits.
            uint2 *c = reinterpret_cast<uint2 *>(wc32) + lane;
            uint32_t s0 = 0, s1 = 0;
#pragma unroll 4
            for (uint32_t q = 0; q < W; ++q) {
                const uint2 x = c[q * (kDigits / 4)];
                s0 += x.x;
                s1 += x.y;
            }
            const uint32_t c0 = s0 & 0xFFFF, c1 = s0 >> 16, c2 = s1 & 0xFFFF, c3 = s1 >> 16;
            const uint32_t e0 = wave_exclusive_scan(c0 + c1 + c2 + c3, lane);
            const uint32_t e1 = e0 + c0, e2 = e1 + c1, e3 = e2 + c2;
            s0 = e0 | (e1 << 16);
            s1 = e2 | (e3 << 16);
#pragma unroll 4
            for (uint32_t q = 0; q < W; ++q) {
                const uint2 x = c[q * (kDigits / 4)];
                c[q * (kDigits / 4)] = make_uint2(s0, s1);
                s0 += x.x;
                s1 += x.y;
            }
            reinterpret_cast<uint4 *>(goff)[lane] =
                make_uint4(pre[0] - e0, pre[1] - e1, pre[2] - e2, pre[3] - e3);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            asm volatile("" : "+v"(k[i]));  // the digit again, not kept since the ranking
            pos[i] = (pos[i] + wc[digit_of(k[i], shift)]) * 4;  // byte offset in exch
            asm volatile("" : "+v"(pos[i]));
            *reinterpret_cast<uint32_t *>(smem + pos[i]) = k[i];
        }
        uint32_t v[ITEMS];
        if constexpr (PAIRS) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const uint32_t p = first + i * 64;
                v[i] = FULL || p < left ? load4<NTL>(vin + p) : 0;
            }
        }
        __syncthreads();
        uint32_t dst[ITEMS];
        constexpr int B = 4;  // values in flight from LDS
#pragma unroll
        for (int i = 0; i < ITEMS; i += B) {
            uint32_t x[B];
#pragma unroll
            for (int j = 0; j < B; ++j) x[j] = exch[t + (i + j) * NT];
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const uint32_t p = t + (i + j) * NT;
                dst[i + j] = goff[digit_of(x[j], shift)] + p;
                if (FULL || p < left) wout[dst[i + j]] = x[j];
            }
            asm volatile("" ::: "memory");
        }
        if constexpr (PAIRS) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) *reinterpret_cast<uint32_t *>(smem + pos[i]) = v[i];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; i += B) {
                uint32_t x[B];
#pragma unroll
                for (int j = 0; j < B; ++j) x[j] = exch[t + (i + j) * NT];
#pragma unroll
                for (int j = 0; j < B; ++j)
                    if (FULL || t + (i + j) * NT < left) vout[dst[i + j]] = x[j];
                asm volatile("" ::: "memory");
            }
        }
    };
    if (base + TILE <= a.n)
        sort_tile(TILE, std::true_type{});
    else
        sort_tile((uint32_t)(a.n - base), std::false_type{});
}

// Tiles by the number of elements: the smallest while larger ones would leave
// CUs without a tile (keys, 2^16: 38 us with 2048, 39 with 4096, 55 with 8192;
// pairs with random payloads, 2^19: 102, 108 and 146 us; 10^6: 129, 126 and 158
// us), the largest, whose runs of a digit are as long as a cache line, once the
// arrays outgrow the caches (pairs, 10^7: 222 us with 4096, 237 with 8192;
// 2^24: 323 and 298 us; 2^28: 7.1 and 5.1 ms). Loads carry the nontemporal hint
// with the largest only: 10^7 pairs lose 3 % by it.
enum class RadixTile { kSmall, kMid, kLarge };
constexpr uint32_t kSmallTile = 2048, kMidTile = 4096, kLargeTile = 8192;
constexpr uint32_t kSmallMax = 1u << 19, kMidMax = 12u << 20;
constexpr uint32_t kUnscannedTiles = 128;  // kSmall: up to so many tiles need no scan
static_assert(kUnscannedTiles * kSmallTile <= kSmallMax, "other tiles are always scanned");

struct RadixShape {
    RadixTile kind;
    uint32_t tile, tiles, stride, parts;
    bool scanned;
};

RadixShape radix_shape(uint32_t n) {
    RadixShape r;
    r.kind = n <= kSmallMax ? RadixTile::kSmall : n <= kMidMax ? RadixTile::kMid : RadixTile::kLarge;
    r.tile = r.kind == RadixTile::kSmall ? kSmallTile
             : r.kind == RadixTile::kMid ? kMidTile
                                         : kLargeTile;
    r.tiles = blocks_for(n, r.tile);
    r.stride = (r.tiles + 15) & ~15u;
    r.parts = r.kind == RadixTile::kLarge ? (r.tiles + 3) / 4 : r.tiles;
    r.scanned = r.tiles > kUnscannedTiles;
    return r;
}

// Scratch layout: pieces aligned to 256 bytes.
constexpr size_t padded_words(size_t words) { return (words + 63) & ~(size_t)63; }

size_t radix_table_words(const RadixShape &r) {
    return padded_words((size_t)kDigits * r.stride) + padded_words(kDigits) +
           padded_words(2 * (size_t)r.parts) + padded_words(1);
}

template <int TILE, int TPB, bool NTL, bool SCANNED>
void count(const RadixArgs &a, hipStream_t s) {
    if (a.pass == 0)
        hipLaunchKernelGGL((radix_count_kernel<TILE, TPB, NTL, true, SCANNED>), dim3(a.parts),
                           dim3(256 * TPB), 0, s, a);
    else
        hipLaunchKernelGGL((radix_count_kernel<TILE, TPB, NTL, false, SCANNED>), dim3(a.parts),
                           dim3(256 * TPB), 0, s, a);
}

template <bool PAIRS, int NT, int ITEMS, bool NTL, bool SCANNED>
void scatter(const RadixArgs &a, hipStream_t s) {
    constexpr size_t lds = radix_lds_bytes<NT, ITEMS>();
    static_assert(lds <= 65536, "dynamic LDS beyond the default limit");
    hipLaunchKernelGGL((radix_scatter_kernel<PAIRS, NT, ITEMS, NTL, SCANNED>), dim3(a.tiles),
                       dim3(NT), lds, s, a);
}

template <bool PAIRS>
hipError_t radix_pass(const RadixShape &r, const RadixArgs &a, hipStream_t s) {
    if (!r.scanned) {
        count<kSmallTile, 1, false, false>(a, s);
        scatter<PAIRS, 256, 8, false, false>(a, s);
        return hipGetLastError();
    }
    switch (r.kind) {
        case RadixTile::kSmall: count<kSmallTile, 1, false, true>(a, s); break;
        case RadixTile::kMid: count<kMidTile, 1, false, true>(a, s); break;
        default: count<kLargeTile, 4, true, true>(a, s); break;
    }
    if (r.tiles <= 1024)
        hipLaunchKernelGGL(radix_scan_kernel<64>, dim3(kDigits), dim3(64), 0, s, a);
    else
        hipLaunchKernelGGL(radix_scan_kernel<1024>, dim3(kDigits), dim3(1024), 0, s, a);
    switch (r.kind) {
        case RadixTile::kSmall: scatter<PAIRS, 256, 8, false, true>(a, s); break;
        case RadixTile::kMid: scatter<PAIRS, 512, 8, false, true>(a, s); break;
        default:
            if constexpr (PAIRS)
                scatter<true, 1024, 8, true, true>(a, s);
            else
                scatter<false, 512, 16, true, true>(a, s);
            break;
    }
    return hipGetLastError();
}

}  // namespace

size_t radix_scratch_words(uint32_t n, bool pairs) {
    return (pairs ? 2 : 1) * padded_words(n) + radix_table_words(radix_shape(n));
}

hipError_t launch_radix_sort(uint32_t *keys, uint32_t *vals, uint32_t n, uint32_t *scratch,
                             hipStream_t s) {
    if (n <= 1) return hipSuccess;
    const RadixShape r = radix_shape(n);
    uint32_t *at = scratch;
    auto take = [&at](size_t words) {
        uint32_t *p = at;
        at += padded_words(words);
        return p;
    };
    uint32_t *tk = take(n), *tv = vals != nullptr ? take(n) : nullptr;
    RadixArgs a{};
    a.n = n;
    a.tiles = r.tiles;
    a.stride = r.stride;
    a.parts = r.parts;
    a.counts = take((size_t)kDigits * r.stride);
    a.totals = take(kDigits);
    a.part = take(2 * (size_t)r.parts);
    a.ctl = take(1);
    for (int word = vals != nullptr ? 0 : 1; word < 2; ++word) {
        a.word[0] = word ? keys : vals;
        a.word[1] = word ? tk : tv;
        a.other[0] = word ? vals : keys;
        a.other[1] = word ? tv : tk;
        for (a.pass = 0; a.pass < (uint32_t)kGroupPasses; ++a.pass) {
            const hipError_t e =
                vals != nullptr ? radix_pass<true>(r, a, s) : radix_pass<false>(r, a, s);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace meld
