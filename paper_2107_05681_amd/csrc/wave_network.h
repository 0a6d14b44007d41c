// Bitonic network of u32 keys, or u64 (key, payload) composites, held 32, 16 or 8 per
// lane, every comparator ascending.
//
// With 32 per lane a wave holds 2^11 keys: element bits 0 .. 4 are the register index, bits
// 5 .. 10 the lane; above that, bits 11 .. 13 are the wave of a workgroup that
// sorts up to 2^14 keys. MELD_AUTO uses it where only the sorted order counts,
// so there is one form, and two things that the paper's forms cannot do:
//   * no direction anywhere: before phase 2^m the keys of the blocks that
//     Figure 1 sorts in descending order are complemented, so that every
//     comparator of the phase is a minimum and a maximum (two operations for two
//     keys, where a direction per lane takes four); going from one phase to the
//     next is one exclusive or per key.
//   * the lane bits never go through LDS. Bits 5 .. 8 are the four DPP
//     exchanges with lane ^ 1, ^ 2, ^ 7 and ^ 8 (7, a half-row mirror, instead of
//     4, which would take two moves), and the kept value is the median of the
//     two and of 0 or ~0: two operations a key. Bits 9 and 10 trade places with
//     a register bit (v_permlane16/32_swap, half an operation a key), are
//     compared there and trade back.
// Bits 11 and up move through LDS, 16 bytes per lane and access.
//
// Bound by VALU issue: 92 operations a key for 2^11 keys, 131 for 2^13.
#pragma once

#include "device_common.h"

namespace meld {

namespace {

constexpr int kWaveE = 32;               // keys per lane
constexpr uint32_t kWaveTile = 64 * kWaveE;

// Register bits of a lane that holds E keys (32, or 16 or 8 where a small array is
// spread over more lanes; the functions below take the number from the array, and
// their element bits count from it: B .. B + 5 are the lane).
template <int E>
constexpr int wave_bits() {
    return E == 32 ? 5 : E == 16 ? 4 : 3;
}

struct WaveLane {
    uint32_t id;      // the lane bits of the lane's elements (bits 5 .. 10 of 32 each)
    uint32_t keep[4];  // 0 where the lane is the lower end of lane bit i, else ~0
};

__device__ __forceinline__ WaveLane wave_lane() {
    const uint32_t lane = threadIdx.x & 63;
    WaveLane w;
    // lane ^ 7 flips id bit 2 alone: the physical bits 0 and 1 carry id bit 2 too.
    w.id = lane ^ ((lane & 4) ? 3u : 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) w.keep[i] = (uint32_t)-(int32_t)((w.id >> i) & 1u);
    return w;
}

// Median of x, y and z: the smaller of x and y for z = 0, the larger for ~0.
__device__ __forceinline__ uint32_t median(uint32_t x, uint32_t y, uint32_t z) {
    const uint32_t mn = x < y ? x : y, mx = x < y ? y : x;
    const uint32_t t = mx < z ? mx : z;
    return mn > t ? mn : t;
}

// Register steps on bit Q. T: u32 keys, or u64 (key, payload) composites.
template <int Q, typename T, int E>
__device__ __forceinline__ void wave_reg_step(T (&e)[E]) {
#pragma unroll
    for (int r = 0; r < E; ++r)
        if ((r & (1 << Q)) == 0) {
            const T x = e[r], y = e[r | (1 << Q)];
            e[r] = x < y ? x : y;
            e[r | (1 << Q)] = x < y ? y : x;
        }
}

// Steps on register bits TOP .. 0.
template <int TOP, typename T, int E>
__device__ __forceinline__ void wave_reg_steps(T (&e)[E]) {
    if constexpr (TOP >= 0) {
        wave_reg_step<TOP>(e);
        wave_reg_steps<TOP - 1>(e);
    }
}

// Phases 2^1 .. 2^(B-1), B register bits: bit M of the register index is the
// direction.
template <int M, int Q, typename T, int E>
__device__ __forceinline__ void wave_first_phases(T (&e)[E]) {
    if constexpr (M < wave_bits<E>()) {
#pragma unroll
        for (int r = 0; r < E; ++r)
            if ((r & (1 << Q)) == 0) {
                const T x = e[r], y = e[r | (1 << Q)];
                const T mn = x < y ? x : y, mx = x < y ? y : x;
                e[r] = (r >> M) & 1 ? mx : mn;
                e[r | (1 << Q)] = (r >> M) & 1 ? mn : mx;
            }
        if constexpr (Q > 0)
            wave_first_phases<M, Q - 1>(e);
        else
            wave_first_phases<M + 1, M>(e);
    }
}

// The step on lane bit B, B <= 3.
template <int B, int E>
__device__ __forceinline__ void wave_lane_step(uint32_t (&e)[E], uint32_t keep) {
    constexpr int ctrl = B == 0 ? 0xB1 : B == 1 ? 0x4E : B == 2 ? 0x141 : 0x128;
#pragma unroll
    for (int r = 0; r < E; ++r)
        e[r] = median(e[r], (uint32_t)__builtin_amdgcn_mov_dpp((int)e[r], ctrl, 0xF, 0xF, true),
                      keep);
}

template <int B, int E>
__device__ __forceinline__ void wave_lane_step(uint64_t (&e)[E], uint32_t keep) {
    constexpr int ctrl = B == 0 ? 0xB1 : B == 1 ? 0x4E : B == 2 ? 0x141 : 0x128;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)e[r], ctrl, 0xF, 0xF, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(e[r] >> 32), ctrl, 0xF, 0xF, true);
        const uint64_t y = (uint64_t)hi << 32 | lo;
        e[r] = (y < e[r]) != (keep != 0) ? y : e[r];
    }
}

// Trades lane bit 4 (SWAP32: 5) for the top register bit.
template <bool SWAP32, int E>
__device__ __forceinline__ void wave_trade(uint32_t (&e)[E]) {
#pragma unroll
    for (int r = 0; r < E / 2; ++r) {
        if constexpr (SWAP32) {
            const auto p = __builtin_amdgcn_permlane32_swap(e[r], e[r + E / 2], false, false);
            e[r] = p[0];
            e[r + E / 2] = p[1];
        } else {
            const auto p = __builtin_amdgcn_permlane16_swap(e[r], e[r + E / 2], false, false);
            e[r] = p[0];
            e[r + E / 2] = p[1];
        }
    }
}

template <bool SWAP32, int E>
__device__ __forceinline__ void wave_trade(uint64_t (&e)[E]) {
    uint32_t lo[E], hi[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        lo[r] = (uint32_t)e[r];
        hi[r] = (uint32_t)(e[r] >> 32);
    }
    wave_trade<SWAP32>(lo);
    wave_trade<SWAP32>(hi);
#pragma unroll
    for (int r = 0; r < E; ++r) e[r] = (uint64_t)hi[r] << 32 | lo[r];
}

// Steps on element bits TOP .. 0 of a wave, B register bits. TOP = B + 5 takes
// three trades for its two upper bits instead of four and leaves bits B + 4 and
// B + 5 in each other's place: bit B + 4 is lane bit 5 then, bit B + 5 lane bit 4.
template <int TOP, typename T, int E>
__device__ __forceinline__ void wave_steps(T (&e)[E], const WaveLane &w) {
    constexpr int B = wave_bits<E>();
    static_assert(TOP <= B + 5, "above the wave");
    if constexpr (TOP == B + 5) {
        wave_trade<true>(e);
        wave_reg_step<B - 1>(e);
        wave_trade<false>(e);
        wave_reg_step<B - 1>(e);
        wave_trade<true>(e);
        wave_steps<B + 3>(e, w);
    } else if constexpr (TOP == B + 4) {
        wave_trade<false>(e);
        wave_reg_step<B - 1>(e);
        wave_trade<false>(e);
        wave_steps<B + 3>(e, w);
    } else if constexpr (TOP >= B) {
        wave_lane_step<TOP - B>(e, w.keep[TOP - B]);
        wave_steps<TOP - 1>(e, w);
    } else {
        wave_reg_steps<TOP>(e);
    }
}

// mask: 0 or ~0.
template <typename T, int E>
__device__ __forceinline__ void wave_flip(T (&e)[E], uint32_t mask) {
#pragma unroll
    for (int r = 0; r < E; ++r) e[r] ^= (T)(int32_t)mask;
}

// The complement of phase 2^M of a sort whose last phase is 2^LAST: all ones
// where bit M of the elements is set, nothing in the last phase. high: bits B
// and up of the lane's elements.
template <int M, int LAST, int B = 5>
__device__ __forceinline__ uint32_t wave_down(uint32_t high) {
    return M < LAST ? (uint32_t)-(int32_t)((high >> (M - B)) & 1u) : 0u;
}

// Phases 2^M .. 2^min(LAST, B + 6) on keys already complemented for phase 2^M.
template <int M, int LAST, typename T, int E>
__device__ __forceinline__ void wave_phases(T (&e)[E], const WaveLane &w, uint32_t high) {
    constexpr int B = wave_bits<E>();
    wave_steps<M - 1>(e, w);
    if constexpr (M < LAST && M < B + 6) {
        wave_flip(e, wave_down<M, LAST, B>(high) ^ wave_down<M + 1, LAST, B>(high));
        wave_phases<M + 1, LAST>(e, w, high);
    }
}

// Position of a tile's element in LDS: four words of padding per 32, so that
// the 16-byte accesses of both layouts are free of bank conflicts. For b a
// multiple of 32, wave_phys(a + b) = wave_phys(a) + wave_phys(b).
__device__ __forceinline__ constexpr uint32_t wave_phys(uint32_t i) { return i + (i >> 5) * 4; }
constexpr uint32_t wave_lds_words(uint32_t tile) { return tile / 32 * 36; }

// The lane's row of 32 elements in LDS, with bits 9 and 10 in each other's
// place (P) or not.
template <bool P>
__device__ __forceinline__ uint32_t *wave_row(uint32_t *s, const WaveLane &w) {
    const uint32_t id = P ? (w.id & 15u) | ((w.id & 16u) << 1) | ((w.id & 32u) >> 1) : w.id;
    return s + id * 36;
}

template <bool P>
__device__ __forceinline__ void wave_to_lds(const uint32_t (&e)[kWaveE], uint32_t *s,
                                            const WaveLane &w) {
    uint4 *row = reinterpret_cast<uint4 *>(wave_row<P>(s, w));
#pragma unroll
    for (int c = 0; c < kWaveE / 4; ++c)
        row[c] = make_uint4(e[4 * c], e[4 * c + 1], e[4 * c + 2], e[4 * c + 3]);
}

template <bool P>
__device__ __forceinline__ void wave_from_lds(uint32_t (&e)[kWaveE], uint32_t *s,
                                              const WaveLane &w) {
    const uint4 *row = reinterpret_cast<const uint4 *>(wave_row<P>(s, w));
#pragma unroll
    for (int c = 0; c < kWaveE / 4; ++c) {
        const uint4 v = row[c];
        e[4 * c] = v.x;
        e[4 * c + 1] = v.y;
        e[4 * c + 2] = v.z;
        e[4 * c + 3] = v.w;
    }
}

// Steps on element bits TOP .. 11 (TOP <= 13) of a tile of 2^LOG elements
// whose waves hold 2^11 each: every lane takes 2^(LOG-11) pieces of
// neighbouring elements, one of each wave's. Bits 9 and 10 are in each other's
// place on entry, and not on return. s: the workgroup's tile.
template <int LOG, int TOP>
__device__ __forceinline__ void wave_cross_steps(uint32_t (&e)[kWaveE], uint32_t *s,
                                                 const WaveLane &w) {
    constexpr int WB = LOG - 11;  // wave bits
    constexpr int GB = 5 - WB;    // low element bits that stay registers
    const uint32_t wave = threadIdx.x / 64;
    uint32_t *own = s + wave * wave_lds_words(kWaveTile);
    wave_to_lds<true>(e, own, w);
    __syncthreads();
    // Piece of 2^GB elements number threadIdx.x of every wave's 2^11.
    uint32_t *p = s + wave_phys((uint32_t)threadIdx.x << GB);
#pragma unroll
    for (int r = 0; r < kWaveE; r += 4) {
        const uint4 v = *reinterpret_cast<const uint4 *>(
            p + (r >> GB) * wave_lds_words(kWaveTile) + (r & ((1 << GB) - 1)));
        e[r] = v.x;
        e[r + 1] = v.y;
        e[r + 2] = v.z;
        e[r + 3] = v.w;
    }
    if constexpr (TOP >= 13) wave_reg_step<GB + 2>(e);
    if constexpr (TOP >= 12) wave_reg_step<GB + 1>(e);
    wave_reg_step<GB>(e);
#pragma unroll
    for (int r = 0; r < kWaveE; r += 4)
        *reinterpret_cast<uint4 *>(p + (r >> GB) * wave_lds_words(kWaveTile) +
                                   (r & ((1 << GB) - 1))) =
            make_uint4(e[r], e[r + 1], e[r + 2], e[r + 3]);
    __syncthreads();
    wave_from_lds<false>(e, own, w);
}

// Phases 2^M .. 2^LOG (M >= 12) on keys complemented for phase 2^(M-1).
template <int M, int LOG>
__device__ __forceinline__ void wave_cross_phases(uint32_t (&e)[kWaveE], uint32_t *s,
                                                  const WaveLane &w, uint32_t high) {
    if constexpr (M <= LOG) {
        wave_flip(e, wave_down<M - 1, LOG>(high) ^ wave_down<M, LOG>(high));
        wave_cross_steps<LOG, M - 1>(e, s, w);
        wave_steps<10>(e, w);
        wave_cross_phases<M + 1, LOG>(e, s, w, high);
    }
}

// Sorts every 2^LOG keys (6 <= LOG <= 14) of the wave, or of the workgroup of
// 2^(LOG-11) waves, from any order into rows of 32 per lane; bits 9 and 10 are
// in each other's place for LOG >= 11. s: 2^LOG elements of LDS for LOG >= 12.
template <int LOG>
__device__ __forceinline__ void wave_sort(uint32_t (&e)[kWaveE], uint32_t *s, const WaveLane &w) {
    const uint32_t high = w.id | (LOG > 11 ? threadIdx.x / 64 << 6 : 0u);
    wave_first_phases<1, 0>(e);
    wave_flip(e, wave_down<5, LOG>(high));
    wave_phases<5, LOG>(e, w, high);
    wave_cross_phases<12, LOG>(e, s, w, high);
}

// The same with E = 8 or 16 keys per lane, which gives each SIMD more waves to
// hide the chain of steps behind.
template <int E, int LOG>
constexpr int wave_group_threads() {
    return LOG > wave_bits<E>() + 6 ? (1 << LOG) / E : 64;
}

// The lane's first element in the workgroup. traded: the two upper lane bits are in
// each other's place.
template <int E>
__device__ __forceinline__ uint32_t wave_group_row(const WaveLane &w, bool traded) {
    const uint32_t id = traded ? (w.id & 15u) | ((w.id & 16u) << 1) | ((w.id & 32u) >> 1) : w.id;
    return ((threadIdx.x & ~63u) | id) * E;
}

// Sixteen bytes at a time between e[0 .. E) and memory aligned to them.
template <typename T, int E>
__device__ __forceinline__ void wave_store_row(T *to, const T (&e)[E]) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int c = 0; c < E; c += 2)
            *reinterpret_cast<ulonglong2 *>(to + c) = make_ulonglong2(e[c], e[c + 1]);
    } else {
#pragma unroll
        for (int c = 0; c < E; c += 4)
            *reinterpret_cast<uint4 *>(to + c) = make_uint4(e[c], e[c + 1], e[c + 2], e[c + 3]);
    }
}
template <typename T, int E>
__device__ __forceinline__ void wave_load_row(T (&e)[E], const T *from) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int c = 0; c < E; c += 2) {
            const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(from + c);
            e[c] = v.x;
            e[c + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int c = 0; c < E; c += 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(from + c);
            e[c] = v.x;
            e[c + 1] = v.y;
            e[c + 2] = v.z;
            e[c + 3] = v.w;
        }
    }
}

// Phases 2^M .. 2^LOG above a wave's on keys complemented for phase 2^(M-1): for the
// steps across waves every lane takes one piece of each wave's keys.
template <int M, int LOG, typename T, int E>
__device__ __forceinline__ void wave_group_cross(T (&e)[E], T *s, const WaveLane &w,
                                                 uint32_t high) {
    if constexpr (M <= LOG) {
        constexpr int B = wave_bits<E>(), TOP = B + 5;
        constexpr int WB = LOG - TOP - 1;  // wave bits
        constexpr int GB = B - WB;         // low element bits that stay registers
        static_assert(GB >= 0, "one exchange per phase");
        wave_flip(e, wave_down<M - 1, LOG, B>(high) ^ wave_down<M, LOG, B>(high));
        wave_store_row(s + wave_phys(wave_group_row<E>(w, true)), e);
        __syncthreads();
        T *p = s + wave_phys((uint32_t)threadIdx.x << GB);
        auto at = [&](int r) -> T & {
            return p[wave_phys((uint32_t)(r >> GB) << (TOP + 1)) + (r & ((1 << GB) - 1))];
        };
#pragma unroll
        for (int r = 0; r < E; ++r) e[r] = at(r);
        if constexpr (M - TOP >= 5) wave_reg_step<GB + 3>(e);
        if constexpr (M - TOP >= 4) wave_reg_step<GB + 2>(e);
        if constexpr (M - TOP >= 3) wave_reg_step<GB + 1>(e);
        wave_reg_step<GB>(e);
#pragma unroll
        for (int r = 0; r < E; ++r) at(r) = e[r];
        __syncthreads();
        wave_load_row(e, s + wave_phys(wave_group_row<E>(w, false)));
        // The next phase's writes go to the lane's own wave's keys, which only that
        // wave reads until the next barrier.
        wave_steps<TOP>(e, w);
        wave_group_cross<M + 1, LOG>(e, s, w, high);
    }
}

// Sorts 2^LOG keys of a workgroup from any order into rows of E per lane
// (wave_group_row; traded for whole waves). s: 2^LOG elements of LDS
// (wave_lds_words) where there is more than one wave.
template <int LOG, typename T, int E>
__device__ __forceinline__ void wave_group_sort(T (&e)[E], T *s, const WaveLane &w) {
    constexpr int B = wave_bits<E>();
    const uint32_t high = (threadIdx.x & ~63u) | w.id;
    wave_first_phases<1, 0>(e);
    wave_flip(e, wave_down<B, LOG, B>(high));
    wave_phases<B, LOG>(e, w, high);
    wave_group_cross<B + 7, LOG>(e, s, w, high);
}

}  // namespace

}  // namespace meld
