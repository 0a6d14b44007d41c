// Merge tails of the keys-only sort: steps j = T/2 .. 1 of a phase k > T on every
// tile of T = 2^L keys (L in 11..14), 32 keys per lane. The direction is the same
// for a whole tile, so the divergent and the melded form coincide: a descending
// tile's keys are complemented, and every comparator is a minimum and a maximum.
//
// Lanes hold elements r * T/32 + thread, so that loads are lane-linear and the top
// five steps register steps; through LDS once (not for T = 2^11) the wave takes
// 2^11 neighbouring keys as r * 64 + lane: the steps down to bit 6 are register
// steps again, bits 5 and 4 trade places with a register bit, bits 3 to 0 are DPP
// medians (wave_network.h), and the keys are stored lane-linear as they stand. With
// 16 keys per lane a tile of 2^14 moves through LDS four times (bitonic.hip): 10^7
// keys, one tail: 23.4 us, 16.5 us so, 17.7 over the first calls (a copy of the 40 MB takes 12.9 us).
#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kPadKey = 0xFFFFFFFFu;

template <int L>
struct MergeWave {
    static constexpr int kThreads = L == 11 ? 256 : 1 << (L - 5);
    static constexpr int kTiles = L == 11 ? 4 : 1;  // per workgroup
};

template <bool NT>
__device__ __forceinline__ uint32_t load_key(const uint32_t *p) {
    return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT>
__device__ __forceinline__ void store_key(uint32_t *p, uint32_t v) {
    if (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

template <int L, bool NT>
__global__ __launch_bounds__(MergeWave<L>::kThreads) void merge_wave_kernel(
    uint32_t *__restrict__ keys, uint32_t n, uint32_t dir, uint32_t m, uint32_t end) {
    extern __shared__ __align__(16) uint32_t s[];
    constexpr uint32_t T = 1u << L, STEP = T / kWaveE;
    const WaveLane w = wave_lane();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const uint32_t b = xcd_run_index<kXcdRunLogMerge>(blockIdx.x, gridDim.x);
    const uint32_t tile = (L == 11 ? b * 4 + wave : b) << L;
    if (tile >= end) return;  // L = 11: a wave, which meets no barrier
    const uint32_t flip = (uint32_t)-(int32_t)(((tile ^ dir) >> m) & 1u);
    const bool whole = tile + T <= n;
    uint32_t e[kWaveE];
    const uint32_t at = L == 11 ? w.id : threadIdx.x;
    if (whole) {
        const uint32_t *k = keys + tile;
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) e[r] = load_key<NT>(k + r * STEP + at);
    } else {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) {
            const uint32_t p = tile + r * STEP + at;
            e[r] = p < n ? keys[p] : kPadKey;
        }
    }
    if (flip != 0) wave_flip(e, ~0u);  // a whole tile: the last one ascends
    wave_reg_steps<4>(e);
    uint32_t first = tile;
    if constexpr (L > 11) {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) s[r * STEP + at] = e[r];
        __syncthreads();
        const uint32_t *own = s + wave * kWaveTile + w.id;
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) e[r] = own[r * 64];
        wave_reg_steps<L - 12>(e);
        first += wave * kWaveTile;
    }
    wave_trade<true>(e);
    wave_reg_step<4>(e);
    wave_trade<false>(e);
    wave_reg_step<4>(e);
    wave_trade<true>(e);
    wave_lane_step<3>(e, w.keep[3]);
    wave_lane_step<2>(e, w.keep[2]);
    wave_lane_step<1>(e, w.keep[1]);
    wave_lane_step<0>(e, w.keep[0]);
    if (flip != 0) wave_flip(e, ~0u);
    // Bits 5 and 4 of the lane are in each other's place.
    const uint32_t id = (w.id & 15u) | ((w.id & 16u) << 1) | ((w.id & 32u) >> 1);
    if (whole) {
        uint32_t *k = keys + first;
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) store_key<NT>(k + r * 64 + id, e[r]);
    } else {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r)
            if (first + r * 64 + id < n) keys[first + r * 64 + id] = e[r];
    }
}

template <int L, bool NT>
hipError_t launch(const SortArray &a, uint32_t m, hipStream_t stream) {
    const uint32_t end = active_end(a.n, m);
    constexpr size_t lds = L == 11 ? 0 : (size_t)sizeof(uint32_t) << L;
    static_assert(lds <= 65536, "within the default limit of dynamic LDS");
    hipLaunchKernelGGL((merge_wave_kernel<L, NT>), dim3(blocks_for(end, MergeWave<L>::kTiles << L)),
                       dim3(MergeWave<L>::kThreads), lds, stream, a.keys, a.n, a.dir, m, end);
    return hipGetLastError();
}

template <int L>
hipError_t launch(const SortArray &a, uint32_t m, hipStream_t stream) {
    return a.nt != 0 ? launch<L, true>(a, m, stream) : launch<L, false>(a, m, stream);
}

}  // namespace

hipError_t launch_merge_wave(const SortArray &a, uint32_t log_t, uint32_t m, hipStream_t stream) {
    switch (log_t) {
        case 11: return launch<11>(a, m, stream);
        case 12: return launch<12>(a, m, stream);
        case 13: return launch<13>(a, m, stream);
        case 14: return launch<14>(a, m, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace meld
