// The loop regions with four consecutive lanes per thread: a candidate of
// MELD_AUTO for the two-sided, the three-way and the per-lane-trips region.
//
// The branch of a lane is a hash of its number, so that a wave of 256 lanes takes
// every way. The forms with a lane per thread therefore issue every step's gather
// once per way, each for part of the wave, and are bound by the address path of
// the vector memory (5.6 cycles a gather of 64 lanes). But the lanes of a wave are
// consecutive, and so are their table entries at a step of one way: here a wave
// loads all 256 of a way's entries by one 16-byte access per thread, from a scalar
// address, and each lane keeps the value of its own way. No gather is issued for
// fewer lanes than there are, index arithmetic is scalar, and the fma order is the
// definition's, so results are bit-identical to the other forms. With trips of its
// own a lane leaves no loop here: the loop runs to the longest, and a lane past its
// last step keeps its value.
//
// 2^23 lanes, 8 to 26 trips a lane, a 2^23-entry table: 184 us with a lane per
// thread, 81 us so; three ways of 10, 10 and 28 trips on 2^24 lanes: 189 and 172 us;
// two sides of 10 trips on 2^24 lanes: 102 and 97 us. The tuner times the forms on the
// same arrays again and again; within its 2 % it may take this one where a lane per
// thread is as fast then (8 and 32 trips: 112 us against 110), and with inputs that
// change it is the faster (138 against 154). What bounds it now is the L2:
// 1.5 GB of the last call's entries come from it in 70 us when the table is there.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "region_steps.h"

namespace meld {

namespace {

constexpr int kQuad = 4;                  // lanes per thread
constexpr uint32_t kQuadWave = 64 * kQuad;  // lanes per wave
constexpr int kQuadBatch = 4;             // steps whose loads are in flight together

struct QuadWay {
    float a;
    uint32_t off, step;
    uint32_t lo, span;  // trips of a lane: lo, or with LANE_TRIPS lo .. lo + span
};
template <int WAYS>
struct QuadWays {
    QuadWay way[WAYS];
    uint32_t kmin;         // steps every lane runs
    uint32_t bound[WAYS];  // where a way's last lane ends, in ascending order
};

typedef float Float4 __attribute__((ext_vector_type(4)));
typedef float Entries4 __attribute__((ext_vector_type(4), aligned(4)));  // at any table entry

// The wave's 256 table entries at NB steps of a way, from `first` on (mod the
// table), four per thread. One check for all of them whether any crosses the
// table's end, so that the loads go out together.
template <int NB>
__device__ __forceinline__ void quad_load(Float4 (&g)[NB], const float *__restrict__ tab,
                                          uint32_t mask, uint32_t first, uint32_t step,
                                          uint32_t lane) {
    uint32_t last = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint32_t at = (first + b * step) & mask;
        last = at > last ? at : last;
    }
    if (mask >= kQuadWave - 1 && last <= mask - (kQuadWave - 1)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            g[b] = *reinterpret_cast<const Entries4 *>(tab + ((first + b * step) & mask) +
                                                       lane * kQuad);
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < kQuad; ++j)
                g[b][j] = tab[(first + b * step + lane * kQuad + j) & mask];
    }
}

// A thread's four lanes.
struct QuadLanes {
    float acc[kQuad], a[kQuad];
    uint32_t way[kQuad], trips[kQuad];
};

// Steps k .. k + NB - 1, which end before or at the last step of every way that
// has one at k. w0: the wave's first lane.
template <int WAYS, int NB>
__device__ __forceinline__ void quad_steps(QuadLanes &l, const QuadWays<WAYS> &ws, uint32_t k,
                                           const float *__restrict__ tab, uint32_t mask,
                                           uint32_t w0, uint32_t lane) {
    Float4 g[WAYS][NB];
#pragma unroll
    for (int q = 0; q < WAYS; ++q)
        if (k < ws.way[q].lo + ws.way[q].span)
            quad_load(g[q], tab, mask, w0 + ws.way[q].off + k * ws.way[q].step, ws.way[q].step,
                      lane);
    auto run = [&](auto check) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < kQuad; ++j) {
                float v = l.way[j] == 0 ? g[0][b][j] : g[1][b][j];
                if constexpr (WAYS == 3) v = l.way[j] == 2 ? g[2][b][j] : v;
                const float r = __builtin_fmaf(l.acc[j], l.a[j], v);
                l.acc[j] = !decltype(check)::value || k + b < l.trips[j] ? r : l.acc[j];
            }
    };
    if (k + NB <= ws.kmin)
        run(std::false_type{});
    else
        run(std::true_type{});
}

template <int WAYS, bool LANE_TRIPS>
__global__ __launch_bounds__(kRegionThreads) void region_quad_kernel(
    const float *__restrict__ x, float *__restrict__ y, uint32_t n, uint32_t lane0,
    const float *__restrict__ tab, uint32_t mask, uint64_t bkey, uint64_t tkey, uint64_t thr0,
    uint64_t thr1, bool vec, QuadWays<WAYS> ws) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(xcd_contiguous_block(blockIdx.x, gridDim.x) * (kRegionThreads / 64) +
              threadIdx.x / 64));
    if ((uint64_t)lane0 + wave * kQuadWave >= n) return;
    const uint32_t w0 = lane0 + wave * kQuadWave;  // the wave's first lane
    const uint32_t i = w0 + lane * kQuad;
    const bool whole = vec && n - w0 >= kQuadWave;
    QuadLanes l;
    if (whole) {
        const float4 v = *reinterpret_cast<const float4 *>(x + i);
        l.acc[0] = v.x;
        l.acc[1] = v.y;
        l.acc[2] = v.z;
        l.acc[3] = v.w;
    } else {
#pragma unroll
        for (int j = 0; j < kQuad; ++j) l.acc[j] = i + j < n && i + j >= w0 ? x[i + j] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < kQuad; ++j) {
        const uint64_t h = mix64(bkey + (i + j)) >> 32;
        const uint32_t way = h < thr0 ? 0u : (WAYS == 2 || h < thr1 ? 1u : 2u);
        float a = way == 0 ? ws.way[0].a : ws.way[1].a;
        uint32_t lo = way == 0 ? ws.way[0].lo : ws.way[1].lo;
        uint32_t span = way == 0 ? ws.way[0].span : ws.way[1].span;
        if constexpr (WAYS == 3) {
            a = way == 2 ? ws.way[2].a : a;
            lo = way == 2 ? ws.way[2].lo : lo;
            span = way == 2 ? ws.way[2].span : span;
        }
        if constexpr (LANE_TRIPS)
            lo += (uint32_t)((mix64(tkey + (i + j)) >> 32) % ((uint64_t)span + 1));
        l.way[j] = way;
        l.a[j] = a;
        l.trips[j] = lo;
    }
    uint32_t k = 0;
#pragma unroll 1
    for (int q = 0; q < WAYS; ++q) {
        const uint32_t end = ws.bound[q];
#pragma unroll 1
        for (; k + kQuadBatch <= end; k += kQuadBatch)
            quad_steps<WAYS, kQuadBatch>(l, ws, k, tab, mask, w0, lane);
        if (k + 2 <= end) {
            quad_steps<WAYS, 2>(l, ws, k, tab, mask, w0, lane);
            k += 2;
        }
        if (k < end) {
            quad_steps<WAYS, 1>(l, ws, k, tab, mask, w0, lane);
            ++k;
        }
    }
    if (whole) {
        *reinterpret_cast<float4 *>(y + i) = make_float4(l.acc[0], l.acc[1], l.acc[2], l.acc[3]);
    } else {
#pragma unroll
        for (int j = 0; j < kQuad; ++j)
            if (i + j < n && i + j >= w0) y[i + j] = l.acc[j];
    }
}

template <int WAYS, bool LANE_TRIPS>
hipError_t launch_quad(const float *x, float *y, uint32_t n, const float *tab, uint32_t mask,
                       uint64_t seed, uint64_t thr0, uint64_t thr1, QuadWays<WAYS> ws,
                       hipStream_t stream) {
    ws.kmin = 0xFFFFFFFFu;
    for (int q = 0; q < WAYS; ++q) {
        ws.kmin = std::min(ws.kmin, ws.way[q].lo);
        ws.bound[q] = ws.way[q].lo + ws.way[q].span;
    }
    std::sort(ws.bound, ws.bound + WAYS);
    const bool vec = (((uintptr_t)x | (uintptr_t)y) & 15) == 0;
    constexpr uint32_t per = kRegionThreads * kQuad;
    for (uint64_t i0 = 0; i0 < n; i0 += kRegionLaunchLanes) {
        const uint32_t len = (uint32_t)(n - i0 < kRegionLaunchLanes ? n - i0 : kRegionLaunchLanes);
        hipLaunchKernelGGL((region_quad_kernel<WAYS, LANE_TRIPS>), dim3(blocks_for(len, per)),
                           dim3(kRegionThreads), 0, stream, x, y, n, (uint32_t)i0, tab, mask,
                           stream_key(seed, 4), stream_key(seed, 11), thr0, thr1, vec, ws);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_region_quad(const float *x, float *y, uint32_t n, const float *tab,
                              uint32_t mask, uint64_t seed, uint64_t thr, RegionSide T,
                              RegionSide F, hipStream_t stream) {
    return launch_quad<2, false>(x, y, n, tab, mask, seed, thr, 0,
                                 {{{T.a, T.off, T.step, T.trips, 0}, {F.a, F.off, F.step, F.trips, 0}}},
                                 stream);
}

hipError_t launch_region3_quad(const float *x, float *y, uint32_t n, const float *tab,
                               uint32_t mask, uint64_t seed, uint64_t thr0, uint64_t thr1,
                               RegionSide W0, RegionSide W1, RegionSide W2, hipStream_t stream) {
    return launch_quad<3, false>(x, y, n, tab, mask, seed, thr0, thr1,
                                 {{{W0.a, W0.off, W0.step, W0.trips, 0},
                                   {W1.a, W1.off, W1.step, W1.trips, 0},
                                   {W2.a, W2.off, W2.step, W2.trips, 0}}},
                                 stream);
}

hipError_t launch_region_lanetrips_quad(const float *x, float *y, uint32_t n, const float *tab,
                                        uint32_t mask, uint64_t seed, uint64_t thr,
                                        RegionSideRange T, RegionSideRange F, hipStream_t stream) {
    return launch_quad<2, true>(x, y, n, tab, mask, seed, thr, 0,
                                {{{T.a, T.off, T.step, T.lo, T.span}, {F.a, F.off, F.step, F.lo, F.span}}},
                                stream);
}

}  // namespace meld
