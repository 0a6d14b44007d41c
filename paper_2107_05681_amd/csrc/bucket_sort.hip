// Sorts buckets of 2^6 .. 2^14 keys in one launch, in registers
// (wave_network.h): what MELD_AUTO runs where every bucket's sorted order is all
// that is asked for.
#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kPadKey = 0xFFFFFFFFu;

// Waves per workgroup: those of one bucket, or four that work side by side.
constexpr int bucket_waves(int log_b) { return log_b <= 11 ? 4 : 1 << (log_b - 11); }

// The 16 bytes at p (a multiple of 4) as far as they lie below n.
__device__ __forceinline__ uint4 load_some(const uint32_t *keys, uint32_t n, uint32_t p) {
    uint4 v = make_uint4(kPadKey, kPadKey, kPadKey, kPadKey);
    if (p + 4 <= n) {
        v = *reinterpret_cast<const uint4 *>(keys + p);
    } else if (p < n) {
        v.x = keys[p];
        if (p + 1 < n) v.y = keys[p + 1];
        if (p + 2 < n) v.z = keys[p + 2];
    }
    return v;
}
__device__ __forceinline__ void store_some(uint32_t *keys, uint32_t n, uint32_t p, uint4 v) {
    if (p + 4 <= n) {
        *reinterpret_cast<uint4 *>(keys + p) = v;
    } else if (p < n) {
        keys[p] = v.x;
        if (p + 1 < n) keys[p + 1] = v.y;
        if (p + 2 < n) keys[p + 2] = v.z;
    }
}

// One wave per 2^11 keys. A lane's first keys may be any of its bucket's, so
// that loads are 16 bytes per lane, neighbouring lanes side by side (4 bytes for
// arrays that are not aligned); the sorted tile goes through LDS to be stored
// the same way. Keys past n are padding, which sorts behind every key.
//
// 2^26 keys in buckets of 2^13 take 212 us (passes of 310 less 98 for the copy of the
// input; a kernel trace averages 260 over the first 13 calls, until the clock settles,
// and ends at 228), the odd-even network with one LDS access per key and step 1070 us;
// buckets of 2^11 155 us, 2^6: 85 us. VALU issue bounds
// the large buckets (131 operations a key at 2^13: 215 us on 1024 SIMDs), the
// transfer the small ones (537 MB).
template <int LOG, bool VEC>
__global__ __launch_bounds__(64 * bucket_waves(LOG)) void bucket_sort_kernel(
    uint32_t *__restrict__ keys, uint32_t n) {
    extern __shared__ __align__(16) uint32_t s[];
    constexpr int W = bucket_waves(LOG);
    constexpr int LB = LOG < 11 ? LOG - 5 : 6;  // log2 of a bucket's lanes in the wave
    const WaveLane w = wave_lane();
    const uint32_t wave = threadIdx.x / 64, lane = threadIdx.x & 63;
    const uint32_t tile = (xcd_contiguous_block(blockIdx.x, gridDim.x) * W + wave) * kWaveTile;
    const uint32_t first = tile + ((w.id >> LB) << (LB + 5));  // the lane's bucket in this wave
    const uint32_t at = w.id & ((1u << LB) - 1);
    const bool full = tile + kWaveTile <= n;  // the same for the whole wave
    uint32_t e[kWaveE];
    if (VEC) {
#pragma unroll
        for (int c = 0; c < kWaveE / 4; ++c) {
            const uint32_t p = first + (((c << LB) + at) << 2);
            const uint4 v = full ? *reinterpret_cast<const uint4 *>(keys + p) : load_some(keys, n, p);
            e[4 * c] = v.x;
            e[4 * c + 1] = v.y;
            e[4 * c + 2] = v.z;
            e[4 * c + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) {
            const uint32_t p = first + ((uint32_t)r << LB) + at;
            e[r] = p < n ? keys[p] : kPadKey;
        }
    }
    wave_sort<LOG>(e, s, w);
    uint32_t *own = s + wave * wave_lds_words(kWaveTile);
    wave_to_lds<(LOG >= 11)>(e, own, w);
    __builtin_amdgcn_wave_barrier();
    if (VEC) {
#pragma unroll
        for (int c = 0; c < kWaveE / 4; ++c) {
            const uint32_t i = (c * 64 + lane) * 4;
            const uint4 v = *reinterpret_cast<const uint4 *>(own + wave_phys(i));
            if (full)
                *reinterpret_cast<uint4 *>(keys + tile + i) = v;
            else
                store_some(keys, n, tile + i, v);
        }
    } else {
#pragma unroll
        for (int r = 0; r < kWaveE; ++r) {
            const uint32_t i = r * 64 + lane;
            if (tile + i < n) keys[tile + i] = own[wave_phys(i)];
        }
    }
}

template <int LOG, bool VEC>
hipError_t launch_bucket(uint32_t *keys, uint32_t n, hipStream_t stream) {
    constexpr int W = bucket_waves(LOG);
    constexpr size_t lds = (size_t)W * wave_lds_words(kWaveTile) * sizeof(uint32_t);
    auto kern = bucket_sort_kernel<LOG, VEC>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(blocks_for(n, W * kWaveTile)), dim3(64 * W), lds, stream, keys,
                       n);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bucket_sort(uint32_t *keys, uint32_t n, uint32_t log_bucket,
                              hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const bool vec = ((uintptr_t)keys & 15) == 0;
#define MELD_BUCKET(L) \
    case L: return vec ? launch_bucket<L, true>(keys, n, stream) \
                       : launch_bucket<L, false>(keys, n, stream);
    switch (log_bucket) {
        MELD_BUCKET(6)
        MELD_BUCKET(7)
        MELD_BUCKET(8)
        MELD_BUCKET(9)
        MELD_BUCKET(10)
        MELD_BUCKET(11)
        MELD_BUCKET(12)
        MELD_BUCKET(13)
        MELD_BUCKET(14)
        default: return hipErrorInvalidValue;
    }
#undef MELD_BUCKET
}

}  // namespace meld
