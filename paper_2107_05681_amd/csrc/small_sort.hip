// Sort of up to 2^14 keys by one workgroup, 8 or 16 keys per lane (wave_network.h): a
// small array is bound by the latency of its chain of steps, and more lanes with
// fewer keys each issue fewer instructions in a row. 1000 keys take 3.4 us (the
// network's tile in LDS: 6.6), 2^11 3.8, 2^12 6.2, where the one compute unit's VALU
// begins to bound it, 2^13 10 to 12, 2^14 20. With the copy of the input, against 32
// keys per lane: 2^11 10.9 -> 8.2, 2^12 11.8 -> 8.4, 2^13 14.0 -> 13.1. 16 keys from 2^13
// on: 8 would take sixteen waves there and a second exchange per upper phase. Pairs are
// sorted as u64 composites, 5 operations a comparator and key where u32 takes 1: with
// the copies 1000 pairs 18.8 -> 12.2, 2^11 21.5 -> 14.8, 2^12 29 -> 20.8.
#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kSmallPad = 0xFFFFFFFFu;

// T: u32 keys, or u64 (key, payload) composites of keys and payload.
template <typename T, int LOG, int E>
__global__ __launch_bounds__((wave_group_threads<E, LOG>())) void small_sort_kernel(
    uint32_t *__restrict__ keys, uint32_t *__restrict__ payload, uint32_t n, bool vec) {
    constexpr int NT = wave_group_threads<E, LOG>();
    constexpr uint32_t LANES = (1u << LOG) / E;  // that hold keys
    __shared__ __align__(16) T s[NT > 64 ? wave_lds_words(1u << LOG) : 4];
    const WaveLane w = wave_lane();
    const uint32_t lane = (threadIdx.x & ~63u) | w.id;
    T e[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t p = r * LANES + lane;  // in any order
        const bool in = lane < LANES && p < n;
        e[r] = in ? keys[p] : kSmallPad;
        if constexpr (sizeof(T) == 8) e[r] = e[r] << 32 | (in ? payload[p] : kSmallPad);
    }
    wave_group_sort<LOG>(e, s, w);
    const uint32_t row = wave_group_row<E>(w, NT > 64 || LANES == 64);
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int r = 0; r < E; ++r)
            if (row + r < n) {
                keys[row + r] = (uint32_t)(e[r] >> 32);
                payload[row + r] = (uint32_t)e[r];
            }
        return;
    }
#pragma unroll
    for (int c = 0; c < E; c += 4) {
        if (vec && row + c + 4 <= n) {
            *reinterpret_cast<uint4 *>(keys + row + c) =
                make_uint4((uint32_t)e[c], (uint32_t)e[c + 1], (uint32_t)e[c + 2],
                           (uint32_t)e[c + 3]);
        } else {
#pragma unroll
            for (int r = c; r < c + 4; ++r)
                if (row + r < n) keys[row + r] = (uint32_t)e[r];
        }
    }
}

template <int LOG, int E>
void launch_small(uint32_t *keys, uint32_t *payload, uint32_t n, hipStream_t stream) {
    const dim3 threads(wave_group_threads<E, LOG>());
    if (payload == nullptr) {
        hipLaunchKernelGGL((small_sort_kernel<uint32_t, LOG, E>), dim3(1), threads, 0, stream,
                           keys, payload, n, ((uintptr_t)keys & 15) == 0);
    } else if constexpr (1u << LOG <= kSmallPairsMax) {
        hipLaunchKernelGGL((small_sort_kernel<uint64_t, LOG, E>), dim3(1), threads, 0, stream,
                           keys, payload, n, false);
    }
}

}  // namespace

hipError_t launch_small_sort(uint32_t *keys, uint32_t *payload, uint32_t n, hipStream_t stream) {
    if (n > (payload ? kSmallPairsMax : kSmallSortMax)) return hipErrorInvalidValue;
    if (n <= 1u << 6)
        launch_small<6, 8>(keys, payload, n, stream);
    else if (n <= 1u << 7)
        launch_small<7, 8>(keys, payload, n, stream);
    else if (n <= 1u << 8)
        launch_small<8, 8>(keys, payload, n, stream);
    else if (n <= 1u << 9)
        launch_small<9, 8>(keys, payload, n, stream);
    else if (n <= 1u << 10)
        launch_small<10, 8>(keys, payload, n, stream);
    else if (n <= 1u << 11)
        launch_small<11, 8>(keys, payload, n, stream);
    else if (n <= 1u << 12)
        launch_small<12, 8>(keys, payload, n, stream);
    else if (n <= 1u << 13)
        launch_small<13, 16>(keys, payload, n, stream);
    else
        launch_small<14, 16>(keys, payload, n, stream);
    return hipGetLastError();
}

}  // namespace meld
