// Sort of up to 2^14 keys by one workgroup, 8 or 16 keys per lane (wave_network.h): a
// small array is bound by the latency of its chain of steps, and more lanes with
// fewer keys each issue fewer instructions in a row. 1000 keys take 3.4 us (the
// network's tile in LDS: 6.6), 2^11 3.8, 2^12 6.2, where the one compute unit's VALU
// begins to bound it, 2^13 10 to 12, 2^14 20. With the copy of the input, against 32
// keys per lane: 2^11 10.9 -> 8.2, 2^12 11.8 -> 8.4, 2^13 14.0 -> 13.1. 16 keys from 2^13
// on: 8 would take sixteen waves there and a second exchange per upper phase.
#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kSmallPad = 0xFFFFFFFFu;

template <int LOG, int E>
__global__ __launch_bounds__((wave_group_threads<E, LOG>())) void small_sort_kernel(
    uint32_t *__restrict__ keys, uint32_t n, bool vec) {
    constexpr int T = wave_group_threads<E, LOG>();
    constexpr uint32_t LANES = (1u << LOG) / E;  // that hold keys
    __shared__ __align__(16) uint32_t s[T > 64 ? wave_lds_words(1u << LOG) : 4];
    const WaveLane w = wave_lane();
    const uint32_t lane = (threadIdx.x & ~63u) | w.id;
    uint32_t e[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t p = r * LANES + lane;  // in any order
        e[r] = lane < LANES && p < n ? keys[p] : kSmallPad;
    }
    wave_group_sort<LOG>(e, s, w);
    const uint32_t row = wave_group_row<E>(w, T > 64 || LANES == 64);
#pragma unroll
    for (int c = 0; c < E; c += 4) {
        if (vec && row + c + 4 <= n) {
            *reinterpret_cast<uint4 *>(keys + row + c) =
                make_uint4(e[c], e[c + 1], e[c + 2], e[c + 3]);
        } else {
#pragma unroll
            for (int r = c; r < c + 4; ++r)
                if (row + r < n) keys[row + r] = e[r];
        }
    }
}

template <int LOG, int E>
void launch_small(uint32_t *keys, uint32_t n, hipStream_t stream) {
    hipLaunchKernelGGL((small_sort_kernel<LOG, E>), dim3(1), dim3(wave_group_threads<E, LOG>()),
                       0, stream, keys, n, ((uintptr_t)keys & 15) == 0);
}

}  // namespace

hipError_t launch_small_sort(uint32_t *keys, uint32_t n, hipStream_t stream) {
    if (n > kSmallSortMax) return hipErrorInvalidValue;
    if (n <= 1u << 6)
        launch_small<6, 8>(keys, n, stream);
    else if (n <= 1u << 7)
        launch_small<7, 8>(keys, n, stream);
    else if (n <= 1u << 8)
        launch_small<8, 8>(keys, n, stream);
    else if (n <= 1u << 9)
        launch_small<9, 8>(keys, n, stream);
    else if (n <= 1u << 10)
        launch_small<10, 8>(keys, n, stream);
    else if (n <= 1u << 11)
        launch_small<11, 8>(keys, n, stream);
    else if (n <= 1u << 12)
        launch_small<12, 8>(keys, n, stream);
    else if (n <= 1u << 13)
        launch_small<13, 16>(keys, n, stream);
    else
        launch_small<14, 16>(keys, n, stream);
    return hipGetLastError();
}

}  // namespace meld
