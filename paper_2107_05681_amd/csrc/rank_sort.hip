// Sort of 2^13 .. 2^17 keys in two launches: runs of 2^13 by a workgroup each
// (wave_network.h), then every key to its rank: its place in its own run plus, by
// binary search, the number of keys before it in each other run. The searches of a
// key do not depend on each other, so that all of them wait for memory together.
// Equal keys of an earlier run come before, of a later run after. The searches grow
// with n times the number of runs, which is why larger arrays go through radix
// passes; runs of 2^11, 2 us faster to sort, would make them four times as many
// (2^16 keys: 40 us).
#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kRankPad = 0xFFFFFFFFu;
constexpr int kRunLog = 13;
constexpr uint32_t kRun = 1u << kRunLog;
constexpr int kRunE = 16;
constexpr int kRunThreads = wave_group_threads<kRunE, kRunLog>();
constexpr int kRankThreads = 256;

// A run per workgroup, written whole: with the padding behind the last key, and in
// the runs past it.
__global__ __launch_bounds__(kRunThreads) void rank_runs_kernel(const uint32_t *__restrict__ keys,
                                                                uint32_t n,
                                                                uint32_t *__restrict__ runs) {
    __shared__ __align__(16) uint32_t s[wave_lds_words(kRun)];
    const WaveLane w = wave_lane();
    const uint32_t t = threadIdx.x, tile = blockIdx.x * kRun;
    uint32_t e[kRunE];
    if (tile + kRun <= n) {
#pragma unroll
        for (int r = 0; r < kRunE; ++r) e[r] = keys[tile + r * kRunThreads + t];
    } else {
#pragma unroll
        for (int r = 0; r < kRunE; ++r) {
            const uint32_t p = tile + r * kRunThreads + t;
            e[r] = p < n ? keys[p] : kRankPad;
        }
    }
    if (tile < n) wave_group_sort<kRunLog>(e, s, w);
    uint4 *to = reinterpret_cast<uint4 *>(runs + tile + wave_group_row<kRunE>(w, true));
#pragma unroll
    for (int c = 0; c < kRunE; c += 4)
        to[c / 4] = make_uint4(e[c], e[c + 1], e[c + 2], e[c + 3]);
}

// One thread per key; the 256 keys of a workgroup are neighbours in one run, so
// that their probes fall on few cache lines. Bound by the fourteen round trips to
// memory of a search, 0.6 us each, and by the address path.
template <int RUNS>
__global__ __launch_bounds__(kRankThreads) void rank_place_kernel(
    const uint32_t *__restrict__ runs, uint32_t n, uint32_t *__restrict__ keys) {
    const uint32_t i = blockIdx.x * kRankThreads + threadIdx.x;
    const uint32_t own = blockIdx.x * kRankThreads >> kRunLog;
    const uint32_t x = runs[i];
    uint32_t pos[RUNS], y[RUNS];
#pragma unroll
    for (int r = 0; r < RUNS; ++r) pos[r] = 0;
    // A key of an earlier run stands before an equal one, of a later run after.
    auto advance = [&](uint32_t by) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r)
            if ((uint32_t)r < own ? y[r] <= x : y[r] < x) pos[r] += by;
    };
#pragma unroll
    for (uint32_t half = kRun / 2; half != 0; half >>= 1) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) y[r] = runs[((uint32_t)r << kRunLog) + pos[r] + half - 1];
        advance(half);
    }
    // Places 0 .. 2^13 - 1 so far; one key of the run is left to look at.
#pragma unroll
    for (int r = 0; r < RUNS; ++r) y[r] = runs[((uint32_t)r << kRunLog) + pos[r]];
    advance(1);
    uint32_t rank = 0;
#pragma unroll
    for (int r = 0; r < RUNS; ++r) rank += (uint32_t)r == own ? i & (kRun - 1) : pos[r];
    if (i < n) keys[rank] = x;
}

template <int RUNS>
void launch_ranks(uint32_t *keys, uint32_t n, uint32_t *runs, hipStream_t stream) {
    hipLaunchKernelGGL(rank_runs_kernel, dim3(RUNS), dim3(kRunThreads), 0, stream,
                       (const uint32_t *)keys, n, runs);
    hipLaunchKernelGGL(rank_place_kernel<RUNS>, dim3(blocks_for(n, kRankThreads)),
                       dim3(kRankThreads), 0, stream, (const uint32_t *)runs, n, keys);
}

}  // namespace

hipError_t launch_rank_sort(uint32_t *keys, uint32_t n, uint32_t *scratch, hipStream_t stream) {
    if (n > kRankSortMax) return hipErrorInvalidValue;
    if (n <= 2 * kRun)
        launch_ranks<2>(keys, n, scratch, stream);
    else if (n <= 4 * kRun)
        launch_ranks<4>(keys, n, scratch, stream);
    else if (n <= 8 * kRun)
        launch_ranks<8>(keys, n, scratch, stream);
    else
        launch_ranks<16>(keys, n, scratch, stream);
    return hipGetLastError();
}

}  // namespace meld
