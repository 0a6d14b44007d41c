// Sort of 2^12 .. 2^17 keys in two launches: runs by a workgroup each
// (wave_network.h), then every key to its rank: its place in its own run plus, by
// search, the number of keys before it in each other run. Equal keys of an earlier run
// come before, of a later run after. A search would be a chain of a round trip to
// memory per level (eleven to thirteen, 0.6 us each); the runs leave a sample of every
// 8 or 16 keys, which fits in LDS for all runs, and what is left of a search is one
// round trip for the keys of one sample.
//
// The searches grow with n times the number of runs, the runs' sort with their length,
// hence longer runs for more keys. Microseconds, runs + places: 2^14 keys in 8 runs
// 4.9 + 3.8 (2 runs searched in memory: 12.2 + 5.3), 2^15 in 16 runs 4.9 + 5.3, 2^16 in
// 16 runs 7.2 + 7.3 (8 runs searched in memory: 12.2 + 11.7), 2^17 in 16 runs 12.8 + 11.1.
//
// Pairs are u64 composites in the runs and samples. With the copies, network against
// ranks: 2^12 29 -> 17.6 us, 2^14 45 -> 18.1, 2^16 67 -> 27.8.
#include "kernels.h"
#include "wave_network.h"

namespace meld {

namespace {

constexpr uint32_t kRankPad = 0xFFFFFFFFu;

// Keys per lane of a run's sort, and how many keys of a run one sample stands for.
template <int LOG>
constexpr int run_e() {
    return LOG > 12 ? 16 : 8;
}
template <int LOG>
constexpr uint32_t sample() {
    return LOG > 11 ? 8 : 16;
}

// A run per workgroup, written whole: with the padding behind the last key, and in
// the runs past it. The last of every sample() keys goes to samples too.
template <typename T, int LOG>
__global__ __launch_bounds__((wave_group_threads<run_e<LOG>(), LOG>())) void rank_runs_kernel(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ payload, uint32_t n,
    T *__restrict__ runs, T *__restrict__ samples) {
    constexpr int E = run_e<LOG>(), NT = wave_group_threads<E, LOG>();
    constexpr uint32_t RUN = 1u << LOG;
    __shared__ __align__(16) T s[wave_lds_words(RUN)];
    const WaveLane w = wave_lane();
    const uint32_t t = threadIdx.x, tile = blockIdx.x * RUN;
    T e[E];
    if (tile + RUN <= n) {
#pragma unroll
        for (int r = 0; r < E; ++r) e[r] = keys[tile + r * NT + t];
        if constexpr (sizeof(T) == 8) {
#pragma unroll
            for (int r = 0; r < E; ++r) e[r] = e[r] << 32 | payload[tile + r * NT + t];
        }
    } else {
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const uint32_t p = tile + r * NT + t;
            e[r] = p < n ? keys[p] : kRankPad;
            if constexpr (sizeof(T) == 8) e[r] = e[r] << 32 | (p < n ? payload[p] : kRankPad);
        }
    }
    if (tile < n) wave_group_sort<LOG>(e, s, w);
    const uint32_t row = tile + wave_group_row<E>(w, true);
    wave_store_row(runs + row, e);
    constexpr uint32_t S = sample<LOG>();
    if constexpr ((uint32_t)E >= S) {
#pragma unroll
        for (uint32_t r = S - 1; r < E; r += S) samples[(row + r) / S] = e[r];
    } else if (row % S + E == S) {
        samples[row / S] = e[E - 1];
    }
}

// K neighbours in one run per workgroup, so that their probes fall on few cache lines
// and LDS words, and a thread for each of them and a share of the runs: the shares keep
// every compute unit busy where there are few keys, and shorten the chain of a thread
// (2^16 keys, 256 to a workgroup: 18.6 us with the copy of the input without shares, 15.1
// with two, 14.6 for 64 keys with eight).
template <typename T, int LOG, int RUNS, int K, int SHARES>
__global__ __launch_bounds__(K *SHARES) void rank_place_kernel(
    const T *__restrict__ runs, const T *__restrict__ samples, uint32_t n,
    uint32_t *__restrict__ keys, uint32_t *__restrict__ payload) {
    constexpr uint32_t RUN = 1u << LOG, S = sample<LOG>(), PER = RUN / S,
                       NT = K * SHARES;
    constexpr uint32_t V = 16 / sizeof(T);  // per 16-byte load
    constexpr int G = RUNS / SHARES;
    __shared__ __align__(16) T s[RUNS * PER];
    __shared__ uint32_t part[SHARES * K];
    const uint32_t t = threadIdx.x, i = blockIdx.x * K + t % K;
    const uint32_t own = blockIdx.x * K >> LOG;
    const uint32_t first = __builtin_amdgcn_readfirstlane(t / K * G);  // of the share's runs
    const T x = runs[i];
#pragma unroll
    for (uint32_t c = 0; c < RUNS * PER; c += NT * V)
        if (RUNS * PER % (NT * V) == 0 || c + t * V < RUNS * PER)
            *reinterpret_cast<uint4 *>(s + c + t * V) =
                *reinterpret_cast<const uint4 *>(samples + c + t * V);
    __syncthreads();
    // A key of an earlier run stands before an equal one, of a later run after.
    auto before = [&](int r, T y) { return first + r < own ? y <= x : y < x; };
    uint32_t pos[G];
#pragma unroll
    for (int r = 0; r < G; ++r) pos[r] = 0;
#pragma unroll
    for (uint32_t half = PER / 2; half != 0; half >>= 1) {
        T y[G];
#pragma unroll
        for (int r = 0; r < G; ++r) y[r] = s[(first + r) * PER + pos[r] + half - 1];
#pragma unroll
        for (int r = 0; r < G; ++r)
            if (before(r, y[r])) pos[r] += half;
    }
    T y[G][S];
#pragma unroll
    for (int r = 0; r < G; ++r) wave_load_row(y[r], runs + (first + r) * RUN + pos[r] * S);
    __builtin_amdgcn_sched_barrier(0);  // every load before the first wait
    uint32_t rank = 0;
#pragma unroll
    for (int r = 0; r < G; ++r) {
        uint32_t at = pos[r] * S;
#pragma unroll
        for (uint32_t c = 0; c < S; ++c) at += (uint32_t)before(r, y[r][c]);
        rank += first + r == own ? i & (RUN - 1) : at;
    }
    if constexpr (SHARES > 1) {
        part[t] = rank;
        __syncthreads();
        if (t >= K) return;
#pragma unroll
        for (int c = 1; c < SHARES; ++c) rank += part[c * K + t];
    }
    if (i < n) {
        if constexpr (sizeof(T) == 8) {
            keys[rank] = (uint32_t)(x >> 32);
            payload[rank] = (uint32_t)x;
        } else {
            keys[rank] = x;
        }
    }
}

template <typename T, int LOG, int RUNS, int K, int SHARES>
void launch_ranks(uint32_t *keys, uint32_t *payload, uint32_t n, uint32_t *scratch,
                  hipStream_t stream) {
    T *runs = reinterpret_cast<T *>(scratch), *samples = runs + ((uint32_t)RUNS << LOG);
    hipLaunchKernelGGL((rank_runs_kernel<T, LOG>), dim3(RUNS),
                       dim3(wave_group_threads<run_e<LOG>(), LOG>()), 0, stream,
                       (const uint32_t *)keys, (const uint32_t *)payload, n, runs, samples);
    hipLaunchKernelGGL((rank_place_kernel<T, LOG, RUNS, K, SHARES>), dim3(blocks_for(n, K)),
                       dim3(K * SHARES), 0, stream, (const T *)runs, (const T *)samples, n, keys,
                       payload);
}

}  // namespace

hipError_t launch_rank_sort(uint32_t *keys, uint32_t *payload, uint32_t n, uint32_t *scratch,
                            hipStream_t stream) {
    if (n > (payload ? kRankPairsMax : kRankSortMax)) return hipErrorInvalidValue;
#define MELD_RANKS(T, ...) launch_ranks<T, __VA_ARGS__>(keys, payload, n, scratch, stream)
    if (payload != nullptr) {
        if (n <= 2u << 11)
            MELD_RANKS(uint64_t, 11, 2, 64, 1);
        else if (n <= 4u << 11)
            MELD_RANKS(uint64_t, 11, 4, 64, 2);
        else if (n <= 8u << 11)
            MELD_RANKS(uint64_t, 11, 8, 64, 4);
        else if (n <= 16u << 11)
            MELD_RANKS(uint64_t, 11, 16, 64, 8);
        else
            MELD_RANKS(uint64_t, 12, 16, 64, 8);
        return hipGetLastError();
    }
    // With the copy of the input, microseconds, 2^11 / 2^12 / 2^13 keys to a run (64 keys
    // to a workgroup, two runs to a thread): 2^14 10.0 / 11.6 / 16.2, 2^15 10.7 / 12.1 /
    // 16.9, 2^16 15.6 / 14.6 / 18.3, 80000 22.0 / 20.5 (24 runs: 18.5) / 23.0, 2^17 25.7 /
    // 26.5 / 27.1 (four runs to a thread and 256 keys: 23.8).
    if (n <= 4u << 11)
        MELD_RANKS(uint32_t, 11, 4, 64, 2);
    else if (n <= 8u << 11)
        MELD_RANKS(uint32_t, 11, 8, 64, 4);
    else if (n <= 16u << 11)
        MELD_RANKS(uint32_t, 11, 16, 64, 8);
    else if (n <= 16u << 12)
        MELD_RANKS(uint32_t, 12, 16, 64, 8);
    else if (n <= 24u << 12)
        MELD_RANKS(uint32_t, 12, 24, 64, 12);
    else
        MELD_RANKS(uint32_t, 13, 16, 256, 4);
#undef MELD_RANKS
    return hipGetLastError();
}

}  // namespace meld
