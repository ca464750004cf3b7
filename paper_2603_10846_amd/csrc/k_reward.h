// Rewards of the two stages and their online normalisation, computed on the device so that a batch
// of verifier outcomes can go straight into the value update.
//   Stage 1 (Sec. 3.3): +1 if the candidate is feasible, -1 otherwise.
//   Stage 2 (Sec. 3.4): -1 if infeasible, else tanh(log b - log l), b the best latency so far, l the
//   measured one (App. A: tanh(log rho), rho the speed-up ratio).
//   Normalisation (Sec. 3.4, App. A "Stability of Online Normalization"): sample t becomes
//   (r_t - mu_{t-1}) / max(sigma_{t-1}, sigma_min), optionally clipped, with mu, sigma the running
//   mean and population deviation of the raw rewards BEFORE it; the statistics (count, sum, sum of
//   squares, fp64) persist in the handle's workspace.
// The dependence of sample t on all earlier ones is a prefix sum.  Up to 1024 samples are one workgroup's; up to 64 blocks of 256 are one
// launch in which a block leaves its sums of (r, r^2) and waits for those of the blocks before it; longer batches are two launches, the
// first for the sums, and in the second a block adds those of the blocks before it.  The raw rewards -- two fp64
// logarithms and a tanh per sample -- are what bounds a block, and the launches (about 3 us each) the host.  us a call, one workgroup walking the batch in
// pieces of 1024 up to 1536 samples (3072 in stage 0) and two launches beyond, and now: stage 1, 1025 samples 9.0, 7.2; 8192 8.9, 7.1; stage 0, 3072 9.6, 7.1.
// All arithmetic in fp64; outputs fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "k_ingest.h"

namespace evk {

constexpr int REWARD_ONE = 1024;          // largest batch of one workgroup
constexpr int REWARD_T = 256;             // samples per block of the other forms
constexpr int REWARD_CHAIN = 64;          // blocks of the one-launch form, a bit each
// Blocks of a pair of launches, at most: every block adds up the sums of all before it, so a pair's work has a part that
// grows with the square of its blocks.  Normalised, 4 M samples 147 -> 133 us, 16.7 M 1267 -> 531, 67 M 17.5 -> 2.2 ms (a batch in one
// pair before; pairs of 2048 blocks take 15 to 20 % longer than these).
constexpr int REWARD_BLOCKS = 8192;

__device__ __forceinline__ double wave_inclusive_sum_d(double x, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

struct RewardArgs {
    const unsigned char* feasible;
    const float* latency;
    const float* best;
    int64_t M;
    double sigma_min, clip;
    double* state;            // count, sum, sum of squares
    double* sums;             // the statistics before the batch (two launches), then two sums per block
    uint64_t* chain;          // one launch: which blocks have left their sums, 32 to a word: the latest call's number << 32 | a bit each
    uint32_t call;            // one launch: its number, of this handle's; larger than any before, never 0
    float* out;
    int stage, normalise;
};
constexpr int REWARD_HEAD = 4;            // doubles in front of the blocks' sums

__device__ __forceinline__ double raw_reward(const RewardArgs& A, int64_t j) {
    if (!A.feasible[j]) return -1.0;
    return A.stage == 0 ? 1.0 : tanh(log((double)A.best[j]) - log((double)A.latency[j]));
}

// Normalised reward of a sample, n samples with the given sums having come before it.
__device__ __forceinline__ double normalised_reward(const RewardArgs& A, double raw, double n, double sum, double sq) {
    const double mu = n > 0.0 ? sum / n : 0.0;
    const double var = n > 0.0 ? sq / n - mu * mu : 0.0;
    const double sigma = var > 0.0 ? sqrt(var) : 0.0;
    double r = (raw - mu) / (sigma > A.sigma_min ? sigma : A.sigma_min);
    if (A.clip > 0.0) r = r > A.clip ? A.clip : (r < -A.clip ? -A.clip : r);
    return r;
}

// Sums over the samples of earlier lanes and over the block, for blocks of W wavefronts (all lanes call it).
template <int W>
__device__ __forceinline__ void block_prefix2(double (*part)[2], int wave, int lane, double x, double y, double& before_x, double& before_y,
                                              double& all_x, double& all_y) {
    const double ix = wave_inclusive_sum_d(x, lane), iy = wave_inclusive_sum_d(y, lane);
    if (lane == 63) { part[wave][0] = ix; part[wave][1] = iy; }
    __syncthreads();
    before_x = ix - x;
    before_y = iy - y;
    all_x = 0.0;
    all_y = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if (w < wave) { before_x += part[w][0]; before_y += part[w][1]; }
        all_x += part[w][0];
        all_y += part[w][1];
    }
}

// At most 1024 samples (more of them unnormalised are the last kernel's).
__global__ __launch_bounds__(REWARD_ONE) void k_shape_rewards(RewardArgs A) {
    __shared__ double part[REWARD_ONE / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool live = tid < A.M;
    const double raw = live ? raw_reward(A, tid) : 0.0;
    if (!A.normalise) {                                              // uniform
        if (live) A.out[tid] = (float)raw;
        return;
    }
    const double n0 = A.state[0], s0 = A.state[1], q0 = A.state[2];  // the statistics before the batch
    double bs, bq, as, aq;
    block_prefix2<REWARD_ONE / 64>(part, wave, lane, raw, raw * raw, bs, bq, as, aq);    // (has a barrier)
    if (live) A.out[tid] = (float)normalised_reward(A, raw, n0 + tid, s0 + bs, q0 + bq);
    if (tid == 0) { A.state[0] = n0 + (double)A.M; A.state[1] = s0 + as; A.state[2] = q0 + aq; }
}

// Up to 64 blocks in one launch.  A block waits for those before it only.  All of the launch's blocks fit on the device many times
// over, so each of them comes to run whatever the others do, and the wait ends.
// No word is cleared, so no wait depends on when: a call raises the words to its own number, which drops the bits of earlier ones, and a later
// number says as much as the bits do.  Were two calls on a handle to overlap, each might take the other's sums, but both would end and leave nothing
// that a later call trips over.  The number comes from the host; a replayed graph would bring an old one, so recorded calls are two launches.
// What blocks hand to each other are their sums, stored and loaded as device-scope atomics, which pass by the caches that differ between
// XCDs; a block's stores have been acknowledged before it says so.
__global__ __launch_bounds__(REWARD_T) void k_reward_chain(RewardArgs A) {
    __shared__ double total[REWARD_T / 64][2], part[REWARD_T / 64][2], earlier[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, block = (int)blockIdx.x;
    const int64_t j = (int64_t)block * REWARD_T + tid;
    const bool live = j < A.M;
    if (tid == 0) (void)__hip_atomic_fetch_max(A.chain + (block >> 5), (uint64_t)A.call << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const double n_old = A.state[0], s_old = A.state[1], q_old = A.state[2];      // (replaced by the last block once all have said so)
    const double raw = live ? raw_reward(A, j) : 0.0;
    const double s = wave_total_d(raw), q = wave_total_d(raw * raw);
    if (lane == 0) { total[wave][0] = s; total[wave][1] = q; }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wave == 0) {                                                 // uniform within a wavefront
        double* mine = A.sums + REWARD_HEAD;
        if (lane < 2)
            __hip_atomic_store(mine + 2 * block + lane, (total[0][lane] + total[1][lane]) + (total[2][lane] + total[3][lane]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) (void)__hip_atomic_fetch_or(A.chain + (block >> 5), 1ull << (block & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // lane 0 watches the word of blocks 0 to 31, lane 1 that of the others
        const uint64_t before = ((1ull << block) - 1ull) >> (lane == 1 ? 32 : 0);
        const uint32_t need = lane < 2 ? (uint32_t)before : 0u;
        bool there = need == 0;
        for (;;) {
            if (!there) {
                const uint64_t w = __hip_atomic_load(A.chain + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                there = (uint32_t)(w >> 32) > A.call || ((uint32_t)(w >> 32) == A.call && ((uint32_t)w & need) == need);
            }
            if (__builtin_amdgcn_ballot_w64(!there) == 0) break;     // uniform
            __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");
        double es = 0.0, eq = 0.0;
        if (lane < block) {
            es = __hip_atomic_load(mine + 2 * lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            eq = __hip_atomic_load(mine + 2 * lane + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        es = wave_total_d(es);
        eq = wave_total_d(eq);
        if (lane == 0) { earlier[0] = es; earlier[1] = eq; }
    }
    double bs, bq, as, aq;
    block_prefix2<REWARD_T / 64>(part, wave, lane, raw, raw * raw, bs, bq, as, aq);       // (has a barrier)
    const double s0 = s_old + earlier[0], q0 = q_old + earlier[1];
    if (live) A.out[j] = (float)normalised_reward(A, raw, n_old + (double)j, s0 + bs, q0 + bq);
    if (block == (int)gridDim.x - 1 && tid == 0) {
        A.state[0] = n_old + (double)A.M;
        A.state[1] = s0 + as;
        A.state[2] = q0 + aq;
    }
}

// First launch of a longer batch: the blocks' sums, and a copy of the statistics (the second launch replaces them
// while other blocks still need the old ones).
__global__ __launch_bounds__(REWARD_T) void k_reward_sums(RewardArgs A) {
    __shared__ double part[REWARD_T / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t j = (int64_t)blockIdx.x * REWARD_T + tid;
    const double raw = j < A.M ? raw_reward(A, j) : 0.0;
    const double s = wave_total_d(raw), q = wave_total_d(raw * raw);
    if (lane == 0) { part[wave][0] = s; part[wave][1] = q; }
    __syncthreads();
    if (tid < 2) A.sums[REWARD_HEAD + 2 * (int64_t)blockIdx.x + tid] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
    if (blockIdx.x == 0 && tid < 3) A.sums[tid] = A.state[tid];
}

__global__ __launch_bounds__(REWARD_T) void k_reward_shape(RewardArgs A) {
    __shared__ double part[REWARD_T / 64][2], earlier[REWARD_T / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t j = (int64_t)blockIdx.x * REWARD_T + tid;
    const bool live = j < A.M;
    const double raw = live ? raw_reward(A, j) : 0.0;
    if (!A.normalise) {                                              // uniform
        if (live) A.out[j] = (float)raw;
        return;
    }
    double s = 0.0, q = 0.0;                                         // sums of the blocks before this one
    for (int64_t k = tid; k < (int64_t)blockIdx.x; k += REWARD_T) {
        s += A.sums[REWARD_HEAD + 2 * k];
        q += A.sums[REWARD_HEAD + 2 * k + 1];
    }
    s = wave_total_d(s);
    q = wave_total_d(q);
    if (lane == 0) { earlier[wave][0] = s; earlier[wave][1] = q; }
    double bs, bq, as, aq;
    block_prefix2<REWARD_T / 64>(part, wave, lane, raw, raw * raw, bs, bq, as, aq);       // (has a barrier)
    const double n0 = A.sums[0];
    const double s0 = A.sums[1] + ((earlier[0][0] + earlier[1][0]) + (earlier[2][0] + earlier[3][0]));
    const double q0 = A.sums[2] + ((earlier[0][1] + earlier[1][1]) + (earlier[2][1] + earlier[3][1]));
    if (live) A.out[j] = (float)normalised_reward(A, raw, n0 + (double)j, s0 + bs, q0 + bq);
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        A.state[0] = n0 + (double)A.M;
        A.state[1] = s0 + as;
        A.state[2] = q0 + aq;
    }
}

}  // namespace evk
