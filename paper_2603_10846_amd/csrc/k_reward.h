// Rewards of the two stages and their online normalisation, computed on the device so that a batch
// of verifier outcomes can go straight into the value update.
//   Stage 1 (Sec. 3.3): +1 if the candidate is feasible, -1 otherwise.
//   Stage 2 (Sec. 3.4): -1 if infeasible, else tanh(log b - log l), b the best latency so far, l the
//   measured one (App. A: tanh(log rho), rho the speed-up ratio).
//   Normalisation (Sec. 3.4, App. A "Stability of Online Normalization"): sample t becomes
//   (r_t - mu_{t-1}) / max(sigma_{t-1}, sigma_min), optionally clipped, with mu, sigma the running
//   mean and population deviation of the raw rewards BEFORE it; the statistics (count, sum, sum of
//   squares, fp64) persist in the handle's workspace.
// The dependence of sample t on all earlier ones is a prefix sum.  A batch of little more than one workgroup's size is one
// launch; a longer one is two: the first leaves every block's sums of (r, r^2), in the second a block adds
// the sums of the blocks before it and scans its own samples.  The raw rewards are computed in both -- two fp64
// logarithms and a tanh per sample are what bounds the kernel, and one workgroup walking the batch in
// pieces of 1024 did them on one compute unit: 8192 samples 45.3 us, 3.3 + 4.2 us in two launches.
// All arithmetic in fp64; outputs fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "k_ingest.h"

namespace evk {

constexpr int REWARD_ONE = 1024;          // samples per piece of the one-launch form
// Largest batch of the one-launch form.  A second launch costs the host about 3.5 us, a second piece what its samples cost
// (one launch / two, us a call): stage 1, 1025 samples 10.1 / 11.5, 1536 11.0 / 11.7, 2000 12.8 / 11.5; stage 0 (no logarithms), 1025
// 8.9 / 12.0, 3000 10.7 / 11.8, 4096 13.2 / 12.1; unnormalised rewards of a longer batch need one launch over all blocks in any case.
__host__ constexpr int64_t reward_one_launch(int stage, int normalise) { return !normalise ? REWARD_ONE : stage == 0 ? 3 * REWARD_ONE : REWARD_ONE + REWARD_ONE / 2; }
constexpr int REWARD_T = 256;             // samples per block of the two-launch form
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
    double* sums;             // two-launch form: the statistics before the batch, then two sums per block
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

// One workgroup walks the batch in pieces of 1024 samples.
__global__ __launch_bounds__(REWARD_ONE) void k_shape_rewards(RewardArgs A) {
    __shared__ double part[2][REWARD_ONE / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double n0 = 0.0, s0 = 0.0, q0 = 0.0;                             // the statistics before the piece
    if (A.normalise) { n0 = A.state[0]; s0 = A.state[1]; q0 = A.state[2]; }
    for (int64_t base = 0; base < A.M; base += REWARD_ONE) {
        const int64_t j = base + tid;
        const bool live = j < A.M;
        const double raw = live ? raw_reward(A, j) : 0.0;
        if (!A.normalise) {                                          // uniform
            if (live) A.out[j] = (float)raw;
            continue;
        }
        double bs, bq, as, aq;
        block_prefix2<REWARD_ONE / 64>(part[(base / REWARD_ONE) & 1], wave, lane, raw, raw * raw, bs, bq, as, aq);    // (has a barrier)
        if (live) A.out[j] = (float)normalised_reward(A, raw, n0 + tid, s0 + bs, q0 + bq);
        n0 += (double)(A.M - base < REWARD_ONE ? A.M - base : REWARD_ONE);
        s0 += as;
        q0 += aq;
    }
    if (A.normalise && tid == 0) { A.state[0] = n0; A.state[1] = s0; A.state[2] = q0; }
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
