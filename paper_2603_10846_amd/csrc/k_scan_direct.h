// Similarity scan of a sparse pass (Sec. 3.2, dense recall): few bank tiles, so latency is what counts.
//
// The matrix-core scan of k_scan_mfma.h walks a tile's k-blocks one after another in one workgroup, about 1 us per
// block however few tiles there are: a pass over 32 tiles leaves most compute units idle and takes as long as one
// tile does.  Here a workgroup takes 16 MR bank rows and 16 MQ queries and its eight wavefronts share the k
// dimension: each forms the products of its own eighth with v_mfma_f32_16x16x32, operands loaded straight from
// global memory into registers (both are stored in operand order: a lane's 16 bytes are 8 consecutive elements of
// its row), several steps' loads in flight, no barrier and no LDS until the partial sums are added once at the end.
// What bounds it: two memory latencies and, with many queries or long rows, the operands a compute unit takes in
// (20 to 30 GB/s).  First pass over 8192 rows, by tiles and so: one query, d = 1024 bf16 17.2 -> 5.6 us; 64 queries
// 20.5 -> 9.4; 64 queries, d = 1024 fp32 33.6 -> 14.8; 32 queries, d = 384 fp16 13.4 -> 4.9.  With up to 16 queries that pass
// prepares them as well (seven queries, 7680 x 200 fp16: 4.2 + 4.0 us in two launches, 4.3 in one).
#pragma once
#include "k_scan_mfma.h"
#include "layout.h"

namespace evk {

constexpr int DIRECT_WAVES = 8;
// Partial sums [wavefront][query][row]; four spare floats per row of queries put the four lane groups of an
// accumulator's store (queries 4 apart) on different banks.
// FIRST: the wavefronts' sums of the queries' squares (fp64) behind them.
template <int MQ, int MR, bool FIRST = false> constexpr int direct_lds_bytes() { return DIRECT_WAVES * 16 * MQ * (16 * MR + 4 + (FIRST ? 2 : 0)) * 4; }

// FIRST: the sparsest pass, with the queries as given (fp32 rows at a multiple of 16 bytes): a lane rounds and splits what it
// needs of them, and adds up its part of their squares; the workgroups behind the scan's prepare the queries for the launches after
// this one.
template <int DT, int MQ, int MR, bool FIRST>
__global__ __launch_bounds__(64 * DIRECT_WAVES) void k_scan_direct(const void* __restrict__ store_, const float* __restrict__ invnorm,
                                                                   const uint16_t* __restrict__ qop, const float* __restrict__ invq,
                                                                   const float* __restrict__ thr, uint32_t* __restrict__ cnt,
                                                                   uint64_t* __restrict__ surv, int64_t N, int nkb, int Bp, int nqt,
                                                                   Level L, Mask mask, int B, PrepArgs prep) {
    static_assert(!FIRST || MQ == 1, "few queries");
    static_assert(MR == 2 || MR == 4, "32 or 64 rows: a wavefront finishes two queries or one at a time");
    constexpr int TQ = 16 * MQ, TR = 16 * MR, TRP = TR + 4, W = DIRECT_WAVES;
    constexpr int DEPTH = DT == 0 ? 2 : 4;                // steps whose loads are in flight together
    extern __shared__ __align__(16) float direct_part[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, grp = lane >> 4;
    if constexpr (FIRST) {
        const int nscan = 8 * ((L.ntiles * (TILE_ROWS / TR) + 7) / 8) * nqt;
        if ((int)blockIdx.x >= nscan) {                   // uniform
            prep_query<DT, 64 * W>(prep, (int)blockIdx.x - nscan, reinterpret_cast<double*>(direct_part));
            return;
        }
    }
    // The query tiles that share rows are neighbours on one XCD: all but the first find the rows in its L2.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int q0 = (slot % nqt) * TQ;
    const int unit = (slot / nqt) * 8 + xcd;
    if (unit >= L.ntiles * (TILE_ROWS / TR)) return;      // uniform
    const int tile_j = unit / (TILE_ROWS / TR), r0 = unit % (TILE_ROWS / TR) * TR;
    const int64_t t = level_tile(L, tile_j);

    // ---- this wavefront's share of the k dimension, in steps of 32 elements ----
    const int steps = 2 * nkb, s0 = steps * wave / W, s1 = steps * (wave + 1) / W;
    f32x4_t acc[MQ][MR];
#pragma unroll
    for (int a = 0; a < MQ; ++a)
#pragma unroll
        for (int b = 0; b < MR; ++b) acc[a][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // rows 16 apart have the same swizzle, and so have the two halves of a k-block up to one bit
    const int lane16 = l16 * KB + swz16(grp, l16) * 8;    // a lane's offset in 16 rows of 16-bit elements, first half
    const int row_elem = (r0 + l16) * KB + grp * 8;       // fp32 stores
    double qsq[MQ];                                       // (in fp64: a query's squares need not fit a float)
    const float* qrow[MQ];
    if constexpr (FIRST) {
#pragma unroll
        for (int a = 0; a < MQ; ++a) {
            const int q = q0 + a * 16 + l16;
            qsq[a] = 0.0;
            qrow[a] = prep.q + (int64_t)(q < B ? q : B - 1) * prep.d;    // (a query past the end: computed, not kept)
        }
    }
    for (int s = s0; s < s1; s += DEPTH) {                // uniform within the wavefront
        u32x4_t x[DEPTH][MR][DT == 0 ? 2 : 1], y[DEPTH][MQ][DT == 0 || FIRST ? 2 : 1];
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int su = s + u < s1 ? s + u : s1 - 1, kb = su >> 1, h = su & 1;   // (past the end: loaded, not used)
            if constexpr (DT == 0) {
                const float* blk = static_cast<const float*>(store_) + (t * nkb + kb) * (int64_t)BLOCK_ELEMS + row_elem + h * 32;
#pragma unroll
                for (int b = 0; b < MR; ++b)
#pragma unroll
                    for (int i = 0; i < 2; ++i) x[u][b][i] = *reinterpret_cast<const u32x4_t*>(blk + b * 16 * KB + i * 4);
#pragma unroll
                for (int a = 0; a < MQ && !FIRST; ++a)
#pragma unroll
                    for (int i = 0; i < 2; ++i) y[u][a][i] = *reinterpret_cast<const u32x4_t*>(qop + qop_row(2 * su + i, Bp) + (q0 + a * 16) * 32 + lane * 8);
            } else {
                const uint16_t* blk = static_cast<const uint16_t*>(store_) + (t * nkb + kb) * (int64_t)BLOCK_ELEMS + r0 * KB;
#pragma unroll
                for (int b = 0; b < MR; ++b) x[u][b][0] = *reinterpret_cast<const u32x4_t*>(blk + b * 16 * KB + (lane16 ^ (h * 32)));
#pragma unroll
                for (int a = 0; a < MQ && !FIRST; ++a) y[u][a][0] = *reinterpret_cast<const u32x4_t*>(qop + qop_row(su, Bp) + (q0 + a * 16) * 32 + lane * 8);
            }
            if constexpr (FIRST) {
                const int e = su * 32 + grp * 8;
#pragma unroll
                for (int a = 0; a < MQ; ++a)
#pragma unroll
                    for (int i = 0; i < 2; ++i) y[u][a][i] = *reinterpret_cast<const u32x4_t*>(qrow[a] + (e < prep.d ? e + i * 4 : 0));
            }
        }
        __builtin_amdgcn_sched_barrier(0);                // all of them requested before the first is used
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (s + u >= s1) break;                       // uniform
            if constexpr (FIRST) {                        // eight fp32 elements -> operands, as k_prep_queries makes them
                const bool in = (s + u) * 32 + grp * 8 < prep.d;
#pragma unroll
                for (int a = 0; a < MQ; ++a) {
                    u32x4_t hi, lo;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const u32x4_t v = y[u][a][i >> 1];
                        const float f0 = in ? __uint_as_float(v[(i & 1) * 2]) : 0.f, f1 = in ? __uint_as_float(v[(i & 1) * 2 + 1]) : 0.f;
                        if constexpr (DT == 0) {
                            float ra, rb;
                            hi[i] = pack_bf16x2_hi(f0, f1, ra, rb);
                            lo[i] = cvt_pk_bf16(ra, rb);
                            const double g0 = f0, g1 = f1;
                            qsq[a] += g0 * g0 + g1 * g1;
                        } else {
                            hi[i] = DT == 1 ? cvt_pk_bf16(f0, f1) : (f2f16_rne(f0) | ((uint32_t)f2f16_rne(f1) << 16));
                            const uint16_t h0 = (uint16_t)hi[i], h1 = (uint16_t)(hi[i] >> 16);
                            const double g0 = DT == 1 ? bf16_to_f(h0) : f16_to_f(h0), g1 = DT == 1 ? bf16_to_f(h1) : f16_to_f(h1);
                            qsq[a] += g0 * g0 + g1 * g1;
                        }
                    }
                    y[u][a][0] = hi;
                    if constexpr (DT == 0) y[u][a][1] = lo;
                }
            }
            if constexpr (DT == 0) {
                // bf16 hi + lo of the rows (the queries are stored split): hi*hi + hi*lo + lo*hi
#pragma unroll
                for (int b = 0; b < MR; ++b) {
                    u32x4_t hi, lo;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const u32x4_t v = x[u][b][i >> 1];
                        float ra, rb;
                        hi[i] = pack_bf16x2_hi(__uint_as_float(v[(i & 1) * 2]), __uint_as_float(v[(i & 1) * 2 + 1]), ra, rb);
                        lo[i] = cvt_pk_bf16(ra, rb);
                    }
#pragma unroll
                    for (int a = 0; a < MQ; ++a) {
                        acc[a][b] = mfma16<1>(y[u][a][1], hi, acc[a][b]);
                        acc[a][b] = mfma16<1>(y[u][a][0], lo, acc[a][b]);
                        acc[a][b] = mfma16<1>(y[u][a][0], hi, acc[a][b]);
                    }
                }
            } else {
#pragma unroll
                for (int a = 0; a < MQ; ++a)
#pragma unroll
                    for (int b = 0; b < MR; ++b) acc[a][b] = mfma16<DT>(y[u][a][0], x[u][b][0], acc[a][b]);
            }
        }
    }
    // ---- the eight partial sums; then a wavefront finishes 64 / TR queries at a time, a lane per row ----
    // (queries are the accumulator's rows, 4 grp + register; bank rows its columns, l16)
#pragma unroll
    for (int a = 0; a < MQ; ++a)
#pragma unroll
        for (int b = 0; b < MR; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) direct_part[(wave * TQ + a * 16 + 4 * grp + r) * TRP + b * 16 + l16] = acc[a][b][r];
    double* qsq_part = reinterpret_cast<double*>(direct_part + W * TQ * TRP);             // [wavefront][query]
    if constexpr (FIRST) {
#pragma unroll
        for (int a = 0; a < MQ; ++a) {
            double v = qsq[a];
            v += __shfl_xor(v, 16, 64); v += __shfl_xor(v, 32, 64);
            if (grp == 0) qsq_part[wave * TQ + a * 16 + l16] = v;
        }
    }
    constexpr int QL = 64 / TR, ITER = (TQ + W * QL - 1) / (W * QL);
    const int row = lane % TR, ql = lane / TR;
    const int64_t id = t * TILE_ROWS + r0 + row;
    const float inve = id < N ? invnorm[id] : 0.f;
    const uint32_t tag = mask.tags && id < N ? mask.tags[id] : 0u;
    float v[ITER], th[ITER], inq[ITER];
    bool keep[ITER], ok[ITER];
    uint32_t base[ITER];
#pragma unroll
    for (int i = 0; i < ITER; ++i) {                      // (requested before the barrier)
        const int qi = (i * W + wave) * QL + ql, q = q0 + qi;
        keep[i] = qi < TQ && q < B && id < N;
        th[i] = FIRST ? 0.f : thr[keep[i] ? q : 0];
        inq[i] = FIRST ? 0.f : invq[keep[i] ? q : 0];
        ok[i] = keep[i] && (!mask.tags || eligible(tag, mask.allow[q], mask.exclude[q]));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
        const int qi = (i * W + wave) * QL + ql, q = q0 + qi;
        v[i] = 0.f;
        if (qi < TQ) {
#pragma unroll
            for (int w = 0; w < W; ++w) v[i] += direct_part[(w * TQ + qi) * TRP + row];
        }
        v[i] *= inve;
        if constexpr (FIRST) {
            double qs = 0.0;
            if (qi < TQ) {
#pragma unroll
                for (int w = 0; w < W; ++w) qs += qsq_part[w * TQ + qi];
            }
            inq[i] = (float)rsqrt_d(qs);
        }
        if (FIRST || L.rho == 0) {
            // sparsest pass: every row is kept, at its own position (0 = empty slot)
            if (keep[i])
                surv[(int64_t)q * L.cap + (int64_t)tile_j * TILE_ROWS + r0 + row] = ok[i] ? pack_key(v[i] * inq[i], (int32_t)id) : 0ull;
        } else {
            keep[i] = ok[i] && v[i] >= th[i];
            const uint64_t m = __builtin_amdgcn_ballot_w64(keep[i]);
            const uint32_t c = QL == 1 ? (uint32_t)__popcll(m) : (uint32_t)__popc((uint32_t)(m >> (32 * ql)));
            base[i] = 0;
            if (row == 0 && c != 0) base[i] = atomicAdd(slot_counter(cnt, q), c);
        }
    }
    if (FIRST || L.rho == 0) return;
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
        const int q = q0 + (i * W + wave) * QL + ql;
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep[i]);
        if (m == 0) continue;                             // uniform within the wavefront
        const uint64_t below = (m >> (TR * ql)) & ((1ull << row) - 1ull);
        const uint32_t pos = (uint32_t)__shfl((int)base[i], TR * ql, 64) + (uint32_t)__popcll(below);
        if (keep[i] && pos < (uint32_t)L.cap) surv[(int64_t)q * L.cap + pos] = pack_key(v[i] * inq[i], (int32_t)id);
    }
}

}  // namespace evk
