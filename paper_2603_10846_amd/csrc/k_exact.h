// Exhaustive selection (mem_retrieve_exact): the pool from similarities accumulated in fp64, whatever the
// bank holds.
//
// The bank is read once per group of up to EXACT_NB queries, in the passes of the ordinary plan: the sparsest
// pass keeps every row, each denser one the rows whose key -- the fp64 similarity rounded to fp32, lower ids
// first among equals -- reaches the query's cut, and after every pass the list is cut back to the k1 best
// keys plus those within two fp32 roundings of the k1-th (or, if that band is crowded, to exactly the k1
// best).  The top-k1 of a union is the top-k1 of the parts' top-k1, so after the last pass the list holds the
// pool.  There is no error margin in a cut, and ties break by id as in the pool itself, so masses of equal
// rows pass a cut no more often than distinct rows do.  A list can still overflow when a pass meets thousands of
// rows that beat everything in the sparser passes (the bank's order decides); such a query is lost, takes
// part in no further pass, and walks the whole bank by itself afterwards (k_exact_walk), range by range with
// lists that cannot overflow.
//
// Four queries over 1M x 1024 bf16 entries: 4.37 ms when every query read the bank for itself in ranges of 7,680
// entries (411 launches), 0.49 ms now, of which the last pass is 0.38 ms for 2.0 GB: bound by fp64 multiply-adds and
// conversions as much as by HBM (fetching two steps ahead instead of one changed nothing).
#pragma once
#include "k_ingest.h"
#include "k_select.h"

namespace evk {

constexpr int EXACT_NB = 8;               // queries per bank read, at most
constexpr int EXACT_ROWS = 64;            // rows a workgroup scores at a time: 16 lanes per row, 4 rows per lane group
constexpr int EXACT_WALK_PARTS = 64;      // workgroups of a lost query, at most

// Per-query words of the exhaustive selection, in the space of the query's fp64 similarities (which are
// written only after the selection): the cut, and the number of workgroups that have walked their part.
__device__ __forceinline__ uint64_t* exact_words(double* exact, int b, int exact_stride) {
    return reinterpret_cast<uint64_t*>(exact + (int64_t)b * exact_stride);
}

// Products of four neighbouring rows r0 .. r0 + 3 of bank tile t with NB queries, accumulated in fp64 by a lane
// group of 16: a lane takes one 16-byte chunk of each row per step (its offset within a k-block is fixed, so a
// step only adds to pointers) and the queries' chunk is read from L2 and widened once for the four rows.
// NB + 1 multiply-adds per element, the last one for the row's squared norm.  Rows past the bank's end lie
// inside the last tile's storage; what they give is the caller's to drop.
template <int DT, int NB>
__device__ __forceinline__ void score_four_rows(const void* store_, const float* const (&qp)[NB], int64_t t, int r0, int sub, int nkb,
                                                double (&dot)[4][NB], double (&ssq)[4]) {
    constexpr int EPC = DT == 0 ? 4 : 8, R = 4;
    constexpr int64_t STEP = 4ll * BLOCK_ELEMS;     // bytes from a lane's chunk to its next: one k-block of fp32, two of 16 bits
    const int steps = DT == 0 ? nkb : (nkb - (sub >> 3) + 1) / 2;
    const unsigned char* xp[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t id = t * TILE_ROWS + r0 + i;
        if constexpr (DT == 0) xp[i] = reinterpret_cast<const unsigned char*>(static_cast<const float*>(store_) + off32(id, sub, nkb));
        else xp[i] = reinterpret_cast<const unsigned char*>(static_cast<const uint16_t*>(store_) + off16(id, sub & 7, nkb) + (sub >> 3) * BLOCK_ELEMS);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        ssq[i] = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) dot[i][j] = 0.0;
    }
    // Two steps' chunks are in flight ahead of the one being used.  Past the end the last chunk is requested
    // again and not used.
    auto fetch = [&](stream_u32x4 (&x)[R], int u) __attribute__((always_inline)) {
        const int64_t off = (u < steps ? u : steps - 1) * STEP;
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = stream_load16(xp[i] + off);
    };
    auto use = [&](const stream_u32x4 (&x)[R], int u) __attribute__((always_inline)) {
#pragma unroll
        for (int e0 = 0; e0 < EPC; e0 += 4) {
            float4 y[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) y[j] = *reinterpret_cast<const float4*>(qp[j] + u * 16 * EPC + e0);
#pragma unroll
            for (int e1 = 0; e1 < 4; ++e1) {
                const int e = e0 + e1;
                double yd[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) yd[j] = e1 == 0 ? y[j].x : e1 == 1 ? y[j].y : e1 == 2 ? y[j].z : y[j].w;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    double xd;
                    if constexpr (DT == 0) xd = __uint_as_float(x[i][e]);
                    else {
                        const uint16_t h = (uint16_t)(x[i][e >> 1] >> (16 * (e & 1)));
                        xd = DT == 1 ? bf16_to_f(h) : f16_to_f(h);
                    }
                    ssq[i] += xd * xd;
#pragma unroll
                    for (int j = 0; j < NB; ++j) dot[i][j] += xd * yd[j];
                }
            }
        }
    };
    if (steps > 0) {                                // (with one 16-bit k-block the upper lanes have no chunk)
        stream_u32x4 xa[R], xb[R], x[R];
        fetch(xa, 0);
        fetch(xb, 1);
        for (int u = 0; u < steps; u += 2) {
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = xa[i];
            fetch(xa, u + 2);
            use(x, u);
            if (u + 1 < steps) {
#pragma unroll
                for (int i = 0; i < R; ++i) x[i] = xb[i];
                fetch(xb, u + 3);
                use(x, u + 1);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        ssq[i] = row16_sum(ssq[i]);
#pragma unroll
        for (int j = 0; j < NB; ++j) dot[i][j] = row16_sum(dot[i][j]);
    }
}

// One pass.  Blocks of the query groups that share rows are neighbours on one XCD, so all but the first find
// them in L2.
template <int DT, int NB>
__global__ __launch_bounds__(256, NB > 4 ? 2 : 3) void k_exact_scan(const void* __restrict__ store_, const float* __restrict__ qf,
                                                    const double* __restrict__ invq64, uint64_t* __restrict__ surv,
                                                    uint32_t* __restrict__ cnt, double* __restrict__ exact, int exact_stride,
                                                    int64_t N, int nkb, int B, int groups, Level L) {
    constexpr int R = 4;
    const int sub = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int q0 = (slot % groups) * NB;
    const int64_t units = (int64_t)L.ntiles * (TILE_ROWS / EXACT_ROWS), walkers = (gridDim.x >> 3) / groups * 8;
    const float* qp[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) qp[j] = qf + (int64_t)(q0 + j < B ? q0 + j : B - 1) * (nkb * KB) + sub * (DT == 0 ? 4 : 8);
    for (int64_t unit = (int64_t)(slot / groups) * 8 + xcd; unit < units; unit += walkers) {
        const int tile_j = (int)(unit / (TILE_ROWS / EXACT_ROWS));
        const int r0 = (int)(unit % (TILE_ROWS / EXACT_ROWS)) * EXACT_ROWS + grp * R;
        const int64_t t = level_tile(L, tile_j);
        double dot[R][NB], ssq[R];
        score_four_rows<DT, NB>(store_, qp, t, r0, sub, nkb, dot, ssq);
        // lane p of a group finishes pair (row p % R, query p / R), and p + 16 after it
#pragma unroll
        for (int p0 = 0; p0 < R * NB; p0 += 16) {
            const int p = p0 + sub, i = p % R, j = p / R, b = q0 + j;
            double dv = 0.0, sv = ssq[0];
#pragma unroll
            for (int k = 1; k < R; ++k) sv = i == k ? ssq[k] : sv;
#pragma unroll
            for (int k = 0; k < 16 && p0 + k < R * NB; ++k) dv = sub == k ? dot[(p0 + k) % R][(p0 + k) / R] : dv;
            const int64_t id = t * TILE_ROWS + r0 + i;
            if (p >= R * NB || b >= B || id >= N) continue;
            const uint64_t key = exact_key(dv * invq64[b] * (1.0 / sqrt(sv)), (int32_t)id);
            uint64_t* list = surv + (int64_t)b * SURV_CAP;
            if (L.rho == 0) {                       // sparsest pass: every row, at its own position
                list[tile_j * TILE_ROWS + r0 + i] = key;
            } else if (key >= exact_words(exact, b, exact_stride)[0]) {
                const uint32_t pos = atomicAdd(slot_counter(cnt, b), 1u);
                if (pos < (uint32_t)SURV_CAP) list[pos] = key;
            }
        }
    }
}

// Between two passes: the list cut back, the cut of the next pass.  (After the last one the tail selects.)
__global__ __launch_bounds__(1024) void k_exact_select(uint64_t* __restrict__ surv, uint32_t* __restrict__ cnt, double* __restrict__ exact,
                                                       int exact_stride, int k1, int keep_max) {
    __shared__ SelectLds sh;
    const int b = (int)blockIdx.x, tid = threadIdx.x;
    uint64_t* list = surv + (int64_t)b * SURV_CAP;
    uint64_t* words = exact_words(exact, b, exact_stride);
    Selected s;
    const uint32_t raw = select_keys(list, slot_counter(cnt, b), k1, EXACT_KEY_MARGIN, false, keep_max, SEL_EXACT, sh, s);
    if (raw > (uint32_t)SURV_CAP) {                 // lost: no key reaches this cut, so the count stays as it is
        if (tid == 0) words[0] = ~0ull;
        return;
    }
    store_kept(s, list);
    if (tid == 0) { *slot_counter(cnt, b) = s.kept; words[0] = s.cut; words[1] = 0ull; }
}

// The lost queries: gridDim.y workgroups each walk a part of the bank, a tile at a time, with a list in LDS of
// the rows that reach the part's own cut; when the list has no room for another tile it is sorted and cut back
// as a pass's list is, which gives the next cut.  Each leaves its best in a share of the query's survivor slots (at
// least keep_of(k1) of them) and the last one to finish selects from the shares.  Queries that are not lost leave at
// once.  Over the 1M x 1024 bank one such query takes 1.5 ms on top of the passes and 64 of them 33 ms, fp64
// arithmetic being the bound (4.5 and 23 ms in all by ranges of 7,680 entries, which every query had to walk).
constexpr int WALK_CAP = 4096;
static_assert(keep_of(BIG_K1_MAX) <= WALK_CAP - TILE_ROWS, "a list that was cut back has room for a tile");
template <int DT>
__global__ __launch_bounds__(1024) void k_exact_walk(const void* __restrict__ store_, const float* __restrict__ qf,
                                                     const double* __restrict__ invq64, uint64_t* __restrict__ surv,
                                                     uint32_t* __restrict__ cnt, double* __restrict__ exact, int exact_stride,
                                                     int64_t N, int nkb, int k1, int keep_max) {
    const int b = (int)blockIdx.x, part = (int)blockIdx.y, parts = (int)gridDim.y, tid = threadIdx.x;
    if (*slot_counter(cnt, b) <= (uint32_t)SURV_CAP) return;       // uniform over the query's workgroups: written only below, by the last of them
    __shared__ uint64_t keys[WALK_CAP];
    __shared__ uint32_t n_s, last_s;
    __shared__ SelectLds sh;
    const int share = SURV_CAP / parts, sub = tid & 15, r0 = (tid >> 4) * 4;
    const int64_t tiles = (N + TILE_ROWS - 1) / TILE_ROWS, first = tiles * part / parts, end = tiles * (part + 1) / parts;
    const float* const qp[1] = {qf + (int64_t)b * nkb * KB + sub * (DT == 0 ? 4 : 8)};
    uint64_t* list = surv + (int64_t)b * SURV_CAP;
    uint64_t cut = 0ull;
    if (tid == 0) n_s = 0;
    __syncthreads();
    for (int64_t t = first; t < end; ++t) {
        double dot[4][1], ssq[4];
        score_four_rows<DT, 1>(store_, qp, t, r0, sub, nkb, dot, ssq);
        if (sub < 4) {
            const double dv = sub == 0 ? dot[0][0] : sub == 1 ? dot[1][0] : sub == 2 ? dot[2][0] : dot[3][0];
            const double sv = sub == 0 ? ssq[0] : sub == 1 ? ssq[1] : sub == 2 ? ssq[2] : ssq[3];
            const int64_t id = t * TILE_ROWS + r0 + sub;
            const uint64_t key = exact_key(dv * invq64[b] * (1.0 / sqrt(sv)), (int32_t)id);
            if (id < N && key >= cut) keys[atomicAdd(&n_s, 1u)] = key;      // there is room for a whole tile
        }
        __syncthreads();
        const int n = (int)n_s;
        __syncthreads();                            // every lane has read it
        if (n > WALK_CAP - TILE_ROWS || t + 1 == end) {       // uniform
            for (int i = n + tid; i < WALK_CAP; i += 1024) keys[i] = 0ull;       // sorts last
            if (tid == 0) n_s = (uint32_t)(n < k1 ? n : k1);
            __syncthreads();
            bitonic_desc(keys, WALK_CAP, tid, 1024, [](uint64_t x, uint64_t y) { return x < y; });
            if (n >= k1) {                          // as between two passes: the k1 best and what lies within two fp32 roundings of the k1-th,
                cut = keys[k1 - 1];                 // or exactly the k1 best when that is more than keep_max
                const uint64_t band = (uint64_t)f2ord(key_sim(cut) - EXACT_KEY_MARGIN) << 32;
                if (keys[keep_max] < band) {        // uniform
                    cut = band;
                    for (int i = k1 + tid; i <= keep_max; i += 1024)
                        if (keys[i] < band && keys[i - 1] >= band) n_s = (uint32_t)i;
                }
            }
        }
    }
    __syncthreads();
    const int have = (int)n_s;
    for (int i = tid; i < share; i += 1024) list[part * share + i] = i < have ? keys[i] : 0ull;
    __threadfence();
    __syncthreads();
    uint64_t* words = exact_words(exact, b, exact_stride);
    if (tid == 0) last_s = atomicAdd(reinterpret_cast<uint32_t*>(words + 1), 1u) == (uint32_t)parts - 1u;
    __syncthreads();
    if (!last_s) return;                            // uniform
    __threadfence();
    Selected s;
    if (tid == 0) last_s = SURV_CAP;
    __syncthreads();
    select_keys(list, &last_s, k1, EXACT_KEY_MARGIN, true, keep_max, SEL_EXACT, sh, s);
    store_kept(s, list);
    if (tid == 0) *slot_counter(cnt, b) = s.kept;
}

}  // namespace evk
