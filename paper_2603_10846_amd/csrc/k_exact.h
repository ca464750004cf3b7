// Exhaustive selection (mem_retrieve_exact): the pool from similarities accumulated in fp64, whatever the
// bank holds.
//
// The bank is read once per group of up to EXACT_NB queries (32 in a pass on the matrix cores), in the passes of the ordinary plan: the sparsest
// pass keeps every row, each denser one the rows whose key -- the fp64 similarity rounded to fp32, lower ids
// first among equals -- reaches the query's cut, and after every pass the list is cut back to the k1 best
// keys plus those within two fp32 roundings of the k1-th (or, if that band is crowded, to exactly the k1
// best).  The top-k1 of a union is the top-k1 of the parts' top-k1, so after the last pass the list holds the
// pool.  There is no error margin in a cut, and ties break by id as in the pool itself, so masses of equal
// rows pass a cut no more often than distinct rows do.  A list can still overflow when a pass meets thousands of
// rows that beat everything in the sparser passes (the bank's order decides); such a query is lost, takes
// part in no further pass, and walks the whole bank afterwards (k_exact_walk), with lists that cannot overflow.
//
// Scoring every row of a denser pass in fp64 is bound by multiply-adds and conversions as much as by HBM (1M x 1024 bf16, four
// queries, last pass: 0.41 ms for 2.0 GB, one query 0.33; fetching two steps ahead instead of one changed nothing) and costs by the
// query.  Where it pays (use_exact_mfma in evomem.hip), such a pass runs on the matrix cores instead: their scan, with a
// threshold below the query's cut by the margin of its rounding, finds the rows that may reach the cut, and only those are scored in
// fp64, so lists and cuts are the same.  Whole call with 4 and 16 queries: 485 -> 386 us, 1245 -> 415 us.  The masses of near-ties inside
// the margin are scored too, 100,000 of them in 585 and 1260 us (526 and 1262 with every row scored); where most of them lie in a few tiles
// the workgroups that have those score alone (20,000 in a run: 550 and 1528, 510 and 1239).
#pragma once
#include "k_ingest.h"
#include "k_select.h"

namespace evk {

constexpr int EXACT_NB = 8;               // queries per bank read, at most
constexpr int EXACT_ROWS = 64;            // rows a workgroup scores at a time: 16 lanes per row, 4 rows per lane group

// Per-query words of the exhaustive selection, in the space of the query's fp64 similarities (which are
// written only after the selection): the cut, and the number of parts of the bank that have been walked.
__device__ __forceinline__ uint64_t* exact_words(double* exact, int b, int exact_stride) {
    return reinterpret_cast<uint64_t*>(exact + (int64_t)b * exact_stride);
}

// What a denser pass on the matrix cores needs besides an ordinary one (k_scan_mfma with EXACT).
struct ExactPass {
    const float* qf;
    const double* invq64;
    double* words;            // see exact_words
    int stride;
    int most_rows;            // of a query that a workgroup scores, once it scores many
};

// Norms of rows and queries that the matrix cores' filter is good for: its thresholds are pairs of bf16, which have fp32's range and 2^-16
// of precision; products of norms are kept from the ends.  All norms that fp16 rows can have fit; zero, infinity and NaN do not.
// (2^-50 .. 2^50, so an inverse norm may be asked about as well.)
__device__ __forceinline__ bool exact_norm_fits(float norm) {
    return __float_as_uint(norm) - __float_as_uint(0x1p-50f) <= __float_as_uint(0x1p50f) - __float_as_uint(0x1p-50f);
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
// margin: of the threshold for a pass on the matrix cores; 0 if there is none ahead.  A query that such a pass cannot filter for is lost to
// it: its norm does not fit, or its cut lies at the rows without a norm.
// A query without a norm has no similarity to any row: its pool are the first rows of the bank, and no pass has to look for them.
__global__ __launch_bounds__(1024) void k_exact_select(uint64_t* __restrict__ surv, uint32_t* __restrict__ cnt, double* __restrict__ exact,
                                                       int exact_stride, int k1, int keep_max, float* __restrict__ thr,
                                                       const float* __restrict__ invq, const double* __restrict__ invq64, float margin) {
    __shared__ SelectLds sh;
    const int b = (int)blockIdx.x, tid = threadIdx.x;
    uint64_t* list = surv + (int64_t)b * SURV_CAP;
    uint64_t* words = exact_words(exact, b, exact_stride);
    const double inv64 = invq64[b];                 // (asked for with the list)
    Selected<SURV_CAP / 1024> s;
    const bool normed = inv64 > 0.0 && inv64 < (double)INFINITY;           // uniform
    const uint32_t found = *slot_counter(cnt, b);
    const uint32_t raw = select_keys(list, slot_counter(cnt, b), k1, EXACT_KEY_MARGIN, false, keep_max, SEL_EXACT, false, sh, s,
                                     [&](int i, uint32_t at) __attribute__((always_inline)) { if (normed && found <= (uint32_t)SURV_CAP) list[at] = s.key[i]; });
    if (!normed) {
        for (int i = tid; i < k1; i += 1024) list[i] = pack_key(-INFINITY, i);  // (with more than one pass the bank holds more rows than a pool)
        if (tid == 0) { *slot_counter(cnt, b) = (uint32_t)k1; words[0] = ~0ull; words[1] = 0ull; }
        return;
    }
    if (raw > (uint32_t)SURV_CAP) {                 // lost: no key reaches this cut, so the count stays as it is
        if (tid == 0) words[0] = ~0ull;
        return;
    }
    if (tid == 0) {
        const bool filtered = exact_norm_fits(invq[b]) && key_sim(s.cut) >= -1.5f;
        *slot_counter(cnt, b) = margin > 0.f && !filtered ? (uint32_t)SURV_CAP + 1u : s.kept;
        words[0] = s.cut;
        words[1] = 0ull;
        thr[b] = (key_sim(s.cut) - margin) / invq[b];
    }
}

// The lost queries walk the bank together, WALK_NB to a group (one at a time while there are only one or two): a
// workgroup scores a part of the bank for its group, with a list in LDS per query of the rows that reach the query's
// cut in this part.  A list without room for another step is sorted and cut back as a pass's list is, which gives the
// next cut.  Each part leaves what it has (at most keep_of(k1) keys) in its share of the survivor slots, and the last
// part of a group to finish merges the shares into the head of the queries' lists, zeros behind.  The counts stay
// as they are, above SURV_CAP, while any workgroup may still look for lost queries; the tail takes such a list as full,
// with empty slots.
// The shares lie in the survivor lists of the query slots that this call does not use, as long as those give a query
// more parts than its own list does: tied to its own 8192 slots a pool of 2048 was walked by four workgroups.
// 1M x 1024 bf16 bank, ms for the whole call: by ranges of 7,680 entries that every query walked; by workgroups of one
// query, 8192 / k1 of them at most; now.  One lost query of one, pool 64 4.0, 1.4, 0.88, pool 2048 5.4, 15.0, 1.1; four of
// four, pool 2048 5.9, 15.3, 1.6; 64 of 64, pool 64 23.2, 24.7, 8.1, pool 2048 24.5, 23.8, 15.9.  fp64 arithmetic is the bound.
constexpr int WALK_T = 512, WALK_ROWS = WALK_T / 4, WALK_NB = 4, WALK_CAP = 4096;
constexpr int WALK_GROUPS = 256;          // workgroups of the launch: one per compute unit
constexpr int WALK_LDS = WALK_NB * WALK_CAP * 8;
static_assert(keep_of(BIG_K1_MAX) <= WALK_CAP - WALK_T, "a list that was cut back has room for a step and for a load of the merge");

struct WalkLds {
    uint64_t cut[WALK_NB];
    uint32_t n[WALK_NB], wave_n[WALK_T / 64], last;
    uint16_t lost[MAX_BATCH];             // the lost queries
};

// Sorts a list of n keys and cuts it back: the k1 best and what lies within two fp32 roundings of the k1-th, or exactly
// the k1 best when that is more than keep_max.  All lanes call it, with the keys written before a barrier; ends with one.
__device__ __forceinline__ void walk_cut_back(uint64_t* keys, int n, int k1, int keep_max, uint32_t* n_out, uint64_t* cut_out) {
    const int tid = threadIdx.x;
    int cap = 2;
    while (cap < n) cap <<= 1;
    for (int i = n + tid; i < cap; i += WALK_T) keys[i] = 0ull;                    // sorts last
    __syncthreads();
    bitonic_desc(keys, cap, tid, WALK_T, [](uint64_t x, uint64_t y) { return x < y; });
    if (n < k1) return;                                                            // uniform, as all that follows
    const uint64_t pivot = keys[k1 - 1], band = (uint64_t)f2ord(key_sim(pivot) - EXACT_KEY_MARGIN) << 32;
    if (n <= keep_max || keys[keep_max] < band) {
        for (int i = k1 + tid; i <= (n < keep_max ? n : keep_max); i += WALK_T)
            if ((i == n || keys[i] < band) && keys[i - 1] >= band) { *n_out = (uint32_t)i; *cut_out = band; }
    } else if (tid == 0) {
        *n_out = (uint32_t)k1;
        *cut_out = pivot;
    }
    __syncthreads();
}

template <int DT, int NB>
__device__ __forceinline__ void walk_lost(const void* store_, const float* qf, const double* invq64, uint64_t* surv, double* exact,
                                          int exact_stride, int64_t N, int nkb, int k1, int B, int lists, int nlost, uint64_t* keys, WalkLds& sh) {
    constexpr int R = 4;
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4, keep = keep_of(k1);
    const int groups = (nlost + NB - 1) / NB;
    const int64_t tiles = (N + TILE_ROWS - 1) / TILE_ROWS, spare = (int64_t)(lists - B) * SURV_CAP / ((int64_t)nlost * keep);
    const bool own = spare <= SURV_CAP / keep;                // the shares in the query's own list
    int64_t parts = own ? SURV_CAP / keep : spare;
    if (parts > WALK_GROUPS / groups) parts = WALK_GROUPS / groups > 1 ? WALK_GROUPS / groups : 1;
    if (parts > tiles) parts = tiles;
    static_assert(WALK_GROUPS <= WALK_T, "a load of the merge sees every share");
    for (int64_t item = blockIdx.x; item < groups * parts; item += gridDim.x) {
        const int g = (int)(item / parts), part = (int)(item % parts);
        const int live = nlost - g * NB < NB ? nlost - g * NB : NB;                // queries of this group
        auto query = [&](int j) __attribute__((always_inline)) { return (int)sh.lost[g * NB + (j < live ? j : live - 1)]; };
        auto share_of = [&](int j) __attribute__((always_inline)) {
            return own ? surv + (int64_t)query(j) * SURV_CAP : surv + (int64_t)B * SURV_CAP + (int64_t)(g * NB + j) * parts * keep;
        };
        auto start = [&]() __attribute__((always_inline)) {                        // empty lists; a valid cut if a pass left one
            if (tid < NB) {
                const uint64_t c = exact_words(exact, query(tid), exact_stride)[0];
                sh.n[tid] = 0;
                sh.cut[tid] = c == ~0ull ? 0ull : c;
            }
            __syncthreads();
        };
        const float* qp[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) qp[j] = qf + (int64_t)query(j) * nkb * KB + sub * (DT == 0 ? 4 : 8);
        start();
        const int64_t first = tiles * part / parts * (TILE_ROWS / WALK_ROWS), end = tiles * (part + 1) / parts * (TILE_ROWS / WALK_ROWS);
        for (int64_t u = first; u < end; ++u) {
            const int64_t t = u / (TILE_ROWS / WALK_ROWS);
            const int r0 = (int)(u % (TILE_ROWS / WALK_ROWS)) * WALK_ROWS + grp * R;
            double dot[R][NB], ssq[R];
            score_four_rows<DT, NB>(store_, qp, t, r0, sub, nkb, dot, ssq);
            // lane p of a group of 16 finishes pair (row p % R, query p / R)
            double dv = 0.0, sv = ssq[0];
            const int i = sub % R, j = sub / R;
#pragma unroll
            for (int k = 1; k < R; ++k) sv = i == k ? ssq[k] : sv;
#pragma unroll
            for (int k = 0; k < R * NB; ++k) dv = sub == k ? dot[k % R][k / R] : dv;
            const int64_t id = t * TILE_ROWS + r0 + i;
            if (j < live && id < N) {
                const uint64_t key = exact_key(dv * invq64[query(j)] * (1.0 / sqrt(sv)), (int32_t)id);
                if (key >= sh.cut[j]) keys[j * WALK_CAP + atomicAdd(&sh.n[j], 1u)] = key;   // there is room for a whole step
            }
            __syncthreads();
            for (int l = 0; l < live; ++l) {                                       // uniform
                const int n = (int)sh.n[l];
                if (n > WALK_CAP - WALK_ROWS || u + 1 == end) walk_cut_back(keys + l * WALK_CAP, n, k1, keep, &sh.n[l], &sh.cut[l]);
            }
            __syncthreads();                                                       // every lane has read the counts
        }
        for (int l = 0; l < live; ++l) {
            uint64_t* share = share_of(l) + (int64_t)part * keep;
            const int n = (int)sh.n[l];
            for (int i = tid; i < keep; i += WALK_T) share[i] = i < n ? keys[l * WALK_CAP + i] : 0ull;
        }
        __threadfence();
        __syncthreads();
        if (tid == 0) sh.last = atomicAdd(reinterpret_cast<uint32_t*>(exact_words(exact, query(0), exact_stride) + 1), 1u) == (uint32_t)parts - 1u;
        __syncthreads();
        if (sh.last) {                                                             // uniform
            __threadfence();
            start();
            for (int l = 0; l < live; ++l) {
                // best ranks of all shares first; they are sorted, so nothing follows a load that brought no key
                const uint64_t* shares = share_of(l);
                const int total = (int)parts * keep;
                int before = 0;
                for (int i0 = 0; i0 < total; i0 += WALK_T) {
                    const int i = i0 + tid;
                    const uint64_t key = i < total ? shares[(i % (int)parts) * keep + i / (int)parts] : 0ull;
                    if (key != 0ull && key >= sh.cut[l]) keys[l * WALK_CAP + atomicAdd(&sh.n[l], 1u)] = key;
                    __syncthreads();
                    const int n = (int)sh.n[l];
                    if (n == before) break;                                        // uniform
                    __syncthreads();                                               // every lane has read the count
                    if (n > WALK_CAP - WALK_T) walk_cut_back(keys + l * WALK_CAP, n, k1, keep, &sh.n[l], &sh.cut[l]);
                    before = (int)sh.n[l];
                    __syncthreads();
                }
                walk_cut_back(keys + l * WALK_CAP, (int)sh.n[l], k1, keep, &sh.n[l], &sh.cut[l]);
                uint64_t* list = surv + (int64_t)query(l) * SURV_CAP;
                const int n = (int)sh.n[l];
                for (int i = tid; i < SURV_CAP; i += WALK_T) list[i] = i < n ? keys[l * WALK_CAP + i] : 0ull;
            }
        }
        __syncthreads();                                                           // the lists are used again
    }
}

template <int DT>
__global__ __launch_bounds__(WALK_T) void k_exact_walk(const void* __restrict__ store_, const float* __restrict__ qf,
                                                       const double* __restrict__ invq64, uint64_t* __restrict__ surv,
                                                       const uint32_t* __restrict__ cnt, double* __restrict__ exact, int exact_stride,
                                                       int64_t N, int nkb, int k1, int B, int lists) {
    extern __shared__ __align__(16) uint64_t walk_keys[];
    __shared__ WalkLds sh;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    int nlost = 0;
    for (int b0 = 0; b0 < B; b0 += WALK_T) {
        const bool lost = b0 + tid < B && *slot_counter(cnt, b0 + tid) > (uint32_t)SURV_CAP;
        const uint64_t m = __builtin_amdgcn_ballot_w64(lost);
        if (lane == 0) sh.wave_n[wave] = (uint32_t)__popcll(m);
        __syncthreads();
        int at = nlost + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
        for (int w = 0; w < WALK_T / 64; ++w) {
            at += w < wave ? (int)sh.wave_n[w] : 0;
            nlost += (int)sh.wave_n[w];
        }
        if (lost) sh.lost[at] = (uint16_t)(b0 + tid);
        __syncthreads();
    }
    if (nlost == 0) return;                                                        // uniform
    if (nlost <= 2) walk_lost<DT, 1>(store_, qf, invq64, surv, exact, exact_stride, N, nkb, k1, B, lists, nlost, walk_keys, sh);
    else walk_lost<DT, WALK_NB>(store_, qf, invq64, surv, exact, exact_stride, N, nkb, k1, B, lists, nlost, walk_keys, sh);
}

}  // namespace evk
