// Last steps of a retrieve (Sec. 3.2), one launch: the selection after the last scan pass, the exact re-scoring of
// the candidates it keeps, the candidate pool C(x) and the value filter.
//
// One workgroup per query, or `parts` of them: each then makes the same selection (from the same list, so with the same
// result, and at the same time), re-scores its share of the candidates, and the last one to finish orders the
// pool.  Nothing waits for another workgroup.  Against separate launches: one query
// over 4096 x 768 fp32 rows with a pool of 32 took 6.1 + 5.1 + 5.2 us in three launches, 10.7 in one.
// What bounds it: about 4 us of barriers and LDS round trips in the selection, which lays out the candidates too, 2 to 5 us in the
// orderings and z-scores; in between the rows, which come at 6.8 TB/s when there are many (128 queries, a pool of 256 of 8 KB: 46 us).
//
// Re-scoring: 16 to 64 lanes per candidate row accumulate in fp64, so that the value filter, which divides by the
// pool's spread, sees exact similarities.  It is a gather of 128-byte pieces that lie a k-block apart; the query lies in
// LDS, requested before the selection.  With the query's chunks read from memory where they are used (a round trip each), always 16
// lanes to a row and sums over the workgroup for the z-scores: one query, 32 x 3 KB 13.5 us, 10.7 now; 64 queries, 64 x 4 KB 24.4, 14.0; one
// query, 128 x 2 KB 19.1, 15.0; 256 queries, 128 x 2 KB 41, 28; 1024 queries, 128 x 3 KB 206, 120; 128 queries, 256 x 8 KB 119, 80;
// 64 queries, 960 x 2 KB 66, 55.  (Two workgroups of 64 registers a lane to a compute unit then, one of 128 now.)
// Ordering: a pool of up to 256 is ordered by counting how many candidates precede each one (four lanes share a
// candidate); for larger ones counting all pairs is too much work, so the entries are spread over 2048 buckets by
// value first -- a monotone map, so only entries of one bucket need comparing -- with a bitonic sort as the way out
// when a bucket holds too many (masses of equal values).
// z-scores over the pool (population deviation, denominator std + 1e-6), score = (1-lambda) z_s + lambda z_q, the
// k2 best by (score desc, id asc) or the k2 slots filled epsilon-greedily (Sec. 3.3).  All in fp64, scores rounded
// to fp32 on output.
#pragma once
#include "k_select.h"

namespace evk {

constexpr int TAIL_T = 1024;
constexpr int TAIL_CROWD = 64;            // entries of one bucket that are still ranked by counting
constexpr int TAIL_PIECE = keep_of(BIG_K1_MAX);   // ids of a crowded band that are laid out at a time

// LDS besides the static part (dynamic), in this order: v0[cap] f64, v1[k1p] f64, i0[cap] i32, i1[k1p] i32, q0[cap] f32, q1[k1p] f32,
// then for pools of more than 256 order[sort_cap] u32; cap = keep_of(k1), k1p = k1 rounded up to 64, sort_cap = cap rounded up to a
// power of two.  The epsilon-greedy draws (two words per slot) take over v0's space.
__host__ __device__ constexpr int tail_pad64(int x) { return (x + 63) & ~63; }
__host__ __device__ constexpr int tail_pow2(int x) { int p = 64; while (p < x) p <<= 1; return p; }
__host__ __device__ constexpr size_t tail_lds(int k1) {
    return (size_t)keep_of(k1) * 16 + (size_t)tail_pad64(k1) * 16 + (k1 > SMALL_K1_MAX ? (size_t)tail_pow2(keep_of(k1)) * 4 : 0);
}
constexpr size_t TAIL_STATIC_LDS = sizeof(SelectLds) + 2 * 16 * 8 + 64;          // besides these, the query's d floats (rounded up to a k-block)
static_assert(TAIL_PIECE * 4 <= tail_lds(1), "a piece of a crowded band's ids lies where the candidates will");

// A NaN similarity or score (a zero-norm or non-finite row or query, a NaN in the Q table: inputs
// for which the results are unspecified) is ranked as -inf, so that the orderings below stay total
// orders: every rank is taken exactly once and every id that is gathered with is a real one.
__device__ __forceinline__ double finite_or_lowest(double v) { return v == v ? v : -INFINITY; }

// (v, id) before (w, jd)?  Written without short-circuit operators: inside the counting loops below
// the arguments come from LDS, and a short-circuit form compiles to a branch per element with the
// second LDS read behind it, so that every element pays two LDS round trips (measured: 200 cycles
// per element, 36 us for a 128-entry pool); this form lets the reads of an unrolled group go out together.
__device__ __forceinline__ bool ranks_before(double v, int32_t id, double w, int32_t jd) {
    return (bool)((int)(v > w) | ((int)(v == w) & (int)(id < jd)));
}

// Sums of two values per lane over the workgroup, in a fixed order.
__device__ __forceinline__ void group_sum2(double (*red)[16], int wave, int lane, double& a, double& b) {
    a = wave_total_d(a);
    b = wave_total_d(b);
    if (lane == 0) { red[0][wave] = a; red[1][wave] = b; }
    __syncthreads();
    a = 0.0;
    b = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) { a += red[0][w]; b += red[1][w]; }
    __syncthreads();
}

// Calls emit(i, r) for every entry i of n, r being its rank by (value desc, id asc).  All lanes take part; the
// inputs were written before a barrier, and emit must not write them.
template <bool BIG, class Emit>
__device__ __forceinline__ void rank_entries(const double* val, const int32_t* ids, int n, uint32_t* order, SelectLds& sh,
                                             Emit emit) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if constexpr (!BIG) {
        // four lanes share an entry, or as many as there are: each counts over every fourth (8th, 16th) other entry
        auto count = [&](auto lanes) __attribute__((always_inline)) {
            constexpr int L = decltype(lanes)::value;
            for (int i = tid / L; i < n; i += TAIL_T / L) {          // trip count uniform within the lanes that share
                const double v = val[i];
                const int32_t id = ids[i];
                int rank = 0;
#pragma unroll 8
                for (int j = tid % L; j < n; j += L) rank += ranks_before(val[j], ids[j], v, id);
                rank += __builtin_amdgcn_update_dpp(0, rank, 0xb1, 0xf, 0xf, true);             // quad_perm 1,0,3,2
                rank += __builtin_amdgcn_update_dpp(0, rank, 0x4e, 0xf, 0xf, true);             // quad_perm 2,3,0,1
                if constexpr (L >= 8) rank += __builtin_amdgcn_update_dpp(0, rank, 0x141, 0xf, 0xf, true);     // row_half_mirror
                if constexpr (L >= 16) rank += __builtin_amdgcn_update_dpp(0, rank, 0x140, 0xf, 0xf, true);    // row_mirror
                if (tid % L == 0) emit(i, rank);
            }
        };
        if (n <= TAIL_T / 16) count(std::integral_constant<int, 16>{});
        else if (n <= TAIL_T / 8) count(std::integral_constant<int, 8>{});
        else count(std::integral_constant<int, 4>{});
    } else {
        constexpr int U = (BIG_K1_MAX + 256 + TAIL_T - 1) / TAIL_T;   // entries per lane
        // Range of the finite values.  It is that of their differences from one of them, rounded to fp32, so it is as good for values that fp32
        // does not tell apart (near-duplicates, a pool of 2048, one query: whole call 94 us with the range of the values themselves, 52 so); a value
        // may lie half a step outside it.
        const double first = val[0], base = first > -INFINITY && first < INFINITY ? first : 0.0;      // (n is not 0, or nothing below counts)
        uint32_t most = 0u, least = 0u;                              // complement of the smallest
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + u * TAIL_T;
            const float v = i < n ? (float)(val[i] - base) : -INFINITY;
            const uint32_t o = f2ord(v);
            most = v > -INFINITY && o > most ? o : most;
            least = v > -INFINITY && ~o > least ? ~o : least;
        }
        most = wave_max_u32(most);
        least = wave_max_u32(least);
        if (lane == 63) { sh.most[wave] = most; sh.least[wave] = least; }
        for (int i = tid; i < SEL_BINS; i += TAIL_T) sh.hist[i] = 0;
        if (tid == 0) sh.count = 0;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            most = sh.most[w] > most ? sh.most[w] : most;
            least = sh.least[w] > least ? sh.least[w] : least;
        }
        const double hi = base + ord2f(most), lo = base + ord2f(~least);
        const double scale = (double)SEL_BINS / (hi - lo);
        uint32_t bin[U], pos[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + u * TAIL_T;
            if (i < n) {
                const double x = (hi - val[i]) * scale;               // grows as the value falls; NaN (no range) goes to the last bucket
                bin[u] = x < 0.0 ? 0u : x < (double)(SEL_BINS - 1) ? (uint32_t)(int)x : (uint32_t)(SEL_BINS - 1);
                pos[u] = atomicAdd(&sh.hist[bin[u]], 1u);
            }
        }
        __syncthreads();
        const uint32_t c0 = sh.hist[2 * tid], c1 = sh.hist[2 * tid + 1];
        if (c0 > TAIL_CROWD || c1 > TAIL_CROWD) sh.count = 1;
        uint32_t total;
        const uint32_t start = group_prefix_u32(c0 + c1, sh.part_a, wave, lane, total);     // (has a barrier)
        sh.hist[2 * tid] = start;
        sh.hist[2 * tid + 1] = start + c0;
        const bool crowd = sh.count != 0;                              // uniform
        __syncthreads();
        if (!crowd) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = tid + u * TAIL_T;
                if (i < n) order[sh.hist[bin[u]] + pos[u]] = (uint32_t)i;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = tid + u * TAIL_T;
                if (i < n) {
                    const uint32_t first = sh.hist[bin[u]], last = bin[u] + 1 < (uint32_t)SEL_BINS ? sh.hist[bin[u] + 1] : (uint32_t)n;
                    const double v = val[i];
                    const int32_t id = ids[i];
                    uint32_t rank = first;
                    for (uint32_t t = first; t < last; ++t) {
                        const uint32_t j = order[t];
                        rank += ranks_before(val[j], ids[j], v, id);
                    }
                    emit(i, (int)rank);
                }
            }
        } else {
            int cap = 2;
            while (cap < n) cap <<= 1;
            for (int i = tid; i < cap; i += TAIL_T) order[i] = (uint32_t)i;
            __syncthreads();
            bitonic_desc(order, cap, tid, TAIL_T, [&](uint32_t x, uint32_t y) {
                const bool lx = (int)x < n, ly = (int)y < n;           // padding sorts last
                if (!lx || !ly) return !lx && ly;
                return ranks_before(val[y], ids[y], val[x], ids[x]);
            });
            for (int r = tid; r < n; r += TAIL_T) emit((int)order[r], r);
        }
    }
}

// Position of the set bit number `want` (from 0) of x, which has more than `want` of them.
__device__ __forceinline__ int nth_set_bit(uint64_t x, int want) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const int c = __popcll(x & ((1ull << w) - 1ull));
        const bool up = want >= c;
        want -= up ? c : 0;
        pos += up ? w : 0;
        x >>= up ? w : 0;
    }
    return pos;
}

struct TailArgs {
    uint64_t* surv;
    const uint32_t* cnt;
    uint32_t* counters;
    uint32_t* flags;
    uint32_t* arrived;        // per query, zero before the launch
    const void* store;
    const float* qf;
    const double* invq64;
    double* exact;            // [B][exact_stride]; used when a query has several workgroups
    uint64_t* spare;          // B lists as long as surv's that nothing else uses, or null
    const float* qstage;
    int32_t* out_ids;
    float* out_scores;
    int32_t* cand_ids;
    float* cand_sims;
    double lambda;
    int nkb, exact_stride, k1, k2, may_have_empty, mode;
    float margin;
    EpsGreedy eg;
};

// The arguments of a kernel whose only parameter is a TailArgs, to be loaded where they are used.  Held from the start, what the
// later steps need fills the scalar registers, and the selections spill theirs to vector lanes (150 reads of spilled
// scalars in the code, 42 this way when it was measured: a pool of 32 over 100 rows 10.9 us instead of 11.2 to 12.2).
typedef const __attribute__((address_space(4))) TailArgs* TailArgsPtr;
__device__ __forceinline__ TailArgsPtr tail_args_from_here() {
    TailArgsPtr p = (TailArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// K: keys of a query's list per lane (8 or 16).  With 16 a lane keeps a few registers in scratch memory (16 to 32 bytes), none with 8.
// 64 queries, a pool of 960 of 2 KB, four workgroups to a query: whole call 179.5 us (193.9 with 60 to 68 bytes, slots filled one by one and
// the buckets' range found with shuffles of fp64 values: 61 us of it here).
template <int DT, bool BIG, int K = SURV_CAP / TAIL_T>
__global__ __launch_bounds__(TAIL_T) void k_tail(TailArgs A) {
    constexpr int CAP = K * TAIL_T;
    extern __shared__ __align__(16) unsigned char tail_smem[];
    __shared__ SelectLds sh;
    __shared__ double red[2][16];
    __shared__ uint32_t last_s;
    const int k1 = A.k1, cap = keep_of(k1), k1p = tail_pad64(k1);
    double* v0 = reinterpret_cast<double*>(tail_smem);
    double* v1 = v0 + cap;
    int32_t* i0 = reinterpret_cast<int32_t*>(v1 + k1p);
    int32_t* i1 = i0 + cap;
    float* q0 = reinterpret_cast<float*>(i1 + k1p);                // the stage's values of the entries in i0, i1
    float* q1 = q0 + cap;
    uint32_t* order = reinterpret_cast<uint32_t*>(q1 + k1p);      // larger pools only
    const int b = (int)blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    float4* yq = reinterpret_cast<float4*>(tail_smem + tail_lds(k1));                      // the query
    int part = (int)blockIdx.y, parts = (int)gridDim.y;
    uint64_t* list = A.surv + (int64_t)b * CAP;

    query_to_lds<DT>(yq, A.qf + (int64_t)b * A.nkb * KB, A.nkb, TAIL_T);                   // (barriers follow)
    // ---- selection ----
    Selected<K> s;
    // (several workgroups each take a share of the same order)
    const uint32_t raw = select_keys(list, slot_counter(A.cnt, b), k1, A.margin, A.may_have_empty != 0, cap, A.mode, parts > 1, sh, s,
                                     [&](int i, uint32_t at) __attribute__((always_inline)) { if (at < (uint32_t)cap) i0[at] = key_id(s.key[i]); });
    const TailArgsPtr mid = tail_args_from_here();
    if (raw > (uint32_t)CAP && mid->mode == SEL_FINAL && part == 0 && tid == 0) { atomicAdd(mid->counters + 1, 1u); mid->flags[b] |= 1u; }
    // The last of the query's workgroups to come here?  All that one workgroup hands to another are the similarities
    // below, and those are stored and loaded as device-scope atomics, which pass by the caches that differ between
    // XCDs; so it is enough that a workgroup's stores have been acknowledged before it arrives.  That is this chip's
    // order, not the language's.  (Device-scope fences instead write back and invalidate a whole L2 per wavefront: this
    // kernel took 71 us with them for 64 queries in two parts, 24 without; an acquire-release arrival by one lane per
    // workgroup costs 3 us of a 42 us call for 64 queries in four parts, a pool of 960.)
    auto last_to_arrive = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) last_s = __hip_atomic_fetch_add(mid->arrived + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)gridDim.y - 1u;
        __syncthreads();
        return last_s != 0;
    };
    auto stays = [&](int i) __attribute__((always_inline)) { return s.key[i] >= s.cut; };
    // A crowded band (uniform, and the same for all of the query's workgroups): every key of it, up to the list's size, gets its
    // similarity accumulated in fp64 and the selection is made again with those, which are then the candidates' similarities.
    // The keys' ids stay in registers, so the similarities can take the place of the query's own list, or, if several
    // workgroups share the work, a list that the call does not use; without one it is left to the workgroup that knows
    // that the others have read theirs.
    // 7000 near rows, us for the whole call with the re-keying left to one workgroup and the candidates gathered once more,
    // and shared: one query, d = 1024 bf16 681, 160; 64 queries, two of them crowded, d = 4096 fp16 2690, 768; 256 queries (one
    // workgroup each), d = 1024 bf16 826, 737; one query, d = 128 bf16 (one workgroup, short rows) 194, 200.  (Rows scored as they
    // are now: this kernel 109 -> 81 us for one query, 196 -> 134 for 64 with two crowded, d = 1024 bf16.)
    const bool crowded = s.crowded && mid->mode == SEL_FINAL;
    if (crowded && parts > 1 && mid->spare == nullptr) {
        if (!last_to_arrive()) return;
        part = 0;
        parts = 1;
    }
    uint64_t* sims = !crowded ? reinterpret_cast<uint64_t*>(mid->exact + (int64_t)b * mid->exact_stride) : parts > 1 ? mid->spare + (int64_t)b * CAP : list;
    int32_t* ids = crowded ? reinterpret_cast<int32_t*>(tail_smem) : i0;            // (a crowded band's in pieces)
    // Crowded: this lane's ids (-1 = none) and their places, two to a word, in the list's order as far as a wavefront's keys go.
    // Neighbours in a list are often neighbours in the bank; in the order of `slot` rows gathered together lie 1024 entries
    // apart (5 to 8 % slower).
    int32_t mine[K];
    uint32_t places[K / 2];
    int kk = (int)s.kept;
    auto lay_out = [&](int c0) __attribute__((always_inline)) {      // the ids at places c0 .. c0 + TAIL_PIECE - 1
#pragma unroll
        for (int i = 0; i < K; ++i) {
            int32_t id = mine[i];
            asm volatile("" : "+v"(id));                             // (kept from one piece to the next, the eight conditions fill the scalar registers)
            const uint32_t at = (places[i / 2] >> (16 * (i % 2)) & 0xffffu) - (uint32_t)c0;
            if (id >= 0 && at < (uint32_t)TAIL_PIECE) ids[at] = id;
        }
        __syncthreads();
    };
    if (crowded) {
#pragma unroll
        for (int i = 0; i < K; ++i) mine[i] = stays(i) ? key_id(s.key[i]) : -1;
        uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.slot);
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint64_t in = __builtin_amdgcn_ballot_w64(mine[i] >= 0);
            const uint32_t at = first + __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));   // at most CAP
            places[i / 2] = i % 2 ? places[i / 2] | at << 16 : at;
            first += (uint32_t)__popcll(in);
        }
#pragma unroll
        for (int i = 0; i < K / 2; ++i) asm volatile("" : "+v"(places[i]));
        lay_out(0);
    }
    // the stage's values of all candidates: requested here, so that the z-scores need not wait for them
    constexpr int UC = ((BIG ? keep_of(BIG_K1_MAX) : KEEP_MAX) + TAIL_T - 1) / TAIL_T;
    float qc[UC];
#pragma unroll
    for (int u = 0; u < UC; ++u) qc[u] = !crowded && tid + u * TAIL_T < kk ? mid->qstage[i0[tid + u * TAIL_T]] : 0.f;

    // ---- exact similarities (of this workgroup's share) ----
    // Lanes per row: as many as leave no lane group without a row (16 at least); with more rows than groups of 16, two rows to a group,
    // which share the query's reads and conversions.  The order of a row's sums follows from it, and copies of a row have to tie exactly:
    // so one number for the whole query, by the largest share of its workgroups, whatever this one's is, and in a crowded band by a whole
    // piece's.  (Sums in one order for every number of lanes, 64 / G partial sums to a lane, would do too but take registers that are not
    // there: 256 queries, 128 x 2 KB 29 -> 38 us, 1024 queries, 128 x 3 KB 124 -> 157; with 32 lanes and two rows in place of 16 a
    // crowded band of 7000 81 -> 91.)
    const int most = ((crowded ? TAIL_PIECE : kk) + parts - 1) / parts;
    for (int c0 = 0;;) {                                             // (one piece unless crowded)
        const int m = !crowded || kk - c0 < TAIL_PIECE ? kk - c0 : TAIL_PIECE;
        const int share = (m - part + parts - 1) / parts;            // rows of this workgroup
        auto score = [&](auto lanes, auto rows) __attribute__((always_inline)) {
            constexpr int G = decltype(lanes)::value, R = decltype(rows)::value, GROUPS = TAIL_T / G;
            const int sub = tid % G, grp = tid / G;
            for (int j0 = 0; j0 < share; j0 += GROUPS * R) {         // uniform
                if (j0 + (wave * 64 / G) * R >= share) break;        // uniform within a wavefront, whose lanes add up across
                int32_t id[R];
                double dot[R], ssq[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int i = j0 + grp * R + r;
                    id[r] = ids[(i < share ? i : 0) * parts + part];
                }
                row_products<DT, G, R>(mid->store, yq, id, sub, mid->nkb, dot, ssq);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int i = j0 + grp * R + r, j = i * parts + part;
                    if (i < share && sub == 0) {
                        const double sim = finite_or_lowest(dot[r] * mid->invq64[b] * (1.0 / sqrt(ssq[r])));
                        if (!crowded && parts == 1) v0[j] = sim;
                        else __hip_atomic_store(sims + c0 + j, __builtin_bit_cast(uint64_t, sim), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        };
        using std::integral_constant;
        if (most <= TAIL_T / 64) score(integral_constant<int, 64>{}, integral_constant<int, 1>{});
        else if (most <= TAIL_T / 32) score(integral_constant<int, 32>{}, integral_constant<int, 1>{});
        else if (most <= TAIL_T / 16) score(integral_constant<int, 16>{}, integral_constant<int, 1>{});
        else score(integral_constant<int, 16>{}, integral_constant<int, 2>{});
        c0 += TAIL_PIECE;
        if (!crowded || c0 >= kk) break;                             // uniform
        __syncthreads();
        lay_out(c0);
    }
    if (parts > 1 && !last_to_arrive()) return;
    auto sim_at = [&](uint32_t at) __attribute__((always_inline)) {
        return __builtin_bit_cast(double, __hip_atomic_load(sims + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    if (crowded) {
        __syncthreads();
        double sim[K];                                               // (all requested at once: behind a condition each it is a round trip each)
#pragma unroll
        for (int i = 0; i < K; ++i) sim[i] = sim_at(mine[i] >= 0 ? places[i / 2] >> (16 * (i % 2)) & 0xffffu : 0u);
#pragma unroll
        for (int i = 0; i < K; ++i) s.key[i] = mine[i] >= 0 ? exact_key(sim[i], mine[i]) : 0ull;
        select_keys(kk, CAP, k1, EXACT_KEY_MARGIN, true, cap, SEL_EXACT, false, sh, s,
                    [&](int i, uint32_t at) __attribute__((always_inline)) { if (at < (uint32_t)cap) { i0[at] = mine[i]; v0[at] = sim[i]; } });
        kk = (int)s.kept;
        for (int i = tid; i < kk; i += TAIL_T) q0[i] = mid->qstage[i0[i]];
    } else {
        if (parts > 1)
            for (int i = tid; i < kk; i += TAIL_T) v0[i] = sim_at((uint32_t)i);
#pragma unroll
        for (int u = 0; u < UC; ++u)
            if (tid + u * TAIL_T < kk) q0[tid + u * TAIL_T] = qc[u];
    }
    __syncthreads();

    const TailArgsPtr late = tail_args_from_here();
    const int k2 = late->k2;
    int32_t* cand_ids = late->cand_ids;
    float* cand_sims = late->cand_sims;
    const double lambda = late->lambda;
    int32_t* out_ids = late->out_ids + (int64_t)b * k2;
    float* out_scores = late->out_scores + (int64_t)b * k2;
    const uint64_t threshold = late->eg.threshold;
    unsigned char* explored = late->eg.explored;
    // ---- the pool: the k1e best by (similarity desc, id asc) -> (v1, i1, q1) ----
    const int k1e = kk < k1 ? kk : k1;
    rank_entries<BIG>(v0, i0, kk, order, sh, [&](int i, int r) __attribute__((always_inline)) {
        if (r < k1e) { v1[r] = v0[i]; i1[r] = i0[i]; q1[r] = q0[i]; }
    });
    __syncthreads();
    // ---- z-scores over the pool ----
    if (cand_ids)
        for (int i = tid; i < k1; i += TAIL_T) {
            cand_ids[(int64_t)b * k1 + i] = i < k1e ? i1[i] : -1;
            cand_sims[(int64_t)b * k1 + i] = i < k1e ? (float)v1[i] : -INFINITY;
        }
    if (k1e > 0) {                                                    // uniform
        if constexpr (!BIG) {
            // Every wavefront that holds a member adds up the whole pool for itself: no barrier (with sums over the workgroup, four
            // of them, this took 2.5 us, 1.2 now).
            constexpr int U = SMALL_K1_MAX / 64;
            if (wave * 64 < k1e) {
                double sim[U], qv[U], sum_s = 0.0, sum_q = 0.0, var_s = 0.0, var_q = 0.0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = lane + 64 * u;
                    sim[u] = i < k1e ? v1[i] : 0.0;
                    qv[u] = i < k1e ? (double)q1[i] : 0.0;
                    sum_s += sim[u];
                    sum_q += qv[u];
                }
                const double mean_s = wave_total_d(sum_s) / k1e, mean_q = wave_total_d(sum_q) / k1e;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool mine = lane + 64 * u < k1e;
                    sim[u] = mine ? sim[u] - mean_s : 0.0;
                    qv[u] = mine ? qv[u] - mean_q : 0.0;
                    var_s += sim[u] * sim[u];
                    var_q += qv[u] * qv[u];
                }
                const double scale_s = 1.0 / (sqrt(wave_total_d(var_s) / k1e) + 1e-6), scale_q = 1.0 / (sqrt(wave_total_d(var_q) / k1e) + 1e-6);
                if (tid < k1e) {                                      // v0 / i0 are reused for the scores
                    v0[tid] = finite_or_lowest((1.0 - lambda) * ((v1[tid] - mean_s) * scale_s) + lambda * (((double)q1[tid] - mean_q) * scale_q));
                    i0[tid] = i1[tid];
                }
            }
        } else {
            constexpr int U = (BIG_K1_MAX + TAIL_T - 1) / TAIL_T;     // pool entries per lane
            double sim[U], qv[U], sum_s = 0.0, sum_q = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = tid + u * TAIL_T;
                sim[u] = i < k1e ? v1[i] : 0.0;
                qv[u] = i < k1e ? (double)q1[i] : 0.0;
                sum_s += sim[u];
                sum_q += qv[u];
            }
            group_sum2(red, wave, lane, sum_s, sum_q);
            const double mean_s = sum_s / k1e, mean_q = sum_q / k1e;
            double var_s = 0.0, var_q = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool mine = tid + u * TAIL_T < k1e;
                sim[u] = mine ? sim[u] - mean_s : 0.0;
                qv[u] = mine ? qv[u] - mean_q : 0.0;
                var_s += sim[u] * sim[u];
                var_q += qv[u] * qv[u];
            }
            group_sum2(red, wave, lane, var_s, var_q);
            const double scale_s = 1.0 / (sqrt(var_s / k1e) + 1e-6), scale_q = 1.0 / (sqrt(var_q / k1e) + 1e-6);
#pragma unroll
            for (int u = 0; u < U; ++u) {                             // v0 / i0 are reused for the scores
                const int i = tid + u * TAIL_T;
                if (i < k1e) {
                    v0[i] = finite_or_lowest((1.0 - lambda) * (sim[u] * scale_s) + lambda * (qv[u] * scale_q));
                    i0[i] = i1[i];
                }
            }
        }
    }
    __syncthreads();
    // ---- the k2 best by (score desc, id asc) ----
    const int k2e = k1e < k2 ? k1e : k2;
    const bool greedy = threshold == 0 && explored == nullptr;
    rank_entries<BIG>(v0, i0, k1e, order, sh, [&](int i, int r) __attribute__((always_inline)) {
        if (greedy) {
            if (r < k2e) { out_ids[r] = i0[i]; out_scores[r] = (float)v0[i]; }
        } else {
            v1[r] = v0[i];
            i1[r] = i0[i];
        }
    });
    for (int i = k2e + tid; i < k2; i += TAIL_T) {
        out_ids[i] = -1;
        out_scores[i] = -INFINITY;
        if (explored) explored[(int64_t)b * k2 + i] = 0;
    }
    if (greedy) return;                                               // uniform
    // ---- epsilon-greedy slot filling (Sec. 3.3) ----
    // The whole pool is laid out in greedy order; every slot's draw is computed by its own lane (the draws
    // depend on the slot number only); then one wavefront fills the slots in order, because which members are
    // still free depends on the slots before.  Lane w holds the free members 64 w .. 64 w + 63 as a bit mask.  The slots between two that
    // explore take the best free members in order, all at once (64 queries, a pool of 960, 32 slots, eps 0.1: whole call 190.5 us slot by slot, 185.9).
    int t = (int)threadIdx.x;                                          // (computed anew: what is kept for these lines is spilled by every call)
    asm volatile("" : "+v"(t));
    const int tl = t & 63;
    uint32_t* word0 = reinterpret_cast<uint32_t*>(v0);                 // v0 holds at least 2 k2 words
    uint32_t* word1 = word0 + k2;
    __syncthreads();                                                   // the ordering has read v0
    for (int j = t; j < k2e; j += TAIL_T) {
        const philox_out r = philox4x32_10((uint32_t)late->eg.step, (uint32_t)(late->eg.step >> 32), (uint32_t)b, (uint32_t)j,
                                           (uint32_t)late->eg.seed, (uint32_t)(late->eg.seed >> 32));
        word0[j] = r.w0;
        word1[j] = r.w1;
    }
    __syncthreads();
    if (t >= 64) return;                                               // uniform within a wavefront
    uint64_t is_free = k1e >= 64 * tl + 64 ? ~0ull : k1e <= 64 * tl ? 0ull : (1ull << (k1e - 64 * tl)) - 1ull;
    auto emit = [&](int slot, int at, bool explore) __attribute__((always_inline)) {
        out_ids[slot] = i1[at];
        out_scores[slot] = (float)v1[at];
        if (explored) explored[(int64_t)b * k2 + slot] = explore ? 1 : 0;
    };
    for (int c0 = 0; c0 < k2e; c0 += 64) {                             // a slot per lane
        const int here = k2e - c0 < 64 ? k2e - c0 : 64;
        const uint32_t w1 = tl < here ? word1[c0 + tl] : 0u;
        const uint64_t explores = __builtin_amdgcn_ballot_w64(tl < here && (uint64_t)word0[c0 + (tl < here ? tl : 0)] < threshold);
        for (int p = 0; p < here;) {                                   // uniform; every turn fills a slot at least
            const int c = __popcll(is_free), upto = (int)wave_inclusive_sum((uint32_t)c), before = upto - c;
            const uint64_t ahead = explores >> p;
            const int run = ahead == 0 || __builtin_ctzll(ahead) > here - p ? here - p : __builtin_ctzll(ahead);
            if (run > 0) {                                             // the run's t-th slot takes the t-th free member
                const int t = tl - p;
                int at = 0;
                for (int done = 0; done < run;) {                      // (a turn for every lane that holds some of them)
                    const int holder = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto > done));
                    const uint64_t mask = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(is_free >> 32), holder) << 32
                                        | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)is_free, holder);
                    const int first = __builtin_amdgcn_readlane(before, holder), last = __builtin_amdgcn_readlane(upto, holder);
                    if (t >= done && t < last) at = 64 * holder + nth_set_bit(mask, t - first);
                    done = last;
                }
                if (t >= 0 && t < run) emit(c0 + tl, at, false);
                if (upto <= run) is_free = 0;
                else if (before < run) is_free &= ~((2ull << nth_set_bit(is_free, run - before - 1)) - 1ull);
                p += run;
            } else {
                const int j = c0 + p;
                const int want = (int)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)w1, p) * (uint32_t)(k1e - j)) >> 32);   // index among the free members
                const int holder = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto > want));       // the first lane that reaches it
                if (tl == holder) {
                    const int bit = nth_set_bit(is_free, want - before);
                    is_free &= ~(1ull << bit);
                    emit(j, 64 * tl + bit, true);
                }
                ++p;
            }
        }
    }
}

}  // namespace evk
