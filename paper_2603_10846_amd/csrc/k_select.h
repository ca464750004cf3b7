// Selection over survivor lists (Sec. 3.2, dense recall), and what it shares with the kernels that follow it.
#pragma once
#include <type_traits>

#include "k_ingest.h"
#include "layout.h"

namespace evk {

// In-LDS bitonic sort, descending, n a power of two, all threads of the workgroup take part.
// Pair p of a stage belongs to thread p % nthreads, so a wavefront always works on the same
// 128-element blocks; a stage with stride j <= 64 stays inside those blocks.  Hence a workgroup
// barrier is needed only next to a stage with a larger stride -- between two small-stride stages
// (and always in a one-wavefront workgroup) the wavefront's own in-order LDS accesses suffice.
template <typename T, typename Less>
__device__ __forceinline__ void bitonic_desc(T* a, int n, int tid, int nthreads, Less less) {
    int prev_j = 1 << 30;                                     // "large": the caller's writes came from any thread
    for (int k = 2; k <= n; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (nthreads > 64 && (j > 64 || prev_j > 64)) __syncthreads();
            else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int p = tid; p < (n >> 1); p += nthreads) {
                int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));   // index with bit j clear
                int l = i | j;
                bool desc = (i & k) == 0;
                T x = a[i], y = a[l];
                if (less(x, y) == desc) { a[i] = y; a[l] = x; }
            }
            prev_j = j;
        }
    __syncthreads();
}

// Maximum over the 64 lanes of a wavefront (all lanes active); lane 63 ends up with the result.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
    auto up = [](uint32_t a, int b) __attribute__((always_inline)) { return (uint32_t)b > a ? (uint32_t)b : a; };
    x = up(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true));   // row_shr:1
    x = up(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true));   // row_shr:2
    x = up(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true));   // row_shr:4
    x = up(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true));   // row_shr:8
    x = up(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, true));   // row_bcast:15 into rows 1 and 3
    x = up(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, true));   // row_bcast:31 into rows 2 and 3
    return x;
}

// Sum over the workgroup's 16 wavefronts of one value per lane, and the sum over the lanes before this one.
// `part` has 16 slots; ends without a barrier (the caller's next barrier protects `part`).
__device__ __forceinline__ uint32_t group_prefix_u32(uint32_t x, uint32_t* part, int wave, int lane, uint32_t& total) {
    const uint32_t incl = wave_inclusive_sum(x);
    if (lane == 63) part[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const uint32_t p = part[w];
        before += w < wave ? p : 0u;
        all += p;
    }
    total = all;
    return before + incl - x;
}

// After a scan pass, for one query: find the k1-th best survivor key (similarity desc, id asc), set the
// next pass's threshold to that similarity minus `margin` (a bound on the scan's fp32 rounding error, so
// that no true member of the pool can be filtered out; pre-divided by the query's inverse norm because the
// scan compares before applying it), and keep every key whose similarity reaches that threshold: these
// seed the next pass and, after the last pass, are the candidates that get re-scored in fp64.  Nothing is
// sorted here -- slot order is irrelevant to every consumer.
// Keys live in registers (8 per lane, 1024 lanes).  The kernel is a chain of barriers and LDS round trips
// with one workgroup per query, so what counts is how many there are.  The first round uses 1024 bins of equal width in
// similarity: the pool is the thin upper tail of a list, so the pivot's bin nearly always holds no more than SEL_SMALL
// keys and those few are ranked by counting.  (Digits of the bit pattern put most keys into a few bins, one per
// exponent and leading bits; they remain for lists that equal widths cannot resolve.)  What every wavefront needs to know -- the
// pivot's bin, the pivot -- every wavefront works out for itself from LDS, which takes less than handing it round behind a barrier:
// four barriers, seven when one wavefront or lane found it for all.
// 16 wavefronts share four SIMDs, so vector instructions count as well: places come from ballots and scalar sums, not from a prefix sum per lane.
// Together, with the tail's: one query over 4096 rows, whole call 18.5 -> 17.9 us; seven over 30,011 (two selections) 30.2 -> 28.5; 32 over 300,007
// (three) 91.2 -> 88.7; 64, pool of 960 193.9 -> 190.5.
// A list that overflowed during the pass (more than SURV_CAP rows reached the threshold; the surplus was
// dropped) is counted and the query is flagged: its pool may then miss members.
// More than keep_max keys inside the margin ("crowded band"; near-duplicate entries do that):
//   SEL_PASS   (between scan passes) every key of the band is kept -- any of them may belong to the pool;
//   SEL_FINAL  (after the last pass) likewise, and the caller replaces the keys' similarities by exactly
//              accumulated ones and selects again with a margin of two fp32 roundings;
//   SEL_EXACT  (that second selection) a band that is still crowded can only be one of ties within
//              fp32 resolution: the k1 best keys are kept, lower ids first among equal similarities.
enum { SEL_PASS = 0, SEL_FINAL = 1, SEL_EXACT = 2 };
constexpr int SEL_DIGIT = 11, SEL_BINS = 1 << SEL_DIGIT;
constexpr int SEL_FIRST = 1024;          // bins of the first round
constexpr int SEL_SMALL = 128, SEL_FEW = 32;
struct SelectLds {
    __align__(16) uint32_t hist[SEL_BINS];
    uint64_t small[SEL_SMALL], pivot;
    uint32_t most[16], least[16];
    uint32_t part_a[16], part_b[16], count, nsmall, kept[2], digit, need;
};
template <int K>         // keys per lane: 8 for a list of 8192, 16 for two
struct Selected {
    uint64_t key[K];     // this lane's keys (0 = none)
    uint64_t cut;        // a key stays iff it is not 0 and not below this
    float tau;           // the threshold that this is (similarity units); meaningless with keep_all
    uint32_t kept;       // how many stay
    uint32_t slot;       // the first place of this wavefront's among them
    bool keep_all;       // fewer keys than the pool has members: all stay and there is no threshold
    bool crowded;
};
// Reads a list into the lanes' registers; returns its count as the scan left it (it may exceed the list's size).  The
// count and the first quarter of the list, which is what a filtering pass fills, are requested together.
template <int K>
__device__ __forceinline__ uint32_t load_keys(const uint64_t* list, const uint32_t* count, Selected<K>& s) {
    const int tid = threadIdx.x;
    uint64_t (&key)[K] = s.key;
#pragma unroll
    for (int i = 0; i < 2; ++i) key[i] = list[i * 1024 + tid];
    const uint32_t raw = (uint32_t)__builtin_amdgcn_readfirstlane((int)*count);
    const int n = raw > (uint32_t)(K * 1024) ? K * 1024 : (int)raw;
#pragma unroll
    for (int i = 2; i < K; ++i) key[i] = 0ull;                        // 0 = empty
#pragma unroll
    for (int i = 2; i < K; ++i)
        if (i * 1024 < n) { int idx = i * 1024 + tid; key[i] = idx < n ? list[idx] : 0ull; }
#pragma unroll
    for (int i = 0; i < 2; ++i) key[i] = i * 1024 + tid < n ? key[i] : 0ull;
    return raw;
}

// The bin of the first round in which the running count of the bins reaches `need`, the rank that is left in it -> need, and how many keys it
// has.  Every wavefront does the same.
__device__ __forceinline__ uint32_t find_bin(const uint32_t* hist, int lane, uint32_t& need, uint32_t& in_bin) {
    constexpr int PER = SEL_FIRST / 64, Q = PER / 4;                         // bins, and pieces of four, to a lane
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {                                            // (each lane from another quarter on: different banks)
        const uint4 v = reinterpret_cast<const uint4*>(hist)[lane * Q + ((j + (lane >> 2)) & (Q - 1))];
        sum += (v.x + v.y) + (v.z + v.w);
    }
    const uint32_t incl = wave_inclusive_sum(sum);
    const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl >= need));
    const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)incl, at) - (uint32_t)__builtin_amdgcn_readlane((int)sum, at);
    const uint32_t c = lane < PER ? hist[at * PER + lane] : 0u;
    const uint32_t upto = before + wave_inclusive_sum(c);
    const int bin = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto >= need));
    in_bin = (uint32_t)__builtin_amdgcn_readlane((int)c, bin);
    need -= (uint32_t)__builtin_amdgcn_readlane((int)upto, bin) - in_bin;
    return (uint32_t)(at * PER + bin);
}

// Selects among the keys in the registers (n of them, or fewer where some are empty; only the first `slots` places of the list
// they were read from may hold one: what lies past them is skipped, a list is seldom full).  place(i, at) is called for this lane's
// keys that stay, with their places (which may lie past keep_max: a crowded band, whose places are good for nothing unless the mode
// says that it stays); a barrier follows.  `ordered`: the places follow from the list alone, not from which wavefront came first.
template <int K, class Place>
__device__ __forceinline__ void select_keys(int n, int slots, int k1, float margin, bool may_have_empty, int keep_max, int mode, bool ordered, SelectLds& sh,
                                            Selected<K>& s, Place place) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const uint64_t (&key)[K] = s.key;
    for (int i = tid; i < SEL_BINS; i += 1024) sh.hist[i] = 0;
    if (tid == 0) { sh.nsmall = 0; sh.kept[0] = 0; sh.kept[1] = 0; }
    uint32_t used = 0;                                // keys of this wavefront
    uint32_t most = 0u, least = 0xffffffffu;          // largest similarity part of a key, and the smallest less one (of no key: itself again)
#pragma unroll
    for (int i = 0; i < K; ++i) {
        if (i * 1024 >= slots) continue;                                 // uniform
        const uint32_t o = (uint32_t)(key[i] >> 32);
        most = o > most ? o : most;
        least = o - 1u < least ? o - 1u : least;
        if (may_have_empty || n < k1) used += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[i] != 0));       // uniform
    }
    most = wave_max_u32(most);
    least = wave_max_u32(~least);
    if (lane == 63) { sh.most[wave] = most; sh.least[wave] = least; sh.part_b[wave] = used; }
    s.crowded = false;
    s.keep_all = false;
    __syncthreads();
    most = 0u;
    least = 0u;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        most = sh.most[w] > most ? sh.most[w] : most;
        least = sh.least[w] > least ? sh.least[w] : least;
    }
    least = ~least + 1u;
    // Places of the keys that stay: a wavefront's lie together, in the order of i and lane.
    auto place_all = [&](int again) __attribute__((always_inline)) {
        uint64_t in[K];
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            in[i] = i * 1024 < slots ? __builtin_amdgcn_ballot_w64(key[i] >= s.cut) : 0ull;
            sum += (uint32_t)__popcll(in[i]);
        }
        if (ordered) {                                                       // uniform
            uint32_t* part = again ? sh.part_b : sh.part_a;
            if (lane == 0) part[wave] = sum;
            __syncthreads();
            s.slot = 0;
            s.kept = 0;
#pragma unroll
            for (int w = 0; w < 16; ++w) {
                const uint32_t p = part[w];
                s.slot += w < wave ? p : 0u;
                s.kept += p;
            }
            if (mode == SEL_EXACT && !again && s.kept > (uint32_t)keep_max) return;          // uniform; these are not the places
            s.slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.slot);
        } else {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&sh.kept[again], sum);
            s.slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        }
        uint32_t at = s.slot;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (in[i] == 0) continue;                                        // uniform within a wavefront
            if (key[i] >= s.cut) place(i, at + __builtin_amdgcn_mbcnt_hi((uint32_t)(in[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in[i], 0u)));
            at += (uint32_t)__popcll(in[i]);
        }
        __syncthreads();
        if (!ordered) s.kept = sh.kept[again];
    };
    if (may_have_empty || n < k1) {                                       // uniform
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) total += sh.part_b[w];
        s.keep_all = total < (uint32_t)k1;
        if (s.keep_all) {
            s.cut = 1ull;
            s.tau = 0.f;
            place_all(0);
            return;
        }
    }
    // The search for the k1-th key.  A round counts the keys per bin (bins in descending order, so that the pivot's bin is
    // found by a prefix sum); a bin of few keys is ranked by counting, else the next round looks into it.
    uint64_t pivot = 0;
    uint32_t need = (uint32_t)k1;
    // ranks the in_bin keys that `in` names; the need-th of them is the pivot
    auto rank_few = [&](uint32_t in_bin, auto in) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i * 1024 < slots && key[i] != 0 && in(i)) sh.small[atomicAdd(&sh.nsmall, 1u)] = key[i];
        __syncthreads();
        // A few of them every wavefront ranks for itself; many (near-duplicates) are ranked once, eight lanes to a key, and the pivot is handed round.
        // (All 16 wavefronts over 96 copies of a row: the exhaustive call's first selection 11.6 us, 8.6 so.)
        if (in_bin > (uint32_t)SEL_FEW) {                                    // uniform
            static_assert(SEL_SMALL * 8 == 1024, "eight lanes to a key");
            const uint64_t mine = sh.small[tid >> 3];
            uint32_t rank = 0;
            for (uint32_t j = tid & 7; j < in_bin; j += 8) rank += sh.small[j] > mine;
            rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, 0xb1, 0xf, 0xf, true);             // quad_perm 1,0,3,2
            rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, 0x4e, 0xf, 0xf, true);             // quad_perm 2,3,0,1
            rank += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rank, 0x141, 0xf, 0xf, true);            // row_half_mirror
            if ((uint32_t)(tid >> 3) < in_bin && rank == need - 1) sh.pivot = mine;                        // keys are distinct
            __syncthreads();
            return sh.pivot;
        }
        const uint64_t mine = sh.small[lane];
        uint32_t rank = 0;
#pragma unroll 8
        for (uint32_t j = 0; j < in_bin; ++j) rank += sh.small[j] > mine;
        const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64((uint32_t)lane < in_bin && rank == need - 1) | 1ull << 63);
        return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), src) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, src);
    };
    // First round: bins of equal width in similarity between the largest and the smallest one (differences and
    // products round monotonically, so a better key never gets a later bin).  The upper tail, where the pivot lies, is thin.
    const float top = ord2f(most), width = (float)SEL_FIRST / (top - ord2f(least));
    bool found = false;
    if (width > 0.f && width < 1e30f && top - ord2f(least) < 1e30f) {        // uniform; not with infinities, NaN or equal similarities
        uint32_t bin[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            bin[i] = 0;
            if (i * 1024 >= slots) continue;                             // uniform
            const float x = (top - key_sim(key[i])) * width;
            bin[i] = x < (float)(SEL_FIRST - 1) ? (uint32_t)x : (uint32_t)(SEL_FIRST - 1);
            if (key[i] != 0) atomicAdd(&sh.hist[bin[i]], 1u);
        }
        __syncthreads();
        uint32_t in_bin;
        const uint32_t at = find_bin(sh.hist, lane, need, in_bin);
        if (in_bin <= (uint32_t)SEL_SMALL) {                                 // uniform
            pivot = rank_few(in_bin, [&](int i) __attribute__((always_inline)) { return bin[i] == at; });
            found = true;
        } else {                                                             // crowded: by digits, from the start
            need = (uint32_t)k1;
            __syncthreads();
            sh.hist[tid] = 0;
            __syncthreads();
        }
    }
    // By digits of 11 bits, from the highest bit on which two keys differ.  Here one lane finds the bin for all: 16 wavefronts that each read 2048
    // bins take longer than two barriers (7000 near-duplicates among 40,000 rows, one query, the selection after the first pass 17.6 -> 14.9 us; 14.1
    // with many keys ranked once, that of the exhaustive call 19.0 -> 14.9).  It clears the bins for the next round.
    auto find_digit = [&](uint32_t& in_bin) __attribute__((always_inline)) {
        __syncthreads();
        const uint2 c = reinterpret_cast<const uint2*>(sh.hist)[tid];
        reinterpret_cast<uint2*>(sh.hist)[tid] = make_uint2(0u, 0u);
        const uint32_t mine = c.x + c.y, incl = wave_inclusive_sum(mine);
        if (lane == 63) sh.part_b[wave] = incl;
        __syncthreads();
        const uint32_t part = lane < 16 ? sh.part_b[lane] : 0u, upto = wave_inclusive_sum(part);
        const int holder = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto >= need));
        if (__builtin_amdgcn_readfirstlane(wave) == holder) {
            const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(upto - part), holder);
            const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(before + incl >= need));
            const uint32_t run = before + incl - mine;                       // (of lane `at`)
            if (lane == at) {
                const bool second = run + c.x < need;
                sh.digit = (uint32_t)(2 * tid + second);
                sh.need = need - run - (second ? c.x : 0u);
                sh.count = second ? c.y : c.x;
            }
        }
        __syncthreads();
        need = sh.need;
        in_bin = sh.count;
        return sh.digit;
    };
    int hi = most != least ? 63 - __builtin_clz(most ^ least) : 31;
    uint64_t prefix = hi < 63 ? (((uint64_t)most << 32) >> (hi + 1)) << (hi + 1) : 0ull;
    while (!found) {
        const int shift = hi >= SEL_DIGIT - 1 ? hi - (SEL_DIGIT - 1) : 0;   // this round ranks bits hi .. shift
        const uint32_t dmask = (1u << (hi - shift + 1)) - 1u;
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i * 1024 < slots && key[i] != 0 && (hi == 63 || (key[i] >> (hi + 1)) == (prefix >> (hi + 1))))
                atomicAdd(&sh.hist[SEL_BINS - 1 - ((uint32_t)(key[i] >> shift) & dmask)], 1u);
        uint32_t in_bin;
        prefix |= (uint64_t)(SEL_BINS - 1 - find_digit(in_bin)) << shift;
        if (shift == 0) { pivot = prefix; break; }                           // all 64 bits are known
        if (in_bin <= (uint32_t)SEL_SMALL) {                                 // uniform
            pivot = rank_few(in_bin, [&](int i) __attribute__((always_inline)) { return (key[i] >> shift) == (prefix >> shift); });
            break;
        }
        hi = shift - 1;
    }
    s.tau = key_sim(pivot) - margin;
    s.cut = (uint64_t)f2ord(s.tau) << 32 | 1u;      // every key with similarity >= tau compares >= cut (no id is 2^32 - 1), an empty one never
    place_all(0);
    if (s.kept <= (uint32_t)keep_max) return;                                // uniform
    s.crowded = true;
    if (mode != SEL_EXACT) return;
    s.cut = pivot;                                  // ties within fp32 resolution: exactly the k1 best
    if (!ordered) {
        __builtin_amdgcn_s_waitcnt(0x0f70);         // vmcnt(0): what place has stored comes before what it stores next
        __syncthreads();
    }
    place_all(1);
}
template <int K, class Place>
__device__ __forceinline__ uint32_t select_keys(const uint64_t* list, const uint32_t* count, int k1, float margin, bool may_have_empty,
                                                int keep_max, int mode, bool ordered, SelectLds& sh, Selected<K>& s, Place place) {
    const uint32_t raw = load_keys(list, count, s);
    const int n = raw > (uint32_t)(K * 1024) ? K * 1024 : (int)raw;
    select_keys(n, n, k1, margin, may_have_empty, keep_max, mode, ordered, sh, s, place);
    return raw;
}

// Between two scan passes: one workgroup per query.
template <int K>
__global__ __launch_bounds__(1024) void k_select(uint64_t* __restrict__ surv, uint32_t* __restrict__ cnt,
                                                 float* __restrict__ thr, const float* __restrict__ invq,
                                                 uint32_t* __restrict__ counters, uint32_t* __restrict__ flags, int k1, float margin,
                                                 int may_have_empty, int keep_max) {
    __shared__ SelectLds sh;
    const int b = (int)blockIdx.x, tid = threadIdx.x;
    uint64_t* list = surv + (int64_t)b * (K * 1024);
    Selected<K> s;
    // the keys that stay go to the list's head (they were all read before a barrier; the count too)
    const uint32_t raw = select_keys(list, slot_counter(cnt, b), k1, margin, may_have_empty != 0, keep_max, SEL_PASS, false, sh, s,
                                     [&](int i, uint32_t at) __attribute__((always_inline)) { list[at] = s.key[i]; });
    if (raw > (uint32_t)(K * 1024) && tid == 0) { atomicAdd(counters + 1, 1u); flags[b] |= 1u; }
    if (tid == 0) {
        *slot_counter(cnt, b) = s.kept;
        thr[b] = (s.keep_all ? -2.0f : s.tau) / invq[b];      // no threshold: a finite floor, see k_prep_queries
    }
}

// A query in LDS as row_products reads it: four elements to an entry, the two halves of a 16-bit store's chunks of eight in planes of
// their own (a wavefront's reads are then 16 bytes apart).  All lanes call it; a barrier has to follow.
template <int DT>
__device__ __forceinline__ void query_to_lds(float4* yq, const float* q, int nkb, int nthreads) {
    constexpr int PLANES = DT == 0 ? 1 : 2;
    const int n4 = nkb * KB / 4;
    for (int f = (int)threadIdx.x; f < n4; f += nthreads) yq[(f % PLANES) * (n4 / PLANES) + f / PLANES] = reinterpret_cast<const float4*>(q)[f];
}

// Products of R stored rows with one query, accumulated in fp64 by G neighbouring lanes (lane `sub` of them takes every G-th 16-byte
// chunk; eight loads in flight); every lane gets the sums.  Products of 16-bit values are exact, so dot / sqrt(ssq) is the
// cosine of the stored vectors up to fp64 rounding.  The query comes from LDS: read from memory where it is used, each of its
// chunks was a round trip of its own, since the loop's exit checks keep the compiler from requesting them together (64 queries, 66
// rows of 1024 fp32 each over four workgroups: 10.6 us of the kernel's 22).
template <int DT, int G, int R>
__device__ __forceinline__ void row_products(const void* store_, const float4* yq, const int32_t (&id)[R], int sub, int nkb, double (&dot)[R],
                                             double (&ssq)[R]) {
    constexpr int EPC = DT == 0 ? 4 : 8, U = 8 / R;      // elements per 16-byte chunk; chunks of a row in flight
    const int nch = nkb * KB / EPC;                      // chunks per row
#pragma unroll
    for (int r = 0; r < R; ++r) { dot[r] = 0.0; ssq[r] = 0.0; }
    for (int first = 0; first < nch; first += G * U) {   // uniform
        uint4 pk[R][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = first + sub + G * u < nch ? first + sub + G * u : nch - 1;     // past the end: the last chunk, dropped below
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (DT == 0) pk[r][u] = *reinterpret_cast<const uint4*>(static_cast<const float*>(store_) + off32(id[r], c, nkb));
                else pk[r][u] = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(store_) + off16(id[r], c, nkb));
            }
        }
        __builtin_amdgcn_sched_barrier(0);               // all of them requested before the first is used
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (first + G * u >= nch) break;             // uniform
            const bool in = first + sub + G * u < nch;
            const int c = in ? first + sub + G * u : nch - 1;
            const float4 y0 = yq[c], y1 = DT == 0 ? y0 : yq[nch + c];
            const float yy[8] = {y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w};
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t w[4] = {in ? pk[r][u].x : 0u, in ? pk[r][u].y : 0u, in ? pk[r][u].z : 0u, in ? pk[r][u].w : 0u};
#pragma unroll
                for (int e = 0; e < EPC; ++e) {
                    double x;
                    if (DT == 0) x = __uint_as_float(w[e & 3]);
                    else {
                        const uint16_t h = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                        x = DT == 1 ? bf16_to_f(h) : f16_to_f(h);
                    }
                    dot[r] += x * (double)yy[e];
                    ssq[r] += x * x;
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        dot[r] = row16_sum(dot[r]);
        ssq[r] = row16_sum(ssq[r]);
#pragma unroll
        for (int o = 16; o < G; o <<= 1) { dot[r] += __shfl_xor(dot[r], o, 64); ssq[r] += __shfl_xor(ssq[r], o, 64); }
    }
}

// The key of a similarity accumulated in fp64, rounded to fp32 (resolution 6e-8); NaN ranks lowest.
__device__ __forceinline__ uint64_t exact_key(double sim, int32_t id) { return pack_key(sim == sim ? (float)sim : -INFINITY, id); }

constexpr float EXACT_KEY_MARGIN = 2.4e-7f;     // two fp32 roundings of a similarity of magnitude <= 1

// One block of the Philox-4x32 counter-based generator with 10 rounds (Salmon et al., SC'11): each
// round multiplies counter words 0 and 2 by fixed odd constants, crosses the high and low halves
// with the other two words and the key, and the key advances by fixed Weyl increments.
struct philox_out { uint32_t w0, w1, w2, w3; };
__device__ __forceinline__ philox_out philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                    uint32_t k0, uint32_t k1) {
    constexpr uint32_t MUL_A = 0xD2511F53u, MUL_B = 0xCD9E8D57u, WEYL_A = 0x9E3779B9u, WEYL_B = 0xBB67AE85u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint32_t a_hi = __umulhi(MUL_A, c0), a_lo = MUL_A * c0;
        const uint32_t b_hi = __umulhi(MUL_B, c2), b_lo = MUL_B * c2;
        c0 = b_hi ^ c1 ^ k0;
        c2 = a_hi ^ c3 ^ k1;
        c1 = b_lo;
        c3 = a_lo;
        k0 += WEYL_A;
        k1 += WEYL_B;
    }
    return {c0, c1, c2, c3};
}

// Parameters of the epsilon-greedy slot filling (Sec. 3.3); threshold 0 and no flag output = greedy.
struct EpsGreedy {
    uint64_t threshold;      // floor(eps * 2^32): a slot explores iff its first random word is below it
    uint64_t seed, step;
    unsigned char* explored; // [B][k2] or null
};

}  // namespace evk
