// Similarity scan on the matrix cores (Sec. 3.2, dense recall): scores[q][n] = <query q, bank row n>,
// never written to memory.  Used for every batch size on 16-bit stores (at a handful of queries the
// arithmetic is idle and the kernel is a streaming engine for the bank) and for more than four
// queries on fp32 stores.
//
// Persistent workgroups of 4 or 8 wavefronts; each owns QT queries and walks over 256-row bank
// tiles.  Per k-block the bank tile's 32 KB block (already in LDS operand order in HBM, see
// layout.h) and the queries' block are staged in LDS (two stages) and consumed by
// v_mfma_f32_16x16x32 (bf16 or f16 operands, fp32 accumulation).  Bank loads run two k-blocks
// ahead of the MFMAs through two register sets, and the (tile, k-block) sequence is flattened, so
// the loads of the next tile are already in flight while a tile's epilogue runs.  Queries are the
// rows of the accumulator tile and bank rows its columns: a lane holds one bank row per 16x16 block.
// Within a k-block the two k-steps are a hand-written software pipeline (see compute()): operand
// fragments are read from LDS a few query blocks ahead, the LDS stores and global loads of the following
// k-blocks issue between the MFMAs, and there is one workgroup barrier per k-block.
//
// 128 or 256 queries to a tile over 16-bit stores (RING): operands go from memory straight to LDS, through rings of three places, and the
// two wavefronts of a SIMD take turns -- one feeds the matrix cores from registers while the other fetches its next fragments and asks for
// what comes two or three blocks later (ring_step()).  Where all wavefronts do all of it side by side, as the smaller tiles do, each load
// holds its wavefront up for some 50 cycles (the address path takes 16 for a 1 KB request) and the other one is no more likely to have
// matrix instructions ready: parts switched off in turn, 1M x 1536 bf16 with 1024 queries, densest pass, 10^6 cycles: fragments and
// matrix instructions alone 27.2, with queries loaded 30.4, with bank rows too 35.2, with the epilogue 37.6; taking turns 29.3, 29.9,
// 31.2, 32.5.  The latency of the bank is hidden either way (rows from HBM, from L2 or none at all: the same cycles).
// What bounds it with 1024 queries is the power limit: without the epilogue that pass takes 4 % fewer cycles and as long, at a clock of
// 1.79 instead of 1.87 GHz, and without loads of the bank, too, it takes 12 % less, at 1.95.  With 256 queries the same parts take time: 1M x 1024
// 420 us, 386 without the epilogue, 327 without bank loads too, the matrix cores busy for 62, 69 and 76 % of the cycles.  Densest pass of 1M x 1536, 1024 queries 2470 ->
// 2230 us (1390 TFLOP/s, on other cards up to 1450; the vendor's product of 16384 x 16384 x 8192 1540), 1M x 1024, 256 queries 460 -> 430.
// One rotation of the k-loop for all workgroups of an XCD when several share its bank tiles: 2150 -> 2130 us.  128 queries (whole calls): 1.1M x 4096 fp16
// 1592 -> 1546 us, 1M x 1024 bf16 391 -> 385, 200,000 x 768 134 -> 129, 1M x 64 100 -> 88, 300,007 x 384 92.0, 92.0.
// Instructions: 16x16x32 move half as many accumulator bytes per product as 32x32x16 ones (256 x 256 x 64 from LDS alone 1.15 and 1.35 us).
//
// fp32 stores: each value is split on the fly into bf16 hi + bf16 lo and the product is
// hi*hi + hi*lo + lo*hi (three MFMAs, relative error of a product about 2^-16); this only has to
// be good enough for the filter, since the value filter re-scores the selected candidates in fp64.
//
// Filter: the accumulators of a tile start at  -threshold[query] * norm[row]  (one extra MFMA per
// block), so after the k-loop a score passes iff its accumulator is non-negative; the epilogue
// collects sign bits, stages the rare survivors in an LDS list and flushes it every few tiles.
// The sparsest pass has no threshold and writes every row's key to the row's own position.
//
// EXACT: a denser pass of the exhaustive selection (k_exact.h).  The filter is the same, what it stages is scored in fp64 before it
// goes to a list.  Padding queries and queries that are lost stage nothing, and neither do zero rows, which are below every cut.
#pragma once
#include <type_traits>

#include "k_exact.h"
#include "k_scan_gemv.h"
#include "layout.h"

namespace evk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

template <int DT>
__device__ __forceinline__ f32x4_t mfma16(u32x4_t a, u32x4_t b, f32x4_t c) {
    if constexpr (DT == 2) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// acc += a * b in acc's own registers.  Given the choice the compiler lets the result wander to other registers, and with
// every register taken by accumulators that ends in spills inside the k-loop.  It does not see that a matrix instruction is
// in flight, so before anything but another one reads acc there has to be a settle().
template <int DT>
__device__ __forceinline__ void mfma16_in_place(f32x4_t& acc, u32x4_t a, u32x4_t b) {
    if constexpr (DT == 2) asm("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
    else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// Wait states that cover the last matrix instruction issued (eight passes at most, 18 wait states with the instruction itself).
__device__ __forceinline__ void mfma_settle() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}


// hi/lo split of two fp32 values for the matrix cores: returns the packed bf16 heads and leaves the
// (exactly representable) remainders a - head(a), b - head(b) in ra, rb.
__device__ __forceinline__ uint32_t pack_bf16x2_hi(float a, float b, float& ra, float& rb) {
    const uint32_t h = cvt_pk_bf16(a, b);
    ra = a - __uint_as_float(h << 16);
    rb = b - __uint_as_float(h & 0xffff0000u);
    return h;
}

// The accumulators of four blocks, as the 16 registers that a lane's survivors are looked for in together.
struct AccGroup { float v[16]; };

// Per-lane choice of one of the 16 registers of a group: register r = 4 * hi + lo of each
// lane's own (lo, hi), given as lane masks (lo == 1, lo == 3, lo >= 2, hi == 1, hi == 3, hi >= 2).  A
// two-level tree of 15 v_cndmask (registers cannot be indexed per lane).  Written as instructions because
// the compiler turns the equivalent C++ selects over elements of an accumulator vector into a
// dynamically indexed vector access, which it expands to a 16-way chain.  The two wait states at the
// top are the ones gfx950 needs between a vector compare writing a mask and a vector instruction reading
// it; the compiler does not add them for instructions it cannot see, and one pair serves all 15.
__device__ __forceinline__ float lane_select16(const AccGroup& g, uint64_t lo1, uint64_t lo3, uint64_t lo23,
                                               uint64_t hi1, uint64_t hi3, uint64_t hi23) {
    const float (&v)[16] = g.v;
    float g0, g1, g2, g3, t;
    asm("s_nop 1\n\t"
        "v_cndmask_b32_e64 %[g0], %[a0], %[a1], %[lo1]\n\t"
        "v_cndmask_b32_e64 %[t], %[a2], %[a3], %[lo3]\n\t"
        "v_cndmask_b32_e64 %[g0], %[g0], %[t], %[lo23]\n\t"
        "v_cndmask_b32_e64 %[g1], %[a4], %[a5], %[lo1]\n\t"
        "v_cndmask_b32_e64 %[t], %[a6], %[a7], %[lo3]\n\t"
        "v_cndmask_b32_e64 %[g1], %[g1], %[t], %[lo23]\n\t"
        "v_cndmask_b32_e64 %[g2], %[a8], %[a9], %[lo1]\n\t"
        "v_cndmask_b32_e64 %[t], %[a10], %[a11], %[lo3]\n\t"
        "v_cndmask_b32_e64 %[g2], %[g2], %[t], %[lo23]\n\t"
        "v_cndmask_b32_e64 %[g3], %[a12], %[a13], %[lo1]\n\t"
        "v_cndmask_b32_e64 %[t], %[a14], %[a15], %[lo3]\n\t"
        "v_cndmask_b32_e64 %[g3], %[g3], %[t], %[lo23]\n\t"
        "v_cndmask_b32_e64 %[g0], %[g0], %[g1], %[hi1]\n\t"
        "v_cndmask_b32_e64 %[g2], %[g2], %[g3], %[hi3]\n\t"
        "v_cndmask_b32_e64 %[g0], %[g0], %[g2], %[hi23]"
        : [g0] "=&v"(g0), [g1] "=&v"(g1), [g2] "=&v"(g2), [g3] "=&v"(g3), [t] "=&v"(t)
        : [a0] "v"(v[0]), [a1] "v"(v[1]), [a2] "v"(v[2]), [a3] "v"(v[3]), [a4] "v"(v[4]), [a5] "v"(v[5]), [a6] "v"(v[6]),
          [a7] "v"(v[7]), [a8] "v"(v[8]), [a9] "v"(v[9]), [a10] "v"(v[10]), [a11] "v"(v[11]), [a12] "v"(v[12]),
          [a13] "v"(v[13]), [a14] "v"(v[14]), [a15] "v"(v[15]), [lo1] "s"(lo1), [lo3] "s"(lo3), [lo23] "s"(lo23),
          [hi1] "s"(hi1), [hi3] "s"(hi3), [hi23] "s"(hi23));
    return g0;
}

// The one non-negative value among the 16 registers of a group, for lanes that have exactly
// one: as signed integers, every value with the sign bit set is below every value without it, so the
// integer maximum of the bit patterns is that value, bit for bit (8 three-operand maxima; no compare
// masks and no per-lane register choice).
__device__ __forceinline__ float only_non_negative(const AccGroup& g) {
    auto bits = [&](int r) __attribute__((always_inline)) { return (int)__float_as_uint(g.v[r]); };
    auto max3 = [](int a, int b, int c) __attribute__((always_inline)) { return max(max(a, b), c); };
    const int t0 = max3(bits(0), bits(1), bits(2)), t1 = max3(bits(3), bits(4), bits(5)), t2 = max3(bits(6), bits(7), bits(8));
    const int t3 = max3(bits(9), bits(10), bits(11)), t4 = max3(bits(12), bits(13), bits(14));
    return __uint_as_float((uint32_t)max(max3(t0, t1, t2), max3(t3, t4, bits(15))));
}

constexpr int STAGE_BANK_BYTES = TILE_ROWS * 128;
constexpr int SCAN_LDS = 160 * 1024;    // of a compute unit
constexpr int SCAN_LIST_TILES = 64;     // a workgroup's list is written out after as many tiles at the latest

// 16-bit stores with 128 or 256 queries to a tile: operands pass through rings in LDS (see ring_step()).
template <int DT, int QT> constexpr bool scan_mfma_ring() { return DT != 0 && QT >= 128; }
constexpr int RING_PLACES = 3;          // (four of bank blocks with 128 queries: 1.1M x 4096 fp16 1546 -> 1557 us a call, 1M x 1024 385 -> 402)
// LDS: the operand stages -- two of a bank block and a query block, or, as rings, three of a bank block and three of half a query
// block --; per-query threshold, inverse norm, survivor count and list base; tiles of the list; counters; the workgroup's survivor list (8 bytes an
// entry), for which the rings leave less room.
// (masked variant: the per-query type masks and excluded groups in addition; EXACT: cuts and inverse norms)
template <int DT, int QT> constexpr int scan_mfma_stage_bytes() {
    return scan_mfma_ring<DT, QT>() ? RING_PLACES * (STAGE_BANK_BYTES + QT * 64) : 2 * (STAGE_BANK_BYTES + QT * 128);
}
template <int DT, int QT, bool MASKED = false, bool EXACT = false> constexpr int scan_mfma_word_bytes() { return QT * 16 + SCAN_LIST_TILES * 4 + 16 + (MASKED ? QT * 8 : EXACT ? QT * 16 : 0); }
// survivor entries a workgroup can stage
template <int DT, int QT, bool MASKED = false, bool EXACT = false> constexpr int scan_mfma_list_cap() {
    return scan_mfma_ring<DT, QT>() ? (SCAN_LDS - scan_mfma_stage_bytes<DT, QT>() - scan_mfma_word_bytes<DT, QT, MASKED, EXACT>()) / 8 : 2048;
}
template <int DT, int QT, bool MASKED = false, bool EXACT = false> constexpr int scan_mfma_lds_bytes() {
    return scan_mfma_stage_bytes<DT, QT>() + scan_mfma_word_bytes<DT, QT, MASKED, EXACT>() + scan_mfma_list_cap<DT, QT, MASKED, EXACT>() * 8;
}
// ... and with BUSY, where the list is written out after every tile.  A list that runs full costs a device-wide atomic per surplus survivor, so many
// survivors to a tile (wide pools, small banks, masks) need room, and what the rings leave is less than that of the smaller tiles.  The place of
// the tile's last bank block is free from the end of the k-loop to the next tile's first loads.  Whole calls, us, lists of 2048 entries / what the
// rings leave / the place: 65,536 x 256 bf16, 256 queries, pool of 256 84, 86, 71; 100,000 x 256 masked, 1024 queries, pool of 128 238, 254, 221.
// (128 queries to a tile: the rings leave more than that, 4830 entries.)
constexpr int BUSY_LIST = STAGE_BANK_BYTES / 8;
template <int DT, int QT, bool MASKED> constexpr bool scan_mfma_busy() { return scan_mfma_ring<DT, QT>() && scan_mfma_list_cap<DT, QT, MASKED>() < BUSY_LIST; }
static_assert(BUSY_LIST >= 2048 && scan_mfma_list_cap<1, 128, true>() >= BUSY_LIST, "rings leave a busy tile's list no less room than two stages did");
static_assert(scan_mfma_lds_bytes<1, 256, true>() <= SCAN_LDS && scan_mfma_lds_bytes<0, 256, true>() <= SCAN_LDS, "one workgroup to a compute unit");

// DT: 0 fp32 store (bf16 split), 1 bf16, 2 f16.  Wave grid WQ x WR, each wave MQ x MR blocks of 16x16.
// gridDim.x is a multiple of 8 * (Bp / QT).
// EXACT: see above; not MASKED, never the sparsest pass, 32 queries to a tile.
// MASKED: typed / masked retrieval -- a row is kept for a query only if the query accepts its tag.
// STREAM: bank rows are loaded with the non-temporal hint (layout.h).  Right whenever a bank tile is read
// by one workgroup only; with several query tiles per bank tile (more than 256 queries) the later readers
// are meant to find the tile in L2, and the hint costs 2 % there (measured: 1397 -> 1366 TFLOP/s at 1024 queries, the sparser passes 10 %).
// BUSY: the list is written out after every tile and lies in a ring's free place.  (A variant of its own: chosen at run time, the kernel for seldom
// written lists took 2 % longer, 2M x 1536, 1024 queries 4960 -> 5100 us, though its k-loop was the same.)
template <int DT, int MQ, int WQ, int MR, int WR, bool MASKED, bool STREAM = true, bool EXACT = false, bool BUSY = false>
__global__ __launch_bounds__(64 * WQ * WR, 2) void k_scan_mfma(const void* __restrict__ store_, const float* __restrict__ invnorm,
                                                   const uint16_t* __restrict__ qop, const float* __restrict__ invq,
                                                   const float* __restrict__ thr, uint32_t* __restrict__ cnt,
                                                   uint64_t* __restrict__ surv, int64_t N, int nkb, int Bp,
                                                   Level L, int flush_every, Mask mask, int B, ExactPass exact) {
    static_assert((WQ * WR == 4 || WQ * WR == 8) && MR * WR == 16, "4 or 8 waves, 256 bank rows per workgroup");
    static_assert(MQ == 2 || MQ == 4 || MQ == 8, "whole groups of query blocks");
    constexpr int NT = 64 * WQ * WR;                   // lanes per workgroup
    constexpr int QT = 16 * MQ * WQ;
    constexpr int BCH = 2048 / NT;                     // 16-byte bank chunks per lane per stage
    constexpr int QCH = QT * 8 / NT;                   // 16-byte query chunks per lane per stage
    constexpr bool RING = scan_mfma_ring<DT, QT>();
    constexpr int QUERY_AT = (RING ? RING_PLACES : 2) * STAGE_BANK_BYTES;        // the stages of queries lie behind those of bank blocks
    constexpr int LIST_CAP = scan_mfma_list_cap<DT, QT, MASKED, EXACT>();
    // Query blocks go straight to LDS in the largest variant, whose registers are all taken; the few pieces of a smaller query tile
    // pass through registers, which look a step further ahead (whole masked call, 32 queries, 300,007 x 384 fp16: 94.8 us, 96.9
    // straight to LDS).
    constexpr bool Q_DIRECT = QT == 256 && !RING;
    // an AccGroup: GB query blocks of BB row blocks, 16 registers (4 * (GB * row block + query block) + register)
    constexpr int GB = MQ < 4 ? MQ : 4, BB = 4 / GB, GROUPS = MQ / GB, RGROUPS = MR / BB;
    // 16-bit float type of the operands that carry thresholds and norms: the store's (bf16 also for fp32 stores, which are split into
    // bf16).  EXACT: always bf16, whose pairs are good to the margin over the whole range of norms that an fp16 row can have.
    constexpr int TT = DT == 2 && !EXACT ? 2 : 1;
    auto enc16 = [](float x) __attribute__((always_inline)) { return TT == 2 ? f2f16_rne(x) : (uint16_t)cvt_pk_bf16(x, x); };
    auto dec16 = [](uint16_t h) __attribute__((always_inline)) { return TT == 2 ? f16_to_f(h) : bf16_to_f(h); };
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wq = wave / WR, wr = wave % WR;
    const int l16 = lane & 15, grp = lane >> 4;
    // Outside the k-loop (tile start, epilogue) lane coordinates are formed afresh: the wavefront's
    // position from scalar registers, the lane index from the lane counter seeded with a zero the
    // compiler cannot see through.  A per-lane value kept from the kernel's start would live on the
    // stack across the k-loop (there is no register to spare), and the wait for its reload is a wait
    // for every load in flight.
    const int wq_u = __builtin_amdgcn_readfirstlane(wq), wr_u = __builtin_amdgcn_readfirstlane(wr);
    auto fresh_lane = [&]() __attribute__((always_inline)) {
        uint32_t z = 0;
        asm volatile("" : "+v"(z));
        return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, z));
    };

    // Workgroup -> (query tile, sequence of bank tiles).  Blocks are dealt to the 8 XCDs round-robin;
    // the nqt workgroups that share a bank tile are neighbours on one XCD and walk the tiles in the
    // same order, so a tile is fetched from HBM once and the other query tiles hit that XCD's L2.
    const int nqt = Bp / QT;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int qt = slot % nqt, group = slot / nqt;
    const int groups = (gridDim.x >> 3) / nqt;         // tile walkers per XCD
    const int q0 = qt * QT;
    // tiles of this workgroup: j = (group + i * groups) * 8 + xcd < L.ntiles
    const int first_j = group * 8 + xcd, stride_j = groups * 8;
    if (first_j >= L.ntiles) return;
    const int my_tiles = (L.ntiles - first_j + stride_j - 1) / stride_j;

    auto sbank = [&](int s) __attribute__((always_inline)) { return smem + s * STAGE_BANK_BYTES; };
    auto sq = [&](int s) __attribute__((always_inline)) { return smem + QUERY_AT + s * QT * 128; };
    constexpr int WORDS_AT = scan_mfma_stage_bytes<DT, QT>();
    uint32_t* thp_s = reinterpret_cast<uint32_t*>(smem + WORDS_AT);    // thresholds as (hi | lo << 16), 16-bit floats
    float* invq_s = reinterpret_cast<float*>(thp_s + QT);
    uint32_t* cnt_s = reinterpret_cast<uint32_t*>(invq_s + QT);
    uint32_t* base_s = cnt_s + QT;
    constexpr uint32_t LIST_AT = WORDS_AT + scan_mfma_word_bytes<DT, QT, MASKED, EXACT>();
    // An entry: accumulator value << 32 | refused << 24 | which of the tiles since the list was empty << 16 | row of the tile << 8 | register of the
    // group, lane group << 4, group of query blocks << 6 (EXACT: queries << 32 | id).
    uint64_t* list_s = reinterpret_cast<uint64_t*>(smem + LIST_AT);
    static_assert(!BUSY || RING, "a place of a ring");
    constexpr uint32_t LIST_ROOM = BUSY ? BUSY_LIST : LIST_CAP;
    constexpr uint32_t REFUSED = 1u << 24;
    auto entry_query = [&](uint32_t m) __attribute__((always_inline)) {
        return (int)(((m >> 6 & 3u) * GB + (m >> 2) % GB) * 16 + (m >> 4 & 3u) * 4 + (m & 3u));
    };
    auto entry_row = [&](uint32_t m) __attribute__((always_inline)) { return (m >> 8 & 0xffu) + (BB > 1 ? (m >> 3 & 1u) * 16 : 0u); };
    uint32_t* tile_s = base_s + QT;                     // the tiles whose survivors the list holds
    uint32_t* total_s = tile_s + SCAN_LIST_TILES;
    uint32_t* allow_s = total_s + 4;                    // masked variant only
    uint32_t* exclude_s = allow_s + QT;
    uint64_t* cut_s = reinterpret_cast<uint64_t*>(total_s + 4);                 // EXACT: cuts and inverse norms of the tile's queries
    double* inv_s = reinterpret_cast<double*>(cut_s + QT);
    uint32_t count = 0;
    uint64_t cut = 0;
    double inv64 = 0.0;
    if constexpr (EXACT) {                              // (asked for together with the thresholds)
        static_assert(QT == 32 && MQ == 2 && MR == 4, "a bit per query, 16 bits per pair of row blocks");
        const int b = q0 + (lane & 31) < B ? q0 + (lane & 31) : 0;
        if (wave == 0) { count = *slot_counter(cnt, b); cut = exact_words(exact.words, b, exact.stride)[0]; inv64 = exact.invq64[b]; }
    }
    for (int i = tid; i < QT; i += NT) {
        const float th = thr[q0 + i];
        const uint16_t hi = enc16(th), lo = enc16(th - dec16(hi));
        thp_s[i] = hi | ((uint32_t)lo << 16);
        invq_s[i] = invq[q0 + i];
        cnt_s[i] = 0;
        if constexpr (MASKED) {                         // padding queries accept nothing
            allow_s[i] = q0 + i < B ? mask.allow[q0 + i] : 0u;
            exclude_s[i] = q0 + i < B ? mask.exclude[q0 + i] : 0u;
        }
    }
    if constexpr (EXACT) {
        // The queries of the tile that rows are looked for, a bit each: not the padding, not the lost, not those that no row can reach.
        if (wave == 0) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(q0 + (lane & 31) < B && count <= (uint32_t)L.cap && cut != ~0ull);
            if (lane == 0) total_s[1] = (uint32_t)m;
            if (lane < 32) { cut_s[lane] = cut; inv_s[lane] = inv64; base_s[lane] = 0; }
        }
    }
    if (tid == 0) { total_s[0] = 0; total_s[2] = 0; total_s[3] = 0; }
    uint32_t live = ~0u;                                // EXACT: see there

    // Accumulators: (re)initialised at the start of every tile by MFMAs with a zero C operand.
    // (An explicit re-zeroing inside the tile loop makes the compiler keep two copies of them.)
    f32x4_t acc[MQ][MR];

    // Steps per tile, made even so that the two register sets / LDS stages are in the same phase at
    // every tile boundary: an odd count gets one dummy step that multiplies the tile's last bank
    // block with an all-zero query block (the query operand holds one such block at index nkb).  (Rings turn by themselves.)
    const int real_steps = DT == 0 ? nkb * 2 : nkb;
    const int nsteps = RING ? real_steps : real_steps + (real_steps & 1);
    u32x4_t gbA[BCH], gbB[BCH], gqA[QCH], gqB[QCH];       // (gq: unless Q_DIRECT)

    // Bank and query loads run two steps ahead of the MFMAs.
    // Each tile walker starts its k-loop at a different k-block (the order of the k-blocks does not
    // matter for a dot product): workgroups run in near lock-step over tiles that are 2^n bytes
    // apart, and without the rotation they would all pull from the same few HBM channels at once.
    // Workgroups that share a walker's tiles start at the same one (RING: all of an XCD, which share the queries too), so that each of them finds in L2 what the first
    // one fetched (L2 misses of a pass over 1M x 1536 with 1024 queries: 104 M lines when they did not, 52 M, of which the bank is
    // 25 M; 2.52 -> 2.46 ms).
    const int rot = (int)((RING && nqt > 1 ? (unsigned)xcd * 3u : (unsigned)first_j * 7u) % (unsigned)real_steps);
    auto rotated = [&](int step) __attribute__((always_inline)) {   // logical step -> k-step actually loaded
        if (step >= real_steps) return step;                          // the dummy step stays last
        int k = step + rot;
        return k >= real_steps ? k - real_steps : k;
    };
    int ld_ti = 0, ld_step = 0, ldq_step = 0;
    // (the cursor step and the loads themselves are separate, so that the loads can be issued one
    // at a time between MFMAs)
    auto gnext_q = [&]() __attribute__((always_inline)) {
        const uint16_t* qb = qop + qop_row(2 * rotated(ldq_step), Bp) + q0 * 32;
        if (++ldq_step == nsteps) ldq_step = 0;
        return qb;
    };
    // A step's queries are two fragment rows (QT * 64 bytes each of this tile's), one behind the other in LDS.
    constexpr int QROW = QT * 4;                       // 16-byte pieces of a row
    const int64_t qrow_elems = qop_row(1, Bp);
    auto gpiece = [&](const uint16_t* base, int i) __attribute__((always_inline)) {
        if constexpr (NT <= QROW) return *reinterpret_cast<const u32x4_t*>(base + i * NT / QROW * qrow_elems + (i * NT % QROW + tid) * 8);
        else return *reinterpret_cast<const u32x4_t*>(base + tid / QROW * qrow_elems + tid % QROW * 8);
    };
    auto gpiece_bank = [&](const uint16_t* base, int i) __attribute__((always_inline)) {
        if constexpr (STREAM) return __builtin_bit_cast(u32x4_t, stream_load16(base + (i * NT + tid) * 8));
        else return *reinterpret_cast<const u32x4_t*>(base + (i * NT + tid) * 8);
    };
    auto gload_q = [&](u32x4_t (&gq)[QCH]) __attribute__((always_inline)) {
        const uint16_t* qb = gnext_q();
#pragma unroll
        for (int i = 0; i < QCH; ++i) gq[i] = gpiece(qb, i);
    };
    // first element of the bank tile the load cursor is on (recomputed only when the cursor moves on
    // to another tile: level_tile() contains an integer division)
    int64_t ld_tile_elem = level_tile(L, first_j) * nkb * (int64_t)BLOCK_ELEMS;
    auto gnext_b = [&]() __attribute__((always_inline)) {     // 16-bit stores only
        const int kb = ld_step < real_steps ? rotated(ld_step) : real_steps - 1;
        const uint16_t* blk = static_cast<const uint16_t*>(store_) + ld_tile_elem + kb * (int64_t)BLOCK_ELEMS;
        if (++ld_step == nsteps) {
            ld_step = 0;
            if (ld_ti + 1 < my_tiles) { ++ld_ti; ld_tile_elem = level_tile(L, first_j + ld_ti * stride_j) * nkb * (int64_t)BLOCK_ELEMS; }
        }
        return blk;
    };
    auto gload = [&](u32x4_t (&gb)[BCH]) __attribute__((always_inline)) {
        if constexpr (DT == 0) {
            const float* blk = static_cast<const float*>(store_) + ld_tile_elem + (rotated(ld_step) >> 1) * (int64_t)BLOCK_ELEMS + (rotated(ld_step) & 1) * 32;
#pragma unroll
            for (int i = 0; i < BCH; ++i) {
                int g = i * NT + tid, r = g >> 3, c4 = g & 7;
                if constexpr (STREAM) gb[i] = __builtin_bit_cast(u32x4_t, stream_load16(blk + r * KB + c4 * 4));
                else gb[i] = *reinterpret_cast<const u32x4_t*>(blk + r * KB + c4 * 4);
            }
            // past the last step the cursor stays on the last tile: the loads issued there are never
            // consumed, but keeping every step free of branches lets the loads stay in flight across it
            if (++ld_step == nsteps) {
                ld_step = 0;
                if (ld_ti + 1 < my_tiles) { ++ld_ti; ld_tile_elem = level_tile(L, first_j + ld_ti * stride_j) * nkb * (int64_t)BLOCK_ELEMS; }
            }
        } else {
            const uint16_t* blk = gnext_b();
#pragma unroll
            for (int i = 0; i < BCH; ++i) gb[i] = gpiece_bank(blk, i);
        }
    };
    auto lstore = [&](int s, u32x4_t (&gb)[BCH], u32x4_t (&gq)[QCH]) __attribute__((always_inline)) {
        if constexpr (DT == 0) {
#pragma unroll
            for (int i = 0; i < BCH; ++i) {
                int g = i * NT + tid, r = g >> 3, c4 = g & 7;
                float f0 = __uint_as_float(gb[i].x), f1 = __uint_as_float(gb[i].y);
                float f2 = __uint_as_float(gb[i].z), f3 = __uint_as_float(gb[i].w);
                float r0, r1, r2, r3;
                u32x2_t hi, lo;
                hi.x = pack_bf16x2_hi(f0, f1, r0, r1); hi.y = pack_bf16x2_hi(f2, f3, r2, r3);
                lo.x = cvt_pk_bf16(r0, r1);
                lo.y = cvt_pk_bf16(r2, r3);
                unsigned char* rowp = sbank(s) + r * 128 + (c4 & 1) * 8;
                *reinterpret_cast<u32x2_t*>(rowp + swz16(c4 >> 1, r) * 16) = hi;
                *reinterpret_cast<u32x2_t*>(rowp + swz16(4 + (c4 >> 1), r) * 16) = lo;
            }
        } else {
#pragma unroll
            for (int i = 0; i < BCH; ++i) *reinterpret_cast<u32x4_t*>(sbank(s) + (i * NT + tid) * 16) = gb[i];
        }
        if constexpr (!Q_DIRECT) {
#pragma unroll
            for (int i = 0; i < QCH; ++i) *reinterpret_cast<u32x4_t*>(sq(s) + (i * NT + tid) * 16) = gq[i];
        }
    };
    // Q_DIRECT: query blocks go from global memory straight to LDS (a lane's 16 bytes land at M0 + 16 * lane, and the
    // block's image in memory is its image in LDS), without registers and LDS stores.  The compiler does not see
    // these loads: what waits for them is the explicit count before the step's barrier.
    const uint32_t lds_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const uint32_t piece_at = (uint32_t)tid * 16u;
    auto qload_to_lds = [&](const uint16_t* qb, int s, int i) __attribute__((always_inline)) {
        const uint32_t to = lds_at + (uint32_t)(QUERY_AT + s * QT * 128 + i * NT * 16) + (uint32_t)__builtin_amdgcn_readfirstlane(wave) * 1024u;
        const uint64_t from = (uint64_t)(qb + i * NT / QROW * qrow_elems + i * NT % QROW * 8);   // (uniform; said so to the compiler)
        const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(from >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)from);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(piece_at), "s"(base) : "memory", "m0");
    };
    // Operand addresses.  Queries: fragments of 1 KB, k-step h in row h of the stage.  Bank row (block*16 + l16), logical chunk
    // c = 4*h + grp of k-step h: byte offset = block*2048 + l16*128 + ((c ^ f(l16)) * 16), the swizzle depending on l16 only.
    // The k-step enters through bit 6 only, so one per-lane offset per operand (the wave's first block folded in)
    // serves every block, both stages and both k-steps; the rest is a compile-time constant.
    const uint32_t offA0 = QUERY_AT + wq * MQ * 1024 + lane * 16, offB0 = l16 * 128 + swz16(grp, l16) * 16 + wr * MR * 2048;
    auto frag_a = [&](int s, int h, int block) __attribute__((always_inline)) {
        return *reinterpret_cast<const u32x4_t*>(smem + offA0 + (s * QT * 128 + h * QT * 64 + block * 1024));
    };
    auto frag_b = [&](int s, uint32_t off, int block) __attribute__((always_inline)) {
        return *reinterpret_cast<const u32x4_t*>(smem + off + (s * STAGE_BANK_BYTES + block * 2048));
    };
    // One step: the MFMAs on LDS stage s, and meanwhile the operands of the next step (registers gb, gq,
    // loaded a step and a half ago) go to stage s ^ 1, and the loads of the step two ahead go to the registers stored in the step before
    // (fp32 stores: of the step three ahead, to the registers just stored).
    // Inverse norms of this lane's MR bank rows of the next tile.  They are requested in the last
    // k-step of a tile (the fragment registers are free by then; across the whole k-loop there is
    // no register to spare, and a value that gets spilled has to be waited for right after its
    // request, which drains every load in flight) and turned into MFMA operands (tile_prepare)
    // after that tile's epilogue, by when they have long arrived.  The rare epilogue paths that
    // need an inverse norm of the current tile read it from memory again.  (RING, which has registers left: behind the last step.)
    float inv_n[MR];
    int tile_now = 0;
    auto load_invnorm = [&](int ti) __attribute__((always_inline)) {
        const int64_t t = level_tile(L, first_j + (ti < my_tiles ? ti : my_tiles - 1) * stride_j);
        const int row0 = (wr_u * MR) * 16 + (fresh_lane() & 15);
#pragma unroll
        for (int b = 0; b < MR; ++b) {
            const int64_t id = t * TILE_ROWS + row0 + b * 16;
            inv_n[b] = invnorm[id < N ? id : N - 1];
        }
    };

    // Operand fragments of the 16-bit path, carried from step to step.  A step has 2 MQ slots (k-step h, query block a); the
    // query fragment of slot g lies in af[g % RA], requested RA slots ahead.
    constexpr int RA = RING ? MQ : MQ < 4 ? MQ : 4, SLOTS = 2 * MQ, BARRIER = 3 * MQ / 2;
    u32x4_t af[RA], bfr[2][MR];
    auto compute = [&](int s, u32x4_t (&gb)[BCH], u32x4_t (&free)[BCH], u32x4_t (&gq)[QCH], auto fetch_next) __attribute__((always_inline)) {
        if constexpr (DT == 0) {
            // hi (chunks 0..3) and lo (4..7) of 32 elements: one k-step of three products
            if constexpr (Q_DIRECT) {
                const uint16_t* nq = gnext_q();                             // the next step's; stage s ^ 1 is free
#pragma unroll
                for (int i = 0; i < QCH; ++i) qload_to_lds(nq, s ^ 1, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            u32x4_t bh[MR], bl[MR];
            u32x4_t al = frag_a(s, 1, 0);
#pragma unroll
            for (int b = 0; b < MR; ++b) bh[b] = frag_b(s, offB0, b);
            u32x4_t ah = frag_a(s, 0, 0);
#pragma unroll
            for (int b = 0; b < MR; ++b) bl[b] = frag_b(s, offB0 ^ 64, b);
#pragma unroll
            for (int a = 0; a < MQ; ++a) {
                u32x4_t al1 = al, ah1 = ah;
                if (MQ < 8 && a + 1 < MQ) { al1 = frag_a(s, 1, a + 1); ah1 = frag_a(s, 0, a + 1); }
#pragma unroll
                for (int b = 0; b < MR; ++b) mfma16_in_place<1>(acc[a][b], al, bh[b]);     // (MR of them apart: no one waits for the one before)
#pragma unroll
                for (int b = 0; b < MR; ++b) mfma16_in_place<1>(acc[a][b], ah, bl[b]);
#pragma unroll
                for (int b = 0; b < MR; ++b) mfma16_in_place<1>(acc[a][b], ah, bh[b]);
                if (MQ == 8 && a + 1 < MQ) { al1 = frag_a(s, 1, a + 1); ah1 = frag_a(s, 0, a + 1); }   // (no registers to have them earlier)
                al = al1;
                ah = ah1;
                if (a == MQ / 2 - 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    lstore(s ^ 1, gb, gq);
                    if constexpr (!Q_DIRECT) gload_q(gq);
                    gload(gb);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
            // A software pipeline written out by hand, one slot per query block a of a k-step: the MFMAs of block a
            // (MR of them), then the LDS read of the fragment RA slots ahead into the registers those MFMAs have just
            // read, then one piece of the side work.  The bank fragments are used by every slot of a k-step and are
            // double buffered instead.  The global loads of bank pieces (first quarter of the slots) and the LDS stores (second and third)
            // issue in the shadow of the MFMAs instead of forming a period without any.  (Behind the barrier, in the last quarter, the loads
            // of all wavefronts met the first fragments' reads: 32 queries, 300,007 x 384 fp16, densest pass 44.6 us, 42.8 now; 64, 196,608 x
            // 1024 bf16 69.3, 67.8.  In kernel traces of whole calls the first of them takes 41 us, masked 46.)
            // The scheduler is fenced per slot to keep this order (left alone it hoists the reads).
            // On entry af and bfr[0] hold the step's first fragments, fetched by the previous step or, for
            // the first step of a tile, by the tile loop (the last step of a tile fetches nothing: the
            // fragments would only occupy registers that the tile epilogue needs).
            constexpr bool FETCH = decltype(fetch_next)::value;
            const uint16_t* nq = gnext_q();
            const uint16_t* nb = gnext_b();
#pragma unroll
            for (int g = 0; g < SLOTS; ++g) {
                const int h = g / MQ, a = g % MQ;
                // The step's only barrier: every wavefront has stored its share of stage s ^ 1 and has received all
                // it reads from stage s.  After the barrier
                // the last quarter's slots still have their operands in registers or requested, and fetch the first
                // fragments of the next step from stage s ^ 1, so the matrix pipe does not wait for LDS.
                if (g == BARRIER) {
                    __syncthreads();
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the bank pieces two steps ahead, into the registers that the last step has stored
                constexpr int Q1 = MQ / 2;                                  // slots of a quarter
                if (g < Q1) {
#pragma unroll
                    for (int i = g * BCH / Q1; i < (g + 1) * BCH / Q1; ++i) free[i] = gpiece_bank(nb, i);
                }
                // bank fragments: those of k-step 1 over the first slots, those of the next step behind the barrier
                constexpr int BPS = (2 * MR + MQ - 1) / MQ;               // per slot
                if (g < MQ / 2) {
#pragma unroll
                    for (int b = g * BPS; b < (g + 1) * BPS && b < MR; ++b) bfr[1][b] = frag_b(s, offB0 ^ 64, b);
                }
                if (FETCH && g >= BARRIER) {
                    // query fragments whose registers were free before stage s ^ 1 could be read
                    if (g == BARRIER) {
#pragma unroll
                        for (int f = SLOTS - RA; f < BARRIER; ++f) af[f % RA] = frag_a(s ^ 1, 0, f + RA - SLOTS);
                    }
#pragma unroll
                    for (int b = (g - BARRIER) * BPS; b < (g - BARRIER + 1) * BPS && b < MR; ++b) bfr[0][b] = frag_b(s ^ 1, offB0, b);
                }
#pragma unroll
                for (int b = 0; b < MR; ++b) mfma16_in_place<DT>(acc[a][b], af[g % RA], bfr[h][b]);
                if (g + RA < SLOTS) {
                    const int f = g + RA;
                    af[g % RA] = frag_a(s, f / MQ, f % MQ);
                } else if (FETCH && g >= BARRIER) {
                    af[g % RA] = frag_a(s ^ 1, 0, g + RA - SLOTS);
                }
                // the bank pieces: stored over the second and third quarter of the slots
                if (g >= Q1 && g < BARRIER) {
#pragma unroll
                    for (int i = (g - Q1) * BCH / (2 * Q1); i < (g - Q1 + 1) * BCH / (2 * Q1); ++i)
                        *reinterpret_cast<u32x4_t*>(sbank(s ^ 1) + (i * NT + tid) * 16) = gb[i];
                }
                // the query pieces: stored over the second quarter, reloaded over the third
                if (g >= Q1 && g < MQ) {
#pragma unroll
                    for (int i = (g - Q1) * QCH / Q1; i < (g - Q1 + 1) * QCH / Q1; ++i)
                        *reinterpret_cast<u32x4_t*>(sq(s ^ 1) + (i * NT + tid) * 16) = gq[i];
                }
                if (g >= MQ && g < BARRIER) {
#pragma unroll
                    for (int i = (g - MQ) * QCH / Q1; i < (g - MQ + 1) * QCH / Q1; ++i) gq[i] = gpiece(nq, i);
                }
                if (!FETCH && g == SLOTS - 1) load_invnorm(tile_now + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // RING: one step (a k-block) of the 16-bit path with 128 or 256 queries to a tile, in two halves of 32 k.  A half is two spells: fetch (8 or
    // 12 fragments from LDS to registers, two or four loads of 1 KB from memory to LDS) and multiply (16 or 32 matrix instructions).  A barrier ends
    // every spell, and the last four wavefronts -- the second one of every SIMD -- are a spell behind the first four, so on each SIMD one
    // multiplies while the other fetches.  The first four load queries, half a block a time, the others bank blocks, so that neither waits
    // for the other's loads (a wavefront's loads are waited for in order).
    //   queries: in the fetch of half i, half i + 2 goes to the place of half i - 1, which the second four have read a spell ago;
    //            it is waited for before the barrier that ends the multiplication of half i + 1 (one batch of QL loads comes after it)
    //   bank:    in the fetches of the two halves of block m, block m + 2 goes to the place of block m - 1; it is waited for
    //            at the end of the fetch of the second half of block m + 1 (eight loads come after it), before the barrier behind which
    //            the first four read it
    // A tile begins with the first four a spell ahead and ends with both done, so the epilogue is everyone's at the same time and its
    // barriers are met by all: both groups pass four barriers a step.
    int wave_opaque = __builtin_amdgcn_readfirstlane(wave);
    auto second = [&]() __attribute__((always_inline)) {       // one of the last four wavefronts?  Compared anew each time: a scalar
        asm volatile("" : "+s"(wave_opaque));                  // compare and branch, not a lane mask kept
        return wave_opaque >= 4;
    };
    const int wave_u = __builtin_amdgcn_readfirstlane(wave) & 3;
    uint32_t at_bank = 0, at_query = 0;                        // ring places of this step's bank block, of this half's queries
    const char* src = nullptr;                                 // this lane's next piece, and where to
    uint32_t dst = 0;
    const uint32_t piece0 = (uint32_t)wave_u * 1024u + (uint32_t)lane * 16u;
    // (per-lane addresses: a scalar one that a vector instruction has made would need five wait states, which nobody would add here)
    auto ring_load = [&](bool bank) __attribute__((always_inline)) {
        const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)dst);
        if (STREAM && bank) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(to), "v"(src) : "memory", "m0");
        else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(to), "v"(src) : "memory", "m0");
        src += 4096;
        dst += 4096;
    };
    constexpr int QL = QT / 64;                                // loads of half a query block, of one of the four
    constexpr auto wait_vm = [](int n) { return 0x0f70 | (n & 15) | (n >> 4) << 14; };       // s_waitcnt vmcnt(n)
    auto ring_step = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (second()) __syncthreads();                       // a spell behind
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t a0 = offA0 + at_query, b0 = (h ? offB0 ^ 64 : offB0) + at_bank;
#pragma unroll
            for (int b = 0; b < MR; ++b) bfr[0][b] = *reinterpret_cast<const u32x4_t*>(smem + b0 + b * 2048);
#pragma unroll
            for (int a = 0; a < MQ; ++a) af[a] = *reinterpret_cast<const u32x4_t*>(smem + a0 + a * 1024);
            __builtin_amdgcn_sched_barrier(0);
            if (second()) {
                if (h == 0) {
                    src = reinterpret_cast<const char*>(gnext_b()) + piece0;
                    dst = lds_at + (at_bank == 0 ? (RING_PLACES - 1) * STAGE_BANK_BYTES : at_bank - STAGE_BANK_BYTES) + wave_u * 1024;
                }
#pragma unroll
                for (int p = 0; p < 4; ++p) ring_load(true);
                if (h == 1) __builtin_amdgcn_s_waitcnt(wait_vm(8 * (RING_PLACES - 2)));
            } else {
                if (h == 0) src = reinterpret_cast<const char*>(gnext_q()) + piece0;
                else src += qrow_elems * 2 - QL * 4096;
                dst = lds_at + QUERY_AT + (at_query == 0 ? (RING_PLACES - 1) * QT * 64 : at_query - QT * 64) + wave_u * 1024;
#pragma unroll
                for (int p = 0; p < QL; ++p) ring_load(false);
            }
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < MQ; ++a)
#pragma unroll
                for (int b = 0; b < MR; ++b) mfma16_in_place<DT>(acc[a][b], af[a], bfr[0][b]);
            __builtin_amdgcn_sched_barrier(0);
            if (!second()) {
                __builtin_amdgcn_s_waitcnt(wait_vm(QL));
                __syncthreads();
            }
            __builtin_amdgcn_sched_barrier(0);
            at_query = at_query == (RING_PLACES - 1) * QT * 64 ? 0u : at_query + QT * 64;
        }
        at_bank = at_bank == (RING_PLACES - 1) * STAGE_BANK_BYTES ? 0u : at_bank + STAGE_BANK_BYTES;
    };

    // Key of a survivor from its accumulator value (score - threshold * norm, see tile_init): the
    // threshold term is added back exactly as the MFMA formed it, then the cosine is taken.
    auto finish_key = [&](float av, int ql, int32_t id, float inv) __attribute__((always_inline)) {
        const float norm = __builtin_amdgcn_rcpf(inv);
        const float nh = dec16(enc16(norm)), nl = dec16(enc16(norm - nh));
        const uint32_t tp = thp_s[ql];
        const float th = dec16((uint16_t)(tp & 0xffffu)), tl = dec16((uint16_t)(tp >> 16));
        const float dot = av + (th * nh + th * nl + tl * nh);
        return pack_key(dot * inv * invq_s[ql], id);
    };

    // Write the workgroup's staged survivors to the per-query lists (all lanes call it together):
    // count the entries of each query with LDS atomics, reserve that many slots with one device-wide
    // integer atomic per query that has any, copy.
    auto flush = [&](uint32_t list_at) __attribute__((always_inline)) {
        const uint64_t* list = reinterpret_cast<const uint64_t*>(smem + list_at);
        const uint32_t total = *total_s < LIST_ROOM ? *total_s : LIST_ROOM;
        for (uint32_t e = tid; e < total; e += NT) {
            const uint32_t m = (uint32_t)list[e];
            if (!(MASKED && (m & REFUSED))) atomicAdd(cnt_s + entry_query(m), 1u);
        }
        __syncthreads();
        for (int i = tid; i < QT; i += NT) {
            uint32_t c = cnt_s[i];
            base_s[i] = c ? atomicAdd(slot_counter(cnt, q0 + i), c) : 0u;
            cnt_s[i] = 0;
        }
        __syncthreads();
        // four entries per lane at a time, so that their inverse-norm reads are in flight together
        for (uint32_t e0 = tid; e0 < total; e0 += 4 * NT) {
            float inv[4];
            uint64_t ent[4];
            int32_t id[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t e = e0 + k * NT;
                ent[k] = list[e < total ? e : e0];
                id[k] = (int32_t)(tile_s[(uint32_t)ent[k] >> 16 & 0xffu] * TILE_ROWS + entry_row((uint32_t)ent[k]));
                inv[k] = invnorm[id[k]];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t e = e0 + k * NT;
                if (e < total && !(MASKED && ((uint32_t)ent[k] & REFUSED))) {
                    const int ql = entry_query((uint32_t)ent[k]);
                    const uint32_t pos = atomicAdd(base_s + ql, 1u);           // (the order in a list is of no account)
                    if (pos < (uint32_t)L.cap) surv[(int64_t)(q0 + ql) * L.cap + pos] = finish_key(__uint_as_float((uint32_t)(ent[k] >> 32)), ql, id[k], inv[k]);
                }
            }
        }
        // Nothing of this is in flight when the k-loop goes on (a wait that the compiler knows of): a register that it has to take
        // for a load's target would otherwise be waited for at the top of every step, and with it every load before it.
        __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0)
        __syncthreads();
        if (tid == 0) *total_s = 0;
        __syncthreads();
    };

    // EXACT: the staged rows are scored again in fp64, 16 lanes to a row and query, and a row whose key reaches the query's cut goes to its
    // list.  About k1 * rho rows per query and pass come here.  A lane group takes the next row that none has taken, and scores it for its
    // queries one after the other, 48 chunks to a step, the next step's on their way while one is used.  Where many queries are near the same rows
    // (masses of near-ties, which only the margin lets through) the groups are at the same query most of the time, so that rows and
    // queries are found in the compute unit's cache.  Against pairs staged
    // one by one and scored one after the other (1M x 1024 bf16, whole call, us, four, 16 and 64 queries): 390, 455, 781 -> 386, 420, 665;
    // 100,000 rows within the margin of all of them 841, 1625, 4559 -> 585, 1260, 3771; 20,000 such rows in a run, whose queries were lost for want
    // of room, 647, 2823, 7417 -> 550, 1528, 2918.  Rows of 64 fp16 pay for the longer code: two queries over 1M, densest pass 53 -> 58.
    // A workgroup that meets most of a query's rows (near-duplicates appended one after the other) would score them alone while the others
    // have none: once it has scored more than 2048 pairs, a query with more than most_rows of them is lost, and walks the bank.
    uint32_t* taken_s = total_s + 2;                           // rows taken; pairs scored; base_s: those of a query
    auto flush_exact = [&]() __attribute__((always_inline)) {
        constexpr int EPC = DT == 0 ? 4 : 8, U = 3;            // elements per 16-byte chunk; chunks to a step
        static_assert(!EXACT || WQ == 1, "a wavefront's number is that of its rows");
        const int lane = fresh_lane(), sub = lane & 15, nch = nkb * KB / EPC;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane((int)*total_s);      // (never more than the list holds)
        // What a lane group fetches next; all that follows is uniform within it.
        struct Step { u32x4_t x[U]; float4 y[U][EPC / 4]; int32_t id; int q, c; };       // c: first chunk; q < 0: none left
        int32_t id = 0;
        uint32_t left = 0;                                     // queries of the row
        int at = 0;
        auto next_pair = [&]() __attribute__((always_inline)) {
            left &= left - 1;
            for (;;) {
                while (left == 0) {
                    uint32_t row = 0;
                    if (sub == 0) row = atomicAdd(taken_s, 1u);
                    row = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)row, 0x150, 0xf, 0xf, true);       // of the first of 16 lanes
                    if (row >= total) return;
                    id = (int32_t)(uint32_t)list_s[row];
                    left = (uint32_t)(list_s[row] >> 32) & live;
                }
                const int q = __builtin_ctz(left);
                if (taken_s[1] <= (uint32_t)LIST_CAP || base_s[q] <= (uint32_t)exact.most_rows) return;
                if (sub == 0) atomicMax(slot_counter(cnt, q0 + q), (uint32_t)L.cap + 1u);
                left &= left - 1;
            }
        };
        auto fetch = [&](Step& st) __attribute__((always_inline)) {
            st.id = id;
            st.q = left != 0 ? __builtin_ctz(left) : -1;
            st.c = at;
            const float4* y = reinterpret_cast<const float4*>(exact.qf + (int64_t)(q0 + (st.q < 0 ? 0 : st.q)) * (nkb * KB));    // (none left: loaded, not used)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = at + sub + 16 * u < nch ? at + sub + 16 * u : nch - 1;     // past the end: loaded, not used
                if constexpr (DT == 0) st.x[u] = *reinterpret_cast<const u32x4_t*>(static_cast<const float*>(store_) + off32(id, c, nkb));
                else st.x[u] = *reinterpret_cast<const u32x4_t*>(static_cast<const uint16_t*>(store_) + off16(id, c, nkb));
#pragma unroll
                for (int i = 0; i < EPC / 4; ++i) st.y[u][i] = y[c * (EPC / 4) + i];
            }
            __builtin_amdgcn_sched_barrier(0);
            at += 16 * U;
            if (at >= nch) { at = 0; next_pair(); }
        };
        double dot = 0.0, ssq = 0.0;
        auto use = [&](const Step& st) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (st.c + sub + 16 * u >= nch) break;
#pragma unroll
                for (int k = 0; k < EPC; ++k) {
                    double xd;
                    if constexpr (DT == 0) xd = __uint_as_float(st.x[u][k]);
                    else xd = DT == 1 ? bf16_to_f((uint16_t)(st.x[u][k >> 1] >> (16 * (k & 1)))) : f16_to_f((uint16_t)(st.x[u][k >> 1] >> (16 * (k & 1))));
                    const float4 yk = st.y[u][k >> 2];
                    const double yd = (k & 3) == 0 ? yk.x : (k & 3) == 1 ? yk.y : (k & 3) == 2 ? yk.z : yk.w;
                    dot += xd * yd;
                    ssq += xd * xd;
                }
            }
            if (st.c + 16 * U < nch) return;
            dot = row16_sum(dot);
            ssq = row16_sum(ssq);
            if (sub == 0) {
                atomicAdd(taken_s + 1, 1u);
                atomicAdd(base_s + st.q, 1u);
                const uint64_t key = exact_key(dot * inv_s[st.q] * (1.0 / sqrt(ssq)), st.id);
                if (key >= cut_s[st.q]) {
                    const uint32_t pos = atomicAdd(slot_counter(cnt, q0 + st.q), 1u);
                    if (pos < (uint32_t)L.cap) surv[(int64_t)(q0 + st.q) * L.cap + pos] = key;
                }
            }
            dot = 0.0;
            ssq = 0.0;
        };
        Step a, b;
        next_pair();
        if (left != 0) {
            fetch(a);
            for (;;) {
                fetch(b);
                use(a);
                if (b.q < 0) break;
                fetch(a);
                use(b);
                if (a.q < 0) break;
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0), as above
        __syncthreads();
        if (taken_s[1] > (uint32_t)LIST_CAP) live &= ~(uint32_t)__builtin_amdgcn_ballot_w64(lane < 32 && base_s[lane & 31] > (uint32_t)exact.most_rows);
        if (tid == 0) { total_s[0] = 0; taken_s[0] = 0; }
        __syncthreads();
    };

    // Start of a tile.  The accumulators are not zeroed but initialised, by one MFMA per block,
    // with  - threshold[query] * norm[row] : the filter  score * invnorm >= threshold  is
    // score - threshold * norm >= 0, so after the k-loop the epilogue only has to look at signs.
    // The operands are a 3-term extension, query side (th, th, tl), bank side -(nh, nl, nh), with
    // threshold = th + tl and norm = nh + nl in the operands' 16-bit type (the dropped tl*nl term and
    // the residuals are ~2^-16 relative, inside the margin).  The sparsest pass has no threshold: its
    // query-side extension is zero and the accumulators start at zero.
    // Norm operands of the tile about to start, from the inverse norms requested a tile earlier.
    // EXACT: rows whose norm these operands cannot carry, a bit per block.  Bits 0 .. 3: they are staged whatever comes out here; bits 4 .. 7:
    // zero rows, which are not; bits 8 .. 11: rows with an infinite inverse norm, zero or not (the epilogue looks).
    uint32_t bx[MR], by[MR], odd = 0;
    auto tile_prepare = [&]() __attribute__((always_inline)) {
        const bool none = fresh_lane() >= 16;                      // only the first chunk of the extension is used
#pragma unroll
        for (int b = 0; b < MR; ++b) {
            const float norm = __builtin_amdgcn_rcpf(inv_n[b]);   // finish_key() forms it the same way
            const uint16_t nh = enc16(norm), nl = enc16(norm - dec16(nh));
            const uint32_t mh = nh ^ 0x8000u, ml = nl ^ 0x8000u;
            bx[b] = none ? 0u : (mh | (ml << 16));
            by[b] = none ? 0u : mh;
        }
        if constexpr (EXACT) {
            odd = 0;
            bool all_fit = true;
#pragma unroll
            for (int b = 0; b < MR; ++b) all_fit = all_fit && exact_norm_fits(inv_n[b]);
            if (__builtin_amdgcn_ballot_w64(!all_fit) != 0) {          // uniform, and seldom
#pragma unroll
                for (int b = 0; b < MR; ++b) odd |= exact_norm_fits(inv_n[b]) ? 0u : inv_n[b] == INFINITY ? 0x110u << b : 1u << b;
            }
        }
    };
    auto tile_init = [&](int ti) __attribute__((always_inline)) {
        const bool use_thr = L.rho != 0;
        const int ln = fresh_lane();
        uint32_t th[MQ];                                           // (all requested before the first is used)
#pragma unroll
        for (int a = 0; a < MQ; ++a) th[a] = thp_s[(wq_u * MQ + a) * 16 + (ln & 15)];
#pragma unroll
        for (int a = 0; a < MQ; ++a) {
            const uint32_t tp = use_thr && ln < 16 ? th[a] : 0u;
            const u32x4_t aext = {(tp & 0xffffu) | (tp << 16), tp >> 16, 0u, 0u};
#pragma unroll
            for (int b = 0; b < MR; ++b) {
                const u32x4_t bext = {bx[b], by[b], 0u, 0u};
                const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
                acc[a][b] = mfma16<TT>(aext, bext, z);
            }
        }
    };

    // ---- per-tile epilogue (all lanes of the workgroup call it together) ----
    int since = 0;                                             // tiles whose survivors the list holds
    auto epilogue = [&](int ti, uint32_t list_at) __attribute__((always_inline)) {
        const int j = first_j + ti * stride_j;
        const int64_t t = level_tile(L, j);
        if (L.rho == 0) {
            // Sparsest pass: no threshold yet, every row is kept.  Slot = position of the row in
            // this pass, so no counter is needed (the count was preset to the pass's valid rows).
#pragma unroll
            for (int b = 0; b < MR; ++b) {
                const int ln = fresh_lane();
                const int rt = (wr_u * MR + b) * 16 + (ln & 15);
                const int64_t id = t * TILE_ROWS + rt;
                if (id < N) {
                    const float inve = invnorm[id];
                    uint32_t tag = 0;
                    if constexpr (MASKED) tag = mask.tags[id];
                    const int64_t pos = (int64_t)j * TILE_ROWS + rt;
#pragma unroll
                    for (int a = 0; a < MQ; ++a) {
                        int opq = 0;
                        asm volatile("" : "+v"(opq));
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int ql = (wq_u * MQ + a) * 16 + 4 * ((ln >> 4) + opq) + r;
                            const bool ok = !MASKED || eligible(tag, allow_s[ql], exclude_s[ql]);
                            surv[(int64_t)(q0 + ql) * L.cap + pos] = ok ? pack_key(acc[a][b][r] * inve * invq_s[ql], (int32_t)id) : 0ull;   // 0 = empty slot
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        } else {
            // Filter against the per-query thresholds.  Survivors (rare) go to a workgroup list in
            // LDS first, so that the global slot counters are bumped once per (workgroup, query)
            // and all at the same time, instead of one dependent device-wide atomic per survivor.
            // The accumulators hold  score - threshold * norm  (see tile_init): survivors are the
            // non-negative values.
            if constexpr (!EXACT) { if (threadIdx.x == 0) tile_s[since] = (uint32_t)t; }     // (a barrier comes before it is read)
            // Pass 1.  Per group and lane a 16-bit mask of the non-negative accumulators, built from the
            // sign bits with one funnel shift per register (no test for "no survivor here"
            // first: at the survivor rates of the dense passes nearly every wavefront has some).
            auto group = [&](int g, int bg) __attribute__((always_inline)) {
                AccGroup v;
#pragma unroll
                for (int r = 0; r < 16; ++r) v.v[r] = acc[g * GB + (r >> 2) % GB][bg * BB + (r >> 2) / GB][r & 3];
                return v;
            };
            uint32_t msk[GROUPS * RGROUPS];
            uint32_t mine = 0;
            const int rows_here = N - t * TILE_ROWS < TILE_ROWS ? (int)(N - t * TILE_ROWS) : TILE_ROWS;
            uint32_t asked = ~0u, staged = 0, dropped = 0;               // EXACT: this lane's queries (16 bits), and its rows that are
            if constexpr (EXACT) {                                       // staged and dropped whatever the accumulators say (8 bits a row block)
                const int g4 = 4 * (fresh_lane() >> 4);
                asked = (live >> g4 & 0xfu) | (live >> (g4 + 12) & 0xf0u);
                asked |= asked << 8;
                // An infinite inverse norm: zeros, or a norm below 2^-74 whose squares vanished, and such a row has a similarity.  (Not in
                // fp16.)  So these rows are looked at, 16 KB by a wavefront at a time: with a row in five zero, 1M x 1024 bf16, four
                // queries, 470 us a call, 398 without any (621 with eight rows and two steps of a loop over their pieces at a time).
                if constexpr (DT != 2) {
                    uint64_t todo = 0, solid = 0;                        // the wavefront's rows, 16 to a block
#pragma unroll
                    for (int b = 0; b < MR; ++b) todo |= (__builtin_amdgcn_ballot_w64((odd >> (8 + b) & 1u) != 0) & 0xffffull) << (16 * b);
                    const int ln = fresh_lane(), nch = nkb * KB / (DT == 0 ? 4 : 8);
                    const int64_t id0 = t * TILE_ROWS + wr_u * MR * 16;  // (past the bank's end: in the tile's storage, not valid below)
                    int c0 = 0;
                    while (todo != 0) {                                  // uniform
                        constexpr int U = 16;
                        u32x4_t x[U];
                        int at[U];                                       // (past the last row: the last piece again)
#pragma unroll
                        for (int i = 0; i < U; ++i) {
                            at[i] = todo != 0 ? __builtin_ctzll(todo) : at[i > 0 ? i - 1 : 0];
                            const int c = c0 + ln < nch ? c0 + ln : nch - 1;
                            if constexpr (DT == 0) x[i] = *reinterpret_cast<const u32x4_t*>(static_cast<const float*>(store_) + off32(id0 + at[i], c, nkb));
                            else x[i] = *reinterpret_cast<const u32x4_t*>(static_cast<const uint16_t*>(store_) + off16(id0 + at[i], c, nkb));
                            c0 += 64;
                            if (c0 >= nch) { c0 = 0; todo &= todo - 1; }
                        }
                        __builtin_amdgcn_sched_barrier(0);               // all of them requested before the first is used
#pragma unroll
                        for (int i = 0; i < U; ++i) {
                            const uint32_t any = (x[i][0] | x[i][1] | x[i][2] | x[i][3]) & (DT == 0 ? 0x7fffffffu : 0x7fff7fffu);
                            solid |= __builtin_amdgcn_ballot_w64(any != 0) != 0 ? 1ull << at[i] : 0ull;
                        }
                    }
#pragma unroll
                    for (int b = 0; b < MR; ++b)
                        if (solid >> (16 * b + (ln & 15)) & 1ull) odd = (odd & ~(0x10u << b)) | 1u << b;
                }
                if (__builtin_amdgcn_ballot_w64(odd != 0) != 0) {        // uniform
                    auto spread = [](uint32_t rows) __attribute__((always_inline)) { return ((rows & 0xfu) * 0x00204081u & 0x01010101u) * 0xffu; };   // bit b -> byte b
                    staged = spread(odd);
                    dropped = spread(odd >> 4);
                }
            }
#pragma unroll
            for (int bg = 0; bg < RGROUPS; ++bg) {
                uint32_t valid = 0;
#pragma unroll
                for (int i = 0; i < BB; ++i)
                    valid |= (wr_u * MR + bg * BB + i) * 16 + (fresh_lane() & 15) < rows_here ? ((1u << (4 * GB)) - 1u) << (4 * GB * i) : 0u;
#pragma unroll
                for (int g = 0; g < GROUPS; ++g) {
                    uint32_t neg = 0;                                    // sign bits, register 15 first
                    const AccGroup v = group(g, bg);
#pragma unroll
                    for (int r = 15; r >= 0; --r) neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(v.v[r]), 31);
                    const uint32_t m = (EXACT ? ((~neg & ~(dropped >> (16 * bg))) | staged >> (16 * bg)) & asked : ~neg) & valid;
                    msk[g * RGROUPS + bg] = m;
                    mine += __popc(m);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // EXACT: the list takes rows, each with the queries that it may reach; so there is room for every row of a tile, and the four
            // lanes that hold a row's queries put them together.
            if constexpr (EXACT) {
                if (__builtin_amdgcn_ballot_w64(mine != 0) != 0) {      // uniform within the wavefront
                    const int ln = fresh_lane(), g = ln >> 4;
                    uint32_t queries = 0;                               // of row 16 * g + (ln & 15) of the wavefront's 64
#pragma unroll
                    for (int b = 0; b < MR; ++b) {
                        const uint32_t m = msk[b / BB] >> (8 * (b % BB)) & 0xffu;       // this lane's of row block b
                        uint32_t all = (m & 0xfu) << (4 * g) | (m >> 4) << (16 + 4 * g);
                        const auto s16 = __builtin_amdgcn_permlane16_swap(all, all, false, false);
                        all = s16[0] | s16[1];
                        const auto s32 = __builtin_amdgcn_permlane32_swap(all, all, false, false);
                        all = s32[0] | s32[1];
                        queries = g == b ? all : queries;
                    }
                    const uint64_t rows = __builtin_amdgcn_ballot_w64(queries != 0);
                    uint32_t at = 0;
                    if (ln == 0) at = atomicAdd(total_s, (uint32_t)__popcll(rows));
                    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(rows & ((1ull << ln) - 1ull));
                    if (queries != 0) list_s[at] = (uint64_t)queries << 32 | (uint32_t)(t * TILE_ROWS + wr_u * MR * 16 + ln);
                }
            }
            // Slots: a prefix sum over the wavefront, one LDS atomic per wavefront for its total.
            else if (__builtin_amdgcn_ballot_w64(mine != 0) != 0) {     // uniform within the wavefront
                const uint32_t incl = wave_inclusive_sum(mine);
                const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                uint32_t wave_base = 0;
                if (fresh_lane() == 0) wave_base = atomicAdd(total_s, sum);
                wave_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_base);
                uint32_t slot = wave_base + incl - mine;
                // what is the same in all of this lane's entries: tile, row in block 0, lane group
                const int ln0 = fresh_lane();
                const uint32_t where0 = (uint32_t)since << 16 | (uint32_t)(wr_u * MR * 16 + (ln0 & 15)) << 8 | (uint32_t)(wq_u * GROUPS << 6) | (uint32_t)(ln0 >> 4) << 4;
                // Pass 2, survivors only, all lanes in parallel: each lane takes the first set bit of its
                // own mask, fetches that accumulator register with a two-level select (registers cannot
                // be indexed per lane) and stages (value, row id, query); the key is finished when the
                // list is flushed.  The first round over the groups is straight-line code, so that the
                // groups' instructions interleave; lanes that hold a second survivor of one group (few)
                // are served by a loop afterwards.
                auto pick = [&](int g, int bg, int r) __attribute__((always_inline)) {
                    const int lo = r & 3, hi = (r >> 2) & 3;
                    return lane_select16(group(g, bg), __builtin_amdgcn_ballot_w64(lo == 1), __builtin_amdgcn_ballot_w64(lo == 3),
                                         __builtin_amdgcn_ballot_w64(lo >= 2), __builtin_amdgcn_ballot_w64(hi == 1),
                                         __builtin_amdgcn_ballot_w64(hi == 3), __builtin_amdgcn_ballot_w64(hi >= 2));
                };
                auto stage_one = [&](int g, int bg, int r, float av) __attribute__((always_inline)) {   // lanes with a survivor
                    const int ln = fresh_lane();
                    const uint32_t rt = (uint32_t)((wr_u * MR + bg * BB + ((r >> 2) & 3) / GB) * 16 + (ln & 15));
                    const int32_t id = (int32_t)(t * TILE_ROWS + rt);
                    const int ql = (wq_u * MQ + g * GB + ((r >> 2) & 3) % GB) * 16 + 4 * (ln >> 4) + (r & 3);
                    bool ok = true;
                    if constexpr (MASKED) ok = eligible(mask.tags[id], allow_s[ql], exclude_s[ql]);
                    if (slot < LIST_ROOM) {
                        *reinterpret_cast<uint64_t*>(smem + list_at + slot * 8u) = (uint64_t)__float_as_uint(av) << 32 | where0 + (uint32_t)(bg * BB * 16 << 8 | g << 6 | r) | (ok ? 0u : REFUSED);   // the slot was reserved before the check
                    } else if (ok) {   // list full (a very loose threshold): fall back to the direct path
                        uint32_t pos = atomicAdd(slot_counter(cnt, q0 + ql), 1u);
                        if (pos < (uint32_t)L.cap) surv[(int64_t)(q0 + ql) * L.cap + pos] = finish_key(av, ql, id, invnorm[id]);
                    }
                    ++slot;
                };
                // First round, the common case kept free of inner branches: lanes with exactly one survivor in
                // a group stage it; lanes with more are left to the loop below, and so is everything when the
                // wavefront's reservation does not fit the list (then no lane needs a room check here).
                uint32_t rest = 0;
                const bool fits = wave_base + sum <= LIST_ROOM;                                // uniform
                // (a group of two row blocks: the rows past the bank's end must not be a group's maximum)
                const bool whole = (t + 1) * TILE_ROWS <= N;                                   // uniform
                unsigned char* pk = smem + list_at + slot * 8u;                                // the lane's next list entry
#pragma unroll
                for (int bg = 0; bg < RGROUPS; ++bg)
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g) {
                        const uint32_t m = msk[g * RGROUPS + bg];
                        const bool take = fits && __popc(m) == 1 && (BB == 1 || whole);
                        if (take) {
                            const int r = __builtin_ctz(m);
                            const float av = only_non_negative(group(g, bg));
                            uint32_t where = where0 + (uint32_t)(bg * BB * 16 << 8 | g << 6) + (uint32_t)r;
                            if constexpr (MASKED) {                                            // the slot was reserved before the check
                                const int ql = entry_query(where);
                                where |= eligible(mask.tags[t * TILE_ROWS + entry_row(where)], allow_s[ql], exclude_s[ql]) ? 0u : REFUSED;
                            }
                            *reinterpret_cast<uint64_t*>(pk) = (uint64_t)__float_as_uint(av) << 32 | where;
                            pk += 8;
                        }
                        const uint32_t left = take ? 0u : m;
                        msk[g * RGROUPS + bg] = left;
                        rest |= left;
                    }
                slot = ((uint32_t)(pk - smem) - list_at) >> 3;
                if (__builtin_amdgcn_ballot_w64(rest != 0) != 0) {
#pragma unroll
                    for (int bg = 0; bg < RGROUPS; ++bg)
#pragma unroll
                        for (int g = 0; g < GROUPS; ++g) {
                            uint32_t m = msk[g * RGROUPS + bg];
                            while (__builtin_amdgcn_ballot_w64(m != 0) != 0) {
                                const int r = __builtin_ctz(m | 0x10000u);
                                const float av = pick(g, bg, r);
                                if (m) stage_one(g, bg, r, av);
                                m &= m - 1;
                            }
                        }
                }
            }
            // The list is carried from tile to tile and written out every `flush_every` tiles (the host
            // sizes that from the expected number of survivors per tile; a surplus takes the direct
            // path above) and once at the end, so the device-wide round trip is paid every few tiles.
            if constexpr (EXACT) {                             // (no wavefront gets to the next tile's epilogue before all have looked)
                __syncthreads();
                static_assert(LIST_CAP / 4 + TILE_ROWS <= LIST_CAP, "room for the rows of another tile");
                if (*total_s > (uint32_t)LIST_CAP / 4 || ti == my_tiles - 1) flush_exact();      // uniform
            } else if (BUSY || since == flush_every - 1 || ti == my_tiles - 1) {  // uniform
                __syncthreads();
                flush(list_at);
                since = 0;
            } else {
                ++since;
            }
        }
    };

    // ---- pipeline over the flattened (tile, k-block) sequence; g counts steps over all tiles ----
    auto phase = [&](int s, u32x4_t (&gb)[BCH], u32x4_t (&free)[BCH], u32x4_t (&gq)[QCH], auto fetch_next) __attribute__((always_inline)) {
        compute(s, gb, free, gq, fetch_next);
        if constexpr (DT == 0) {
            if constexpr (Q_DIRECT) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(BCH) : "memory");   // the query block: only the bank pieces came after it
            __syncthreads();
        }
    };
    if constexpr (RING) {
        static_assert(NT == 512, "four wavefronts for the queries, four for the bank");
        if (second()) {
#pragma unroll
            for (int i = 0; i < RING_PLACES - 1; ++i) {
                src = reinterpret_cast<const char*>(gnext_b()) + piece0;
                dst = lds_at + i * STAGE_BANK_BYTES + wave_u * 1024;
                for (int p = 0; p < 8; ++p) ring_load(true);
            }
            __builtin_amdgcn_s_waitcnt(wait_vm(8 * (RING_PLACES - 2)));
        } else {
            src = reinterpret_cast<const char*>(gnext_q()) + piece0;
            dst = lds_at + QUERY_AT + wave_u * 1024;
            for (int p = 0; p < QL; ++p) ring_load(false);
            src += qrow_elems * 2 - QL * 4096;
            for (int p = 0; p < QL; ++p) ring_load(false);
            __builtin_amdgcn_s_waitcnt(wait_vm(QL));
        }
        __syncthreads();
        load_invnorm(0);
        tile_prepare();
        for (int ti = 0; ti < my_tiles; ++ti) {
            tile_init(ti);
            int st = nsteps;
            do ring_step(); while (--st > 0);
            load_invnorm(ti + 1);
            mfma_settle();
            // All have read the tile's last bank block: the second four before the barrier that ended their last fetch.  What they load to its place
            // next they ask for behind the next tile's first barrier, which nobody reaches before it has left the epilogue.
            epilogue(ti, !BUSY ? LIST_AT : at_bank == 0 ? (uint32_t)((RING_PLACES - 1) * STAGE_BANK_BYTES) : at_bank - (uint32_t)STAGE_BANK_BYTES);
            tile_prepare();
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // blocks past the end still land in this workgroup's LDS
        return;
    }
    if constexpr (Q_DIRECT) {
        const uint16_t* qb = gnext_q();
#pragma unroll
        for (int i = 0; i < QCH; ++i) qload_to_lds(qb, 0, i);
    } else {
        gload_q(gqA);
    }
    gload(gbA);
    if constexpr (!Q_DIRECT) gload_q(gqB);
    gload(gbB);
    lstore(0, gbA, gqA);
    if constexpr (!Q_DIRECT) gload_q(gqA);
    if constexpr (DT == 0) gload(gbA);
    if constexpr (Q_DIRECT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if constexpr (EXACT) {
        live = (uint32_t)__builtin_amdgcn_readfirstlane((int)total_s[1]);
        if (live == 0) return;                          // uniform: all have read the same word
    }
    load_invnorm(0);
    tile_prepare();
    for (int ti = 0; ti < my_tiles; ++ti) {
        tile_init(ti);
        tile_now = ti;
        if constexpr (DT == 0) load_invnorm(ti + 1);
        if constexpr (DT != 0) {
#pragma unroll
            for (int a = 0; a < RA; ++a) af[a] = frag_a(0, 0, a);
#pragma unroll
            for (int b = 0; b < MR; ++b) bfr[0][b] = frag_b(0, offB0, b);
        }
        for (int st = 0; st < nsteps - 2; st += 2) {
            phase(0, gbB, gbA, gqB, std::true_type{});
            phase(1, gbA, gbB, gqA, std::true_type{});
        }
        phase(0, gbB, gbA, gqB, std::true_type{});
        phase(1, gbA, gbB, gqA, std::false_type{});
        mfma_settle();
        epilogue(ti, LIST_AT);
        tile_prepare();
    }
    if constexpr (Q_DIRECT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // query blocks past the end still land in this workgroup's LDS
}

}  // namespace evk
