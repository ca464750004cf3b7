// Ingest kernels: append rows to the tiled store, read them back, prepare a batch of queries.
#pragma once
#include "layout.h"

namespace evk {

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// x + (x of the lane that is N places further round in its row of 16 lanes)
template <int N>
__device__ __forceinline__ double add_row_ror(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 + N, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 + N, 0xf, 0xf, true);
    return x + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double row16_sum(double x) { return add_row_ror<1>(add_row_ror<2>(add_row_ror<4>(add_row_ror<8>(x)))); }

// 1 / sqrt(x), far below a float's rounding: the hardware's approximation, good to about a float, and one Newton step.  (With the
// library's square root and division seven queries over 30,011 x 200 fp16 take 30.35 us instead of 30.15.)
__device__ __forceinline__ double rsqrt_d(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    return y * (1.5 - 0.5 * x * y * y);
}

// Sum over the 64 lanes of a wavefront (all lanes active), the same in every lane: within rows of 16 lanes by
// rotations, then the four rows' sums.
__device__ __forceinline__ double wave_total_d(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, row16_sum(x));
    auto row = [&](int lane) __attribute__((always_inline)) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    };
    return (row(0) + row(16)) + (row(32) + row(48));
}

// Memory growth rule of Sec. 3.1: entry first_id + row gets embedding emb[row], rounded to the
// store's element type; the inverse L2 norm of the *stored* values is kept beside it (fp32, used
// only by the scan's filter; the value filter recomputes norms in fp64) and both Q tables get their
// initial value.  One wavefront per row.  A lane takes 4 consecutive elements per step: its 16-byte
// load is one contiguous 1 KB read per wavefront, its 8-byte store half of a 16-byte chunk of the
// tiled store (two neighbouring lanes fill a chunk), four steps in flight at a time.  Both are streamed
// (non-temporal, see layout.h).
template <typename ST>  // BF16, F16 (uint16_t storage) ; fp32 handled by the overload below
__global__ __launch_bounds__(256) void k_append16(const float* __restrict__ emb, int64_t n, int d, int nkb,
                                                  int64_t first_id, uint16_t* __restrict__ store,
                                                  float* __restrict__ invnorm, float* __restrict__ qtab,
                                                  int64_t capacity, const float* __restrict__ q0d,
                                                  const float* __restrict__ q0r) {
    int lane = threadIdx.x & 63;
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= n) return;
    int64_t id = first_id + row;
    const float* src = emb + row * (int64_t)d;
    float ssq = 0.f;
    const int ngroups = nkb * 16;                       // groups of 4 elements, padding included
    for (int g0 = lane; g0 < ngroups; g0 += 4 * 64) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int g = g0 + 64 * u;
            v[u] = (g < ngroups && g * 4 < d) ? stream_load_float4(src + g * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int g = g0 + 64 * u;
            if (g >= ngroups) break;
            const uint16_t h0 = ST::enc(v[u].x), h1 = ST::enc(v[u].y), h2 = ST::enc(v[u].z), h3 = ST::enc(v[u].w);
            const float w0 = ST::dec(h0), w1 = ST::dec(h1), w2 = ST::dec(h2), w3 = ST::dec(h3);
            ssq += w0 * w0; ssq += w1 * w1; ssq += w2 * w2; ssq += w3 * w3;
            uint2 pk;
            pk.x = h0 | ((uint32_t)h1 << 16); pk.y = h2 | ((uint32_t)h3 << 16);
            stream_store8(store + off16(id, g >> 1, nkb) + (g & 1) * 4, pk.x, pk.y);
        }
    }
    ssq = wave_sum_f(ssq);
    if (lane == 0) {
        invnorm[id] = (float)(1.0 / sqrt((double)ssq));
        qtab[id] = q0d ? q0d[row] : 0.f;
        qtab[capacity + id] = q0r ? q0r[row] : 0.f;
    }
}

__global__ __launch_bounds__(256) void k_append32(const float* __restrict__ emb, int64_t n, int d, int nkb,
                                                  int64_t first_id, float* __restrict__ store,
                                                  float* __restrict__ invnorm, float* __restrict__ qtab,
                                                  int64_t capacity, const float* __restrict__ q0d,
                                                  const float* __restrict__ q0r) {
    int lane = threadIdx.x & 63;
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= n) return;
    int64_t id = first_id + row;
    const float* src = emb + row * (int64_t)d;
    float ssq = 0.f;
    for (int c4 = lane; c4 < nkb * 16; c4 += 64) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c4 * 4 < d) a = stream_load_float4(src + c4 * 4);
        ssq += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
        stream_store_float4(store + off32(id, c4, nkb), a);
    }
    ssq = wave_sum_f(ssq);
    if (lane == 0) {
        invnorm[id] = (float)(1.0 / sqrt((double)ssq));
        qtab[id] = q0d ? q0d[row] : 0.f;
        qtab[capacity + id] = q0r ? q0r[row] : 0.f;
    }
}

// Stored rows first .. first+n widened to fp32, row-major [n][d].
template <typename ST>
__global__ __launch_bounds__(256) void k_read_rows16(const uint16_t* __restrict__ store, int64_t first, int64_t n,
                                                     int d, int nkb, float* __restrict__ dst) {
    int lane = threadIdx.x & 63;
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= n) return;
    for (int c8 = lane; c8 * 8 < d; c8 += 64) {
        uint4 pk = *reinterpret_cast<const uint4*>(store + off16(first + row, c8, nkb));
        uint32_t w[4] = {pk.x, pk.y, pk.z, pk.w};
        float* o = dst + row * (int64_t)d + c8 * 8;
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[2 * i] = ST::dec((uint16_t)(w[i] & 0xffff)); o[2 * i + 1] = ST::dec((uint16_t)(w[i] >> 16)); }
    }
}
__global__ __launch_bounds__(256) void k_read_rows32(const float* __restrict__ store, int64_t first, int64_t n,
                                                     int d, int nkb, float* __restrict__ dst) {
    int lane = threadIdx.x & 63;
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= n) return;
    for (int c4 = lane; c4 * 4 < d; c4 += 64)
        *reinterpret_cast<float4*>(dst + row * (int64_t)d + c4 * 4) =
            *reinterpret_cast<const float4*>(store + off32(first + row, c4, nkb));
}

// Read-only pass over the stored rows, nothing else: every 16-byte piece of the store is loaded once and
// folded into a checksum.  It measures what a scan of this bank can reach at best on the machine at
// hand (the similarity scan of Sec. 3.2 has to read the same bytes once per retrieve).
// Access pattern of the scan itself: a workgroup takes whole contiguous 64 KB pieces, round-robin, each
// lane 16 independent 16-byte loads (one load instruction of the workgroup covers 4 KB).
__global__ __launch_bounds__(256) void k_read_probe(const uint4* __restrict__ p, int64_t n16, uint32_t* __restrict__ checksum) {
    constexpr int PIECE = 4096;                          // 16-byte units per 64 KB piece
    const int64_t pieces = n16 / PIECE;
    uint32_t acc = 0;
    for (int64_t c = blockIdx.x; c < pieces; c += gridDim.x) {
        const uint4* q = p + c * PIECE + threadIdx.x;
        uint4 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) { const stream_u32x4 t = stream_load16(q + u * 256); v[u] = make_uint4(t.x, t.y, t.z, t.w); }
#pragma unroll
        for (int u = 0; u < 16; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (int64_t i = pieces * PIECE + (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (int64_t)gridDim.x * 256) {
        const uint4 v = p[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc ^= __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) atomicXor(checksum, acc);
}

// Query preparation (Sec. 3.2, the query side of dense retrieval): round each query to the store's
// element type, keep it widened (fp32, row-major, zero-padded to the k-block multiple) for the
// GEMV scan and the fp64 re-score, and as fragments for the matrix cores (qop_row in layout.h; for fp32
// stores the query is split as hi + lo in bf16, so that the scan can use bf16 MFMA), with an all-zero
// k-block behind the last one, plus its inverse norm (fp32 and fp64).  Also resets the per-query threshold and presets the
// survivor count to the number of rows of the sparsest scan pass, which keeps every row.
// Slots >= B become all-zero queries that never pass a filter.
//
// It takes as long as a launch does (3 to 5 us), and the first scan pass needs of it only what a workgroup can make of the
// queries itself.  So where that pass has variants that read the queries as given (FIRST in k_scan_direct.h and k_scan_gemv.h)
// these workgroups ride in its launch, and what they write is for the launches after it.
struct PrepArgs {
    const float* q;                // [B][d]
    float* qf;
    uint16_t* qop;
    float* invq;
    double* invq64;
    float* thr;
    uint32_t* cnt;
    uint32_t* flags;
    uint32_t cnt0;
    int B, Bpad, d, nkb;
    int aligned;                   // the queries lie at a multiple of 16 bytes (their rows are multiples of 32 bytes)
    int operands;                  // qop is read (not by the VALU scan, whose Bpad need not be whole fragments)
};
// Eight consecutive elements of a query as given, from element e0 (a multiple of 8) on; zeros past its end.
template <bool ALIGNED>
__device__ __forceinline__ void load_query8(const float* row, int e0, int d, float (&v)[8]) {
    const bool in = e0 < d;                                     // d is a multiple of 8
    const float* p = row + (in ? e0 : 0);
    if constexpr (ALIGNED) {
        const float4 x = *reinterpret_cast<const float4*>(p), y = *reinterpret_cast<const float4*>(p + 4);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = p[i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = in ? v[i] : 0.f;
}
// Chunk c8 (eight consecutive elements) of query b, rounded to the store's type (h: 16-bit types, two to a word) and widened again; slots >= B are all-zero.
template <int DT>
__device__ __forceinline__ void prep_values(const PrepArgs& A, int b, int c8, float (&v)[8], uint32_t (&h)[4]) {
    const float* row = A.q + (int64_t)(b < A.B ? b : 0) * A.d;
    if (A.aligned) load_query8<true>(row, c8 * 8, b < A.B ? A.d : 0, v);
    else load_query8<false>(row, c8 * 8, b < A.B ? A.d : 0, v);
    if constexpr (DT != 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = DT == 1 ? cvt_pk_bf16(v[2 * i], v[2 * i + 1]) : f2f16_rne(v[2 * i]) | (uint32_t)f2f16_rne(v[2 * i + 1]) << 16;
            const uint16_t lo = (uint16_t)h[i], hi = (uint16_t)(h[i] >> 16);
            v[2 * i] = DT == 1 ? bf16_to_f(lo) : f16_to_f(lo);
            v[2 * i + 1] = DT == 1 ? bf16_to_f(hi) : f16_to_f(hi);
        }
    }
}
__device__ __forceinline__ double prep_squares(const float (&v)[8]) {
    double ssq = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) ssq += (double)v[i] * (double)v[i];
    return ssq;
}
template <int DT>
__device__ __forceinline__ void prep_store(const PrepArgs& A, int b, int c8, const float (&v)[8], const uint32_t (&h)[4]) {
    const int kb = c8 >> 3, c = c8 & 7, Bpad = A.Bpad;
    if constexpr (DT == 0) {
        // fp32 store: operand = bf16 hi + bf16 lo
        if (A.operands) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                hi[i] = cvt_pk_bf16(v[2 * i], v[2 * i + 1]);
                lo[i] = cvt_pk_bf16(v[2 * i] - bf16_to_f((uint16_t)hi[i]), v[2 * i + 1] - bf16_to_f((uint16_t)(hi[i] >> 16)));
            }
            const int64_t u = (kb * 2 + (c >> 2)) * 2;                  // heads; remainders in the row behind
            *reinterpret_cast<uint4*>(A.qop + qop_row(u, Bpad) + qop_in_row(b, c & 3)) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(A.qop + qop_row(u + 1, Bpad) + qop_in_row(b, c & 3)) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
    } else {
        *reinterpret_cast<uint4*>(A.qop + qop_row(kb * 2 + (c >> 2), Bpad) + qop_in_row(b, c & 3)) = make_uint4(h[0], h[1], h[2], h[3]);
    }
    float* o = A.qf + (int64_t)b * A.nkb * KB + c8 * 8;
    *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
// one all-zero k-block behind the last one: the MFMA scan pairs it with a repeated bank block
// when it pads an odd number of k-steps to an even one, and after the last pass its words count the
// workgroups of the tail.  Eight lanes to a query.
template <int DT>
__device__ __forceinline__ void prep_zero_block(const PrepArgs& A, int b, int lane) {
    *reinterpret_cast<uint4*>(A.qop + ((int64_t)(DT == 0 ? 2 * A.nkb : A.nkb) * A.Bpad + b) * KB + lane * 8) = make_uint4(0, 0, 0, 0);
}
__device__ __forceinline__ void prep_words(const PrepArgs& A, int b, double ssq) {
    const bool live = b < A.B;
    const double inv = live ? 1.0 / sqrt(ssq) : 0.0;
    A.invq64[b] = inv;
    A.invq[b] = (float)inv;
    // "No threshold yet" is a finite floor below every reachable value (the scan compares
    // dot * invnorm, which lies in [-|q|, |q|]); empty slots get a threshold their all-zero query
    // can never reach.  Finite values keep the scan's arithmetic free of inf - inf.
    A.thr[b] = live ? (float)(-2.0 / inv) : 1.0f;
    *slot_counter(A.cnt, b) = live ? A.cnt0 : 0u;     // rows the sparsest pass will write without counting
    A.flags[b] = 0u;                 // per-query status of this retrieve (bit 0: a survivor list overflowed)
}
// One query, by all NT lanes of a workgroup; red has a word per wavefront.  Without STORE only its norm and its words.
template <int DT, int NT, bool STORE = true>
__device__ __forceinline__ void prep_query(const PrepArgs& A, int b, double* red) {
    const int tid = threadIdx.x;
    double ssq = 0.0;
    for (int c8 = tid; c8 < A.nkb * 8; c8 += NT) {
        float v[8];
        uint32_t h[4];
        prep_values<DT>(A, b, c8, v, h);
        ssq += prep_squares(v);
        if constexpr (STORE) prep_store<DT>(A, b, c8, v, h);
    }
    if (tid < 8) prep_zero_block<DT>(A, b, tid);
    ssq = wave_total_d(ssq);
    if ((tid & 63) == 0) red[tid >> 6] = ssq;
    __syncthreads();
    if (tid == 0) {
        ssq = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) ssq += red[w];
        prep_words(A, b, ssq);
    }
}
// A query to a workgroup.
template <int DT>
__global__ __launch_bounds__(256) void k_prep_queries(PrepArgs A) {
    __shared__ double red[4];
    prep_query<DT, 256>(A, (int)blockIdx.x, red);
}
// The first Bpad workgroups take a query each, for its norm and its words, and the others 16 queries' part of the k dimension each, which they
// write as whole fragments.  (A query's own pieces of a fragment are 16 bytes, 256 apart.)  Both read the queries, so with whole rounds of
// groups they are on the same XCD.
constexpr int PREP_SLICE = 16;           // chunks of 16 queries to a workgroup
inline int prep_fragment_workgroups(int Bpad, int nkb) { return Bpad + Bpad / 16 * ((nkb * 8 + PREP_SLICE - 1) / PREP_SLICE); }
// Which of the two, in us, a query to a workgroup / this: fp32, 64 queries of 1024 2.9, 2.6; 256 of 1024 4.3, 3.7; 512 of 4096 9.4, 6.7; 1024 of
// 2048 9.7, 6.9, of 4096 17.7, 10.0 (9.5 when a query's operands lay together).  16 bits, whose queries are rounded twice so: 256 of 4096 5.8, 6.8; 1024 of
// 1024 5.9, 6.3, of 2048 7.0, 7.1, of 4096 11.6, 9.3 (8.2).
inline bool prep_by_fragments(bool f32, int Bpad, int nkb) { return f32 || (int64_t)Bpad * nkb >= 1024 * 48; }
template <int DT>
__global__ __launch_bounds__(256) void k_prep_fragments(PrepArgs A) {
    __shared__ double red[4];
    const int i = (int)blockIdx.x, j = i >> 3, tid = threadIdx.x;
    if (i < A.Bpad) {                                                   // uniform
        prep_query<DT, 256, false>(A, A.Bpad % 128 == 0 ? ((i & 7) + 8 * (j >> 4)) * 16 + (j & 15) : i, red);
        return;
    }
    static_assert(16 * PREP_SLICE == 256, "a chunk to a lane");
    const uint32_t groups = (uint32_t)A.Bpad / 16, k = (uint32_t)(i - A.Bpad);
    const int b = (int)(k % groups) * 16 + (tid & 15), c8 = (int)(k / groups) * PREP_SLICE + (tid >> 4);
    if (c8 < A.nkb * 8) {
        float v[8];
        uint32_t h[4];
        prep_values<DT>(A, b, c8, v, h);
        prep_store<DT>(A, b, c8, v, h);
    }
}

}  // namespace evk
