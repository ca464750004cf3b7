// Host side of the evomem C ABI (include/evomem.h): argument checks, workspace carving, the scan
// plan, kernel dispatch.  Every step of the method runs in the kernels included below.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/evomem.h"
#include "k_ingest.h"
#include "k_scan_gemv.h"
#include "k_scan_mfma.h"
#include "k_scan_direct.h"
#include "k_select.h"
#include "k_exact.h"
#include "k_tail.h"
#include "k_reward.h"
#include "k_startpoint.h"
#include "k_update.h"
#include "layout.h"

using namespace evk;

static_assert(MEM_MAX_K1 == evk::BIG_K1_MAX && MEM_MAX_B == evk::MAX_BATCH, "header and kernels disagree on the largest pool or batch");

namespace {

constexpr int MAX_PROFILE = 4096;
constexpr int GEMV_MAX_B = 4;       // fp32 stores: at most this many queries use the VALU scan

constexpr int MAX_DEVICES = 16;     // per-device set-up flags and scratch addresses are kept in arrays of this size

constexpr int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Calls f with the store type as a compile-time constant (0 fp32, 1 bf16, 2 fp16: the kernels' DT).
template <class F>
void with_store_type(int dtype, F&& f) {
    if (dtype == MEM_F32) f(std::integral_constant<int, 0>{});
    else if (dtype == MEM_BF16) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, 2>{});
}

struct Workspace {   // byte offsets into a scratch area (the caller's workspace, or the library's own array)
    size_t counters, qf, qop, invq, invq64, thr, cnt, flags, surv, exact, total;
};

// A retrieve pads its batch to a multiple of its query tile (32 .. 256 queries), so the per-query
// arrays are sized for max_B rounded up to `bpad` (256 covers every tile).
constexpr Workspace carve(int d, int dtype, int max_B, int max_k1, int bpad = 256) {
    const int64_t dpad = round_up(d, KB), Bp = round_up(max_B, bpad);
    const size_t sizes[10] = {256, (size_t)Bp * dpad * 4,
                              (size_t)Bp * (dpad + KB) * (dtype == MEM_F32 ? 4 : 2),   // + one all-zero k-block
                              (size_t)Bp * 4, (size_t)Bp * 8, (size_t)Bp * 4, (size_t)Bp * CNT_STRIDE * 4, (size_t)Bp * 4,
                              (size_t)Bp * SURV_CAP * 8, (size_t)Bp * keep_of(max_k1) * 8};
    size_t at[11] = {};
    for (int i = 0; i < 10; ++i) at[i + 1] = (size_t)round_up((int64_t)(at[i] + sizes[i]), 256);
    return Workspace{at[0], at[1], at[2], at[3], at[4], at[5], at[6], at[7], at[8], at[9], at[10]};
}

// Where a retrieve keeps its intermediate results.
struct Scratch {
    unsigned char* base;
    Workspace w;
    int exact_stride;      // fp64 similarities per query
    int lists() const { return (int)((w.exact - w.surv) / (SURV_CAP * sizeof(uint64_t))); }    // survivor lists, at least one per query
};

// Limits of mem_retrieve_static and the library's own scratch array for it (see the header).
constexpr int STATIC_MAX_B = 64, STATIC_MAX_K1 = 256, STATIC_MAX_D = 2048;
constexpr Workspace STATIC_W = carve(STATIC_MAX_D, MEM_F32, STATIC_MAX_B, STATIC_MAX_K1, STATIC_MAX_B);
constexpr size_t STATIC_SCRATCH_BYTES = STATIC_W.total;
static_assert(STATIC_SCRATCH_BYTES <= (6u << 20), "the built-in scratch array is meant to stay small");

bool shape_ok(int d, int dtype, int64_t capacity) {
    return d >= 8 && d <= 16384 && d % 8 == 0 && dtype >= MEM_F32 && dtype <= MEM_F16 && capacity >= 1 &&
           capacity <= 2147483647ll - 256;
}


}  // namespace

struct evomem {
    int d, dtype, nkb, device, max_B, max_k1;
    int64_t capacity, N;
    void* store;
    float* invnorm;
    float* q;
    unsigned char* ws;
    Workspace w;
    bool lds_attr_set;
    // profiling
    bool prof_on;
    int prof_n;
    uint32_t* tags = nullptr;   // per-entry tags of typed / masked retrieval (caller's buffer), or null
    const uint32_t* last_flags = nullptr;   // per-query status words of the latest retrieve (in the scratch it used)
    int last_B = 0;
    uint32_t reward_calls = 0;  // number of the latest batch of rewards in one chained launch (after 2^32 - 1 of them: two launches)
    std::vector<hipEvent_t> ev;
    std::vector<int64_t> prof_rows;
};

// Clears a few words on the stream (a kernel, not a memset: callers may record their calls into a HIP graph).
__global__ void k_clear_words(uint32_t* p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

#define HIPCHK(x) do { if ((x) != hipSuccess) return MEM_EHIP; } while (0)
#define LAUNCHCHK() do { if (hipGetLastError() != hipSuccess) return MEM_EHIP; } while (0)

extern "C" {

size_t mem_store_bytes(int d, int dtype, int64_t capacity) {
    if (!shape_ok(d, dtype, capacity)) return 0;
    return (size_t)round_up(capacity, TILE_ROWS) * (size_t)round_up(d, KB) * (dtype == MEM_F32 ? 4 : 2);
}

size_t mem_workspace_bytes(int d, int dtype, int64_t capacity, int max_B, int max_k1) {
    if (!shape_ok(d, dtype, capacity) || max_B < 1 || max_B > MEM_MAX_B || max_k1 < 1 || max_k1 > MEM_MAX_K1) return 0;
    return carve(d, dtype, max_B, max_k1).total;
}

int mem_create(evomem_t** out, int d, int dtype, int64_t capacity, void* store_dev, float* invnorm_dev,
               float* q_dev, void* workspace_dev, size_t workspace_bytes, int max_B, int max_k1, int device) {
    if (!out) return MEM_EINVAL;
    *out = nullptr;
    if (!shape_ok(d, dtype, capacity) || !store_dev || !invnorm_dev || !q_dev || !workspace_dev) return MEM_EINVAL;
    if (max_B < 1 || max_B > MEM_MAX_B || max_k1 < 1 || max_k1 > MEM_MAX_K1 || device < 0 || device >= MAX_DEVICES) return MEM_EINVAL;
    if (((uintptr_t)store_dev | (uintptr_t)workspace_dev) & 255) return MEM_EINVAL;
    Workspace w = carve(d, dtype, max_B, max_k1);
    if (workspace_bytes < w.total) return MEM_EWORKSPACE;
    evomem* h = new (std::nothrow) evomem();
    if (!h) return MEM_EHIP;
    h->d = d; h->dtype = dtype; h->nkb = (int)(round_up(d, KB) / KB); h->device = device;
    h->max_B = max_B; h->max_k1 = max_k1; h->capacity = capacity; h->N = 0;
    h->store = store_dev; h->invnorm = invnorm_dev; h->q = q_dev;
    h->ws = static_cast<unsigned char*>(workspace_dev); h->w = w;
    h->lds_attr_set = false; h->prof_on = false; h->prof_n = 0;
    if (hipSetDevice(device) != hipSuccess || hipMemsetAsync(h->ws + w.counters, 0, 256, nullptr) != hipSuccess ||
        hipStreamSynchronize(nullptr) != hipSuccess) {
        delete h;
        return MEM_EHIP;
    }
    *out = h;
    return MEM_OK;
}

int mem_destroy(evomem_t* h) {
    if (!h) return MEM_EINVAL;
    for (hipEvent_t e : h->ev) (void)hipEventDestroy(e);
    delete h;
    return MEM_OK;
}

int mem_size(const evomem_t* h, int64_t* n_out) {
    if (!h || !n_out) return MEM_EINVAL;
    *n_out = h->N;
    return MEM_OK;
}

int mem_append(evomem_t* h, const float* emb_dev, int64_t n, const float* q0d, const float* q0r,
               int64_t* first_id_out, void* hip_stream) {
    if (!h || n < 0 || (n > 0 && !emb_dev)) return MEM_EINVAL;
    if (h->N + n > h->capacity) return MEM_ECAPACITY;
    if (first_id_out) *first_id_out = h->N;
    if (n == 0) return MEM_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    dim3 grid((unsigned)((n + 3) / 4)), block(256);
    if (h->dtype == MEM_F32)
        hipLaunchKernelGGL(k_append32, grid, block, 0, st, emb_dev, n, h->d, h->nkb, h->N, (float*)h->store,
                           h->invnorm, h->q, h->capacity, q0d, q0r);
    else if (h->dtype == MEM_BF16)
        hipLaunchKernelGGL(k_append16<BF16>, grid, block, 0, st, emb_dev, n, h->d, h->nkb, h->N, (uint16_t*)h->store,
                           h->invnorm, h->q, h->capacity, q0d, q0r);
    else
        hipLaunchKernelGGL(k_append16<F16>, grid, block, 0, st, emb_dev, n, h->d, h->nkb, h->N, (uint16_t*)h->store,
                           h->invnorm, h->q, h->capacity, q0d, q0r);
    LAUNCHCHK();
    h->N += n;
    return MEM_OK;
}

int mem_read_q(evomem_t* h, int stage, int64_t first, int64_t n, float* dst_dev, void* hip_stream) {
    if (!h || (stage != 0 && stage != 1) || first < 0 || n < 0 || first + n > h->N || (n > 0 && !dst_dev)) return MEM_EINVAL;
    if (n == 0) return MEM_OK;
    HIPCHK(hipMemcpyAsync(dst_dev, h->q + stage * h->capacity + first, (size_t)n * 4, hipMemcpyDeviceToDevice,
                          static_cast<hipStream_t>(hip_stream)));
    return MEM_OK;
}

int mem_read_rows(evomem_t* h, int64_t first, int64_t n, float* dst_dev, void* hip_stream) {
    if (!h || first < 0 || n < 0 || first + n > h->N || (n > 0 && !dst_dev)) return MEM_EINVAL;
    if (n == 0) return MEM_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    dim3 grid((unsigned)((n + 3) / 4)), block(256);
    if (h->dtype == MEM_F32)
        hipLaunchKernelGGL(k_read_rows32, grid, block, 0, st, (const float*)h->store, first, n, h->d, h->nkb, dst_dev);
    else if (h->dtype == MEM_BF16)
        hipLaunchKernelGGL(k_read_rows16<BF16>, grid, block, 0, st, (const uint16_t*)h->store, first, n, h->d, h->nkb, dst_dev);
    else
        hipLaunchKernelGGL(k_read_rows16<F16>, grid, block, 0, st, (const uint16_t*)h->store, first, n, h->d, h->nkb, dst_dev);
    LAUNCHCHK();
    return MEM_OK;
}

int mem_counters(evomem_t* h, int64_t* skipped_ids, int64_t* overflows) {
    if (!h) return MEM_EINVAL;
    uint32_t c[2] = {0, 0};
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMemcpy(c, h->ws + h->w.counters, 8, hipMemcpyDeviceToHost));
    if (skipped_ids) *skipped_ids = c[0];
    if (overflows) *overflows = c[1];
    return MEM_OK;
}

int mem_read_probe(evomem_t* h, uint32_t* checksum_dev, int64_t* bytes_out, void* hip_stream) {
    if (!h || !checksum_dev) return MEM_EINVAL;
    const int64_t bytes = round_up(h->N, TILE_ROWS) * (int64_t)h->nkb * KB * (h->dtype == MEM_F32 ? 4 : 2);
    if (bytes_out) *bytes_out = bytes;
    if (bytes == 0) return MEM_OK;
    int cus = 0;
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h->device));
    // two workgroups per compute unit: measured 6.2 TB/s on a 24 GB store, against 5.7-5.8 TB/s with four or eight
    hipLaunchKernelGGL(k_read_probe, dim3((unsigned)(cus * 2)), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       (const uint4*)h->store, bytes / 16, checksum_dev);
    LAUNCHCHK();
    return MEM_OK;
}

int mem_profile_enable(evomem_t* h, int on) {
    if (!h) return MEM_EINVAL;
    if (on && h->ev.empty()) {
        h->ev.resize(2 * MAX_PROFILE);
        h->prof_rows.resize(MAX_PROFILE);
        for (size_t i = 0; i < h->ev.size(); ++i)
            if (hipEventCreate(&h->ev[i]) != hipSuccess) {       // leave no half-built set behind
                for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(h->ev[j]);
                h->ev.clear();
                h->prof_rows.clear();
                return MEM_EHIP;
            }
    }
    h->prof_on = on != 0;      // the records kept so far stay until they are read
    return MEM_OK;
}

int mem_profile_read(evomem_t* h, int capacity, int* n_out, float* ms_out, int64_t* rows_out) {
    if (!h || capacity < 0 || !n_out || (capacity > 0 && (!ms_out || !rows_out))) return MEM_EINVAL;
    HIPCHK(hipDeviceSynchronize());
    int n = h->prof_n < capacity ? h->prof_n : capacity;
    for (int i = 0; i < n; ++i) {
        HIPCHK(hipEventElapsedTime(&ms_out[i], h->ev[2 * i], h->ev[2 * i + 1]));
        rows_out[i] = h->prof_rows[i];
    }
    *n_out = n;
    h->prof_n = 0;
    return MEM_OK;
}

// Is the stream being recorded into a graph?  (Yes too where it can't be told: the default stream while another one records.)
static bool recording(hipStream_t st) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// the normaliser's statistics live in the zero-initialised counter block: double[2 stages][3] at byte 64
static double* reward_state(evomem_t* h, int stage) { return reinterpret_cast<double*>(h->ws + h->w.counters + 64) + 3 * stage; }

int mem_shape_rewards(evomem_t* h, int stage, const unsigned char* feasible_dev, const float* latency_dev,
                      const float* best_latency_dev, int64_t M, int normalise, float sigma_min, float clip,
                      float* rewards_out_dev, void* hip_stream) {
    if (!h || (stage != 0 && stage != 1) || M < 0 || (normalise && !(sigma_min > 0.f)) || !(clip >= 0.f)) return MEM_EINVAL;
    if (M == 0) return MEM_OK;
    if (!feasible_dev || !rewards_out_dev || (stage == 1 && (!latency_dev || !best_latency_dev))) return MEM_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    // (the chain's two words lie in the zero-initialised counter block, behind the statistics; its calls are numbered from 1)
    RewardArgs A{feasible_dev, latency_dev, best_latency_dev, M, (double)sigma_min, (double)clip, reward_state(h, stage),
                 reinterpret_cast<double*>(h->ws + h->w.surv), reinterpret_cast<uint64_t*>(h->ws + h->w.counters + 128), h->reward_calls + 1,
                 rewards_out_dev, stage, normalise};
    if (normalise && M > REWARD_ONE && M <= (int64_t)REWARD_CHAIN * REWARD_T && A.call != 0 && !recording(st)) {
        h->reward_calls = A.call;
        hipLaunchKernelGGL(k_reward_chain, dim3((unsigned)((M + REWARD_T - 1) / REWARD_T)), dim3(REWARD_T), 0, st, A);
        LAUNCHCHK();
        return MEM_OK;
    }
    if (M <= REWARD_ONE) {
        hipLaunchKernelGGL(k_shape_rewards, dim3(1), dim3(REWARD_ONE), 0, st, A);
        LAUNCHCHK();
        return MEM_OK;
    }
    // the blocks' sums lie where the survivor lists of a retrieve lie (calls on a handle are ordered)
    static_assert((REWARD_HEAD + 2ll * REWARD_BLOCKS) * sizeof(double) <= 256ll * SURV_CAP * sizeof(uint64_t), "a workspace has at least 256 lists");
    const int64_t most = normalise ? (int64_t)REWARD_BLOCKS * REWARD_T : (int64_t)1 << 30;
    for (int64_t off = 0; off < M; off += most) {
        A.feasible = feasible_dev + off;
        if (stage == 1) { A.latency = latency_dev + off; A.best = best_latency_dev + off; }
        A.out = rewards_out_dev + off;
        A.M = M - off < most ? M - off : most;
        const dim3 grid((unsigned)((A.M + REWARD_T - 1) / REWARD_T)), block(REWARD_T);
        if (normalise) {
            hipLaunchKernelGGL(k_reward_sums, grid, block, 0, st, A);
            LAUNCHCHK();
        }
        hipLaunchKernelGGL(k_reward_shape, grid, block, 0, st, A);
        LAUNCHCHK();
    }
    return MEM_OK;
}

int mem_reward_stats(evomem_t* h, int stage, double* count, double* mean, double* sigma) {
    if (!h || (stage != 0 && stage != 1) || !count || !mean || !sigma) return MEM_EINVAL;
    double st[3];
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMemcpy(st, reward_state(h, stage), sizeof(st), hipMemcpyDeviceToHost));
    *count = st[0];
    *mean = st[0] > 0 ? st[1] / st[0] : 0.0;
    const double var = st[0] > 0 ? st[2] / st[0] - (*mean) * (*mean) : 0.0;
    *sigma = var > 0 ? sqrt(var) : 0.0;
    return MEM_OK;
}

int mem_reward_stats_reset(evomem_t* h, int stage, void* hip_stream) {
    if (!h || (stage != 0 && stage != 1)) return MEM_EINVAL;
    hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, static_cast<hipStream_t>(hip_stream),
                       reinterpret_cast<uint32_t*>(reward_state(h, stage)), (int)(3 * sizeof(double) / sizeof(uint32_t)));
    LAUNCHCHK();
    return MEM_OK;
}

int mem_restore(evomem_t* h, int64_t n) {
    if (!h || n < 0) return MEM_EINVAL;
    if (n > h->capacity) return MEM_ECAPACITY;
    h->N = n;
    return MEM_OK;
}

const char* mem_strerror(int s) {
    switch (s) {
        case MEM_OK: return "ok";
        case MEM_EINVAL: return "invalid argument";
        case MEM_ECAPACITY: return "bank capacity exceeded";
        case MEM_EWORKSPACE: return "workspace too small";
        case MEM_EHIP: return "HIP runtime error";
        case MEM_ESTATE: return "handle in unusable state";
        default: return "unknown status";
    }
}

}  // extern "C"

namespace {

// Scan plan: tile strides of the passes, sparsest first.  The sparsest pass has no threshold, so it
// may cover at most SURV_CAP rows, and it is made as large as that allows (a larger sample gives the
// next pass a tighter threshold).  Each denser pass divides the stride by `ratio`, chosen so that
// about k1 * ratio rows (a quarter of the survivor slots) are expected to pass its threshold; the
// step up to the sparsest pass is whatever factor <= ratio fills its row budget.
// (at most 24 passes: every step divides the stride by at least 2 and a bank has fewer than 2^23 tiles;
// kept in a fixed array so that a retrieve allocates nothing on the host either)
constexpr int MAX_LEVELS = 24;
struct Plan { int n; Level lv[MAX_LEVELS]; };
Plan plan_levels(int64_t N, int k1, int cap) {
    const int nt = (int)((N + TILE_ROWS - 1) / TILE_ROWS);
    const int cap_tiles = cap / TILE_ROWS;
    int ratio = cap / (4 * k1);
    if (ratio > 16) ratio = 16;
    if (ratio < 2) ratio = 2;
    int strides[MAX_LEVELS] = {1}, ns = 1;
    for (;;) {
        const int U = (nt + strides[ns - 1] - 1) / strides[ns - 1];
        if (U <= cap_tiles) break;
        const int need = (U + cap_tiles - 1) / cap_tiles;          // >= 2
        strides[ns] = strides[ns - 1] * (need < ratio ? need : ratio);
        ++ns;
    }
    Plan p{};
    for (int i = ns - 1; i >= 0; --i) {
        Level L;
        L.stride = strides[i];
        L.cap = cap;
        const int U = (nt + L.stride - 1) / L.stride;
        if (i == ns - 1) { L.rho = 0; L.ntiles = U; }
        else { L.rho = strides[i + 1] / strides[i]; L.ntiles = U - (U + L.rho - 1) / L.rho; }
        if (L.ntiles > 0) p.lv[p.n++] = L;
    }
    return p;
}

template <int DT, int MQ, int WQ, int MR, int WR, bool MASKED, bool STREAM = true, bool EXACT = false, bool BUSY = false>
int launch_mfma(evomem* h, const Scratch& sc, hipStream_t st, int Bp, const Level& L, int k1, const Mask& mask, int B) {
    constexpr int QT = 16 * MQ * WQ;
    constexpr int lds = scan_mfma_lds_bytes<DT, QT, MASKED, EXACT>();
    auto kern = k_scan_mfma<DT, MQ, WQ, MR, WR, MASKED, STREAM, EXACT, BUSY>;
    static int resident[MAX_DEVICES] = {};          // workgroups of this kernel the whole device holds at once
    if (!resident[h->device]) {
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        int per_cu = 0, cus = 0;
        HIPCHK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), 64 * WQ * WR, lds));
        HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h->device));
        if (per_cu < 1 || cus < 8) return MEM_EHIP;
        resident[h->device] = per_cu * cus;
    }
    // persistent launch: per XCD, `groups` tile walkers for each of the nqt query tiles
    const int nqt = Bp / QT;
    int groups = resident[h->device] / 8 / nqt;
    if (groups < 1) groups = 1;
    if (groups > (L.ntiles + 7) / 8) groups = (L.ntiles + 7) / 8;
    dim3 grid((unsigned)(8 * nqt * groups)), block(64 * WQ * WR);
    // A pass is expected to keep about k1 * rho rows per query; spread over its tiles that is the
    // number of survivors a workgroup stages per tile.  It writes its list out at evenly spaced tiles,
    // as seldom as keeps the expected fill under 55 % of the list (a surplus takes the direct path).
    const double per_tile = L.rho ? (double)k1 * L.rho * QT / L.ntiles : 1.0;
    const int tiles_per_wg = (int)((L.ntiles + 8 * groups - 1) / (8 * groups));
    int n_flush = (int)std::ceil(tiles_per_wg * (per_tile + 1.0) / (0.55 * scan_mfma_list_cap<DT, QT, MASKED, EXACT>()));
    if (n_flush < 1) n_flush = 1;
    int flush_every = (tiles_per_wg + n_flush - 1) / n_flush;
    if (flush_every < 1) flush_every = 1;
    if (flush_every > SCAN_LIST_TILES) flush_every = SCAN_LIST_TILES;
    if constexpr (scan_mfma_busy<DT, QT, MASKED>() && !BUSY) {        // (an expected tile fills more than half of the list, or there is only one)
        if (flush_every == 1 && L.rho != 0) return launch_mfma<DT, MQ, WQ, MR, WR, MASKED, STREAM, EXACT, true>(h, sc, st, Bp, L, k1, mask, B);
    }
    unsigned char* ws = sc.base;
    hipLaunchKernelGGL(kern, grid, block, lds, st, (const void*)h->store, (const float*)h->invnorm,
                       (const uint16_t*)(ws + sc.w.qop), (const float*)(ws + sc.w.invq), (const float*)(ws + sc.w.thr),
                       (uint32_t*)(ws + sc.w.cnt), (uint64_t*)(ws + sc.w.surv), h->N, h->nkb, Bp, L, flush_every, mask, B,
                       ExactPass{(const float*)(ws + sc.w.qf), (const double*)(ws + sc.w.invq64), (double*)(ws + sc.w.exact), sc.exact_stride, (int)(h->N / 500)});
    LAUNCHCHK();
    return MEM_OK;
}

template <int DT, bool MASKED>
int launch_mfma_dt(evomem* h, const Scratch& sc, hipStream_t st, int Bp, int qt, const Level& L, int k1, const Mask& mask, int B) {
    switch (qt) {
        case 32: return launch_mfma<DT, 2, 1, 4, 4, MASKED>(h, sc, st, Bp, L, k1, mask, B);
        case 64:
            // fp32 stores: 8 wavefronts, so that one wavefront's hi/lo split (vector ALU) overlaps the
            // MFMAs of the other one on its SIMD (0.054 -> 0.047 ms on the 65,536 x 1024 bank, with 32x32x16 instructions)
            if constexpr (DT == 0) return launch_mfma<DT, 2, 2, 4, 4, MASKED>(h, sc, st, Bp, L, k1, mask, B);
            else return launch_mfma<DT, 4, 1, 4, 4, MASKED>(h, sc, st, Bp, L, k1, mask, B);
        case 128: return launch_mfma<DT, 4, 2, 4, 4, MASKED>(h, sc, st, Bp, L, k1, mask, B);   // 8 wavefronts, 64 x 64 each
        default:                                                                               // 8 wavefronts, 128 x 64 each
            // several query tiles share every bank tile through L2: no streaming hint on the bank loads then
            return Bp > qt ? launch_mfma<DT, 8, 2, 4, 4, MASKED, false>(h, sc, st, Bp, L, k1, mask, B)
                           : launch_mfma<DT, 8, 2, 4, 4, MASKED, true>(h, sc, st, Bp, L, k1, mask, B);
    }
}
template <bool MASKED>
int launch_mfma_any(evomem* h, const Scratch& sc, hipStream_t st, int Bp, int qt, const Level& L, int k1, const Mask& mask, int B) {
    return h->dtype == MEM_F32 ? launch_mfma_dt<0, MASKED>(h, sc, st, Bp, qt, L, k1, mask, B)
         : h->dtype == MEM_BF16 ? launch_mfma_dt<1, MASKED>(h, sc, st, Bp, qt, L, k1, mask, B)
                                : launch_mfma_dt<2, MASKED>(h, sc, st, Bp, qt, L, k1, mask, B);
}

template <int NB>
int launch_gemv(evomem* h, const Scratch& sc, hipStream_t st, int B, const Level& L, const Mask& mask, const PrepArgs* prep) {
    unsigned char* ws = sc.base;
    // Workgroups per tile.  Measured with 16 and with 4 (us): one query, 205 tiles of 768 28.8, 32.2, 476 tiles of 72 16.6, 14.4;
    // four queries, 52 tiles of 768 16.5, 18.0, 205 tiles of 768 41.4, 36.6.
    const int wgs = L.ntiles <= (NB <= 2 ? 256 : 64) ? 16 : L.ntiles < 1024 ? 4 : 1;
    dim3 grid((unsigned)(wgs * L.ntiles)), block(256);
    const float* invq = (const float*)(ws + sc.w.invq);
    const float* thr = (const float*)(ws + sc.w.thr);
    const float* qf = (const float*)(ws + sc.w.qf);
    uint32_t* cnt = (uint32_t*)(ws + sc.w.cnt);
    uint64_t* surv = (uint64_t*)(ws + sc.w.surv);
    if (prep) {                                                     // the first pass: at most 32 tiles, or 64 with two lists to a query
        hipLaunchKernelGGL((k_scan_gemv32<NB, 1, true>), dim3((unsigned)(16 * L.ntiles + prep->Bpad)), block, 0, st, (const float*)h->store,
                           (const float*)h->invnorm, qf, invq, thr, cnt, surv, h->N, h->nkb, B, L, mask, *prep);
        LAUNCHCHK();
        return MEM_OK;
    }
    if (wgs == 16)
        hipLaunchKernelGGL((k_scan_gemv32<NB, 1>), grid, block, 0, st, (const float*)h->store, (const float*)h->invnorm, qf, invq,
                           thr, cnt, surv, h->N, h->nkb, B, L, mask, PrepArgs{});
    else if (wgs == 4)
        hipLaunchKernelGGL((k_scan_gemv32<NB, 4>), grid, block, 0, st, (const float*)h->store, (const float*)h->invnorm, qf, invq,
                           thr, cnt, surv, h->N, h->nkb, B, L, mask, PrepArgs{});
    else
        hipLaunchKernelGGL((k_scan_gemv32<NB, 16>), grid, block, 0, st, (const float*)h->store, (const float*)h->invnorm, qf, invq,
                           thr, cnt, surv, h->N, h->nkb, B, L, mask, PrepArgs{});
    LAUNCHCHK();
    return MEM_OK;
}

// One sparse pass: 32 or 64 rows and 16 .. 64 queries to a workgroup.
template <int DT, int MQ, int MR, bool FIRST>
int launch_direct(evomem* h, const Scratch& sc, hipStream_t st, int Bp, const Level& L, const Mask& mask, int B, const PrepArgs* prep) {
    constexpr int lds = direct_lds_bytes<MQ, MR, FIRST>();
    auto kern = k_scan_direct<DT, MQ, MR, FIRST>;
    if constexpr (lds > 64 * 1024) {
        static bool lds_set[MAX_DEVICES] = {};
        if (!lds_set[h->device]) {
            HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            lds_set[h->device] = true;
        }
    }
    const int nqt = (B + 16 * MQ - 1) / (16 * MQ), units = L.ntiles * (TILE_ROWS / (16 * MR));
    unsigned char* ws = sc.base;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * ((units + 7) / 8) * nqt + (FIRST ? Bp : 0))), dim3(64 * DIRECT_WAVES), lds, st, (const void*)h->store, (const float*)h->invnorm,
                       (const uint16_t*)(ws + sc.w.qop), (const float*)(ws + sc.w.invq), (const float*)(ws + sc.w.thr),
                       (uint32_t*)(ws + sc.w.cnt), (uint64_t*)(ws + sc.w.surv), h->N, h->nkb, Bp, nqt, L, mask, B, prep ? *prep : PrepArgs{});
    LAUNCHCHK();
    return MEM_OK;
}
// Rows and queries (tr and tq) of a direct workgroup: 32 rows while that makes enough workgroups of a sparse pass.
constexpr int direct_tq(int B) { return B <= 16 ? 16 : B <= 32 ? 32 : 64; }
constexpr int direct_tr(int B) { return B <= 64 ? 32 : 64; }
// Direct or tile by tile?  Either way a compute unit was seen to take in 20 to 30 GB/s of operands in such a pass (mid-size
// fp32 bank, 64 queries: 393 KB in 12.8 us, as 128-byte requests of 420 cycles, some forty in flight on average), so
// what decides is how many rows and queries the busiest one reads.  The direct scan pays for its tail (partial sums, counters) on top, hence the quarter.  Measured, direct against by tiles
// (us; share of the operands the direct scan reads): 32 tiles of 1024 bf16, one query 5.6 / 17.2 (0.17), 64 queries 9.4 / 17.5
// (0.33), 256 queries 20.8 / 20.0 (0.89); 64 tiles, 64 queries 20.0 / 21.0 (0.67); 128 tiles, 64 queries 34 / 23 (1.2);
// 45 tiles of 4096 fp16, 128 queries 79 / 66 (0.89); 32 tiles of 1024 fp32, 64 queries 14.8 / 33.6 (0.33).
bool use_direct(const Level& L, int B, int Bp, int qt) {
    const int tq = direct_tq(B), tr = direct_tr(B);
    const int64_t direct = ((int64_t)L.ntiles * (TILE_ROWS / tr) * ((B + tq - 1) / tq) + 255) / 256 * (tr + tq);
    const int64_t tiles = ((int64_t)L.ntiles * (Bp / qt) + 255) / 256 * (TILE_ROWS + qt);
    return direct * 4 <= tiles * 3;
}
int launch_direct_any(evomem* h, const Scratch& sc, hipStream_t st, int Bp, const Level& L, const Mask& mask, int B, const PrepArgs* first) {
    int rc = MEM_OK;
    with_store_type(h->dtype, [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        rc = B <= 16   ? (first ? launch_direct<DT, direct_tq(16) / 16, direct_tr(16) / 16, true>(h, sc, st, Bp, L, mask, B, first)
                                : launch_direct<DT, direct_tq(16) / 16, direct_tr(16) / 16, false>(h, sc, st, Bp, L, mask, B, nullptr))
             : B <= 32 ? launch_direct<DT, direct_tq(32) / 16, direct_tr(32) / 16, false>(h, sc, st, Bp, L, mask, B, nullptr)
             : B <= 64 ? launch_direct<DT, direct_tq(64) / 16, direct_tr(64) / 16, false>(h, sc, st, Bp, L, mask, B, nullptr)
                       : launch_direct<DT, direct_tq(256) / 16, direct_tr(256) / 16, false>(h, sc, st, Bp, L, mask, B, nullptr);
    });
    return rc;
}

// One pass of the exhaustive selection.  Queries share a bank read in groups: of eight when there are more than
// four, else of the smallest power of two that holds them (an unused slot would cost as much as a query).
int launch_exact_scan(evomem* h, const Scratch& sc, hipStream_t st, int B, const Level& L) {
    unsigned char* ws = sc.base;
    const int64_t oct_units = ((int64_t)L.ntiles * (TILE_ROWS / EXACT_ROWS) + 7) / 8;    // row units per XCD
    auto launch = [&](auto dt, auto nb) {
        constexpr int DT = decltype(dt)::value, NB = decltype(nb)::value;
        const int groups = (B + NB - 1) / NB;
        int64_t walkers = 2048 / groups < 1 ? 1 : 2048 / groups;                           // per XCD; at most 16,384 workgroups or one per unit
        if (walkers > oct_units) walkers = oct_units;
        hipLaunchKernelGGL((k_exact_scan<DT, NB>), dim3((unsigned)(8 * walkers * groups)), dim3(256), 0, st, (const void*)h->store,
                           (const float*)(ws + sc.w.qf), (const double*)(ws + sc.w.invq64), (uint64_t*)(ws + sc.w.surv),
                           (uint32_t*)(ws + sc.w.cnt), (double*)(ws + sc.w.exact), sc.exact_stride, h->N, h->nkb, B, groups, L);
    };
    with_store_type(h->dtype, [&](auto dt) {
        if (B == 1) launch(dt, std::integral_constant<int, 1>{});
        else if (B == 2) launch(dt, std::integral_constant<int, 2>{});
        else if (B <= 4) launch(dt, std::integral_constant<int, 4>{});
        else launch(dt, std::integral_constant<int, EXACT_NB>{});
    });
    LAUNCHCHK();
    return MEM_OK;
}

// A denser pass of it on the matrix cores (32 queries to a tile): the ordinary scan finds the rows that may reach a query's cut,
// and those few are scored in fp64.  Scoring every row in fp64 costs by the query, and a group of queries reads the bank once.
// Whole calls, us, in fp64 and so: 1M x 1024 bf16, one query 394, 390; 2 430, 382; 4 485, 386; 8 682, 406; 16 1245, 415; 64 4552, 665;
// 390,000 x 1024 fp32, 4 339, 341; 5 365, 340; 16 621, 353; 60,000 x 768 bf16 (220 tiles), 4 58.8, 60.7; 5 70.8, 62.4; 16 92.8, 67.4.
// The fewer the queries the more fp64 waits for memory too, and the more the idle workgroups of a last round of tiles count: 300,000 x
// 4096 fp16 (1098 tiles, 4.3 to a workgroup), 4 512, 549; 8 732, 554; 16 1310, 610; 100,000 (366, 1.4), 8 283, 336; 16 468, 299; 1M x 256
// fp16 (3662, 14.3), 4 184, 146.  So two to four want many tiles and rounds of nine tenths, five to eight one round or rounds of four fifths.
// A staged row cost 1.8 times what it costs in a pass that scores a group of eight, 2.6 times for four, when this was drawn (about as much
// since a row is staged once for its queries), and the scan itself half to three quarters of such a pass, so what a pass is expected to stage (k1 * rho rows a query) may be a fifth or a seventeenth of the rows
// times groups; large pools over short passes stay in fp64.  1024 bf16, all in fp64 and so, us: 500,000 rows, pool of 600, 5 queries 416, 346, 16
// 661, 377; pool of 2048, 5 544, 490; 200,000 rows, pool of 600, 16 319, 263; 100,000 rows: the same, no pass qualifies.
bool use_exact_mfma(int dtype, const Level& L, int B, int k1) {
    const int64_t n = L.ntiles, places = (n + 255) / 256 * 256;
    if (L.rho == 0 || B == 1) return false;
    const int64_t staged = (int64_t)k1 * L.rho * B, scored = n * TILE_ROWS * ((B + EXACT_NB - 1) / EXACT_NB);
    if (staged * (B <= 4 ? 17 : 5) > scored) return false;
    if (B <= 4) return dtype != MEM_F32 && n >= 1024 && places * 9 <= n * 10;
    if (B <= EXACT_NB && n > 256 && places * 4 > n * 5) return false;
    return n * ((B + 31) / 32) >= 128;
}
int launch_exact_mfma(evomem* h, const Scratch& sc, hipStream_t st, int Bp, const Level& L, int k1, int B) {
    int rc = MEM_OK;
    const Mask none{nullptr, nullptr, nullptr};
    with_store_type(h->dtype, [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        rc = B > 32 ? launch_mfma<DT, 2, 1, 4, 4, false, false, true>(h, sc, st, Bp, L, k1, none, B)
                    : launch_mfma<DT, 2, 1, 4, 4, false, true, true>(h, sc, st, Bp, L, k1, none, B);
    });
    return rc;
}

// What the passes of the exhaustive selection lost (most calls: nothing, and the launch ends at once).
template <int DT>
int launch_exact_walk(evomem* h, const Scratch& sc, hipStream_t st, int B, int k1) {
    auto kern = k_exact_walk<DT>;
    static bool lds_set[MAX_DEVICES] = {};
    if (!lds_set[h->device]) {
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, WALK_LDS));
        lds_set[h->device] = true;
    }
    unsigned char* ws = sc.base;
    hipLaunchKernelGGL(kern, dim3(WALK_GROUPS), dim3(WALK_T), WALK_LDS, st, (const void*)h->store, (const float*)(ws + sc.w.qf),
                       (const double*)(ws + sc.w.invq64), (uint64_t*)(ws + sc.w.surv), (const uint32_t*)(ws + sc.w.cnt),
                       (double*)(ws + sc.w.exact), sc.exact_stride, h->N, h->nkb, k1, B, sc.lists());
    LAUNCHCHK();
    return MEM_OK;
}

}  // namespace

extern "C" int mem_plan_levels(int64_t N, int k1, int* stride, int* rho, int* ntiles, int max_levels) {
    if (N < 1 || N > 2147483647ll - 256 || k1 < 1 || k1 > MEM_MAX_K1 || !stride || !rho || !ntiles || max_levels < 1) return -1;
    const Plan p = plan_levels(N, k1, SURV_CAP);
    for (int i = 0; i < p.n && i < max_levels; ++i) { stride[i] = p.lv[i].stride; rho[i] = p.lv[i].rho; ntiles[i] = p.lv[i].ntiles; }
    return p.n;
}

static int retrieve_impl(evomem_t* h, const float* queries_dev, int B, int stage, int k1, int k2, float lambda,
                         int32_t* out_ids_dev, float* out_scores_dev, int32_t* out_cand_ids_dev,
                         float* out_cand_sims_dev, void* hip_stream, const EpsGreedy& eg, const Mask& mask,
                         const Scratch& sc, int max_B, int max_k1, bool exhaustive = false) {
    if (!h || B < 0 || B > max_B || (stage != 0 && stage != 1) || k1 < 1 || k2 < 1 || k2 > k1 || k1 > max_k1)
        return MEM_EINVAL;
    if (!(lambda >= 0.f && lambda <= 1.f)) return MEM_EINVAL;
    if ((out_cand_ids_dev == nullptr) != (out_cand_sims_dev == nullptr)) return MEM_EINVAL;
    if (B == 0) return MEM_OK;
    if (!queries_dev || !out_ids_dev || !out_scores_dev) return MEM_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    unsigned char* ws = sc.base;
    const bool gemv = B <= GEMV_MAX_B && h->dtype == MEM_F32;
    // query tile of the MFMA scan and padded batch
    int qt = B <= 32 ? 32 : B <= 64 ? 64 : B <= 128 ? 128 : 256;
    const int Bp = gemv ? B : (int)round_up(B, qt);
    float* qf = (float*)(ws + sc.w.qf);
    uint16_t* qop = (uint16_t*)(ws + sc.w.qop);
    float* invq = (float*)(ws + sc.w.invq);
    double* invq64 = (double*)(ws + sc.w.invq64);
    float* thr = (float*)(ws + sc.w.thr);
    uint32_t* cnt = (uint32_t*)(ws + sc.w.cnt);
    uint32_t* flags = (uint32_t*)(ws + sc.w.flags);
    uint64_t* surv = (uint64_t*)(ws + sc.w.surv);
    double* exact = (double*)(ws + sc.w.exact);
    const int exact_stride = sc.exact_stride;
    h->last_flags = flags;
    h->last_B = B;
    uint32_t* counters = (uint32_t*)(ws + sc.w.counters);

    // A pool of more than 256 leaves a list of 8192 little room for what a denser pass brings (a list is meant to be filled to a
    // quarter), and the passes become many: 1024 tiles with a pool of 960 take six.  While three quarters of the lists would lie idle,
    // a query gets two of them: three passes (64 queries, 262,144 x 1024 bf16, whole call 235.6 -> 203.0 us).  Smaller pools would
    // save no pass that is worth a selection over twice the keys.
    const bool two = k1 > SMALL_K1_MAX && !exhaustive && sc.lists() >= 4 * B;
    const int cap = two ? 2 * SURV_CAP : SURV_CAP;
    Plan plan{};
    uint32_t cnt0 = 0;      // valid rows of the sparsest pass (a prefix of its last tile may be all that exists)
    if (h->N > 0) {
        plan = plan_levels(h->N, k1, cap);
        const Level& L0 = plan.lv[0];
        const int64_t last = level_tile(L0, L0.ntiles - 1) * TILE_ROWS;
        const int64_t in_last = h->N - last < TILE_ROWS ? h->N - last : TILE_ROWS;
        cnt0 = (uint32_t)((int64_t)(L0.ntiles - 1) * TILE_ROWS + in_last);
    }
    // a sparse pass has few bank tiles: give each workgroup fewer queries, so that more
    // workgroups share the pass and each one's k-loop is shorter
    auto tile_of = [&](const Level& L) {
        int lqt = qt;
        while (lqt > 32 && (int64_t)L.ntiles * (Bp / lqt) < 128) lqt >>= 1;
        return lqt;
    };
    auto direct = [&](const Level& L) { return !gemv && use_direct(L, B, Bp, tile_of(L)); };
    const PrepArgs prep{queries_dev, qf, qop, invq, invq64, thr, cnt, flags, cnt0, B, Bp, h->d, h->nkb, ((uintptr_t)queries_dev & 15) == 0, !gemv};
    // The queries are prepared in the launch of the first pass where that pass reads them as given: for few queries.  With more, what a
    // workgroup converts of them costs what the launch saves.  Whole calls, us, in a launch of their own and fused: one query,
    // 4096 x 768 fp32 22.1, 19.0; seven, 30,011 x 200 fp16 33.2, 30.7; one, 1M x 1024 bf16 359.9, 355.8; 32, 300,007 x 384 fp16
    // masked 92.6, 92.7; 64, 65,536 x 1024 fp32 83.5, 84.0; 64, 262,144 x 1024 bf16 235.6, 238.1.
    const bool fused = plan.n > 0 && !exhaustive && prep.aligned && (gemv || (B <= 16 && direct(plan.lv[0])));
    if (!fused) {
        with_store_type(h->dtype, [&](auto dt) {
            constexpr int DT = decltype(dt)::value;
            if (!gemv && prep_by_fragments(DT == 0, Bp, h->nkb)) hipLaunchKernelGGL(k_prep_fragments<DT>, dim3((unsigned)prep_fragment_workgroups(Bp, h->nkb)), dim3(256), 0, st, prep);
            else hipLaunchKernelGGL(k_prep_queries<DT>, dim3(Bp), dim3(256), 0, st, prep);
        });
        LAUNCHCHK();
    }

    // rounding margin of the scan's fp32 similarities
    float eps = (float)(h->nkb * KB) * 5.97e-8f + 1e-6f;
    if (h->dtype == MEM_F32 && !gemv) eps += 2e-5f;      // bf16 hi/lo split of fp32 values
    if (!gemv) eps += 2e-5f;                             // threshold * norm carried as 16-bit hi/lo pairs
    const float margin = 2.f * eps;

    if (h->N > 0 && exhaustive) {
        bool mfma_ahead = false;
        for (int li = 0; li < plan.n; ++li) mfma_ahead = mfma_ahead || use_exact_mfma(h->dtype, plan.lv[li], B, k1);
        for (int li = 0; li < plan.n; ++li) {
            const Level& L = plan.lv[li];
            const int rc = use_exact_mfma(h->dtype, L, B, k1) ? launch_exact_mfma(h, sc, st, Bp, L, k1, B) : launch_exact_scan(h, sc, st, B, L);
            if (rc != MEM_OK) return rc;
            if (li == plan.n - 1) break;
            hipLaunchKernelGGL(k_exact_select, dim3(B), dim3(1024), 0, st, surv, cnt, exact, exact_stride, k1, keep_of(k1), thr, (const float*)invq,
                               (const double*)invq64, mfma_ahead ? margin : 0.f);
            LAUNCHCHK();
        }
        if (plan.n > 1) {                                            // (a single pass never overflows)
            int rc = MEM_OK;
            with_store_type(h->dtype, [&](auto dt) {
                rc = launch_exact_walk<decltype(dt)::value>(h, sc, st, B, k1);
            });
            if (rc != MEM_OK) return rc;
        }
    }
    if (h->N > 0 && !exhaustive) {
        for (int li = 0; li < plan.n; ++li) {
            const Level& L = plan.lv[li];
            const bool prof = h->prof_on && h->prof_n < MAX_PROFILE;
            if (prof) HIPCHK(hipEventRecord(h->ev[2 * h->prof_n], st));
            int rc;
            const PrepArgs* first = fused && li == 0 ? &prep : nullptr;
            if (gemv) {
                rc = B == 1 ? launch_gemv<1>(h, sc, st, B, L, mask, first) : B == 2 ? launch_gemv<2>(h, sc, st, B, L, mask, first) : launch_gemv<4>(h, sc, st, B, L, mask, first);
            } else if (direct(L)) {
                rc = launch_direct_any(h, sc, st, Bp, L, mask, B, first);
            } else {
                rc = mask.tags ? launch_mfma_any<true>(h, sc, st, Bp, tile_of(L), L, k1, mask, B) : launch_mfma_any<false>(h, sc, st, Bp, tile_of(L), L, k1, mask, B);
            }
            if (rc != MEM_OK) return rc;
            if (prof) {
                HIPCHK(hipEventRecord(h->ev[2 * h->prof_n + 1], st));
                int64_t rows = (int64_t)L.ntiles * TILE_ROWS;
                h->prof_rows[h->prof_n++] = rows;
            }
            if (li == plan.n - 1) break;                                // the last selection is the tail's
            hipLaunchKernelGGL(two ? k_select<16> : k_select<8>, dim3(B), dim3(1024), 0, st, surv, cnt, thr, (const float*)invq, counters, flags, k1, margin,
                               mask.tags != nullptr, keep_of(k1));
            LAUNCHCHK();
        }
    }
    // Few queries: a query's candidates are shared by several workgroups, as long as that leaves a compute unit to each
    // and more than 96 KB of rows to gather.  Measured with 1, 2, 4 and 8: one query, 128 x 2 KB 20.0, 17.9, 15.2, 14.4 us;
    // 64 queries, 64 x 4 KB 17.1, 15.2, 14.8, 20.7; 128 queries, 256 x 8 KB 110, 80, 92, 110; 64 queries, 960 x 2 KB 93, 68, 54,
    // 62; one query, 32 x 3 KB 10.9, 12.4, 12.0, 12.0.
    TailArgs ta{};
    ta.eg = eg;
    ta.surv = surv; ta.cnt = cnt; ta.counters = counters; ta.flags = flags;
    ta.arrived = reinterpret_cast<uint32_t*>(qop + (int64_t)(h->dtype == MEM_F32 ? 2 * h->nkb : h->nkb) * Bp * KB);
    ta.store = h->store; ta.qf = qf; ta.invq64 = invq64; ta.exact = exact; ta.spare = (int64_t)sc.lists() * SURV_CAP >= 2ll * B * cap ? surv + (int64_t)B * cap : nullptr; ta.qstage = h->q + (int64_t)stage * h->capacity;
    ta.out_ids = out_ids_dev; ta.out_scores = out_scores_dev; ta.cand_ids = out_cand_ids_dev; ta.cand_sims = out_cand_sims_dev;
    ta.lambda = (double)lambda; ta.nkb = h->nkb; ta.exact_stride = exact_stride; ta.k1 = k1; ta.k2 = k2;
    ta.may_have_empty = mask.tags != nullptr || exhaustive; ta.mode = exhaustive ? SEL_EXACT : SEL_FINAL; ta.margin = exhaustive ? EXACT_KEY_MARGIN : margin;
    const int64_t gather = (int64_t)k1 * h->nkb * KB * (h->dtype == MEM_F32 ? 4 : 2);
    int parts = 1;
    while (parts < 8 && B * parts * 2 <= 256 && gather / parts > 96 * 1024) parts <<= 1;
    const bool big = k1 > SMALL_K1_MAX;
    const size_t lds = tail_lds(k1) + (size_t)h->nkb * KB * 4;        // and the query
    static_assert(tail_lds(BIG_K1_MAX) + 16384 * 4 + TAIL_STATIC_LDS <= 160 * 1024, "the largest pool with the longest rows");
    if (lds + TAIL_STATIC_LDS > 64 * 1024) {
        static bool lds_set[MAX_DEVICES] = {};
        if (!lds_set[h->device]) {
            bool ok = true;
            for (const void* k : {reinterpret_cast<const void*>(k_tail<0, true>), reinterpret_cast<const void*>(k_tail<1, true>), reinterpret_cast<const void*>(k_tail<2, true>),
                                  reinterpret_cast<const void*>(k_tail<0, true, 16>), reinterpret_cast<const void*>(k_tail<1, true, 16>), reinterpret_cast<const void*>(k_tail<2, true, 16>),
                                  reinterpret_cast<const void*>(k_tail<0, false>), reinterpret_cast<const void*>(k_tail<1, false>), reinterpret_cast<const void*>(k_tail<2, false>)})
                ok = ok && hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(tail_lds(BIG_K1_MAX) + 16384 * 4)) == hipSuccess;
            if (!ok) return MEM_EHIP;
            lds_set[h->device] = true;
        }
    }
    with_store_type(h->dtype, [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        const dim3 grid((unsigned)B, (unsigned)parts), block(TAIL_T);
        if (two) hipLaunchKernelGGL((k_tail<DT, true, 16>), grid, block, lds, st, ta);
        else if (big) hipLaunchKernelGGL((k_tail<DT, true>), grid, block, lds, st, ta);
        else hipLaunchKernelGGL((k_tail<DT, false>), grid, block, lds, st, ta);
    });
    LAUNCHCHK();
    return MEM_OK;
}

// the scratch area a handle was created with
static Scratch own_scratch(const evomem* h) { return Scratch{h->ws, h->w, keep_of(h->max_k1)}; }

extern "C" int mem_retrieve(evomem_t* h, const float* queries_dev, int B, int stage, int k1, int k2, float lambda,
                            int32_t* out_ids_dev, float* out_scores_dev, int32_t* out_cand_ids_dev,
                            float* out_cand_sims_dev, void* hip_stream) {
    if (!h) return MEM_EINVAL;
    const EpsGreedy greedy{0, 0, 0, nullptr};
    return retrieve_impl(h, queries_dev, B, stage, k1, k2, lambda, out_ids_dev, out_scores_dev, out_cand_ids_dev,
                         out_cand_sims_dev, hip_stream, greedy, Mask{nullptr, nullptr, nullptr}, own_scratch(h), h->max_B, h->max_k1);
}

// The library's own scratch area for mem_retrieve_static: one array per GPU, in that GPU's memory for
// as long as the library is loaded.  In host code the array's name only stands for the symbol; its
// device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
static unsigned char* scratch_ptr[MAX_DEVICES] = {};

extern "C" int mem_retrieve_static(evomem_t* h, const float* queries_dev, int B, int stage, int k1, int k2, float lambda,
                                   int32_t* out_ids_dev, float* out_scores_dev, int32_t* out_cand_ids_dev,
                                   float* out_cand_sims_dev, void* hip_stream) {
    if (!h) return MEM_EINVAL;
    if (h->nkb * KB > STATIC_MAX_D) return MEM_EINVAL;            // B and k1 are checked against their limits below
    int cur = -1;
    HIPCHK(hipGetDevice(&cur));
    if (cur != h->device) return MEM_ESTATE;
    if (!scratch_ptr[cur]) {                                      // first call on this device
        unsigned char* p = nullptr;
        HIPCHK(hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)));
        if (!p) return MEM_EHIP;
        // the counter block must start at zero; everything else is written before it is read in every call
        hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, static_cast<hipStream_t>(hip_stream),
                           reinterpret_cast<uint32_t*>(p + STATIC_W.counters), 64);
        LAUNCHCHK();
        scratch_ptr[cur] = p;
    }
    const EpsGreedy greedy{0, 0, 0, nullptr};
    return retrieve_impl(h, queries_dev, B, stage, k1, k2, lambda, out_ids_dev, out_scores_dev, out_cand_ids_dev,
                         out_cand_sims_dev, hip_stream, greedy, Mask{nullptr, nullptr, nullptr},
                         Scratch{scratch_ptr[cur], STATIC_W, keep_of(STATIC_MAX_K1)}, STATIC_MAX_B, STATIC_MAX_K1);
}

extern "C" int mem_retrieve_exact(evomem_t* h, const float* queries_dev, int B, int stage, int k1, int k2, float lambda,
                                  int32_t* out_ids_dev, float* out_scores_dev, int32_t* out_cand_ids_dev,
                                  float* out_cand_sims_dev, void* hip_stream) {
    if (!h) return MEM_EINVAL;
    const EpsGreedy greedy{0, 0, 0, nullptr};
    return retrieve_impl(h, queries_dev, B, stage, k1, k2, lambda, out_ids_dev, out_scores_dev, out_cand_ids_dev,
                         out_cand_sims_dev, hip_stream, greedy, Mask{nullptr, nullptr, nullptr}, own_scratch(h), h->max_B, h->max_k1, true);
}

extern "C" int mem_retrieve_flags(evomem_t* h, uint32_t* out_flags_dev, int B, void* hip_stream) {
    if (!h || B < 0 || (B > 0 && !out_flags_dev)) return MEM_EINVAL;
    if (B == 0) return MEM_OK;
    if (!h->last_flags || B > h->last_B) return MEM_ESTATE;      // no retrieve yet, or a smaller one
    HIPCHK(hipMemcpyAsync(out_flags_dev, h->last_flags, sizeof(uint32_t) * (size_t)B, hipMemcpyDeviceToDevice,
                          static_cast<hipStream_t>(hip_stream)));
    return MEM_OK;
}

extern "C" int mem_retrieve_eps(evomem_t* h, const float* queries_dev, int B, int stage, int k1, int k2, float lambda,
                                float eps, uint64_t seed, uint64_t step, int32_t* out_ids_dev, float* out_scores_dev,
                                int32_t* out_cand_ids_dev, float* out_cand_sims_dev, unsigned char* out_explored_dev,
                                void* hip_stream) {
    if (!h) return MEM_EINVAL;
    if (!(eps >= 0.f && eps <= 1.f)) return MEM_EINVAL;
    const EpsGreedy eg{(uint64_t)((double)eps * 4294967296.0), seed, step, out_explored_dev};
    return retrieve_impl(h, queries_dev, B, stage, k1, k2, lambda, out_ids_dev, out_scores_dev, out_cand_ids_dev,
                         out_cand_sims_dev, hip_stream, eg, Mask{nullptr, nullptr, nullptr}, own_scratch(h), h->max_B, h->max_k1);
}

extern "C" int mem_attach_tags(evomem_t* h, uint32_t* tags_dev) {
    if (!h || !tags_dev) return MEM_EINVAL;
    HIPCHK(hipMemset(tags_dev, 0, sizeof(uint32_t) * (size_t)h->capacity));
    h->tags = tags_dev;
    return MEM_OK;
}

extern "C" int mem_set_tags(evomem_t* h, int64_t first, int64_t n, const uint32_t* tags_dev, void* hip_stream) {
    if (!h || first < 0 || n < 0 || first + n > h->N) return MEM_EINVAL;
    if (!h->tags) return MEM_ESTATE;
    if (n == 0) return MEM_OK;
    if (!tags_dev) return MEM_EINVAL;
    HIPCHK(hipMemcpyAsync(h->tags + first, tags_dev, sizeof(uint32_t) * (size_t)n, hipMemcpyDeviceToDevice,
                          static_cast<hipStream_t>(hip_stream)));
    return MEM_OK;
}

extern "C" int mem_retrieve_masked(evomem_t* h, const float* queries_dev, int B, int stage, int k1, int k2, float lambda,
                                   const uint32_t* allow_types_dev, const uint32_t* exclude_group_dev,
                                   int32_t* out_ids_dev, float* out_scores_dev, int32_t* out_cand_ids_dev,
                                   float* out_cand_sims_dev, void* hip_stream) {
    if (!h) return MEM_EINVAL;
    if (!h->tags) return MEM_ESTATE;
    if (B > 0 && (!allow_types_dev || !exclude_group_dev)) return MEM_EINVAL;
    const EpsGreedy greedy{0, 0, 0, nullptr};
    return retrieve_impl(h, queries_dev, B, stage, k1, k2, lambda, out_ids_dev, out_scores_dev, out_cand_ids_dev,
                         out_cand_sims_dev, hip_stream, greedy, Mask{h->tags, allow_types_dev, exclude_group_dev}, own_scratch(h),
                         h->max_B, h->max_k1);
}

extern "C" int mem_select_by_q(evomem_t* h, const int32_t* set_ids_dev, int64_t n_ids, const int64_t* set_offsets_dev,
                               int G, int stage, float eps, uint64_t seed, uint64_t step, int32_t* out_ids_dev,
                               float* out_q_dev, unsigned char* out_explored_dev, void* hip_stream) {
    if (!h || G < 0 || n_ids < 0 || (stage != 0 && stage != 1) || !(eps >= 0.f && eps <= 1.f)) return MEM_EINVAL;
    if (G == 0) return MEM_OK;
    if (!set_offsets_dev || !out_ids_dev || !out_q_dev || (n_ids > 0 && !set_ids_dev)) return MEM_EINVAL;
    const EpsGreedy eg{(uint64_t)((double)eps * 4294967296.0), seed, step, out_explored_dev};
    hipLaunchKernelGGL(k_select_by_q, dim3((unsigned)G), dim3(SP_LANES), 0, static_cast<hipStream_t>(hip_stream),
                       set_ids_dev, n_ids, set_offsets_dev, (const float*)(h->q + (int64_t)stage * h->capacity), h->N, eg,
                       out_ids_dev, out_q_dev, (uint32_t*)(h->ws + h->w.counters));
    LAUNCHCHK();
    return MEM_OK;
}

extern "C" int mem_update_q(evomem_t* h, const int32_t* ids_dev, int64_t M, int stage, const float* rewards_dev,
                            float alpha, void* hip_stream) {
    if (!h || M < 0 || (stage != 0 && stage != 1) || !(alpha > 0.f && alpha <= 1.f)) return MEM_EINVAL;
    if (M == 0) return MEM_OK;
    if (!ids_dev || !rewards_dev) return MEM_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint32_t* counters = (uint32_t*)(h->ws + h->w.counters);
    static bool lds_set[MAX_DEVICES] = {};          // the kernel's LDS list can exceed the default 64 KB limit
    if (!lds_set[h->device]) {
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_update_q), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)upd_lds(UPD_CHUNK)));
        lds_set[h->device] = true;
    }
    for (int64_t off = 0; off < M; off += UPD_CHUNK) {
        int m = (int)(M - off < UPD_CHUNK ? M - off : UPD_CHUNK);
        const int lg = upd_log2_buckets(m);
        hipLaunchKernelGGL(k_update_q, dim3(1u << lg), dim3(1024), upd_lds(m), st, ids_dev + off, rewards_dev + off, m,
                           h->q + (int64_t)stage * h->capacity, h->N, alpha, counters, lg);
        LAUNCHCHK();
    }
    return MEM_OK;
}
