// C ABI of the IDKM library: argument validation, scratch management and the
// scheduling of passes over W.  All arithmetic of the method runs in the kernels.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstddef>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <algorithm>
#include <string>
#include <thread>
#include <vector>

#include "../../include/idkm.h"
#include "common.hpp"
#include "dispatch.h"
#include "persist_small.hpp"
#include "persist_lane.hpp"

namespace idkm {

KernelFn small_kernel_0(int, int, int);
KernelFn small_kernel_1(int, int, int);
KernelFn lane_kernel_0(int, int, int);
KernelFn lane_kernel_1(int, int, int);

KernelFn small_kernel(int K, int D, int dist, int pass) {
    return dist == DIST_L2 ? small_kernel_0(K, D, pass) : small_kernel_1(K, D, pass);
}
PersistFns persist_lane_kernel_0(int, int, bool, bool);
PersistFns persist_lane_kernel_1(int, int, bool, bool);
PersistFns persist_lane_kernel(int KPL, int D, int dist, bool bwd, bool matrix) {
    return dist == DIST_L2 ? persist_lane_kernel_0(KPL, D, bwd, matrix) : persist_lane_kernel_1(KPL, D, bwd, matrix);
}
KernelFn lane_kernel(int KPL, int D, int dist, int pass) {
    return dist == DIST_L2 ? lane_kernel_0(KPL, D, pass) : lane_kernel_1(KPL, D, pass);
}

constexpr int MAX_K = 1024, MAX_D = 8, MAX_KD = 4096;
constexpr int MAX_NACC = MAX_K * 5 > MAX_KD + MAX_K ? MAX_K * 5 : MAX_KD + MAX_K;  // k (d+1) <= kd + k

// ---------------------------------------------------------------- small utility kernels

__global__ void k_init_forward(Args a, const float* C0, double tol, int max_iter) {
    const int kd = a.k * a.d;
    for (int idx = threadIdx.x; idx < kd; idx += blockDim.x) {
        float c = C0[idx];
        a.Cd[idx] = (double)c;
        a.Cf[idx] = c;
    }
    if (threadIdx.x == 0) {
        Ctrl* c = a.ctrl;
        c->abort_flag = 0;
        c->done = 0;
        c->iters = 0;
        c->converged = 0;
        c->empty = 0;
        c->nonfinite = 0;
        c->max_iter = max_iter;
        c->residual = 0.0;
        c->tol = tol;
        c->b_done = 1;
    }
}

__global__ void k_init_backward(Args a, int mode, double tol, int max_iter, double alpha, int basis) {
    Ctrl* c = a.ctrl;
    c->abort_flag = 0;
    c->nonfinite = 0;  // (a forward on the persistent path does not pass through k_init_forward)
    c->b_done = 0;
    c->b_iters = 0;
    c->b_converged = 0;
    c->b_attempt = 0;
    c->b_grow = 0;
    c->b_halvings = 0;
    c->b_max_iter = max_iter;
    c->b_mode = mode;
    c->b_alpha = alpha;
    c->b_prev = __builtin_inf();
    c->b_vnorm = 0.0;
    c->b_residual = 0.0;
    c->b_tol = tol;
    const int kd = a.k * a.d;
    c->k_R = kd < basis ? kd : basis;
    c->k_phase = 0;
    c->k_j = 0;
    c->k_stall = 0;
    c->k_beta = 0.0;
}

__global__ void k_reset_launch_seq(Ctrl* c) { c->launch_seq = 0; }
__global__ void k_add_launch_seq(Ctrl* c, unsigned int n) { c->launch_seq += n; }

// Hs = (g / n) / tau from a caller-supplied float32 cotangent; arms one raw (dF/dC)^T pass.
__global__ void k_set_g(Args a, const float* g) {
    const int kd = a.k * a.d;
    for (int idx = threadIdx.x; idx < kd; idx += blockDim.x) {
        double gv = (double)g[idx];
        a.gd[idx] = gv;
        a.vd[idx] = 0.0;
        store_h(a, idx, gv);
    }
    if (threadIdx.x == 0) {
        Ctrl* c = a.ctrl;
        c->b_done = 0;
        c->b_iters = 0;
        c->b_attempt = 0;
        c->b_grow = 0;
        c->b_halvings = 0;
        c->b_max_iter = 1;
        c->b_alpha = 1.0;
        c->b_prev = __builtin_inf();
        c->b_vnorm = 0.0;
        c->b_tol = 0.0;
    }
}

__global__ void k_fill_u64(unsigned long long* p, size_t n, unsigned long long v) {
    for (size_t i = threadIdx.x + (size_t)blockIdx.x * blockDim.x; i < n; i += (size_t)blockDim.x * gridDim.x) p[i] = v;
}

__global__ void k_f64_to_f32(const double* src, float* dst, int n) {
    for (int i = threadIdx.x + blockIdx.x * blockDim.x; i < n; i += blockDim.x * gridDim.x) dst[i] = (float)src[i];
}

}  // namespace idkm

using namespace idkm;

namespace {
struct Deferred;
}

struct idkm_ctx {
    int device = 0;
    std::string err;
    idkm_path path = IDKM_PATH_AUTO;
    // device scratch
    Ctrl* ctrl = nullptr;
    Ctrl* h_ctrl = nullptr;  // pinned host mirror
    unsigned int* tickets = nullptr;  // arrival counters of the stream path, zero between launches
    unsigned int stream_launches = 0; // upper bound of Ctrl::launch_seq
    int gmres_basis = 64;             // basis length of IDKM_BWD_GMRES before a restart (idkm_set_gmres_basis, <= GM_RMAX)
    double *Cd = nullptr, *nd = nullptr, *Fd = nullptr, *gd = nullptr, *vd = nullptr, *ud = nullptr;
    float *Cf = nullptr, *Ff = nullptr, *Hs = nullptr;
    double *stage = nullptr, *tot = nullptr;
    double* partials = nullptr;
    size_t partials_cap = 0;  // in doubles
    double* kry = nullptr;    // Krylov workspace of IDKM_BWD_GMRES (allocated on first use)
    size_t kry_cap = 0;       // in doubles
    // persistent path
    int num_cu = 0;
    bool coop = false;
    bool coop_launch = false;  // IDKM_COOPERATIVE=1 launches the persistent kernels cooperatively
    int min_vec_per_thread = 4;  // vectors per thread before another workgroup is added (IDKM_MIN_VPT)
    bool tree_exchange = true;   // two-level (die-local, then cross-die) exchange for full-device teams (IDKM_TREE=0: off)
    bool tree_remote = false;    // IDKM_TREE=2: hop 1 with device-scope stores, as for workgroups that are not on their leader's die
    // idkm_set_kernel_timing: events recorded on the caller's stream right before and after a persistent launch
    bool timing = false;
    bool timed = false;          // ev0 / ev1 bracket the last persistent launch
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    hipEvent_t ev_order = nullptr;  // see join_running (created on first use)
    unsigned long long* xbuf = nullptr;  // exchange words: buf1 [2][PT][XLINE], then buf2 [2][XBCAST]
    size_t xbuf_words = 0;
    unsigned int seq_base = 0;
    unsigned long long* lane_xbuf = nullptr;  // exchange words of the lane<->codeword persistent kernels (lazy)
    size_t lane_words = 0;                    // ... of this size
    unsigned long long* rag_xbuf = nullptr;   // exchange words of the ragged codebooks' persistent kernels (lazy)
    unsigned int* abort_word = nullptr;  // device
    PResult* h_res = nullptr;            // pinned host; device memory when res_on_device
    bool res_on_device = false;          // the context of idkm_forward_noalloc: the kernel reports into device memory
    PResult res_copy;                    // ... and the host reads this copy of it
    int last_empty = 0;                  // empty clusters seen by the last forward
    // a persistent launch whose result has not been collected yet (batched calls defer the wait)
    bool defer_wait = false;
    int pending_kind = 0;  // 0 none, 1 forward, 2 backward
    unsigned int pending_id = 0;
    hipStream_t pending_stream = nullptr;
    std::vector<Deferred>* sink = nullptr;  // set by a batched call: persistent launches are handed over, not issued
    std::map<const void*, std::pair<size_t, int>> checked;  // kernel -> (largest LDS size set, blocks per CU at that size)
    std::map<const void*, bool> row_lds;                    // row <-> vector passes whose dynamic LDS limit has been set
    std::map<const void*, size_t> static_lds;               // bytes of static LDS of the kernels whose dynamic LDS is sized against it
    unsigned int spin_limit = 1u << 20;
    bool use_matrix = true;           // d = 4, 17 <= k <= 256: matrix-core kernels where they exist
    size_t tile_limit = 144 * 1024;   // largest tile of W (and dL/dWq) a persistent workgroup of the lane<->vector family keeps in LDS
#ifdef IDKM_TRACE
    long long* trace = nullptr;
#endif
    // forward state
    bool has_forward = false;
    bool has_backward = false;  // a backward has been issued since the last forward: vd, gd hold its v and g
    const float* W = nullptr;
    int64_t m = 0;
    int d = 0, k = 0, dist = 0;
    float tau = 0.f;
};

namespace {

idkm_status fail(idkm_ctx* ctx, idkm_status s, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return s;
}

#define HIP_TRY(ctx, expr)                                                                         \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) {                                                                    \
            (void)hipGetLastError(); /* or the next launch's check would find it again */          \
            return fail(ctx, IDKM_ERR_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
        }                                                                                          \
    } while (0)

// Distance between two 32-bit words (not of one array), in words.
unsigned long long words_between(const unsigned int* from, const unsigned int* to) {
    return (unsigned long long)(((intptr_t)reinterpret_cast<uintptr_t>(to) - (intptr_t)reinterpret_cast<uintptr_t>(from)) / 4);
}

struct Geometry {
    bool small;    // lane<->vector family
    int kpl;       // lane<->codeword family: codewords per lane
    int nwg;       // workgroups per pass
    int64_t vec_per_wg;
    // d = 4, 17 <= k <= 256: the forward loop and the squared energy's (dF/dC)^T pass have a matrix-core form
    bool matrix = false;
    int nwg_m = 0;
    int64_t vec_per_wg_m = 0;
    int kb = 0;  // > 0: the row <-> vector passes (d in {1, 2, 8}, k <= 256), 16 kb codewords
    int64_t wg_most = 0;  // ... their largest grid
    bool several = false; // ... and whether it is smaller than the number of tiles
};

bool pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }

// Which kernel family serves (k, d), and how a pass is cut into workgroups.
idkm_status plan(idkm_ctx* ctx, int64_t m, int k, int d, Geometry* g) {
    if (k > MAX_K || d > MAX_D || (int64_t)k * d > MAX_KD)
        return fail(ctx, IDKM_ERR_UNSUPPORTED, "shape exceeds idkm_limits (k<=1024, d<=8, k*d<=4096)");
    if (!(d == 1 || d == 2 || d == 4 || d == 8)) return fail(ctx, IDKM_ERR_UNSUPPORTED, "d must be 1, 2, 4 or 8");
    g->small = (k >= 2 && k <= 16 && pow2(k) && d <= 4);
    if (g->small) {
        int64_t vpt = (m + (int64_t)WG * 1024 - 1) / ((int64_t)WG * 1024);
        if (vpt < 1) vpt = 1;
        if (vpt > 32) vpt = 32;
        g->vec_per_wg = (int64_t)WG * vpt;
        g->kpl = 0;
    } else {
        int kpl = (k + 63) / 64, p = 1;
        while (p < kpl) p <<= 1;
        g->kpl = p;
        if (p * (d + 1) > 80) return fail(ctx, IDKM_ERR_UNSUPPORTED, "ceil(k/64)*(d+1) must be <= 80");
        // about 1024 workgroups for mid-sized layers, never more than 2048 (their partials are reduced afterwards)
        int64_t vpw = (m + 4095) / 4096;
        if (vpw < 1) vpw = 1;
        if (vpw > 512) vpw = (m + 8191) / 8192 > 512 ? (m + 8191) / 8192 : 512;
        g->vec_per_wg = vpw * (WG / 64);
        if (d != 4 && k <= 256) {
            // row <-> vector passes: as many tiles for each compute unit, all of about the same size (at least a step for each
            // wavefront), and one workgroup a tile until the device is full; from there on a workgroup takes several in turn,
            // so that the partial sums to reduce, and their workspace, stay bounded (at most 1024 workgroups)
            g->kb = 1;
            while (16 * g->kb < k) g->kb <<= 1;
            const int64_t cus = ctx->num_cu > 0 ? ctx->num_cu : 1, most = row_tile_vectors(d);
            // workgroups of a repeated pass that a compute unit holds: tile, tables and the wavefronts' sums
            const int64_t lds = most * d * 4 + (int64_t)16 * g->kb * (8 * d + (RST / 64) * 4 * (d + 1));
            const int64_t resident = std::max<int64_t>(1, std::min<int64_t>(2048 / RST, (int64_t)(160 * 1024) / lds));
            int64_t tiles = (m + cus * most - 1) / (cus * most);  // of a compute unit
            if (tiles > resident) tiles = (tiles + resident - 1) / resident * resident;
            int64_t v = (m + cus * tiles - 1) / (cus * tiles);
            if (v < 64) v = 64;
            g->vec_per_wg = (v + 15) / 16 * 16;
            g->wg_most = cus * resident;
        }
    }
    int64_t nwg = (m + g->vec_per_wg - 1) / g->vec_per_wg;
    if (g->wg_most == 0 && nwg > 0x3fffffff) return fail(ctx, IDKM_ERR_UNSUPPORTED, "m too large");
    if (g->wg_most > 0 && nwg > g->wg_most) {
        nwg = g->wg_most;
        g->several = true;
    }
    g->nwg = (int)nwg;
    g->matrix = false;
    if (!g->small && d == 4 && g->kpl <= 4 && ctx->use_matrix) {
        // one workgroup of 512 threads per compute unit and round where the layer allows it; a chunk is a whole
        // number of 16-vector steps for each of the 8 wavefronts and at most 46 KB of LDS
        int64_t v = (m + ctx->num_cu - 1) / (ctx->num_cu > 0 ? ctx->num_cu : 1);
        v = (v + 127) / 128 * 128;
        if (v > 2304) v = 2304;
        const int64_t n = (m + v - 1) / v;
        if (n <= nwg) {  // the partial-sum buffer is sized for nwg workgroups
            g->matrix = true;
            g->vec_per_wg_m = v;
            g->nwg_m = (int)n;
        }
    }
    return IDKM_OK;
}

idkm_status ensure_partials(idkm_ctx* ctx, size_t need) {
    if (need <= ctx->partials_cap) return IDKM_OK;
    if (ctx->partials) {
        (void)hipDeviceSynchronize();  // earlier launches may still read the old buffer
        (void)hipFree(ctx->partials);
        ctx->partials = nullptr;
        ctx->partials_cap = 0;
    }
    if (hipMalloc(&ctx->partials, need * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, IDKM_ERR_ALLOC, "hipMalloc of the partial-sum buffer failed");
    }
    // stamped words: sequence number 0 is never used, so a cleared buffer holds no valid word
    HIP_TRY(ctx, hipMemset(ctx->partials, 0, need * sizeof(double)));
    ctx->partials_cap = need;
    return IDKM_OK;
}

Args base_args(idkm_ctx* ctx) {
    Args a;
    std::memset(&a, 0, sizeof(a));
    a.W = ctx->W;
    a.m = ctx->m;
    a.k = ctx->k;
    a.d = ctx->d;
    a.tau = ctx->tau;
    a.inv_tau = 1.0f / ctx->tau;
    a.nscale = (float)(-1.4426950408889634 / (double)ctx->tau);
    a.escale = (ctx->dist == DIST_SQL2) ? (float)std::sqrt(1.4426950408889634 / (double)ctx->tau)
                                        : (float)(1.4426950408889634 / (double)ctx->tau);
    a.ctrl = ctx->ctrl;
    a.tickets = ctx->tickets;
    a.Cd = ctx->Cd;
    a.Cf = ctx->Cf;
    a.nd = ctx->nd;
    a.Fd = ctx->Fd;
    a.Ff = ctx->Ff;
    a.gd = ctx->gd;
    a.vd = ctx->vd;
    a.ud = ctx->ud;
    a.Hs = ctx->Hs;
    a.partials = ctx->partials;
    a.kry = ctx->kry;
    a.stage = ctx->stage;
    a.tot = ctx->tot;
    return a;
}

idkm_status launch_pass(idkm_ctx* ctx, const Geometry& g, int pass, Args& a, hipStream_t s) {
    KernelFn fn = g.small ? small_kernel(ctx->k, ctx->d, ctx->dist, pass)
                  : g.kb  ? (ctx->dist == DIST_L2 ? row_kernel_0(g.kb, ctx->d, pass, g.several) : row_kernel_1(g.kb, ctx->d, pass, g.several))
                          : lane_kernel(g.kpl, ctx->d, ctx->dist, pass);
    KernelFn fn_m = g.matrix ? mfma_lane_kernel(g.kpl, ctx->dist, pass) : nullptr;
    if (!fn && !fn_m) return fail(ctx, IDKM_ERR_UNSUPPORTED, "no kernel for this (k, d)");
    const int nwg = fn_m ? g.nwg_m : g.nwg;
    a.vec_per_wg = fn_m ? g.vec_per_wg_m : g.vec_per_wg;
    if (++ctx->stream_launches > 0x7fff0000u) {
        // the sequence numbers that stamp the partial sums would wrap: start over from a cleared buffer
        hipLaunchKernelGGL(k_fill_u64, dim3(256), dim3(256), 0, s, reinterpret_cast<unsigned long long*>(ctx->partials),
                           ctx->partials_cap, 0ull);
        hipLaunchKernelGGL(k_reset_launch_seq, dim3(1), dim3(1), 0, s, ctx->ctrl);
        HIP_TRY(ctx, hipGetLastError());
        ctx->stream_launches = 1;
    }
    if (fn_m)
        hipLaunchKernelGGL(fn_m, dim3(nwg), dim3(mfma_lane_threads(g.kpl, ctx->dist, pass)), (size_t)(a.vec_per_wg + 16) * 20, s, a);
    else if (g.kb) {
        const int tensors = pass == PASS_B1 || pass == PASS_B3 ? 2 : 1;
        const size_t lds = (size_t)a.vec_per_wg * ctx->d * sizeof(float) * tensors;
        bool& set = ctx->row_lds[(const void*)fn];
        if (!set) {  // (the limit is the kernel's, not the context's: always the most that any call needs)
            HIP_TRY(ctx, hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)(row_tile_vectors(ctx->d) * ctx->d * sizeof(float) * tensors)));
            set = true;
        }
        hipLaunchKernelGGL(fn, dim3(nwg), dim3(RST), lds, s, a);
    } else
        hipLaunchKernelGGL(fn, dim3(nwg), dim3(WG), 0, s, a);
    HIP_TRY(ctx, hipGetLastError());
    if (!g.small && pass != PASS_B3) {
        // this family carries k (d+1) sums per workgroup: a many-workgroup reduction, then a one-workgroup tail
        const int nacc = ctx->k * ((pass == PASS_FWD || pass == PASS_FIN) ? ctx->d + 1 : ctx->d);
        launch_reduce_rows(a, nacc, nwg, pass, s);
        HIP_TRY(ctx, hipGetLastError());
        hipLaunchKernelGGL(lane_tail_kernel(pass), dim3(1), dim3(ctx->k * ctx->d >= 512 ? 1024 : WG), 0, s, a);
        HIP_TRY(ctx, hipGetLastError());
    }
    return IDKM_OK;
}

constexpr size_t XBUF1_WORDS = (size_t)2 * PT * XLINE;
constexpr size_t XBUF3_WORDS = (size_t)2 * DIES * XLINE;  // two-level exchange: totals of the dies
constexpr size_t XBUF_WORDS = XBUF1_WORDS + (size_t)2 * XBCAST + XBUF3_WORDS + DIES;
// Lines of the ragged codebooks, whose sums take two words (see SumWords).  A buffer of their own: with xbuf three times as
// large it came to lie elsewhere, and the solves that do not use the rest took 1 to 3 % longer (same code, same bits).
constexpr size_t RAG_WORDS = 2 * (XBUF1_WORDS + XBUF3_WORDS);
constexpr size_t LDS_TILE_MAX = 144 * 1024;  // bytes of LDS a persistent workgroup may use for its tile

struct PersistPlan {
    PersistFn fn;
    PersistBatchFn fn_batch;
    int grid, per, threads;
    bool lane;  // lane<->codeword family: own exchange buffers
    size_t lds;
    bool small_team = false;  // a team of eight for a layer that one workgroup could hold
};
// A persistent solve that a batched call will launch together with others.
struct Deferred {
    idkm_ctx* ctx;
    PersistPlan pp;
    Args a;
    PArgs pa;
};
constexpr size_t LDS_PER_CU = 160 * 1024;
constexpr size_t LANE_TILE_MAX = 94 * 1024;                       // the lane kernels keep ~55 KB of static LDS
// Exchange words of the large-codebook kernels: a line per workgroup (buf1), the totals of the dies (buf3) and the grid totals,
// a copy per die (buf4), in two words a sum, and the die of every workgroup.  Most sums k (d + 1) of a pass, and words of
// a workgroup's line: d <= 4 1536 and as many; d = 8 (k <= 256) 2304 and twice that (float64 sums).
struct LaneBuf {
    size_t line, buf3;
    explicit LaneBuf(int d) : line(d == 8 ? 4608 : 1536), buf3((size_t)2 * DIES * 2 * (d == 8 ? 2304 : 1536)) {}
    size_t buf1() const { return (size_t)2 * PT * line; }
    size_t words() const { return buf1() + 2 * buf3 + PT; }
};

// Bytes of static LDS of a kernel (all of a compute unit's if the runtime does not say).
size_t static_lds_of(idkm_ctx* ctx, const void* fn) {
    size_t& fixed = ctx->static_lds[fn];
    if (fixed == 0) {
        hipFuncAttributes at;
        fixed = (hipFuncGetAttributes(&at, fn) == hipSuccess) ? at.sharedSizeBytes : LDS_PER_CU;
        (void)hipGetLastError();
    }
    return fixed;
}

// The lane<->vector family's part of plan_persistent.
bool plan_small(idkm_ctx* ctx, bool bwd, PersistPlan* pp, const void* dwq, int mode, int max_iter, bool alone) {
    const int k = ctx->k, d = ctx->d;
    const int64_t m = ctx->m;
    // A codebook whose size is not a power of two runs in the kernels for the next one, the surplus codewords' weights held
    // at zero: 512,000 scalar weights under three codewords (23 evaluations, 56 (dF/dC)^T passes) take 333 us there and
    // 3117 in the lane<->codeword kernels, which use 3 of 64 lanes and a 6-step wavefront sum per vector (28.7 us per
    // evaluation, 42 per pass).  These kernels know the two-level exchange only; without it, and where the tile does not
    // fit, the lane<->codeword kernels stay.
    const bool ragged = k >= 3 && k < 16 && !pow2(k);
    const int K = pow2_at_least(k);
    if (k < 2 || k > 16 || d > 4 || K * (d + 1) > XLINE || (ragged && !ctx->tree_exchange)) return false;
    const PersistFns fs = !ragged ? (ctx->dist == DIST_L2 ? persist_kernel_0(k, d, bwd) : persist_kernel_1(k, d, bwd))
                          : ctx->dist == DIST_L2 ? persist_kernel_ragged_0(K, d, bwd)
                                                 : persist_kernel_ragged_1(K, d, bwd);
    pp->fn = fs.one;
    pp->fn_batch = fs.batch;
    if (!pp->fn) return false;
    pp->threads = ctx->sink ? PT : bwd ? bwd_threads(K, d) : fwd_threads();
    pp->lane = false;
    const int64_t chunk = (int64_t)ctx->min_vec_per_thread * PT;
    int64_t g = (m + chunk - 1) / chunk;  // a few vectors per thread before adding workgroups
    // Up to 16 vectors for each of PT threads one workgroup alone needs no exchange through memory (2.6 to 4.8 us a pass in a team of
    // eight whatever m is), but walks through all vectors itself.  Where the lines lie (us per evaluation, one workgroup against
    // eight; m = 1024 / 1500 / 2048 / 3072 / 4096, plain norm): k = 4, d = 1 0.95 / 1.0 / 1.3 / 1.4 / 1.7 against 2.3; k = 8, d = 1 1.4 / 1.6 /
    // 1.8 / 2.3 / 2.6 against 2.6; k = 16, d = 1 2.1 / 2.4 / 2.9 / 3.7 / 4.5 against 2.9 to 3.1; k = 8, d = 2 2.0 / 2.4 / 2.9 / 3.7 / 4.6 against
    // 2.9 to 3.1 (squared energy 1.7 / 2.0 / 2.3 / 2.8 / 3.3); k = 4, d = 4 1.7 / 2.0 / 2.3 / 2.9 / 3.4 against 3.0; k = 8, d = 4 2.5 / 2.9 / 3.6 /
    // 4.8 / 5.8 against 3.2 to 3.4; k = 16, d = 2 3.3 / 4.1 / 5.0 / 6.7 / 8.5 against 3.6 to 4.0; k = 16, d = 4 4.3 / 5.4 / 6.5 / 8.6 / 11.0 against
    // 4.4 to 4.8.  Jacobian-free backward, whole launch: k = 4, d = 1 8.1 / 8.6 / 8.7 / 10.1 / 11.0 against 8.6; k = 8, d = 1 8.8 / 10.9 /
    // 10.4 / 12.6 / 14.3 against 8.6; k = 16, d = 1 11.5 / 12.9 / 15.4 / 18.9 / 22.5 against 9.6 to 10.3; k = 16, d = 4 23 / 30 / 33 / 43 / 53 against 12.6 to 15.6.
    // (The totals of one workgroup are float64, which adds 0.1 us from 16 sums on.)  Batched launches hide the exchange behind other layers
    // and keep one workgroup, as do the modes that are solved in one place, and calls whose result nobody may wait for
    // (idkm_forward_noalloc).  One workgroup waits for nobody: a team that gave up a wait is solved again by one (`alone`).
    if (m <= (int64_t)16 * PT) {
        const int64_t v = (m + PT - 1) / PT;
        const int kd = K * d;
        int from = 99;  // vectors per thread from which the team of eight is faster
        if (bwd)
            from = kd >= 16 ? 4 : (kd >= 8 && K > 2) ? 6 : kd >= 4 ? 10 : 99;
        else if (K >= 8)
            from = kd >= 64 ? 5 : kd >= 32 ? (K == 16 ? 6 : 8) : kd >= 16 ? (K == 16 ? 8 : 12) : 99;
        else if (kd >= 16)
            from = 14;
        const bool one = alone || ctx->sink || ctx->res_on_device || !ctx->tree_exchange || mode == IDKM_BWD_DENSE || mode == IDKM_BWD_GMRES;
        g = (!one && v >= from) ? DIES : 1;
        pp->small_team = g > 1;
    }
    if (g < 1) g = 1;
    // (a team of 2 to 7 workgroups would take the one-level exchange; 8 smaller workgroups take the two-level one)
    if (ctx->tree_exchange && g > 1 && g < DIES) g = DIES;
    if (g > ctx->num_cu) g = ctx->num_cu;
    if (g > PT) g = PT;  // a reducer reads one workgroup per thread
    int64_t per = (m + g - 1) / g;
    per = (per + 3) / 4 * 4;
    const size_t lds = (size_t)per * d * sizeof(float) * (bwd ? 2 : 1);
    pp->grid = (int)((m + per - 1) / per);
    pp->per = (int)per;
    pp->lds = ctx->sink ? (size_t)per * d * sizeof(float) : lds;  // (a batched backward keeps dL/dWq in memory)
    // The operator as a matrix: for the modes that solve a system, where every workgroup receives the totals and where it pays.
    const bool matrix = bwd && (mode == IDKM_BWD_IMPLICIT || mode == IDKM_BWD_GMRES) && pair_shape(K, d, ctx->dist) &&
                        pair_solve_pays(K, d, max_iter) && (pp->grid == 1 || (ctx->tree_exchange && pp->grid >= TREE_MIN_G));
    if (matrix && lds <= ctx->tile_limit) {
        // (its kernel has more static LDS than the one that runs pass by pass, up to 10 KB with many sums; where the tile, and the
        // state of a Krylov solve behind it, no longer fit beside it, the passes serve the call)
        const size_t state = mode == IDKM_BWD_GMRES ? 16 + gm_state_bytes(K * d, gm_basis_length(ctx->gmres_basis, k * d)) : 0;
        if (pp->lds + state + static_lds_of(ctx, (const void*)fs.pairs) <= LDS_PER_CU) {
            pp->fn = fs.pairs;
            pp->fn_batch = fs.pairs_batch;
        }
    }
    const bool fits = lds <= ctx->tile_limit && pp->lds + static_lds_of(ctx, (const void*)pp->fn) <= LDS_PER_CU;
    if (ragged && (!fits || (pp->grid > 1 && pp->grid < TREE_MIN_G))) return false;
    if (!fits) {
        // the layer does not fit on chip: the same solve with W (and dL/dWq) read from memory in every pass.  Not
        // inside a batched launch (such a layer fills the device on its own), and only from 16-byte aligned tensors.
        const PersistFns fg = persist_kernel_global(k, d, ctx->dist, bwd);
        const bool aligned = (reinterpret_cast<uintptr_t>(ctx->W) & 15u) == 0 &&
                             (!bwd || (dwq && (reinterpret_cast<uintptr_t>(dwq) & 15u) == 0));
        // Forward solves take it under IDKM_PATH_AUTO too: an evaluation costs one exchange instead of a launch and a last
        // workgroup that adds a thousand workgroups' sums (stream path against this, us per evaluation: 16.8 M scalar weights, plain norm k = 2
        // 23.1 / 17.2, k = 16 79 / 66, squared energy k = 4 28.6 / 18.5, k = 8 45.6 / 38.4; 60 M k = 4 77 / 55; 4 M 4-vectors k = 4 25.8 /
        // 17.7, k = 16 62 / 44).  Backwards, two passes over the layer whatever the codebook, are within 5 % of each other
        // up to k = 4 and up to 20 % slower here beyond (k = 8 and 16, 133 / 148 and 223 / 253 for a Jacobian-free call): the
        // stream path unless the caller asks for this one.
        if (!fg.one || ctx->sink || !aligned || (bwd && ctx->path != IDKM_PATH_PERSISTENT)) return false;
        pp->fn = matrix ? fg.pairs : fg.one;
        pp->fn_batch = nullptr;
        pp->threads = global_threads(k, d, bwd);
        pp->lds = 0;
    }
    return true;
}

// Can (m, k, d) run as one persistent launch with `tiles` resident tensors (1: W; 2: W and dL/dWq)?
// matrix_ok: the matrix-core kernels may serve the call (every pass of both energies has a matrix-core form).
// dwq: the backward's upstream gradient (a layer too large for LDS is streamed from memory with 16-byte loads, which
// W and dL/dWq must allow).
// mode, max_iter: the backward's (BWD_JFB where there is none).  alone: small layers in one workgroup.
bool plan_persistent(idkm_ctx* ctx, bool bwd, PersistPlan* pp, bool matrix_ok = true, const void* dwq = nullptr, int mode = IDKM_BWD_JFB,
                     int max_iter = 1, bool alone = false) {
    pp->small_team = false;
    if (!ctx->coop || ctx->num_cu < 1) return false;
    const int k = ctx->k, d = ctx->d;
    const int64_t m = ctx->m;
    if (plan_small(ctx, bwd, pp, dwq, mode, max_iter, alone)) return true;
    pp->small_team = false;
    if (!(k >= 2 && k <= 16 && pow2(k) && d <= 4)) {
        // lane<->codeword family
        int kpl = (k + 63) / 64, p = 1;
        while (p < kpl) p <<= 1;
        // d = 8: the forward solve alone, under IDKM_PATH_AUTO alone (the explicit persistent path is not offered for d > 4).
        // 20 evaluations, stream path against this one, us: k = 16 from 300 to 10,000 vectors 280-295 / 135-168, k = 64
        // 300-334 / 232-284, k = 100 and 128 at 4,097 364-368 / 340-370, at 64,000 520 / 335; beyond 128 codewords a small team's
        // workgroups wait for longer slices of the totals: k = 160 and 256 at 4,097 468-487 / 593-667, at 10,000 491-513 / 547-579,
        // at 16,000 534-567 / 535-573, at 24,000 562-599 / 534-558, at 290,000 (k = 256) 1496 / 1370.  Layers of up to 4096 vectors
        // stay on the stream path, which idkm_info has always reported for them, though up to 128 codewords they would gain.
        const bool row8 = d == 8 && k <= 256 && !bwd && m > (k <= 128 ? 4096 : 16000) && ctx->path == IDKM_PATH_AUTO;
        if (!row8 && (d > 4 || p * d > 16 || p * (d + 1) > 24)) return false;
        int64_t g = (m + 255) / 256;  // at least 16 vectors per wavefront before adding workgroups
        if (g < 1) g = 1;
        if (g > 1 && g < DIES) g = DIES;  // (one workgroup per die: they all add in parallel)
        if (g > ctx->num_cu) g = ctx->num_cu;
        if (g > PT) g = PT;
        int64_t per = (m + g - 1) / g;
        per = (per + 3) / 4 * 4;
        // d <= 2 and k <= 256: the row <-> vector kernels (589,824 scalar weights under 64 codewords, 30 evaluations and a
        // Jacobian-free backward: 550 us against 1260 in the lane <-> codeword form they replaced, 671 when that was all that
        // had changed); beyond 256 codewords their tables do not fit the registers
        const bool row = row8 || (d <= 2 && k <= 256);
        PersistFns fl;
        if (row) {
            int kb = 1;
            while (16 * kb < k) kb <<= 1;
            fl = ctx->dist == DIST_L2 ? persist_row_kernel_0(kb, d, bwd) : persist_row_kernel_1(kb, d, bwd);
        } else {
            fl = persist_lane_kernel(p, d, ctx->dist, bwd, matrix_ok && ctx->use_matrix);
        }
        size_t lds = (size_t)per * d * sizeof(float) * (bwd ? 2 : 1);
        if (fl.matrix) {
            // tile padded by 16 vectors, then one float per vector (dL/dWq is not kept); these kernels hold more
            // static LDS than the vector-ALU ones.  A tile too large for what is left goes to the vector-ALU kernel.
            const size_t lds_m = (size_t)(per + 16) * (d + 1) * sizeof(float);
            if (static_lds_of(ctx, (const void*)fl.one) + lds_m <= LDS_PER_CU) {
                pp->fn = fl.one;
                pp->fn_batch = fl.batch;
                pp->grid = (int)((m + per - 1) / per);
                pp->per = (int)per;
                pp->lds = lds_m;
                pp->threads = fl.threads;
                pp->lane = true;
                return true;
            }
            fl = persist_lane_kernel(p, d, ctx->dist, bwd, false);
        }
        pp->fn = fl.one;
        pp->fn_batch = fl.batch;
        if (!pp->fn) return false;
        size_t most = LANE_TILE_MAX;
        if (row8) {
            most = std::min(most, LDS_PER_CU - std::min(static_lds_of(ctx, (const void*)pp->fn), LDS_PER_CU));
        }
        if (lds > most) return false;
        pp->grid = (int)((m + per - 1) / per);
        pp->per = (int)per;
        pp->lds = lds;
        pp->threads = row ? fl.threads : LT;
        pp->lane = true;
        return true;
    }
    return false;
}

// Teams that calls of this process have on a device.  The workgroups of a team wait for one another, so all of them have to be resident:
// what one launch asks for is checked against the device where it is planned, what several streams ask for together is added up
// here.  Two teams that got half of their workgroups each would wait until the waits expire, 0.2 s, and be solved again on the stream path
// (threads with a stream and a context each, 300 steps of solve and Jacobian-free gradient, s: 300,000 weights, k = 16, three threads 37, with this
// list 0.13; 2.4 M, k = 4, three 0.50 / 0.105; 16.8 M, k = 4, three, 100 steps 0.75 / 0.15).  A call leaves the list before it returns: it is never
// longer than there are calls in progress, and a stream in it belongs to one of them.  Not in it: idkm_forward_noalloc, whose launches
// may be recorded into a graph, and teams of one, which wait for nobody.
struct Team {
    const void* owner;
    hipStream_t stream;
    double share;  // of the device
    bool last;     // starts when all that stand before it in the list are over
};
struct DeviceTeams {
    std::mutex mutex;
    std::vector<Team> running;
};
constexpr int TEAM_DEVICES = 64;
DeviceTeams g_teams[TEAM_DEVICES];

DeviceTeams* teams_of(int device) { return device >= 0 && device < TEAM_DEVICES ? &g_teams[device] : nullptr; }

// Share of a device that holds `capacity` workgroups of a kernel, the same number on each die (workgroup b goes to die b mod DIES).
double device_share(int64_t grid, int64_t capacity) { return (double)((grid + DIES - 1) / DIES * DIES) / (double)std::max<int64_t>(capacity, 1); }

// With the list locked, adds what is about to be enqueued on s to it.  Where there is no room beside the teams of other calls, waits for
// some of them to return for about the time of a solve, and otherwise puts s behind them with events, so that no call depends on
// another's thread (events alone: 0.18 instead of 0.13 s and 0.15 instead of 0.105 in the first two examples above).  A failure leaves the order to
// chance, as with other processes on the device: the waits in the kernels are bounded.
constexpr auto JOIN_WAIT = std::chrono::microseconds(300);
void join_running(DeviceTeams& t, std::unique_lock<std::mutex>& lock, const void* owner, double share, hipStream_t s, hipEvent_t* ev) {
    auto room = [&] {
        double load = share;
        for (const Team& r : t.running) load += r.share;
        return load <= 1.0 + 1e-9;
    };
    bool full = !room();
    if (full) {
        const auto until = std::chrono::steady_clock::now() + JOIN_WAIT;
        while (full && std::chrono::steady_clock::now() < until) {
            lock.unlock();
            std::this_thread::yield();
            lock.lock();
            full = !room();
        }
    }
    if (full) {
        size_t from = 0;  // the first whose end is not implied by a later one's
        for (size_t i = 0; i < t.running.size(); ++i)
            if (t.running[i].last) from = i;
        if (!*ev && hipEventCreateWithFlags(ev, hipEventDisableTiming) != hipSuccess) *ev = nullptr;
        for (size_t i = from; *ev && i < t.running.size(); ++i)
            if (t.running[i].stream != s && hipEventRecord(*ev, t.running[i].stream) == hipSuccess) (void)hipStreamWaitEvent(s, *ev, 0);
        (void)hipGetLastError();
    }
    t.running.push_back({owner, s, share, full});
}

void leave_device(int device, const void* owner) {
    DeviceTeams* t = teams_of(device);
    if (!t) return;
    std::lock_guard<std::mutex> lock(t->mutex);
    t->running.erase(std::remove_if(t->running.begin(), t->running.end(), [&](const Team& r) { return r.owner == owner; }), t->running.end());
}

idkm_status enqueue_persistent(idkm_ctx* ctx, const PersistPlan& pp, Args& a, PArgs& pa, hipStream_t s) {
    if (ctx->timing) HIP_TRY(ctx, hipEventRecord(ctx->ev0, s));
    if (ctx->coop_launch) {
        void* args[] = {(void*)&a, (void*)&pa};
        HIP_TRY(ctx, hipLaunchCooperativeKernel((const void*)pp.fn, dim3(pp.grid), dim3(pp.threads), args, pp.lds, s));
    } else {
        // plain launch: the grid fits the device, every wait in the kernel is bounded
        hipLaunchKernelGGL(pp.fn, dim3(pp.grid), dim3(pp.threads), pp.lds, s, a, pa);
        HIP_TRY(ctx, hipGetLastError());
    }
    if (ctx->timing) {
        HIP_TRY(ctx, hipEventRecord(ctx->ev1, s));
        ctx->timed = true;
    }
    return IDKM_OK;
}

idkm_status launch_persistent(idkm_ctx* ctx, const PersistPlan& pp, Args& a, PArgs pa, unsigned int exchanges,
                              hipStream_t s) {
    if (pp.grid > PT || ctx->xbuf_words < XBUF_WORDS) return fail(ctx, IDKM_ERR_DEVICE, "exchange buffer too small");
    if (ctx->seq_base > 0xffffffffu - exchanges - 2u) {  // stamps would wrap: start over from clean buffers
        hipLaunchKernelGGL(k_fill_u64, dim3(64), dim3(256), 0, s, ctx->xbuf, ctx->xbuf_words, 0ull);
        HIP_TRY(ctx, hipGetLastError());
        if (ctx->lane_xbuf) {
            hipLaunchKernelGGL(k_fill_u64, dim3(256), dim3(256), 0, s, ctx->lane_xbuf, ctx->lane_words, 0ull);
            HIP_TRY(ctx, hipGetLastError());
        }
        if (ctx->rag_xbuf) {
            hipLaunchKernelGGL(k_fill_u64, dim3(64), dim3(256), 0, s, ctx->rag_xbuf, RAG_WORDS, 0ull);
            HIP_TRY(ctx, hipGetLastError());
        }
        ctx->seq_base = 0;
    }
    if (pp.lane) {
        const LaneBuf lb(ctx->d);
        if (ctx->lane_words < lb.words()) {
            if (ctx->lane_xbuf) (void)hipFree(ctx->lane_xbuf);  // (waits for what still runs)
            ctx->lane_xbuf = nullptr;
            ctx->lane_words = 0;
            if (hipMalloc(&ctx->lane_xbuf, lb.words() * sizeof(unsigned long long)) != hipSuccess) {
                (void)hipGetLastError();
                return fail(ctx, IDKM_ERR_ALLOC, "hipMalloc of the exchange buffer failed");
            }
            ctx->lane_words = lb.words();
            hipLaunchKernelGGL(k_fill_u64, dim3(256), dim3(256), 0, s, ctx->lane_xbuf, ctx->lane_words, 0ull);
            HIP_TRY(ctx, hipGetLastError());
        }
        pa.buf1 = ctx->lane_xbuf;
        pa.buf3 = ctx->lane_xbuf + lb.buf1();
        pa.buf4 = pa.buf3 + lb.buf3;
        pa.tab = pa.buf4 + lb.buf3;
        pa.tree = (ctx->tree_exchange && !ctx->tree_remote) ? 1 : 2;  // 2: every store of hop 1 at device scope
    } else {
        pa.buf1 = ctx->xbuf;
        pa.buf2 = ctx->xbuf + XBUF1_WORDS;
        pa.buf3 = pa.buf2 + (size_t)2 * XBCAST;
        pa.tab = pa.buf3 + XBUF3_WORDS;
        if (!pow2(ctx->k)) {
            if (!ctx->rag_xbuf) {
                if (hipMalloc(&ctx->rag_xbuf, RAG_WORDS * sizeof(unsigned long long)) != hipSuccess) {
                    (void)hipGetLastError();
                    return fail(ctx, IDKM_ERR_ALLOC, "hipMalloc of the exchange buffer failed");
                }
                hipLaunchKernelGGL(k_fill_u64, dim3(64), dim3(256), 0, s, ctx->rag_xbuf, RAG_WORDS, 0ull);
                HIP_TRY(ctx, hipGetLastError());
            }
            pa.buf1 = ctx->rag_xbuf;
            pa.buf3 = pa.buf1 + 2 * XBUF1_WORDS;
        }
        // teams of DIES workgroups or more: hop 1 stays inside each die (the explicit-Jacobian mode keeps the plain
        // exchange, its one reduction ends in workgroup 0).  Also inside a batched launch: a team's workgroups are
        // consecutive in the grid, so its first DIES lie on DIES different dies and member i shares its die with member
        // i mod DIES wherever the team starts (checked by every workgroup at the start of the launch, as always)
        pa.tree = (ctx->tree_exchange && pp.grid >= TREE_MIN_G && pa.mode != BWD_DENSE) ? (ctx->tree_remote ? 2 : 1) : 0;
    }
    pa.seq_base = ctx->seq_base;
    pa.spin_limit = ctx->spin_limit;
    pa.per = pp.per;
    pa.abort_word = ctx->abort_word;
    pa.out = ctx->h_res;
    if (ctx->res_on_device) {
        static_assert(sizeof(PResult) % sizeof(unsigned long long) == 0, "PResult is cleared in 64-bit words");
        hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, s, reinterpret_cast<unsigned long long*>(ctx->h_res),
                           sizeof(PResult) / sizeof(unsigned long long), 0ull);
        HIP_TRY(ctx, hipGetLastError());
    } else {
        std::memset(ctx->h_res, 0, sizeof(PResult));
    }
#ifdef IDKM_TRACE
    pa.trace = ctx->trace;
#endif
    if (ctx->sink) {
        // part of a batched call: the batch launches this solve together with others of its shape
        ctx->sink->push_back(Deferred{ctx, pp, a, pa});
        ctx->pending_id = ctx->seq_base + 1u;
        ctx->pending_stream = s;
        ctx->seq_base += exchanges;
        return IDKM_OK;
    }
    // attribute and occupancy are queried once per (kernel, LDS size); later launches reuse the answer
    auto& checked = ctx->checked[(const void*)pp.fn];
    if (checked.second == 0 || checked.first < pp.lds) {
        HIP_TRY(ctx, hipFuncSetAttribute((const void*)pp.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pp.lds));
        int nb = 0;
        HIP_TRY(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)pp.fn, pp.threads, pp.lds));
        if (nb < 1) return fail(ctx, IDKM_ERR_DEVICE, "persistent workgroup does not fit a compute unit");
        checked.first = pp.lds;
        checked.second = nb;
    }
    if ((int64_t)checked.second * ctx->num_cu < pp.grid)
        return fail(ctx, IDKM_ERR_DEVICE, "persistent grid would not be co-resident");
    // (one workgroup waits for nobody)
    DeviceTeams* teams = pp.grid > 1 && !ctx->res_on_device ? teams_of(ctx->device) : nullptr;
    std::unique_lock<std::mutex> lock;
    if (teams) {
        const double share = device_share(pp.grid, (int64_t)checked.second * ctx->num_cu);
        lock = std::unique_lock<std::mutex>(teams->mutex);
        join_running(*teams, lock, ctx, share, s, &ctx->ev_order);
    }
    const idkm_status st = enqueue_persistent(ctx, pp, a, pa, s);
    if (st != IDKM_OK) {
        if (teams) teams->running.pop_back();
        return st;
    }
    ctx->pending_id = ctx->seq_base + 1u;
    ctx->pending_stream = s;
    ctx->seq_base += exchanges;
    return IDKM_OK;
}

// Waits for the persistent launch recorded in ctx->pending_* and turns what the kernel reported (pinned host
// memory: one wait, no copy) into a status and an idkm_info.
idkm_status finish_persistent(idkm_ctx* ctx, idkm_info* info) {
    const int kind = ctx->pending_kind;
    if (!kind) return IDKM_OK;
    ctx->pending_kind = 0;
    if (ctx->res_on_device)
        HIP_TRY(ctx, hipMemcpyAsync(&ctx->res_copy, ctx->h_res, sizeof(PResult), hipMemcpyDeviceToHost, ctx->pending_stream));
    const hipError_t waited = hipStreamSynchronize(ctx->pending_stream);
    leave_device(ctx->device, ctx);
    HIP_TRY(ctx, waited);
    const PResult& c = ctx->res_on_device ? ctx->res_copy : *ctx->h_res;
    if (c.done != ctx->pending_id || c.aborted == ctx->pending_id) return fail(ctx, IDKM_ERR_DEVICE, "a grid-wide wait hit its limit");
    if (kind == 1) {
        for (int r = 0; r < c.nred && r < 16; ++r)
            if (c.fin[r] != ctx->pending_id) return fail(ctx, IDKM_ERR_DEVICE, "a grid-wide wait hit its limit");
        int empty = 0, bad = c.nonfinite;
        for (int r = 0; r < 16; ++r) {
            empty += c.empty[r];
            bad |= c.bad[r];
        }
        if (bad) return fail(ctx, IDKM_ERR_NONFINITE, "the codebook became non-finite");
        ctx->has_forward = true;
        ctx->last_empty = empty;
        if (info) {
            info->iters = c.iters;
            info->converged = c.converged;
            info->residual = c.residual;
            info->empty_clusters = empty;
            info->path = IDKM_PATH_PERSISTENT;
            info->alpha = 0.0;
        }
    } else {
        if (c.nonfinite) return fail(ctx, IDKM_ERR_NONFINITE, "the cotangent became non-finite");
        if (info) {
            info->iters = c.iters;
            info->converged = c.converged;
            info->residual = c.residual;
            info->empty_clusters = ctx->last_empty;
            info->path = IDKM_PATH_PERSISTENT;
            info->alpha = c.alpha;
        }
    }
    return IDKM_OK;
}

idkm_status read_ctrl(idkm_ctx* ctx, hipStream_t s) {
    HIP_TRY(ctx, hipMemcpyAsync(ctx->h_ctrl, ctx->ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, s));
    HIP_TRY(ctx, hipStreamSynchronize(s));
    if (ctx->h_ctrl->abort_flag) return fail(ctx, IDKM_ERR_DEVICE, "partial sums of a pass did not arrive");
    return IDKM_OK;
}

idkm_status finish_persistent(idkm_ctx* ctx, idkm_info* info);

idkm_status check_common(idkm_ctx* ctx) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    ctx->err.clear();
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    if (ctx->pending_kind) (void)finish_persistent(ctx, nullptr);  // never leave an earlier launch uncollected
    ctx->err.clear();
    return IDKM_OK;
}

idkm_status validate_problem(idkm_ctx* ctx, const float* W, int64_t m, int d, const float* C, int k, float tau) {
    if (!W || !C) return fail(ctx, IDKM_ERR_INVALID_ARG, "W and the codebook must be non-NULL");
    if (m < 1 || d < 1 || k < 1) return fail(ctx, IDKM_ERR_INVALID_ARG, "m, d, k must be >= 1");
    if ((int64_t)k > m) return fail(ctx, IDKM_ERR_INVALID_ARG, "k must be <= m");
    if (!(tau > 0.f) || !std::isfinite(tau)) return fail(ctx, IDKM_ERR_INVALID_ARG, "tau must be finite and > 0");
    return IDKM_OK;
}

// Most vectors a thread of PASS_BP adds up in float32, as in the pass that forms the explicit Jacobian (runs of 32 give the same errors of v and g at
// 16.8 and 60 M weights, k = 2, 4, 8; twice the workgroups whose sums the last one adds cost 3 us at k = 4 and 23 at k = 8).
constexpr int64_t PAIR_RUN = 64;

// Runs `pass` repeatedly in growing chunks until the device-side flag says the solve is over.
template <class DoneFn>
idkm_status run_until_done(idkm_ctx* ctx, const Geometry& g, int pass, Args& a, hipStream_t s, int64_t budget,
                           DoneFn done) {
    int chunk = 8;
    int64_t launched = 0;
    while (launched < budget) {
        int n = (int)((budget - launched < chunk) ? (budget - launched) : chunk);
        for (int t = 0; t < n; ++t) {
            idkm_status st = launch_pass(ctx, g, pass, a, s);
            if (st != IDKM_OK) return st;
        }
        launched += n;
        idkm_status st = read_ctrl(ctx, s);
        if (st != IDKM_OK) return st;
        if (done(*ctx->h_ctrl)) break;
        if (chunk < 64) chunk *= 2;
    }
    return IDKM_OK;
}

}  // namespace

extern "C" {

int32_t idkm_version(void) { return 200; }

void idkm_limits(idkm_limits_t* out) {
    if (!out) return;
    out->max_k = MAX_K;
    out->max_d = MAX_D;
    out->max_kd = MAX_KD;
}

const char* idkm_status_string(idkm_status s) {
    switch (s) {
        case IDKM_OK: return "ok";
        case IDKM_ERR_INVALID_ARG: return "invalid argument";
        case IDKM_ERR_ALLOC: return "allocation failed";
        case IDKM_ERR_DEVICE: return "device error";
        case IDKM_ERR_NONFINITE: return "non-finite result";
        case IDKM_ERR_NO_FORWARD: return "no forward state";
        case IDKM_ERR_UNSUPPORTED: return "unsupported shape";
    }
    return "unknown";
}

idkm_status idkm_create(idkm_ctx** out, int device_id) {
    if (!out) return IDKM_ERR_INVALID_ARG;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return IDKM_ERR_DEVICE;
    if (device_id < 0 || device_id >= ndev) return IDKM_ERR_INVALID_ARG;
    if (hipSetDevice(device_id) != hipSuccess) return IDKM_ERR_DEVICE;
    idkm_ctx* c = new (std::nothrow) idkm_ctx();
    if (!c) return IDKM_ERR_ALLOC;
    c->device = device_id;
    bool ok = true;
    ok &= hipMalloc(&c->ctrl, sizeof(Ctrl)) == hipSuccess;
    if (ok) ok &= hipMemset(c->ctrl, 0, sizeof(Ctrl)) == hipSuccess;
    ok &= hipHostMalloc(&c->h_ctrl, sizeof(Ctrl)) == hipSuccess;
    ok &= hipMalloc(&c->Cd, MAX_KD * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->Fd, MAX_KD * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->gd, MAX_KD * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->vd, MAX_KD * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->ud, MAX_KD * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->nd, MAX_K * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->Cf, MAX_KD * sizeof(float)) == hipSuccess;
    ok &= hipMalloc(&c->Ff, MAX_KD * sizeof(float)) == hipSuccess;
    ok &= hipMalloc(&c->Hs, MAX_KD * sizeof(float)) == hipSuccess;
    ok &= hipMalloc(&c->stage, (MAX_NACC + 2 * WG) * sizeof(double)) == hipSuccess;
    ok &= hipMalloc(&c->tot, MAX_NACC * sizeof(double)) == hipSuccess;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device_id) == hipSuccess) {
        c->num_cu = prop.multiProcessorCount;
        c->coop = prop.cooperativeLaunch != 0;
    }
    if (const char* e = std::getenv("IDKM_COOPERATIVE")) c->coop_launch = (e[0] == '1');
    if (const char* e = std::getenv("IDKM_TREE")) {
        c->tree_exchange = (e[0] != '0');
        c->tree_remote = (e[0] == '2');
    }
    if (const char* e = std::getenv("IDKM_MIN_VPT")) {
        int v = std::atoi(e);
        if (v >= 1 && v <= 1024) c->min_vec_per_thread = v;
    }
    ok &= hipMalloc(&c->tickets, TICKET_WORDS * sizeof(unsigned int)) == hipSuccess;
    if (ok) ok &= hipMemset(c->tickets, 0, TICKET_WORDS * sizeof(unsigned int)) == hipSuccess;
    ok &= hipMalloc(&c->abort_word, 2 * sizeof(unsigned long long)) == hipSuccess;
    ok &= hipHostMalloc(&c->h_res, sizeof(PResult)) == hipSuccess;
    if (ok) {
        std::memset(c->h_res, 0, sizeof(PResult));
        void* res = nullptr;  // as the kernels see it
        ok &= hipHostGetDevicePointer(&res, c->h_res, 0) == hipSuccess;
        if (ok) {
            const unsigned long long words[2] = {0ull, words_between(c->abort_word, &static_cast<PResult*>(res)->aborted)};
            ok &= hipMemcpy(c->abort_word, words, sizeof(words), hipMemcpyHostToDevice) == hipSuccess;
        }
    }
    c->xbuf_words = XBUF_WORDS;
    ok &= hipMalloc(&c->xbuf, c->xbuf_words * sizeof(unsigned long long)) == hipSuccess;
    if (ok) ok &= hipMemset(c->xbuf, 0, c->xbuf_words * sizeof(unsigned long long)) == hipSuccess;
    if (ok) ok &= hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        idkm_destroy(c);
        return IDKM_ERR_ALLOC;
    }
    *out = c;
    return IDKM_OK;
}

idkm_status idkm_destroy(idkm_ctx* c) {
    if (!c) return IDKM_ERR_INVALID_ARG;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    void* dev[] = {c->ctrl, c->Cd, c->Fd, c->gd, c->vd, c->ud, c->nd, c->Cf, c->Ff, c->Hs, c->stage, c->tot, c->partials, c->kry, c->tickets, c->xbuf, c->lane_xbuf, c->rag_xbuf, c->abort_word};
    for (void* p : dev)
        if (p) (void)hipFree(p);
    leave_device(c->device, c);
    if (c->ev_order) (void)hipEventDestroy(c->ev_order);
    if (c->ev0) (void)hipEventDestroy(c->ev0);
    if (c->ev1) (void)hipEventDestroy(c->ev1);
    if (c->h_ctrl) (void)hipHostFree(c->h_ctrl);
    if (c->h_res) (void)hipHostFree(c->h_res);
    delete c;
    return IDKM_OK;
}

const char* idkm_last_error(const idkm_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

idkm_status idkm_set_path(idkm_ctx* ctx, idkm_path path) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    if (path != IDKM_PATH_AUTO && path != IDKM_PATH_STREAM && path != IDKM_PATH_PERSISTENT)
        return fail(ctx, IDKM_ERR_INVALID_ARG, "unknown path");
    ctx->path = path;
    return IDKM_OK;
}

idkm_status idkm_set_tile_limit(idkm_ctx* ctx, int64_t bytes) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    if (bytes < 0 || (size_t)bytes > LDS_TILE_MAX) return fail(ctx, IDKM_ERR_INVALID_ARG, "tile limit must be in [0, 147456]");
    ctx->tile_limit = (size_t)bytes;
    return IDKM_OK;
}

idkm_status idkm_set_matrix_cores(idkm_ctx* ctx, int32_t enable) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    ctx->use_matrix = enable != 0;
    return IDKM_OK;
}

idkm_status idkm_set_gmres_basis(idkm_ctx* ctx, int32_t basis) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    if (basis < 1 || basis > GM_RMAX) return fail(ctx, IDKM_ERR_INVALID_ARG, "basis must be in [1, 256]");
    ctx->gmres_basis = basis;
    return IDKM_OK;
}

idkm_status idkm_advance_sequence(idkm_ctx* ctx, uint32_t n, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    // as if n more exchanges (persistent path) and n more launches (stream path) had been made
    const uint64_t sb = (uint64_t)ctx->seq_base + n;
    ctx->seq_base = sb > 0xfffffff0ull ? 0xfffffff0u : (unsigned int)sb;
    const uint64_t sl = (uint64_t)ctx->stream_launches + n;
    const unsigned int capped = sl > 0x7ffeff00ull ? 0x7ffeff00u : (unsigned int)sl;
    hipLaunchKernelGGL(k_add_launch_seq, dim3(1), dim3(1), 0, (hipStream_t)hip_stream, ctx->ctrl, capped - ctx->stream_launches);
    HIP_TRY(ctx, hipGetLastError());
    ctx->stream_launches = capped;
    return IDKM_OK;
}

idkm_status idkm_set_kernel_timing(idkm_ctx* ctx, int32_t enable) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (enable && !ctx->ev0) {
        HIP_TRY(ctx, hipEventCreate(&ctx->ev0));
        HIP_TRY(ctx, hipEventCreate(&ctx->ev1));
    }
    ctx->timing = enable != 0;
    ctx->timed = false;
    return IDKM_OK;
}

idkm_status idkm_last_kernel_ms(idkm_ctx* ctx, float* ms_out) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (!ms_out) return fail(ctx, IDKM_ERR_INVALID_ARG, "ms_out must be non-NULL");
    if (!ctx->timing || !ctx->timed)
        return fail(ctx, IDKM_ERR_INVALID_ARG, "no timed persistent launch: enable idkm_set_kernel_timing and make a call on the persistent path first");
    HIP_TRY(ctx, hipEventSynchronize(ctx->ev1));
    HIP_TRY(ctx, hipEventElapsedTime(ms_out, ctx->ev0, ctx->ev1));
    return IDKM_OK;
}

idkm_status idkm_set_spin_limit(idkm_ctx* ctx, uint32_t polls) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    ctx->spin_limit = polls;
    return IDKM_OK;
}

idkm_status idkm_forward(idkm_ctx* ctx, const float* W, int64_t m, int32_t d, const float* C0, int32_t k, float tau,
                         float tol, int32_t max_iter, idkm_dist dist, float* C_out, float* A_out, float* Wq_out,
                         int32_t* assign_out, idkm_info* info, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    ctx->has_forward = false;
    ctx->has_backward = false;
    ctx->timed = false;
    st = validate_problem(ctx, W, m, d, C0, k, tau);
    if (st != IDKM_OK) return st;
    if (!C_out) return fail(ctx, IDKM_ERR_INVALID_ARG, "C_out must be non-NULL");
    if (!(tol >= 0.f)) return fail(ctx, IDKM_ERR_INVALID_ARG, "tol must be >= 0");
    if (max_iter < 1) return fail(ctx, IDKM_ERR_INVALID_ARG, "max_iter must be >= 1");
    if (dist != IDKM_DIST_L2 && dist != IDKM_DIST_SQL2) return fail(ctx, IDKM_ERR_INVALID_ARG, "unknown dist");
    Geometry g;
    st = plan(ctx, m, k, d, &g);
    if (st != IDKM_OK) return st;
    st = ensure_partials(ctx, (size_t)g.nwg * (size_t)k * (d + 1));
    if (st != IDKM_OK) return st;
    hipStream_t s = (hipStream_t)hip_stream;

    ctx->W = W;
    ctx->m = m;
    ctx->d = d;
    ctx->k = k;
    ctx->dist = (int)dist;
    ctx->tau = tau;
    Args a = base_args(ctx);

    PersistPlan pp;
    const bool persistent = ctx->path != IDKM_PATH_STREAM && plan_persistent(ctx, false, &pp);
    if (ctx->path == IDKM_PATH_PERSISTENT && !persistent)
        return fail(ctx, IDKM_ERR_UNSUPPORTED, "the persistent path needs k <= 512, d <= 4 and, for k > 16, the tile of W to fit in LDS");
    if (persistent) {
        a.C_out = C_out;
        a.A_out = A_out;
        a.Wq_out = Wq_out;
        a.assign_out = assign_out;
        PArgs pa;
        std::memset(&pa, 0, sizeof(pa));
        pa.C0 = C0;
        pa.tol = (double)tol;
        pa.max_iter = (int)max_iter;
        for (bool again = true; again;) {
            st = launch_persistent(ctx, pp, a, pa, (unsigned int)max_iter + 1u, s);
            if (st == IDKM_OK) {
                ctx->pending_kind = 1;
                if (ctx->defer_wait) return IDKM_OK;
                st = finish_persistent(ctx, info);
            }
            again = st == IDKM_ERR_DEVICE && pp.small_team && plan_persistent(ctx, false, &pp, true, nullptr, IDKM_BWD_JFB, 1, true);
            if (again) ctx->err.clear();
        }
        // Under IDKM_PATH_AUTO a persistent attempt that could not run to its end -- the grid was not co-resident
        // (other work occupies compute units) or a bounded wait expired -- is answered by the stream path, which
        // depends on nothing but its own launches; an explicit IDKM_PATH_PERSISTENT reports the error.
        if (st != IDKM_ERR_DEVICE || ctx->path != IDKM_PATH_AUTO) return st;
        ctx->err.clear();
        a.C_out = nullptr;
        a.A_out = nullptr;
        a.Wq_out = nullptr;
        a.assign_out = nullptr;
    }

    hipLaunchKernelGGL(k_init_forward, dim3(1), dim3(WG), 0, s, a, C0, (double)tol, (int)max_iter);
    HIP_TRY(ctx, hipGetLastError());

    st = run_until_done(ctx, g, PASS_FWD, a, s, max_iter, [](const Ctrl& c) { return c.done != 0; });
    if (st != IDKM_OK) return st;
    if (ctx->h_ctrl->nonfinite) return fail(ctx, IDKM_ERR_NONFINITE, "the codebook became non-finite");

    a.C_out = C_out;
    a.A_out = A_out;
    a.Wq_out = Wq_out;
    a.assign_out = assign_out;
    st = launch_pass(ctx, g, PASS_FIN, a, s);
    if (st != IDKM_OK) return st;
    ctx->has_forward = true;
    if (info) {
        int iters = ctx->h_ctrl->iters, conv = ctx->h_ctrl->converged;
        double res = ctx->h_ctrl->residual;
        st = read_ctrl(ctx, s);
        if (st != IDKM_OK) return st;
        info->iters = iters;
        info->converged = conv;
        info->residual = res;
        info->empty_clusters = ctx->h_ctrl->empty;
        ctx->last_empty = ctx->h_ctrl->empty;
        info->path = IDKM_PATH_STREAM;
        info->alpha = 0.0;
        if (ctx->h_ctrl->nonfinite) {
            ctx->has_forward = false;
            return fail(ctx, IDKM_ERR_NONFINITE, "non-finite masses in the evaluation at C*");
        }
    }
    return IDKM_OK;
}

idkm_status idkm_backward(idkm_ctx* ctx, const float* dWq, idkm_bwd_mode mode, float tol, int32_t max_iter,
                          float alpha, float* dW_out, idkm_info* info, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    ctx->timed = false;
    if (!ctx->has_forward) return fail(ctx, IDKM_ERR_NO_FORWARD, "idkm_backward needs a successful idkm_forward first");
    if (!dWq || !dW_out) return fail(ctx, IDKM_ERR_INVALID_ARG, "dWq and dW_out must be non-NULL");
    if (mode != IDKM_BWD_IMPLICIT && mode != IDKM_BWD_JFB && mode != IDKM_BWD_DENSE && mode != IDKM_BWD_GMRES)
        return fail(ctx, IDKM_ERR_INVALID_ARG, "unknown mode");
    if (!(tol >= 0.f)) return fail(ctx, IDKM_ERR_INVALID_ARG, "tol must be >= 0");
    if (max_iter < 1) return fail(ctx, IDKM_ERR_INVALID_ARG, "max_iter must be >= 1");
    if (!(alpha > 0.f && alpha <= 1.f)) return fail(ctx, IDKM_ERR_INVALID_ARG, "alpha must be in (0,1]");
    Geometry g;
    st = plan(ctx, ctx->m, ctx->k, ctx->d, &g);
    if (st != IDKM_OK) return st;
    st = ensure_partials(ctx, (size_t)g.nwg * (size_t)ctx->k * (ctx->d + 1));
    if (st != IDKM_OK) return st;
    hipStream_t s = (hipStream_t)hip_stream;
    if (mode == IDKM_BWD_GMRES) {
        const int kd = ctx->k * ctx->d;
        const size_t need = gm_doubles(kd < ctx->gmres_basis ? kd : ctx->gmres_basis, kd);
        if (ctx->kry_cap < need) {
            if (ctx->kry) {
                HIP_TRY(ctx, hipStreamSynchronize(s));
                (void)hipFree(ctx->kry);
                ctx->kry = nullptr;
                ctx->kry_cap = 0;
            }
            if (hipMalloc((void**)&ctx->kry, need * sizeof(double)) != hipSuccess) {
                (void)hipGetLastError();
                return fail(ctx, IDKM_ERR_ALLOC, "hipMalloc of the Krylov workspace failed");
            }
            ctx->kry_cap = need;
        }
    }
    Args a = base_args(ctx);
    a.G = dWq;
    a.dW_out = dW_out;
    ctx->has_backward = true;

    if (mode == IDKM_BWD_DENSE) {
        if (!g.small || ctx->k * ctx->d > DENSE_MAX_KD)
            return fail(ctx, IDKM_ERR_UNSUPPORTED, "the dense backward needs k in {2,4,8,16} and k*d <= 16");
        const int kd = ctx->k * ctx->d;
        // when the K D (K D + D + 1) sums fit one exchange line the persistent kernel does it in one launch
        // (and batched calls can share that launch between layers)
        PersistPlan ppd;
        if (kd * kd + kd * ctx->d + kd <= XDENSE && ctx->path != IDKM_PATH_STREAM && plan_persistent(ctx, true, &ppd, true, dWq, (int)mode)) {
            PArgs pa;
            std::memset(&pa, 0, sizeof(pa));
            pa.tol = 0.0;
            pa.max_iter = 1;
            pa.mode = (int)mode;
            pa.alpha = 1.0;
            st = launch_persistent(ctx, ppd, a, pa, 1u, s);
            if (st == IDKM_OK) {
                ctx->pending_kind = 2;
                if (ctx->defer_wait) return IDKM_OK;
                st = finish_persistent(ctx, info);
            }
            if (st != IDKM_ERR_DEVICE || ctx->path != IDKM_PATH_AUTO) return st;
            ctx->err.clear();  // as in idkm_forward: the stream path answers instead
        }
        // otherwise two launches whatever the path: (v, dF/dC*) + direct solve, then the final pass
        const size_t nacc = (size_t)kd * kd + (size_t)kd * ctx->d + kd;
        Geometry gj = g;
        int64_t vpt = (ctx->m + (int64_t)WG * 256 - 1) / ((int64_t)WG * 256);  // about one workgroup per CU
        if (vpt < 1) vpt = 1;
        if (vpt > 64) vpt = 64;
        gj.vec_per_wg = (int64_t)WG * vpt;
        gj.nwg = (int)((ctx->m + gj.vec_per_wg - 1) / gj.vec_per_wg);
        st = ensure_partials(ctx, (size_t)gj.nwg * nacc);
        if (st != IDKM_OK) return st;
        a.partials = ctx->partials;
        hipLaunchKernelGGL(k_init_backward, dim3(1), dim3(1), 0, s, a, (int)mode, 0.0, 1, 1.0, 1);
        HIP_TRY(ctx, hipGetLastError());
        st = launch_pass(ctx, gj, PASS_BJ, a, s);
        if (st != IDKM_OK) return st;
        st = launch_pass(ctx, g, PASS_B3, a, s);
        if (st != IDKM_OK) return st;
        if (info) {
            st = read_ctrl(ctx, s);
            if (st != IDKM_OK) return st;
            const Ctrl& c = *ctx->h_ctrl;
            info->iters = 0;
            info->converged = c.b_converged;
            info->residual = 0.0;
            info->empty_clusters = ctx->last_empty;
            info->path = IDKM_PATH_STREAM;
            info->alpha = 1.0;
            if (c.nonfinite) return fail(ctx, IDKM_ERR_NONFINITE, "I - dF/dC* is singular or non-finite");
        }
        return IDKM_OK;
    }

    PersistPlan pp;
    bool persistent = ctx->path != IDKM_PATH_STREAM && plan_persistent(ctx, true, &pp, true, dWq, (int)mode, (int)max_iter);
    // The minimal-residual solve keeps O(k d R) state.  Inside the persistent kernel every workgroup holds all of it
    // (in LDS, behind its tiles), which takes a team where every workgroup receives the grid totals (one workgroup, or
    // the two-level exchange of a full-device team), k d <= 64 and room for the state beside the tiles; everything
    // else runs it in the pass tail of the stream path.
    unsigned int gm_off = 0;
    if (persistent && mode == IDKM_BWD_GMRES) {
        const int kd = ctx->k * ctx->d;
        persistent = !pp.lane && kd <= 64 && (pow2(ctx->k) || ctx->path == IDKM_PATH_AUTO) &&
                     (pp.grid == 1 || (ctx->tree_exchange && !ctx->sink && pp.grid >= TREE_MIN_G));
        if (persistent) {
            gm_off = (unsigned int)((pp.lds + 15) / 16 * 16);
            // (the kernel's rows are as long as its padded codebook; the basis has one vector per unknown at most)
            const size_t lds = gm_off + gm_state_bytes(pow2_at_least(ctx->k) * ctx->d, gm_basis_length(ctx->gmres_basis, kd));
            if (static_lds_of(ctx, (const void*)pp.fn) + lds <= LDS_PER_CU)
                pp.lds = lds;
            else
                persistent = false;
        }
    }
    if (ctx->path == IDKM_PATH_PERSISTENT && !persistent)
        return fail(ctx, IDKM_ERR_UNSUPPORTED, mode == IDKM_BWD_GMRES
                        ? "IDKM_BWD_GMRES under IDKM_PATH_PERSISTENT needs k in {2,4,8,16} (under IDKM_PATH_AUTO every k in 2 .. 16 may run in one launch), k*d <= 64, a team of one or of at least 8 workgroups and room in LDS for its basis beside the tiles"
                        : "the persistent path needs k <= 512, d <= 4 and the tiles of W and dWq to fit in LDS");
    if (persistent) {
        const uint64_t ex = 1ull + (mode == IDKM_BWD_IMPLICIT ? (uint64_t)max_iter * 7ull
                                                               : (mode == IDKM_BWD_GMRES ? (uint64_t)max_iter + 3ull : 0ull));
        if (ex < 0x7fffffffull) {
            PArgs pa;
            std::memset(&pa, 0, sizeof(pa));
            pa.tol = (double)tol;
            pa.max_iter = (int)max_iter;
            pa.mode = (int)mode;
            pa.alpha = (double)alpha;
            pa.gm_basis = ctx->gmres_basis;
            pa.gm_off = gm_off;
            for (bool again = true; again;) {
                st = launch_persistent(ctx, pp, a, pa, (unsigned int)ex, s);
                if (st == IDKM_OK) {
                    ctx->pending_kind = 2;
                    if (ctx->defer_wait) return IDKM_OK;
                    st = finish_persistent(ctx, info);
                }
                again = st == IDKM_ERR_DEVICE && pp.small_team && plan_persistent(ctx, true, &pp, true, dWq, (int)mode, (int)max_iter, true);
                if (again) ctx->err.clear();
            }
            if (st != IDKM_ERR_DEVICE || ctx->path != IDKM_PATH_AUTO) return st;
            ctx->err.clear();  // as in idkm_forward: the stream path answers instead
        }
    }
    hipLaunchKernelGGL(k_init_backward, dim3(1), dim3(1), 0, s, a, (int)mode, (double)tol, (int)max_iter, (double)alpha,
                       ctx->gmres_basis);
    HIP_TRY(ctx, hipGetLastError());
    const bool pairs = mode == IDKM_BWD_IMPLICIT && g.small && pair_shape(ctx->k, ctx->d, ctx->dist) &&
                       pair_solve_pays(ctx->k, ctx->d, (int)max_iter);
    if (pairs) {
        // v and the operator in one pass, whose last workgroup runs the whole iteration (about four workgroups per compute unit:
        // it adds the sums of all of them)
        Geometry gp = g;
        gp.vec_per_wg = (int64_t)WG * std::min<int64_t>(PAIR_RUN, std::max<int64_t>(1, (ctx->m + (int64_t)WG * 1024 - 1) / ((int64_t)WG * 1024)));
        gp.nwg = (int)((ctx->m + gp.vec_per_wg - 1) / gp.vec_per_wg);
        st = ensure_partials(ctx, (size_t)gp.nwg * (size_t)pair_sums(ctx->k, ctx->d, ctx->dist));
        if (st != IDKM_OK) return st;
        a.partials = ctx->partials;
        st = launch_pass(ctx, gp, PASS_BP, a, s);
    } else {
        st = launch_pass(ctx, g, PASS_B1, a, s);
    }
    if (st != IDKM_OK) return st;
    if (mode == IDKM_BWD_IMPLICIT && !pairs) {
        // every attempt (alpha, alpha/2, ...) may use max_iter passes; at most 7 attempts
        st = run_until_done(ctx, g, PASS_B2, a, s, (int64_t)max_iter * 7, [](const Ctrl& c) { return c.b_done != 0; });
        if (st != IDKM_OK) return st;
    } else if (mode == IDKM_BWD_GMRES) {
        st = run_until_done(ctx, g, PASS_B2, a, s, (int64_t)max_iter + 2, [](const Ctrl& c) { return c.b_done != 0; });
        if (st != IDKM_OK) return st;
    }
    st = launch_pass(ctx, g, PASS_B3, a, s);
    if (st != IDKM_OK) return st;
    if (info) {
        st = read_ctrl(ctx, s);
        if (st != IDKM_OK) return st;
        const Ctrl& c = *ctx->h_ctrl;
        info->iters = c.b_iters;
        info->converged = c.b_converged;
        info->residual = c.b_residual;
        info->empty_clusters = ctx->last_empty;
        info->path = IDKM_PATH_STREAM;
        info->alpha = c.b_alpha;
        if (c.nonfinite) return fail(ctx, IDKM_ERR_NONFINITE, "the cotangent became non-finite");
    }
    return IDKM_OK;
}

idkm_status idkm_get_cotangents(idkm_ctx* ctx, double* v_out, double* g_out, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (!ctx->has_forward || !ctx->has_backward)
        return fail(ctx, IDKM_ERR_NO_FORWARD, "idkm_get_cotangents needs an idkm_backward after the last idkm_forward");
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t bytes = (size_t)ctx->k * ctx->d * sizeof(double);
    if (v_out) HIP_TRY(ctx, hipMemcpyAsync(v_out, ctx->vd, bytes, hipMemcpyDeviceToHost, s));
    if (g_out) HIP_TRY(ctx, hipMemcpyAsync(g_out, ctx->gd, bytes, hipMemcpyDeviceToHost, s));
    HIP_TRY(ctx, hipStreamSynchronize(s));
    return IDKM_OK;
}

idkm_status idkm_calibrate(idkm_ctx* ctx, int32_t kind, const float* buf, int64_t n_floats, double* result,
                           void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (!result || kind < 0 || kind > 11) return fail(ctx, IDKM_ERR_INVALID_ARG, "kind must be 0 .. 11 and result non-NULL");
    if (kind == 2 && (!buf || n_floats < 4 || (reinterpret_cast<uintptr_t>(buf) & 15u) != 0))
        return fail(ctx, IDKM_ERR_INVALID_ARG, "the streaming read needs a 16-byte aligned buffer");
    hipStream_t s = (hipStream_t)hip_stream;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_TRY(ctx, hipEventCreate(&e0));
    HIP_TRY(ctx, hipEventCreate(&e1));
    const int grid = ctx->num_cu * 8;  // eight wavefronts per SIMD
    const int iters = 4096;
    float* sink = reinterpret_cast<float*>(ctx->tot);
    double work = 0.0;
    for (int rep = 0; rep < 2; ++rep) {  // the first repetition warms up
        HIP_TRY(ctx, hipEventRecord(e0, s));
        if (kind == 0) {
            launch_cal_fma(sink, grid, iters, s);
            work = (double)grid * 256.0 * iters * 16.0;  // lane operations
        } else if (kind >= 9) {
            // the matrix / vector mix (and the matrix instruction alone) with more wavefronts per SIMD: can the vector
            // work of other wavefronts run while a matrix instruction holds the pipeline?
            const int wgs = ctx->num_cu * (kind == 10 ? 4 : 2);  // 512 threads each: 4 or 8 wavefronts per SIMD
            launch_cal_mfma(sink, wgs, iters, kind == 11 ? 0 : 1, s);
            work = (double)wgs * 8.0 * iters * 8.0 * 1024.0;  // multiply-adds
        } else if (kind >= 6) {
            // one workgroup of 512 threads per compute unit: two wavefronts per SIMD, as in the kernel that uses them
            launch_cal_mfma(sink, ctx->num_cu, iters, kind - 6, s);
            work = (double)ctx->num_cu * 8.0 * iters * 8.0 * (kind == 8 ? 256.0 : 1024.0);  // multiply-adds
        } else if (kind == 1 || kind >= 3) {
            const int fmas = kind == 1 ? 0 : (kind == 3 ? 1 : (kind == 4 ? 2 : 4));
            launch_cal_exp(sink, grid, iters, fmas, s);
            work = (double)grid * 256.0 * iters * 8.0;  // exponentials
        } else {
            launch_cal_read(buf, (size_t)n_floats, grid * 2, sink, s);
            work = (double)(n_floats / 4 * 4) * 4.0;     // bytes
        }
        HIP_TRY(ctx, hipGetLastError());
        HIP_TRY(ctx, hipEventRecord(e1, s));
        HIP_TRY(ctx, hipEventSynchronize(e1));
    }
    float ms = 0.f;
    HIP_TRY(ctx, hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *result = work / ((double)ms * 1e-3);
    return IDKM_OK;
}

int32_t idkm_code_bits(int32_t k) {
    if (k < 1) return 0;
    int b = 1;
    while ((1 << b) < k) ++b;
    return b;
}

int64_t idkm_code_words(int64_t m, int32_t k) {
    if (m < 0 || k < 1 || k > 1024) return -1;
    return (m * idkm_code_bits(k) + 31) / 32;
}

idkm_status idkm_pack_codes(idkm_ctx* ctx, const int32_t* assign, int64_t m, int32_t k, uint32_t* words_out,
                            void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (m < 0 || k < 1 || k > 1024) return fail(ctx, IDKM_ERR_INVALID_ARG, "need m >= 0 and 1 <= k <= 1024");
    if (m == 0) return IDKM_OK;
    if (!assign || !words_out) return fail(ctx, IDKM_ERR_INVALID_ARG, "assign and words_out must be non-NULL");
    if ((reinterpret_cast<uintptr_t>(assign) & 15u) != 0) return fail(ctx, IDKM_ERR_INVALID_ARG, "assign must be 16-byte aligned");
    if (m > ((int64_t)1 << 36)) return fail(ctx, IDKM_ERR_INVALID_ARG, "m too large");
    launch_pack_codes(assign, m, idkm_code_bits(k), words_out, idkm_code_words(m, k), (hipStream_t)hip_stream);
    HIP_TRY(ctx, hipGetLastError());
    return IDKM_OK;
}

idkm_status idkm_unpack_quantize(idkm_ctx* ctx, const uint32_t* words, int64_t m, const float* C, int32_t k, int32_t d,
                                 float* Wh_out, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (m < 0 || k < 1 || k > 1024 || d < 1 || d > 64) return fail(ctx, IDKM_ERR_INVALID_ARG, "need m >= 0, 1 <= k <= 1024, 1 <= d <= 64");
    if (m == 0) return IDKM_OK;
    if (!words || !C || !Wh_out) return fail(ctx, IDKM_ERR_INVALID_ARG, "words, C and Wh_out must be non-NULL");
    if (m > ((int64_t)1 << 36)) return fail(ctx, IDKM_ERR_INVALID_ARG, "m too large");
    launch_unpack_quantize(words, idkm_code_words(m, k), m, idkm_code_bits(k), C, k, d, Wh_out, (hipStream_t)hip_stream);
    HIP_TRY(ctx, hipGetLastError());
    return IDKM_OK;
}

#ifdef IDKM_TRACE
// development builds only: device buffer of 2*64*8 int64 clock stamps filled by the persistent forward kernel
idkm_status idkm_debug_trace(idkm_ctx* ctx, long long* dev_buf) {
    if (!ctx) return IDKM_ERR_INVALID_ARG;
    ctx->trace = dev_buf;
    return IDKM_OK;
}
#endif

}  // extern "C"

struct idkm_batch {
    int device = 0;
    int num_cu = 0;
    std::vector<idkm_ctx*> ctx;
    std::vector<Deferred> deferred;
    // launch tables: pinned host staging and their device copies
    BatchItem *h_items = nullptr, *d_items = nullptr;
    unsigned short *h_map = nullptr, *d_map = nullptr;
    size_t map_cap = 0;
    std::map<std::pair<const void*, size_t>, int> blocks_per_cu;  // (kernel, LDS rounded up to 1 KiB) -> occupancy
    std::map<const void*, size_t> lds_attr;                       // kernel -> dynamic LDS limit set so far
    int launches = 0;                                             // of the last batched call
    std::string err;
};

namespace {

idkm_status batch_fail(idkm_batch* b, idkm_status st, const std::string& msg) {
    b->err = msg;
    return st;
}

// Workgroups of `fn` with `lds` bytes of dynamic LDS that the device holds at once (0 on error).
int64_t batch_capacity(idkm_batch* b, const void* fn, int threads, size_t lds) {
    const size_t rounded = (lds + 1023) / 1024 * 1024;
    auto key = std::make_pair(fn, rounded);
    auto it = b->blocks_per_cu.find(key);
    if (it == b->blocks_per_cu.end()) {
        size_t& attr = b->lds_attr[fn];
        if (attr < rounded) {
            if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)rounded) != hipSuccess) {
                (void)hipGetLastError();
                return 0;
            }
            attr = rounded;
        }
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, rounded) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        it = b->blocks_per_cu.emplace(key, nb).first;
    }
    return (int64_t)it->second * b->num_cu;
}

// Launches the deferred solves: solves of one kernel shape share launches, each launch as large as the device
// can hold at once (every team's workgroups must be resident together, since they wait for one another).
idkm_status batch_launch(idkm_batch* b, hipStream_t s) {
    std::vector<Deferred>& q = b->deferred;
    b->launches = 0;
    if (q.empty()) return IDKM_OK;
    // largest tiles first: a launch reserves the LDS of its largest tile for every workgroup, so layers of a size belong together
    std::stable_sort(q.begin(), q.end(), [](const Deferred& x, const Deferred& y) { return x.pp.lds > y.pp.lds; });
    struct Part {
        PersistBatchFn fn;
        int threads;
        size_t lds;
        int64_t grid;
        size_t item, map;  // where its tables begin
        double share;      // of the device
    };
    std::vector<Part> parts;
    std::vector<char> taken(q.size(), 0);
    size_t item_off = 0, map_off = 0;
    for (size_t first = 0; first < q.size(); ++first) {
        if (taken[first]) continue;
        const void* fn = (const void*)q[first].pp.fn_batch;
        const int threads = q[first].pp.threads;
        size_t i = first;
        while (i < q.size()) {
            // one launch: members i.. of this shape while the grid stays co-resident
            const size_t item_begin = item_off, map_begin = map_off;
            size_t lds = 0;
            int64_t total = 0;
            for (; i < q.size(); ++i) {
                if (taken[i] || (const void*)q[i].pp.fn_batch != fn) continue;
                const size_t lds_new = std::max(lds, q[i].pp.lds);
                const int64_t cap = batch_capacity(b, fn, threads, lds_new);
                if (cap < q[i].pp.grid) return batch_fail(b, IDKM_ERR_DEVICE, "persistent grid would not be co-resident");
                if (total + q[i].pp.grid > cap || total + q[i].pp.grid > 65535) break;  // full: next launch
                if (map_off + (size_t)q[i].pp.grid > b->map_cap) return batch_fail(b, IDKM_ERR_DEVICE, "launch table overflow");
                BatchItem& it = b->h_items[item_off];
                it.a = q[i].a;
                it.p = q[i].pa;
                it.wg_begin = (int)total;
                it.wg_count = q[i].pp.grid;
                for (int w = 0; w < q[i].pp.grid; ++w) b->h_map[map_off + w] = (unsigned short)(item_off - item_begin);
                map_off += (size_t)q[i].pp.grid;
                item_off += 1;
                total += q[i].pp.grid;
                lds = lds_new;
                taken[i] = 1;
            }
            if (total == 0) break;
            parts.push_back({q[first].pp.fn_batch, threads, lds, total, item_begin, map_begin,
                             device_share(total, batch_capacity(b, fn, threads, lds))});
        }
    }
    // (the launches run one after the other: the largest decides what the call takes of the device)
    DeviceTeams* teams = teams_of(b->device);
    std::unique_lock<std::mutex> lock;
    if (teams) {
        double share = 0.0;
        for (const Part& p : parts) share = std::max(share, p.share);
        lock = std::unique_lock<std::mutex>(teams->mutex);
        join_running(*teams, lock, b, share, s, &b->ctx[0]->ev_order);
    }
    // the tables of all launches travel in two copies in front of the first one (a pair of copies before every launch cost the
    // 21 tensors of ResNet18 eight round trips through the copy queue a call)
    if (hipMemcpyAsync(b->d_items, b->h_items, item_off * sizeof(BatchItem), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(b->d_map, b->h_map, map_off * sizeof(unsigned short), hipMemcpyHostToDevice, s) != hipSuccess)
        return batch_fail(b, IDKM_ERR_DEVICE, "copy of the launch tables failed");
    for (const Part& p : parts) {
        hipLaunchKernelGGL(p.fn, dim3((unsigned)p.grid), dim3(p.threads), p.lds, s, (const BatchItem*)(b->d_items + p.item),
                           (const unsigned short*)(b->d_map + p.map));
        if (hipGetLastError() != hipSuccess) return batch_fail(b, IDKM_ERR_DEVICE, "batched launch failed");
        b->launches += 1;
    }
    return IDKM_OK;
}

// Collects the deferred solves after batch_launch (or abandons them if the launch failed).
idkm_status batch_collect(idkm_batch* b, idkm_status launched, int32_t n, idkm_info* infos, idkm_status* statuses, hipStream_t s) {
    idkm_status first = launched;
    // (a call that fails half way has launches and copies of its tables on their way)
    if (!b->deferred.empty()) {
        (void)hipStreamSynchronize(s);
        if (launched != IDKM_OK) (void)hipGetLastError();  // (what failed has been reported; the stream path starts without it)
    }
    leave_device(b->device, b);
    for (int i = 0; i < n; ++i) {
        idkm_ctx* c = b->ctx[i];
        if (statuses[i] == IDKM_OK && c->pending_kind) {
            if (launched == IDKM_OK) {
                statuses[i] = finish_persistent(c, &infos[i]);
            } else {
                c->pending_kind = 0;
                statuses[i] = launched;
                c->err = b->err;
            }
        }
        if (statuses[i] != IDKM_OK && first == IDKM_OK) {
            first = statuses[i];
            b->err = "layer " + std::to_string(i) + ": " + c->err;
        }
    }
    b->deferred.clear();
    return first;
}

}  // namespace

extern "C" {

idkm_status idkm_batch_create(idkm_batch** out, int device_id, int32_t n_layers) {
    if (!out) return IDKM_ERR_INVALID_ARG;
    *out = nullptr;
    if (n_layers < 1 || n_layers > 1024) return IDKM_ERR_INVALID_ARG;
    idkm_batch* b = new (std::nothrow) idkm_batch();
    if (!b) return IDKM_ERR_ALLOC;
    b->device = device_id;
    for (int i = 0; i < n_layers; ++i) {
        idkm_ctx* c = nullptr;
        idkm_status st = idkm_create(&c, device_id);
        if (st != IDKM_OK) {
            idkm_batch_destroy(b);
            return st;
        }
        b->ctx.push_back(c);
    }
    b->num_cu = b->ctx[0]->num_cu;
    b->map_cap = (size_t)n_layers * PT;  // a team has at most PT workgroups
    const bool ok = hipHostMalloc((void**)&b->h_items, (size_t)n_layers * sizeof(BatchItem), hipHostMallocDefault) == hipSuccess &&
                    hipHostMalloc((void**)&b->h_map, b->map_cap * sizeof(unsigned short), hipHostMallocDefault) == hipSuccess &&
                    hipMalloc((void**)&b->d_items, (size_t)n_layers * sizeof(BatchItem)) == hipSuccess &&
                    hipMalloc((void**)&b->d_map, b->map_cap * sizeof(unsigned short)) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        idkm_batch_destroy(b);
        return IDKM_ERR_ALLOC;
    }
    *out = b;
    return IDKM_OK;
}

idkm_status idkm_batch_destroy(idkm_batch* b) {
    if (!b) return IDKM_ERR_INVALID_ARG;
    (void)hipSetDevice(b->device);
    (void)hipDeviceSynchronize();
    for (idkm_ctx* c : b->ctx) (void)idkm_destroy(c);
    if (b->h_items) (void)hipHostFree(b->h_items);
    if (b->h_map) (void)hipHostFree(b->h_map);
    if (b->d_items) (void)hipFree(b->d_items);
    if (b->d_map) (void)hipFree(b->d_map);
    delete b;
    return IDKM_OK;
}

const char* idkm_batch_last_error(const idkm_batch* b) { return b ? b->err.c_str() : "null batch"; }

int32_t idkm_batch_launches(const idkm_batch* b) { return b ? b->launches : -1; }

idkm_ctx* idkm_batch_context(idkm_batch* b, int32_t i) {
    return (b && i >= 0 && i < (int32_t)b->ctx.size()) ? b->ctx[i] : nullptr;
}

idkm_status idkm_batch_forward(idkm_batch* b, const idkm_fwd_desc* layers, int32_t n, idkm_info* infos,
                               idkm_status* statuses, void* hip_stream) {
    if (!b || !layers || !infos || !statuses || n < 1 || n > (int32_t)b->ctx.size()) return IDKM_ERR_INVALID_ARG;
    b->err.clear();
    b->deferred.clear();
    if (hipSetDevice(b->device) != hipSuccess) return IDKM_ERR_DEVICE;
    for (int i = 0; i < n; ++i) {
        idkm_ctx* c = b->ctx[i];
        const idkm_fwd_desc& L = layers[i];
        std::memset(&infos[i], 0, sizeof(idkm_info));
        c->defer_wait = true;
        c->sink = &b->deferred;
        statuses[i] = idkm_forward(c, L.W, L.m, L.d, L.C0, L.k, L.tau, L.tol, L.max_iter, (idkm_dist)L.dist, L.C_out,
                                   L.A_out, L.Wq_out, L.assign_out, &infos[i], hip_stream);
        c->defer_wait = false;
        c->sink = nullptr;
    }
    const idkm_status launched = batch_launch(b, (hipStream_t)hip_stream);
    idkm_status first = batch_collect(b, launched, n, infos, statuses, (hipStream_t)hip_stream);
    if (first != IDKM_OK) {
        // layers whose persistent solve could not run to its end are solved again, one by one, on the stream path
        // (contexts left at IDKM_PATH_AUTO only)
        first = IDKM_OK;
        for (int i = 0; i < n; ++i) {
            idkm_ctx* c = b->ctx[i];
            const idkm_fwd_desc& L = layers[i];
            if (statuses[i] == IDKM_ERR_DEVICE && c->path == IDKM_PATH_AUTO) {
                c->path = IDKM_PATH_STREAM;
                statuses[i] = idkm_forward(c, L.W, L.m, L.d, L.C0, L.k, L.tau, L.tol, L.max_iter, (idkm_dist)L.dist, L.C_out,
                                           L.A_out, L.Wq_out, L.assign_out, &infos[i], hip_stream);
                c->path = IDKM_PATH_AUTO;
            }
            if (statuses[i] != IDKM_OK && first == IDKM_OK) {
                first = statuses[i];
                b->err = "layer " + std::to_string(i) + ": " + c->err;
            }
        }
        if (first == IDKM_OK) b->err.clear();
    }
    return first;
}

idkm_status idkm_batch_backward(idkm_batch* b, const idkm_bwd_desc* layers, int32_t n, idkm_info* infos,
                                idkm_status* statuses, void* hip_stream) {
    if (!b || !layers || !infos || !statuses || n < 1 || n > (int32_t)b->ctx.size()) return IDKM_ERR_INVALID_ARG;
    b->err.clear();
    b->deferred.clear();
    if (hipSetDevice(b->device) != hipSuccess) return IDKM_ERR_DEVICE;
    for (int i = 0; i < n; ++i) {
        idkm_ctx* c = b->ctx[i];
        const idkm_bwd_desc& L = layers[i];
        std::memset(&infos[i], 0, sizeof(idkm_info));
        c->defer_wait = true;
        c->sink = &b->deferred;
        statuses[i] = idkm_backward(c, L.dWq, (idkm_bwd_mode)L.mode, L.tol, L.max_iter, L.alpha, L.dW_out, &infos[i],
                                    hip_stream);
        c->defer_wait = false;
        c->sink = nullptr;
    }
    const idkm_status launched = batch_launch(b, (hipStream_t)hip_stream);
    idkm_status first = batch_collect(b, launched, n, infos, statuses, (hipStream_t)hip_stream);
    if (first != IDKM_OK) {
        first = IDKM_OK;  // as in idkm_batch_forward
        for (int i = 0; i < n; ++i) {
            idkm_ctx* c = b->ctx[i];
            const idkm_bwd_desc& L = layers[i];
            if (statuses[i] == IDKM_ERR_DEVICE && c->path == IDKM_PATH_AUTO) {
                c->path = IDKM_PATH_STREAM;
                statuses[i] = idkm_backward(c, L.dWq, (idkm_bwd_mode)L.mode, L.tol, L.max_iter, L.alpha, L.dW_out, &infos[i],
                                            hip_stream);
                c->path = IDKM_PATH_AUTO;
            }
            if (statuses[i] != IDKM_OK && first == IDKM_OK) {
                first = statuses[i];
                b->err = "layer " + std::to_string(i) + ": " + c->err;
            }
        }
        if (first == IDKM_OK) b->err.clear();
    }
    return first;
}

idkm_status idkm_step_F(idkm_ctx* ctx, const float* W, int64_t m, int32_t d, const float* C, int32_t k, float tau,
                        idkm_dist dist, float* Cplus_out, float* n_out, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    ctx->has_forward = false;
    ctx->has_backward = false;
    st = validate_problem(ctx, W, m, d, C, k, tau);
    if (st != IDKM_OK) return st;
    if (!Cplus_out) return fail(ctx, IDKM_ERR_INVALID_ARG, "Cplus_out must be non-NULL");
    if (dist != IDKM_DIST_L2 && dist != IDKM_DIST_SQL2) return fail(ctx, IDKM_ERR_INVALID_ARG, "unknown dist");
    Geometry g;
    st = plan(ctx, m, k, d, &g);
    if (st != IDKM_OK) return st;
    st = ensure_partials(ctx, (size_t)g.nwg * (size_t)k * (d + 1));
    if (st != IDKM_OK) return st;
    hipStream_t s = (hipStream_t)hip_stream;
    ctx->W = W;
    ctx->m = m;
    ctx->d = d;
    ctx->k = k;
    ctx->dist = (int)dist;
    ctx->tau = tau;
    Args a = base_args(ctx);
    hipLaunchKernelGGL(k_init_forward, dim3(1), dim3(WG), 0, s, a, C, 0.0, 1);
    HIP_TRY(ctx, hipGetLastError());
    st = launch_pass(ctx, g, PASS_FIN, a, s);
    if (st != IDKM_OK) return st;
    HIP_TRY(ctx, hipMemcpyAsync(Cplus_out, ctx->Ff, sizeof(float) * k * d, hipMemcpyDeviceToDevice, s));
    if (n_out) {
        hipLaunchKernelGGL(k_f64_to_f32, dim3(1), dim3(WG), 0, s, ctx->nd, n_out, (int)k);
        HIP_TRY(ctx, hipGetLastError());
    }
    ctx->has_forward = true;
    return IDKM_OK;
}

idkm_status idkm_step_JCT(idkm_ctx* ctx, const float* gvec, float* out, void* hip_stream) {
    idkm_status st = check_common(ctx);
    if (st != IDKM_OK) return st;
    if (!ctx->has_forward) return fail(ctx, IDKM_ERR_NO_FORWARD, "idkm_step_JCT needs idkm_step_F or idkm_forward first");
    if (!gvec || !out) return fail(ctx, IDKM_ERR_INVALID_ARG, "g and out must be non-NULL");
    Geometry g;
    st = plan(ctx, ctx->m, ctx->k, ctx->d, &g);
    if (st != IDKM_OK) return st;
    st = ensure_partials(ctx, (size_t)g.nwg * (size_t)ctx->k * (ctx->d + 1));
    if (st != IDKM_OK) return st;
    hipStream_t s = (hipStream_t)hip_stream;
    Args a = base_args(ctx);
    hipLaunchKernelGGL(k_set_g, dim3(1), dim3(WG), 0, s, a, gvec);
    HIP_TRY(ctx, hipGetLastError());
    st = launch_pass(ctx, g, PASS_B2, a, s);
    if (st != IDKM_OK) return st;
    hipLaunchKernelGGL(k_f64_to_f32, dim3(1), dim3(WG), 0, s, ctx->ud, out, ctx->k * ctx->d);
    HIP_TRY(ctx, hipGetLastError());
    return IDKM_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- the entry point that allocates nothing

namespace {

// Everything the persistent forward kernel needs beyond the caller's tensors: the exchange words of the grid-wide
// sums, the O(k d) solver state it leaves behind, the abort word and the block it reports into.
struct StaticScratch {
    unsigned long long xbuf[XBUF_WORDS];
    double Cd[64], Fd[64], nd[16];
    float Cf[64], Ff[64];
    unsigned int abort_word;
    unsigned int pad_;
    unsigned long long abort_away;  // way to res.aborted (see PArgs::abort_word)
    PResult res;
};
constexpr size_t STATIC_SCRATCH_BYTES = (sizeof(StaticScratch) + 255) / 256 * 256;
constexpr int STATIC_MAX_DEVICES = 64;

}  // namespace

// One copy per GPU the library runs on, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the address the kernels get is the one that call returns for the current device.
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {

struct StaticDevice {
    bool ready = false;
    idkm_ctx ctx;  // a host-side context whose device pointers all point into this device's copy of `scratch`
};
StaticDevice g_static[STATIC_MAX_DEVICES];
std::mutex g_static_mutex;
std::string g_static_err;

}  // namespace

extern "C" {

const char* idkm_noalloc_last_error(void) { return g_static_err.c_str(); }

idkm_status idkm_forward_noalloc(int device_id, const float* W, int64_t m, int32_t d, const float* C0, int32_t k,
                                 float tau, float tol, int32_t max_iter, idkm_dist dist, float* C_out, float* A_out,
                                 float* Wq_out, int32_t* assign_out, idkm_info* info, void* hip_stream) {
    std::lock_guard<std::mutex> lock(g_static_mutex);
    g_static_err.clear();
    auto bad = [&](idkm_status st, const std::string& msg) {
        g_static_err = msg;
        return st;
    };
    if (device_id < 0 || device_id >= STATIC_MAX_DEVICES) return bad(IDKM_ERR_INVALID_ARG, "device_id out of range");
    if (hipSetDevice(device_id) != hipSuccess) {
        (void)hipGetLastError();
        return bad(IDKM_ERR_DEVICE, "hipSetDevice failed");
    }
    hipStream_t s = (hipStream_t)hip_stream;
    StaticDevice& sd = g_static[device_id];
    idkm_ctx* ctx = &sd.ctx;
    if (!sd.ready) {
        // once per device, with that device current: the address of this device's copy of the array
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return bad(IDKM_ERR_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        }
        StaticScratch* sc = reinterpret_cast<StaticScratch*>(ptr);
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device_id) != hipSuccess || cus < 1) {
            (void)hipGetLastError();
            return bad(IDKM_ERR_DEVICE, "hipDeviceGetAttribute failed");
        }
        ctx->device = device_id;
        ctx->num_cu = cus;
        ctx->coop = true;  // plain launches of a grid that the occupancy query shows to be co-resident
        ctx->xbuf = sc->xbuf;
        ctx->xbuf_words = XBUF_WORDS;
        ctx->Cd = sc->Cd;
        ctx->Fd = sc->Fd;
        ctx->nd = sc->nd;
        ctx->Cf = sc->Cf;
        ctx->Ff = sc->Ff;
        ctx->abort_word = &sc->abort_word;
        ctx->h_res = &sc->res;
        ctx->res_on_device = true;
        ctx->seq_base = 0;
        // the stamps start from a cleared array (sequence number 0 is never used); a fill kernel, not a memset
        hipLaunchKernelGGL(k_fill_u64, dim3(64), dim3(256), 0, s, reinterpret_cast<unsigned long long*>(ptr),
                           STATIC_SCRATCH_BYTES / sizeof(unsigned long long), 0ull);
        hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, s, &sc->abort_away, (size_t)1,
                           words_between(&sc->abort_word, &sc->res.aborted));
        static_assert(offsetof(StaticScratch, abort_away) == offsetof(StaticScratch, abort_word) + 8, "the word behind the abort word");
        if (hipGetLastError() != hipSuccess) return bad(IDKM_ERR_DEVICE, "clearing the scratch array failed");
        sd.ready = true;
    }
    ctx->err.clear();
    ctx->pending_kind = 0;
    idkm_status st = validate_problem(ctx, W, m, d, C0, k, tau);
    if (st == IDKM_OK && !C_out) st = fail(ctx, IDKM_ERR_INVALID_ARG, "C_out must be non-NULL");
    if (st == IDKM_OK && !(tol >= 0.f)) st = fail(ctx, IDKM_ERR_INVALID_ARG, "tol must be >= 0");
    if (st == IDKM_OK && max_iter < 1) st = fail(ctx, IDKM_ERR_INVALID_ARG, "max_iter must be >= 1");
    if (st == IDKM_OK && dist != IDKM_DIST_L2 && dist != IDKM_DIST_SQL2) st = fail(ctx, IDKM_ERR_INVALID_ARG, "unknown dist");
    if (st != IDKM_OK) return bad(st, ctx->err);
    const bool shape_ok = k >= 2 && k <= 16 && pow2(k) && (d == 1 || d == 2 || d == 4);
    if (!shape_ok || m * d > IDKM_NOALLOC_MAX_WEIGHTS)
        return bad(IDKM_ERR_UNSUPPORTED, "idkm_forward_noalloc serves k in {2,4,8,16}, d in {1,2,4} and m*d <= " +
                                             std::to_string((long long)IDKM_NOALLOC_MAX_WEIGHTS) +
                                             " (the layer is held in LDS)");
    ctx->W = W;
    ctx->m = m;
    ctx->d = d;
    ctx->k = k;
    ctx->dist = (int)dist;
    ctx->tau = tau;
    ctx->path = IDKM_PATH_AUTO;
    Args a = base_args(ctx);
    a.C_out = C_out;
    a.A_out = A_out;
    a.Wq_out = Wq_out;
    a.assign_out = assign_out;
    PersistPlan pp;
    if (!plan_persistent(ctx, false, &pp) || pp.lane || pp.lds == 0 || pp.lds > LDS_TILE_MAX)
        return bad(IDKM_ERR_UNSUPPORTED, "idkm_forward_noalloc: the layer does not fit this device's LDS");
    PArgs pa;
    std::memset(&pa, 0, sizeof(pa));
    pa.C0 = C0;
    pa.tol = (double)tol;
    pa.max_iter = (int)max_iter;
    st = launch_persistent(ctx, pp, a, pa, (unsigned int)max_iter + 1u, s);
    if (st != IDKM_OK) return bad(st, ctx->err);
    if (!info) return IDKM_OK;  // enqueued; nothing waits
    ctx->pending_kind = 1;
    st = finish_persistent(ctx, info);
    if (st != IDKM_OK) return bad(st, ctx->err);
    return IDKM_OK;
}

}  // extern "C"
