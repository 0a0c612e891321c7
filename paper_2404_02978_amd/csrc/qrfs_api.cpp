// qrfs_api.cpp -- the C ABI of libqrfs: argument checks, the context and
// its device workspace, and the host-side orchestration of the kernels.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <numeric>
#include <string>

#include "qrfs.h"
#include "qrfs_internal.hpp"

namespace qrfs {
qrfs_status proposal_check_ready(const qrfs_proposal* p);
hipError_t proposal_sample(const qrfs_proposal* p, uint64_t s0x, uint64_t s0y, uint64_t index,
                           int64_t n_sets, int64_t K, double* fx, double* fy, double* area,
                           hipStream_t st);
}  // namespace qrfs

struct qrfs_context {
    int device = 0;
    void* ws = nullptr;
    size_t ws_size = 0;
    size_t ws_cap = 0;          // 0: unbounded
    int wide_path = 0;          // QRFS_TUNE_WIDE_PATH
    int64_t range_freqs = 2048;  // QRFS_TUNE_RANGE_FREQS
    size_t tile_cap = (size_t)2 << 30;  // QRFS_TUNE_TILE_BYTES
    // What eager calls alone use: partial sums of frequency ranges, and the tiles
    // of two-phase problems that do not fill the device.  In blocks of its own, so
    // that such a call never replaces the workspace, which a captured graph may
    // hold.  Every block is at least twice as long as the one before, which is kept
    // until destroy: work in flight may still use it, and to free it would wait for
    // the device.
    void* scratch = nullptr;
    size_t scratch_size = 0;
    size_t scratch_total = 0;  // with the outgrown blocks
    void* outgrown[40] = {};
    int n_outgrown = 0;
    int grid_slot = -1;  // the context's word for grid answers (-1: none), see grid_word
};

// Scratch of the allocation-free structure-function entry point: a static
// device array (each GPU the library runs on holds its own copy until the
// process ends), never allocated or freed by the library.  In host code
// `scratch` names a host-side stand-in; kernels get the device address that
// hipGetSymbolAddress returns for the current device, kept per device.
constexpr size_t kScratchBytes = (size_t)64 << 20;
// Behind it, the words in which calls note whether their points form a grid: one
// for each context, then a ring for captured calls.
constexpr unsigned kGridSlots = 512, kGridRing = 512;
static __device__ __align__(256) unsigned char
    scratch[kScratchBytes + (kGridSlots + kGridRing) * sizeof(unsigned long long)];

namespace {

constexpr int kMaxDevices = 256;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
bool g_grid_slots[kMaxDevices][kGridSlots] = {};  // taken by a context

thread_local std::string g_detail;

qrfs_status fail(qrfs_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_detail = buf;
    return s;
}

qrfs_status ok() {
    g_detail.clear();
    return QRFS_OK;
}

// Makes ctx->device current for the duration of a call.
struct DeviceGuard {
    int prev = -1;
    bool okay = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        okay = prev == dev || hipSetDevice(dev) == hipSuccess;
        if (prev == dev) prev = -1;  // nothing to restore
    }
    ~DeviceGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

qrfs_status hip_fail(hipError_t e, const char* what) {
    return fail(QRFS_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

bool aligned8(const void* p) { return ((uintptr_t)p & 7u) == 0; }

// Looks up the device address of `scratch` on `device` (which must be
// current) once per device.
hipError_t scratch_setup(int device) {
    if (device < 0 || device >= kMaxDevices) return hipSuccess;  // entry point then refuses
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

qrfs_status sf_sets_enqueue(const qrfs::SfPlan& plan, char* base, int64_t K, const double* fx,
                            const double* fy, const double* w, int64_t nB, const double* bx,
                            const double* by, int64_t R, int64_t R_block, const qrfs_rng* rng,
                            int32_t precision, double* sf, double* sf_stderr, hipStream_t stream);

void* scratch_ptr(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_ptr[device];
}

// A context's word among the device's (-1: all taken).
int take_grid_slot(int device) {
    if (device < 0 || device >= kMaxDevices) return -1;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    for (unsigned i = 0; i < kGridSlots; ++i)
        if (!g_grid_slots[device][i]) {
            g_grid_slots[device][i] = true;
            return (int)i;
        }
    return -1;
}

void give_grid_slot(int device, int slot) {
    if (slot < 0) return;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    g_grid_slots[device][slot] = false;
}

// The word and an id for one call (word NULL: it cannot ask).  Eager calls of a
// context may not overlap, so its word is theirs from the question to the last
// kernel that reads the answer.  Captured ones have none of their own: a graph may
// outlive the context, and calls of any graph, thread and stream share the ring
// (see GridWord).
qrfs::GridWord grid_word(const qrfs_context* ctx, bool captured) {
    static std::atomic<unsigned long long> next{0}, id{1};
    char* base = (char*)scratch_ptr(ctx->device);
    if (!base || (!captured && ctx->grid_slot < 0)) return {};
    const unsigned long long i =
        captured ? kGridSlots + next.fetch_add(1) % kGridRing : (unsigned long long)ctx->grid_slot;
    return {(unsigned long long*)(base + kScratchBytes) + i, id.fetch_add(1)};
}

#define CHECK_PTR(p)                                                                 \
    do {                                                                             \
        if ((p) == nullptr) return fail(QRFS_ERR_INVALID_ARG, "%s is NULL", #p);     \
        if (!aligned8(p)) return fail(QRFS_ERR_INVALID_ARG, "%s is not 8-byte aligned", #p); \
    } while (0)

// Frees the scratch blocks; nothing may be in flight.
void free_scratch(qrfs_context* ctx) {
    for (int i = 0; i < ctx->n_outgrown; ++i) (void)hipFree(ctx->outgrown[i]);
    if (ctx->scratch) (void)hipFree(ctx->scratch);
    ctx->scratch = nullptr;
    ctx->scratch_size = ctx->scratch_total = 0;
    ctx->n_outgrown = 0;
}

// Longest scratch block that the context's cap has room for.
size_t scratch_room(const qrfs_context* ctx) {
    if (!ctx->ws_cap) return SIZE_MAX;
    const size_t held = ctx->ws_size + ctx->scratch_total;
    const size_t room = held < ctx->ws_cap ? ctx->ws_cap - held : 0;
    return room > ctx->scratch_size ? room : ctx->scratch_size;
}

// Scratch of at least `bytes` for an eager call, or NULL where the cap or the
// memory has no room: the caller does without.  Waits for nothing.
char* scratch_block(qrfs_context* ctx, size_t bytes) {
    if (bytes <= ctx->scratch_size) return (char*)ctx->scratch;
    if (bytes > scratch_room(ctx) || ctx->n_outgrown == 40) return nullptr;
    size_t sz = (size_t)1 << 20;
    if (sz < 2 * ctx->scratch_size) sz = 2 * ctx->scratch_size;
    if (sz < bytes) sz = bytes;
    if (sz > scratch_room(ctx)) sz = bytes;
    // this stream is not being captured, but another may be, here or in another
    // thread: an allocation is no part of that
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, sz);
    if (e != hipSuccess && sz > bytes) e = hipMalloc(&p, sz = bytes);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (ctx->scratch) ctx->outgrown[ctx->n_outgrown++] = ctx->scratch;
    ctx->scratch = p;
    ctx->scratch_size = sz;
    ctx->scratch_total += sz;
    return (char*)p;
}

qrfs_status ensure_workspace(qrfs_context* ctx, size_t bytes) {
    if (bytes <= ctx->ws_size) return QRFS_OK;
    if (ctx->ws_cap && bytes > ctx->ws_cap)
        return fail(QRFS_ERR_OUT_OF_MEMORY, "workspace of %zu bytes exceeds the context cap of %zu",
                    bytes, ctx->ws_cap);
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize before workspace growth");
    if (ctx->ws) (void)hipFree(ctx->ws);
    ctx->ws = nullptr;
    ctx->ws_size = 0;
    size_t sz = bytes < ((size_t)1 << 20) ? ((size_t)1 << 20) : bytes;
    if (ctx->ws_cap && sz > ctx->ws_cap) sz = bytes;
    // the workspace comes first: the scratch gives way to it
    if (ctx->ws_cap && sz + ctx->scratch_total > ctx->ws_cap) free_scratch(ctx);
    e = hipMalloc(&ctx->ws, sz);
    if (e != hipSuccess && ctx->scratch) {
        (void)hipGetLastError();
        free_scratch(ctx);
        e = hipMalloc(&ctx->ws, sz);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(QRFS_ERR_OUT_OF_MEMORY, "workspace of %zu bytes: %s", sz, hipGetErrorString(e));
    }
    ctx->ws_size = sz;
    return QRFS_OK;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

qrfs_status check_psd(const qrfs_psd* psd) {
    if (!psd) return fail(QRFS_ERR_INVALID_ARG, "psd is NULL");
    if (psd->model != QRFS_PSD_KOLMOGOROV && psd->model != QRFS_PSD_VON_KARMAN)
        return fail(QRFS_ERR_INVALID_ARG, "unknown PSD model %d", psd->model);
    if (!(psd->r0 > 0.0) || !std::isfinite(psd->r0))
        return fail(QRFS_ERR_INVALID_ARG, "r0 must be > 0 (got %g)", psd->r0);
    if (psd->model == QRFS_PSD_VON_KARMAN && (!(psd->L0 > 0.0) || !std::isfinite(psd->L0)))
        return fail(QRFS_ERR_INVALID_ARG, "von Karman L0 must be > 0 (got %g)", psd->L0);
    if (!std::isfinite(psd->c)) return fail(QRFS_ERR_INVALID_ARG, "PSD constant is not finite");
    if (!(psd->wavelength >= 0.0) || !std::isfinite(psd->wavelength))
        return fail(QRFS_ERR_INVALID_ARG, "wavelength must be >= 0 (got %g)", psd->wavelength);
    return QRFS_OK;
}

qrfs_status check_ap(const qrfs_aperture* ap) {
    if (!(ap->D > 0.0) || !std::isfinite(ap->D))
        return fail(QRFS_ERR_INVALID_ARG, "aperture D must be > 0 (got %g)", ap->D);
    if (!(ap->d >= 0.0) || !(ap->d < ap->D))
        return fail(QRFS_ERR_INVALID_ARG, "obstruction d must satisfy 0 <= d < D (got %g, D=%g)",
                    ap->d, ap->D);
    return QRFS_OK;
}

qrfs_status check_sampler(const qrfs_sampler* s, int64_t K) {
    if (!s) return fail(QRFS_ERR_INVALID_ARG, "sampler is NULL");
    const int sc = s->scheme;
    if (sc == QRFS_SAMPLER_LEARNED) return qrfs::proposal_check_ready(s->proposal);
    if (sc == QRFS_SAMPLER_R2_CARTESIAN || sc == QRFS_SAMPLER_RANDOM_CARTESIAN ||
        sc == QRFS_SAMPLER_JITTER) {
        if (s->N <= 0) return fail(QRFS_ERR_INVALID_ARG, "Cartesian N must be > 0 (got %d)", s->N);
        if (!(s->df > 0.0) || !std::isfinite(s->df))
            return fail(QRFS_ERR_INVALID_ARG, "Cartesian df must be > 0 (got %g)", s->df);
        if (sc == QRFS_SAMPLER_JITTER && K != (int64_t)s->N * s->N)
            return fail(QRFS_ERR_INVALID_ARG, "jittered grid needs K = N^2 (K=%lld, N=%d)",
                        (long long)K, s->N);
    } else if (sc == QRFS_SAMPLER_R2_LOGPOLAR || sc == QRFS_SAMPLER_RANDOM_LOGPOLAR) {
        if (!(s->fmin > 0.0) || !(s->fmax > s->fmin) || !std::isfinite(s->fmax))
            return fail(QRFS_ERR_INVALID_ARG, "log-polar band needs 0 < fmin < fmax (got %g, %g)",
                        s->fmin, s->fmax);
    } else if (sc == QRFS_SAMPLER_R2_DISC || sc == QRFS_SAMPLER_RANDOM_DISC) {
        if (!(s->fmax > 0.0) || !std::isfinite(s->fmax))
            return fail(QRFS_ERR_INVALID_ARG, "disc radius fmax must be > 0 (got %g)", s->fmax);
    } else {
        return fail(QRFS_ERR_INVALID_ARG, "unknown sampler scheme %d", sc);
    }
    return QRFS_OK;
}

qrfs_status check_sum_common(int64_t K, int64_t P, int64_t R, int64_t R_block,
                             const qrfs_rng* rng, const double* coef, int32_t precision) {
    if (K <= 0) return fail(QRFS_ERR_INVALID_ARG, "K must be > 0 (got %lld)", (long long)K);
    if (P <= 0) return fail(QRFS_ERR_INVALID_ARG, "number of points must be > 0 (got %lld)", (long long)P);
    if (R <= 0) return fail(QRFS_ERR_INVALID_ARG, "R must be > 0 (got %lld)", (long long)R);
    if (R_block < 1 || R_block > R)
        return fail(QRFS_ERR_INVALID_ARG, "R_block must be in [1, R] (got %lld, R=%lld)",
                    (long long)R_block, (long long)R);
    if (K > ((int64_t)1 << 33))
        return fail(QRFS_ERR_INVALID_ARG, "K too large for the 32-bit Philox block counter");
    if (precision != QRFS_PREC_FP64 && precision != QRFS_PREC_FP32 &&
        precision != QRFS_PREC_SPLIT_BF16 && precision != QRFS_PREC_BF16X6 &&
        precision != QRFS_PREC_FP16X3)
        return fail(QRFS_ERR_INVALID_ARG, "unknown precision %d", precision);
    if (!coef) {
        if (!rng) return fail(QRFS_ERR_INVALID_ARG, "rng is NULL and no coefficients were given");
        if (rng->mode != QRFS_COEF_GAUSS_CS && rng->mode != QRFS_COEF_EQ3)
            return fail(QRFS_ERR_INVALID_ARG, "unknown coefficient mode %d", rng->mode);
    } else if (!aligned8(coef)) {
        return fail(QRFS_ERR_INVALID_ARG, "coef is not 8-byte aligned");
    }
    return QRFS_OK;
}

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// R2 sampling with any scheme: sets [0, n_sets) starting at `index`
hipError_t sample_any(const qrfs_sampler* s, uint64_t index, int64_t n_sets, int64_t K,
                      double* fx, double* fy, double* area, hipStream_t st) {
    if (s->scheme == QRFS_SAMPLER_LEARNED)
        return qrfs::proposal_sample(s->proposal, s->seed_x, s->seed_y, index, n_sets, K, fx, fy,
                                     area, st);
    return qrfs::launch_sample(s->scheme, s->seed_x, s->seed_y, index, n_sets, K, s->N, s->df,
                               s->fmin, s->fmax, fx, fy, area, st);
}

// Frequencies and weights of n_sets sets for a pipeline that needs no cell
// areas: one fused kernel for the R2, pseudo-random and jittered samplers;
// the learned sampler writes its areas to `area` and the weights follow.
// f32: weights for FP32-class sums (qrfs_weights' precision argument).
hipError_t sample_weights_any(const qrfs_sampler* s, uint64_t index, int64_t n_sets, int64_t K,
                              const qrfs_psd* psd, double c, const qrfs_aperture* ap, int f32,
                              double* fx, double* fy, double* area, double* w, hipStream_t st) {
    const int has_ap = ap ? 1 : 0;
    const double D = ap ? ap->D : 0.0, d = ap ? ap->d : 0.0;
    if (s->scheme == QRFS_SAMPLER_LEARNED) {
        hipError_t e = sample_any(s, index, n_sets, K, fx, fy, area, st);
        if (e != hipSuccess) return e;
        return qrfs::launch_weights(psd->model, c, psd->r0, psd->L0, has_ap, D, d, f32,
                                    n_sets * K, fx, fy, area, w, st);
    }
    return qrfs::launch_sample_weights(s->scheme, s->seed_x, s->seed_y, index, n_sets, K, s->N,
                                       s->df, s->fmin, s->fmax, psd->model, c, psd->r0, psd->L0,
                                       has_ap, D, d, f32, fx, fy, w, st);
}

using qrfs::kMaxLaunchBlocks;

// Runs launch_sum over all sets, splitting the grid so no launch exceeds
// kMaxLaunchBlocks blocks.
qrfs_status run_sum(int precision, int basis, int epi, qrfs::SumArgs a, int64_t n_sets,
                    hipStream_t st) {
    const int64_t per_set = qrfs::sum_blocks_per_set(precision, basis, a);
    const int64_t rts = a.partial
                            ? qrfs::sf_row_tiles_per_set(precision, a.K, a.R, a.R_block, a.P)
                            : 0;
    int64_t max_sets = kMaxLaunchBlocks / (per_set > 0 ? per_set : 1);
    if (max_sets < 1) return fail(QRFS_ERR_INVALID_ARG, "problem too large for one set");
    const double* fx0 = a.fx;
    const double* fy0 = a.fy;
    const double* w0 = a.w;
    double* part0 = a.partial;
    for (int64_t s0 = 0; s0 < n_sets; s0 += max_sets) {
        int64_t s1 = s0 + max_sets < n_sets ? s0 + max_sets : n_sets;
        a.set0 = s0;
        a.set1 = s1;
        a.fx = fx0 + s0 * a.K;
        a.fy = fy0 + s0 * a.K;
        a.w = w0 + s0 * a.K;
        if (part0) a.partial = part0 + s0 * rts * a.P * 2;
        hipError_t e = qrfs::launch_sum(precision, basis, epi, a, st);
        if (e != hipSuccess) return hip_fail(e, "kernel launch");
    }
    return QRFS_OK;
}

// Whether the stream is being captured (or that cannot be told).
bool is_capturing(hipStream_t st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return cap != hipStreamCaptureStatusNone;
}

// Partial sums of the frozen-flow estimator in blocks of `rows` realisations.
size_t temporal_part_bytes(int64_t R, int64_t M, int rows) {
    return align256((size_t)cdiv(R, rows) * M * 2 * sizeof(double));
}

// The estimator's workspace, with `fixed` bytes besides, and its blocks' rows: the
// longer blocks halve the partial sums where the workspace is capped, cannot grow
// (under capture) or finds no memory.
qrfs_status temporal_workspace(qrfs_context* ctx, int64_t R, int64_t M, size_t fixed,
                               hipStream_t st, int* rows) {
    *rows = qrfs::TEMPORAL_ROWS;
    const size_t bytes = fixed + temporal_part_bytes(R, M, *rows);
    qrfs_status s = QRFS_ERR_OUT_OF_MEMORY;
    if (!(bytes > ctx->ws_size && is_capturing(st))) s = ensure_workspace(ctx, bytes);
    if (s != QRFS_ERR_OUT_OF_MEMORY) return s;
    *rows = qrfs::TEMPORAL_ROWS_CAPPED;
    return ensure_workspace(ctx, fixed + temporal_part_bytes(R, M, *rows));
}

// Most scratch that the partial sums of a stored contraction take.
constexpr size_t kSplitCap = (size_t)256 << 20;
size_t split_room(const qrfs_context* ctx) {
    return scratch_room(ctx) < kSplitCap ? scratch_room(ctx) : kSplitCap;
}

// Stored sums in the fused kernels.  Where their tiles leave compute units
// idle, K is cut into ranges whose partial sums go through the scratch; not
// beyond the context's cap, and not while the stream is being captured (a
// graph must not hold memory that a later call may replace): then one range,
// which needs none.
// sp: the split for split_room, or ksplit = 0.
qrfs_status fused_sum(qrfs_context* ctx, int precision, int basis, qrfs::SumArgs a,
                      qrfs::StoreSplit sp, int64_t n_sets, hipStream_t st) {
    if (sp.ksplit == 0)
        sp = qrfs::store_split(precision, basis, a.K, a.R, a.R_block, a.P, split_room(ctx));
    char* part = nullptr;
    if (sp.ksplit > 1) {
        part = is_capturing(st) ? nullptr : scratch_block(ctx, sp.bytes);
        if (!part) sp = qrfs::store_split(precision, basis, a.K, a.R, a.R_block, a.P, 0);
    }
    a.ksplit = sp.ksplit;
    a.kspan = sp.kspan;
    a.phi_part = part;
    // narrow sets: fields on a regular grid go through its product structure, if
    // the points are one (the general kernel sees the same answer).  A grid of at
    // least 171 points (the fewest whose padded tiles can pass) saves up to 5/6 of
    // the time in binary64, half in FP32; a no costs 4 us: asked where that is
    // under 5 % of the call (in binary64 the estimate falls short by a quarter), or
    // where ranges have saved twice as much
    const bool fp64 = precision == QRFS_PREC_FP64;
    const double pad = qrfs::grid_max_pad(fp64, a.R_block);
    if (basis == qrfs::BASIS_PHASE && pad > 0.0 && a.P >= 171 && a.P <= ((int64_t)1 << 24) &&
        (sp.us > (fp64 ? 60.0 : 80.0) ||
         (sp.ksplit > 1 && sp.us > (fp64 ? 25.0 : 60.0) &&
          sp.us + 8.0 <
              qrfs::store_split(precision, basis, a.K, a.R, a.R_block, a.P, 0).us))) {
        qrfs::SepArgs b{};
        b.K = a.K;
        b.fx = a.fx;
        b.fy = a.fy;
        b.w = a.w;
        b.R = a.R;
        b.R_block = a.R_block;
        b.P = a.P;
        b.seed = a.seed;
        b.counter = a.counter;
        b.mode = a.mode;
        b.coef = a.coef;
        b.px = a.px;
        b.py = a.py;
        b.out = a.out;
        a.grid = grid_word(ctx, is_capturing(st));
        const hipError_t e =
            a.grid.word ? qrfs::launch_grid_sum(precision == QRFS_PREC_FP64, b, pad, a.grid, st)
                        : hipSuccess;
        if (e != hipSuccess) return hip_fail(e, "grid sum launch");
    }
    qrfs_status s = run_sum(precision, basis, qrfs::EPI_STORE, a, n_sets, st);
    if (s || sp.ksplit == 1) return s;
    hipError_t e = qrfs::launch_split_sum(precision == QRFS_PREC_FP64, part, sp.ksplit,
                                          a.R * a.P, a.out, a.grid, st);
    if (e != hipSuccess) return hip_fail(e, "partial-sum launch");
    return QRFS_OK;
}

// Sizes of the two-phase contraction of a problem.
struct WidePlan {
    int KCH;             // frequencies per chunk
    int64_t nch, nkv;    // chunks, padded contraction length
    size_t row32;        // bytes of 32 rows of coefficient tiles
    int64_t cts, rts_set;
    size_t scale_bytes;  // FP16X3: one scale per set
    int64_t sets_piece, rows_piece;  // sets, or rows of one set, per piece
    size_t tile_bytes;   // of the coefficient tiles of a piece
    int ksplit;          // frequency ranges (one piece only) and
    int64_t split_ch;    // their chunks
    size_t part_bytes;   // of partial sums
    size_t bytes() const { return tile_bytes + 256 + scale_bytes; }  // beside the partial sums
};

// ksplit: frequency ranges asked for; fewer where their partial sums exceed
// kSplitCap or the context's cap, or the coefficient tiles need pieces.
qrfs_status wide_plan(const qrfs_context* ctx, int precision, int64_t K, int64_t P, int64_t R,
                      int64_t R_block, int ksplit, WidePlan& p) {
    p.KCH = qrfs::wide_chunk(precision);
    p.nch = cdiv(K, p.KCH);
    p.nkv = p.nch * 2 * p.KCH;
    p.row32 = qrfs::wide_frag_bytes_per_row32(precision, p.nkv);
    p.cts = cdiv(P, 256);
    p.rts_set = cdiv(R_block, 256);
    const int64_t n_sets = cdiv(R, R_block);
    // coefficient tiles take at most ctx->tile_cap of workspace per piece
    // (one 256-row block of one set at least); behind them the store sink
    // (256 B) and, for FP16X3, one scale per set
    p.scale_bytes =
        precision == QRFS_PREC_FP16X3 ? align256((size_t)n_sets * sizeof(double)) : 0;
    size_t cap = ctx->tile_cap;
    const size_t extra = 512 + p.scale_bytes;
    if (ctx->ws_cap && ctx->ws_cap < cap + extra)
        cap = ctx->ws_cap > extra ? ctx->ws_cap - extra : 0;
    const size_t set_bytes = (size_t)p.rts_set * 8 * p.row32;
    p.sets_piece = 1;
    p.rows_piece = R_block;
    if (set_bytes <= cap) {
        p.sets_piece = (int64_t)(cap / set_bytes);
        const int64_t max_blocks = kMaxLaunchBlocks;
        if (p.sets_piece * p.rts_set * p.cts > max_blocks)
            p.sets_piece = max_blocks / (p.rts_set * p.cts);
        if (p.sets_piece < 1) return fail(QRFS_ERR_INVALID_ARG, "problem too large for one set");
        if (p.sets_piece > n_sets) p.sets_piece = n_sets;
    } else {
        int64_t tiles = (int64_t)(cap / (8 * p.row32));
        p.rows_piece = (tiles < 1 ? 1 : tiles) * 256;
    }
    p.tile_bytes = align256((size_t)p.sets_piece * cdiv(p.rows_piece, 256) * 8 * p.row32);
    p.ksplit = 1;
    p.split_ch = p.nch;
    p.part_bytes = 0;
    const size_t one = (size_t)R * P * sizeof(float);
    if (p.sets_piece == n_sets && p.rows_piece >= R_block) {
        while (ksplit > 1 && ((size_t)ksplit * one > kSplitCap ||
                              (ctx->ws_cap && p.bytes() + (size_t)ksplit * one > ctx->ws_cap)))
            --ksplit;
        if (ksplit > 1) {
            p.split_ch = cdiv(p.nch, ksplit);
            p.split_ch += p.split_ch & 1;
            p.ksplit = (int)cdiv(p.nch, p.split_ch);
            p.part_bytes = p.ksplit > 1 ? (size_t)p.ksplit * one : 0;
        }
    }
    return QRFS_OK;
}

// Whether a problem has the tiles to fill the chip with the two-phase kernel
// and the columns and rows to amortise it.
bool wide_fills(int64_t P, int64_t R, int64_t R_block) {
    return P >= 1024 && R_block >= 128 &&
           cdiv(R, R_block) * cdiv(R_block, 256) * cdiv(P, 256) >= 512;
}

// Frequencies that the two-phase kernel sums in FP32 before it adds them into
// the output.  Problems that fill the chip, and any when this kernel is asked
// for: ctx->range_freqs, and all of K in split-BF16, whose operand rounding is
// the larger error.  Others come here
// from the fused kernels, which fold their sums every 32 frequencies, and keep
// those kernels' accuracy: errors against binary64 at K = 1200, 4096, 10007 and
// 40000 are 2.2, 2.9, 4.0 and 7.4e-7 (BF16x6, one fused launch), here 2.2, 2.4,
// 3.2 and 7.0e-7 in ranges of K / 80 frequencies within [64, 512] (9.7e-7 at
// 10007 in ranges of 2048); FP16x3, with half the products, 2.4, 2.4, 3.3 and
// 4.3e-7 in ranges of K / 32 within [128, 512] (fused 2.2, 2.8, 3.9, 7.2e-7).
int64_t wide_range(const qrfs_context* ctx, int precision, int64_t K, int64_t P, int64_t R,
                   int64_t R_block) {
    if (ctx->wide_path == 2 || wide_fills(P, R, R_block))
        return precision == QRFS_PREC_SPLIT_BF16 ? K : ctx->range_freqs;
    if (precision == QRFS_PREC_SPLIT_BF16) return ctx->range_freqs < 2048 ? ctx->range_freqs : 2048;
    const bool f16 = precision == QRFS_PREC_FP16X3;
    const int64_t least = f16 ? 128 : 64;
    int64_t r = K / (f16 ? 32 : 80);
    r = r < least ? least : (r > 512 ? 512 : r);
    return r < ctx->range_freqs ? r : ctx->range_freqs;
}

// Fewest frequencies from which a problem that does not fill the device may go to
// the two-phase kernel: from there on its error is no larger than the fused
// kernel's in one range, which grows with K.  Below, the weighted coefficients and
// the short ranges' sums show: RMS error at K = 600, 1300, 1800, 2500, 3300 in units
// of the fused kernel's, 300 rows x 6400 points, piston 1.15, 1.05, 1.02, 0.96, 0.90
// and tilt 1.16, 1.07, 1.03, 0.97, 0.91 (FP32; less in BF16x6); FP16x3: phase 1.15,
// -, 1.00, 0.92, piston 1.14, 1.03, 1.01, 0.93, 0.86, tilt 1.26, 1.14, 1.10, 1.02,
// 0.96; phases of BF16x6 0.99 at 1200.  FP16x3 differences never: the basis itself
// has small values there, which the fused kernel scales with the amplitude and fp16
// cuts off here (1.03 to 1.05 for baselines of 0.1 m and less).
int64_t wide_least_freqs(int precision, int basis, bool tilt) {
    const bool f16 = precision == QRFS_PREC_FP16X3;
    if (basis == qrfs::BASIS_DIFF && f16) return INT64_MAX;
    if (basis == qrfs::BASIS_PISTON) return tilt ? 3300 : 2500;
    return f16 ? 1800 : 1200;
}

// Whether, and in how many frequency ranges, the two-phase kernel contracts
// this problem.  Forced by the context, or MFMA precisions by the estimated
// times of both kernels (us).  Two-phase: a 256 x 256 tile takes a compute
// unit wide_tile_ns per frequency, mostly for its basis, and every coefficient
// is drawn once (2.3 ps per padded row and frequency).  Fused: see store_split
// (coefficients redrawn per column tile).  At 100 realisations (50 per set) of
// 2500 points x 4096 frequencies in FP16x3 the fused kernel takes 139 us and
// this one 66, at ten apertures x 1e4 realisations 115 and 433.  A further range
// has to gain 5 %, this kernel 10 %: the estimates are no better.  Captured calls
// keep to problems that fill the chip whatever the path: a call that needs no
// workspace must not take one under capture.
// `sp` receives the fused kernels' ranges and time where they were estimated.
bool use_wide(const qrfs_context* ctx, int precision, int basis, bool tilt, int64_t K, int64_t P,
              int64_t R, int64_t R_block, bool caller_coef, hipStream_t st, int* ksplit,
              qrfs::StoreSplit* sp) {
    *ksplit = 1;
    if (precision == QRFS_PREC_FP64 || ctx->wide_path == 1) return false;
    // FP16X3 scales the coefficient tiles by the largest value the generators
    // can draw; caller-given coefficients contract in the fused kernel
    if (precision == QRFS_PREC_FP16X3 && caller_coef) return false;
    if (P > ((int64_t)1 << 22)) return false;  // 256 rows of output within 32-bit tile offsets
    const int64_t tiles = cdiv(R, R_block) * cdiv(R_block, 256) * cdiv(P, 256);
    const bool full = wide_fills(P, R, R_block);
    if (ctx->wide_path == 2) return true;  // as asked, in one range whatever the cap
    if (is_capturing(st)) return full;
    if (!full && (R_block <= 8 || K < wide_least_freqs(precision, basis, tilt))) return false;
    *sp = qrfs::store_split(precision, basis, K, R, R_block, P, split_room(ctx));
    const double fused = sp->us;
    double best = 1e300;
    const double coef = 2.3e-6 * (double)(cdiv(R, R_block) * cdiv(R_block, 256) * 256) * (double)K;
    const double one_us = 2.0 / 4e6 * (double)R * (double)P * sizeof(float);  // written and read
    const int64_t range = wide_range(ctx, precision, K, P, R, R_block);
    // the fullest tile of a set, and the mean over its row tiles
    const int64_t rest = R_block % 256;
    const double most = qrfs::wide_tile_ns(precision, basis, R_block);
    const double mean = (most * (double)(R_block / 256) +
                         (rest ? qrfs::wide_tile_ns(precision, basis, rest) : 0.0)) /
                        (double)cdiv(R_block, 256);
    for (int k = 1; k <= 32 && (k == 1 || (int64_t)k * 64 <= K); ++k) {  // as in store_split
        if (k > 1 && (size_t)k * R * P * sizeof(float) > kSplitCap) break;
        const int64_t rounds = cdiv(tiles * k, 256);
        const double ns = rounds > 1 ? std::fmax(most, mean * (double)rounds) : most;
        // each range after a block's first is added into its tile in memory
        const int64_t adds = cdiv(cdiv(K, (int64_t)k), range) - 1;
        const double us = ns * 1e-3 * (double)K / k + coef + 12.0 + (double)(adds * k) * one_us +
                          (k > 1 ? 8.0 + k * one_us : 0.0);
        if (us < 0.95 * best) {
            best = us;
            *ksplit = k;
        }
    }
    if (full) return true;
    WidePlan p;
    if (best > 0.9 * fused || wide_plan(ctx, precision, K, P, R, R_block, *ksplit, p) != QRFS_OK)
        return false;
    // the fused kernel needs no memory: it stays where this one's would exceed
    // the cap
    return p.bytes() + p.part_bytes <= scratch_room(ctx);
}

// Two-phase contraction (EPI_STORE) over all sets: per piece, the
// coefficient tiles, then one contraction launch, which sums ranges of
// wide_range frequencies in FP32 and adds each into the output.  The tiles of
// problems that fill the device, and of any when this kernel is asked for, lie in
// the workspace; all else in the scratch.
qrfs_status wide_sum(qrfs_context* ctx, int precision, int basis, qrfs::SumArgs a,
                     int64_t n_sets, int ksplit, hipStream_t st) {
    WidePlan p;
    qrfs_status s = wide_plan(ctx, precision, a.K, a.P, a.R, a.R_block, ksplit, p);
    if (s) return s;
    const int KCH = p.KCH;
    const int64_t nch = p.nch, sets_piece = p.sets_piece, rows_piece = p.rows_piece;
    char *base, *part;
    if (ctx->wide_path == 2 || wide_fills(a.P, a.R, a.R_block)) {
        s = ensure_workspace(ctx, p.bytes());
        if (s) return s;
        base = (char*)ctx->ws;
        part = p.ksplit > 1 ? scratch_block(ctx, p.part_bytes) : nullptr;
        if (p.ksplit > 1 && !part) {  // no room for partial sums: one range
            s = wide_plan(ctx, precision, a.K, a.P, a.R, a.R_block, 1, p);
            if (s) return s;
        }
    } else {
        base = scratch_block(ctx, p.bytes() + p.part_bytes);
        part = base ? base + p.bytes() : nullptr;
    }
    if (!base)
        return fail(QRFS_ERR_OUT_OF_MEMORY, "scratch of %zu bytes", p.bytes() + p.part_bytes);
    double* ascale = (double*)(base + p.tile_bytes + 256);
    if (precision == QRFS_PREC_FP16X3) {
        hipError_t e = qrfs::launch_wide_scale(a.w, a.K, n_sets, ascale, st);
        if (e != hipSuccess) return hip_fail(e, "tile scale launch");
    }
    a.ksplit = p.ksplit;
    a.phi_part = part;
    // accumulation ranges, an even number of chunks each
    const int64_t range = wide_range(ctx, precision, a.K, a.P, a.R, a.R_block);
    int64_t rch = cdiv(range, KCH);
    rch += rch & 1;
    const double* fx0 = a.fx;
    const double* fy0 = a.fy;
    const double* w0 = a.w;
    qrfs::WideArgs wa{};
    wa.nkv = p.nkv;
    wa.cts = p.cts;
    wa.split_ch = p.split_ch;
    wa.ctile = base;
    wa.sink = (float*)(base + p.tile_bytes);
    for (int64_t s0 = 0; s0 < n_sets; s0 += sets_piece) {
        const int64_t s1 = s0 + sets_piece < n_sets ? s0 + sets_piece : n_sets;
        for (int64_t off = 0; off < a.R_block; off += rows_piece) {
            // the last set may end before this row range
            if (s1 - s0 == 1 && s0 * a.R_block + off >= a.R) break;
            wa.s = a;
            wa.s.set0 = s0;
            wa.s.set1 = s1;
            wa.s.fx = fx0 + s0 * a.K;
            wa.s.fy = fy0 + s0 * a.K;
            wa.s.w = w0 + s0 * a.K;
            wa.ascale = ascale + s0;
            wa.row_off = off;
            wa.rows = off + rows_piece < a.R_block ? rows_piece : a.R_block - off;
            wa.rts = cdiv(wa.rows, 256);
            wa.rt32 = wa.rts * 8;
            hipError_t e = qrfs::launch_wide_coef(precision, wa, st);
            if (e != hipSuccess) return hip_fail(e, "coefficient tile launch");
            wa.ch0 = 0;
            wa.ch1 = nch;
            wa.range_ch = rch;
            wa.accumulate = 0;
            e = qrfs::launch_wide_sum(precision, basis, wa, st);
            if (e != hipSuccess) return hip_fail(e, "two-phase contraction launch");
        }
    }
    if (p.ksplit > 1) {
        hipError_t e = qrfs::launch_split_sum(false, a.phi_part, p.ksplit, a.R * a.P, a.out,
                                              {}, st);
        if (e != hipSuccess) return hip_fail(e, "partial-sum launch");
    }
    return QRFS_OK;
}


qrfs_status sum_entry(qrfs_context* ctx, int basis, int64_t K, const double* fx,
                      const double* fy, const double* w, int64_t P, const double* px,
                      const double* py, const double* apD, const double* apd, int64_t R,
                      int64_t R_block, const qrfs_rng* rng, const double* coef,
                      int32_t precision, void* out, void* stream,
                      const double* grad_u = nullptr) {
    qrfs_status s = check_sum_common(K, P, R, R_block, rng, coef, precision);
    if (s) return s;
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(w);
    CHECK_PTR(px);
    CHECK_PTR(py);
    if (basis == qrfs::BASIS_PISTON) {
        CHECK_PTR(apD);
        CHECK_PTR(apd);
    }
    if (!out) return fail(QRFS_ERR_INVALID_ARG, "output is NULL");
    if (((uintptr_t)out & (precision == QRFS_PREC_FP64 ? 7u : 3u)) != 0)
        return fail(QRFS_ERR_INVALID_ARG, "output is misaligned");
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    qrfs::SumArgs a{};
    a.K = K;
    a.fx = fx;
    a.fy = fy;
    a.w = w;
    a.P = P;
    a.px = px;
    a.py = py;
    a.apD = apD;
    a.apd = apd;
    a.R = R;
    a.R_block = R_block;
    a.seed = rng ? rng->seed : 0;
    a.counter = rng ? rng->counter : 0;
    a.mode = rng ? rng->mode : 0;
    a.coef = coef;
    a.out = out;
    a.partial = nullptr;
    a.ksplit = 1;
    a.kspan = K;
    a.phi_part = nullptr;
    if (grad_u) {
        a.grad = 1;
        a.gx = 2.0 * M_PI * grad_u[0];
        a.gy = 2.0 * M_PI * grad_u[1];
    }
    int ksplit = 1;
    qrfs::StoreSplit sp{};
    bool wide = use_wide(ctx, precision, basis, grad_u != nullptr, K, P, R, R_block,
                         coef != nullptr, (hipStream_t)stream, &ksplit, &sp);
    if (wide) {
        s = wide_sum(ctx, precision, basis, a, cdiv(R, R_block), ksplit, (hipStream_t)stream);
        // no memory for its tiles (nothing is enqueued yet): the fused kernel
        // takes what it took before such problems came here
        wide = !(s == QRFS_ERR_OUT_OF_MEMORY && ctx->wide_path == 0 && !wide_fills(P, R, R_block));
    }
    if (!wide)
        s = fused_sum(ctx, precision, basis, a, sp, cdiv(R, R_block), (hipStream_t)stream);
    if (s) return s;
    return ok();
}

}  // namespace

namespace qrfs {
// shared with the batch layer
qrfs_status api_fail(qrfs_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_detail = buf;
    return s;
}
qrfs_status api_ok() { return ok(); }
int64_t api_context_range_freqs(const qrfs_context* ctx) { return ctx->range_freqs; }
int api_context_device(const qrfs_context* ctx) { return ctx->device; }
}  // namespace qrfs

extern "C" {

const char* qrfs_error_string(qrfs_status s) {
    switch (s) {
        case QRFS_OK: return "success";
        case QRFS_ERR_INVALID_ARG: return "invalid argument";
        case QRFS_ERR_OUT_OF_MEMORY: return "out of device memory";
        case QRFS_ERR_DEVICE: return "device (HIP runtime) error";
        case QRFS_ERR_UNSUPPORTED: return "unsupported";
        case QRFS_ERR_NOT_CONVERGED: return "not converged";
        default: return "unknown status";
    }
}

const char* qrfs_last_error_detail(void) { return g_detail.c_str(); }

int32_t qrfs_abi_version(void) { return QRFS_ABI_VERSION; }

qrfs_status qrfs_context_create(qrfs_context** out, int32_t device, size_t workspace_cap_bytes) {
    if (!out) return fail(QRFS_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess) return hip_fail(e, "hipGetDeviceCount");
    if (device < 0 || device >= n)
        return fail(QRFS_ERR_INVALID_ARG, "device %d out of range (%d devices)", device, n);
    {
        DeviceGuard g(device);
        if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", device);
        e = scratch_setup(device);
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress of the static scratch");
    }
    qrfs_context* c = new (std::nothrow) qrfs_context();
    if (!c) return fail(QRFS_ERR_OUT_OF_MEMORY, "host allocation of the context");
    c->device = device;
    c->ws_cap = workspace_cap_bytes;
    c->grid_slot = take_grid_slot(device);
    *out = c;
    return ok();
}

qrfs_status qrfs_context_set_tuning(qrfs_context* ctx, int32_t key, int64_t value) {
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    if (key == QRFS_TUNE_WIDE_PATH) {
        if (value < 0 || value > 2)
            return fail(QRFS_ERR_INVALID_ARG, "wide path must be 0, 1 or 2 (got %lld)", (long long)value);
        ctx->wide_path = (int)value;
    } else if (key == QRFS_TUNE_RANGE_FREQS) {
        if (value < 0 || value > ((int64_t)1 << 33))
            return fail(QRFS_ERR_INVALID_ARG, "range of %lld frequencies", (long long)value);
        ctx->range_freqs = value == 0 ? 2048 : value;
    } else if (key == QRFS_TUNE_TILE_BYTES) {
        if (value < 0) return fail(QRFS_ERR_INVALID_ARG, "tile cap of %lld bytes", (long long)value);
        ctx->tile_cap = value == 0 ? ((size_t)2 << 30) : (size_t)value;
    } else {
        return fail(QRFS_ERR_INVALID_ARG, "unknown tuning key %d", key);
    }
    return ok();
}

qrfs_status qrfs_context_destroy(qrfs_context* ctx) {
    if (!ctx) return ok();
    qrfs_status st = QRFS_OK;
    {
        DeviceGuard g(ctx->device);
        if (ctx->ws || ctx->scratch) {
            hipError_t e = hipDeviceSynchronize();
            if (e != hipSuccess) st = hip_fail(e, "hipDeviceSynchronize in destroy");
            if (ctx->ws) (void)hipFree(ctx->ws);
            free_scratch(ctx);
        }
    }
    give_grid_slot(ctx->device, ctx->grid_slot);
    delete ctx;
    return st ? st : ok();
}

qrfs_status qrfs_sample_frequencies(qrfs_context* ctx, qrfs_sampler* s, int64_t n_sets,
                                    int64_t K, double* fx, double* fy, double* area,
                                    void* stream) {
    qrfs_status st = check_sampler(s, K);
    if (st) return st;
    if (K <= 0 || n_sets <= 0)
        return fail(QRFS_ERR_INVALID_ARG, "K and n_sets must be > 0 (got %lld, %lld)",
                    (long long)K, (long long)n_sets);
    if (n_sets > INT64_MAX / K || n_sets * K > QRFS_MAX_POINTS_PER_CALL)
        return fail(QRFS_ERR_INVALID_ARG, "n_sets * K = %lld exceeds %lld points per call",
                    (long long)(n_sets > INT64_MAX / K ? INT64_MAX : n_sets * K),
                    (long long)QRFS_MAX_POINTS_PER_CALL);
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(area);
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipError_t e = sample_any(s, s->index, n_sets, K, fx, fy, area, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "sampler launch");
    s->index += (uint64_t)(n_sets * K);
    return ok();
}

// The precision argument of the weight entry points: any known precision,
// FP64 for binary64 weights, the others for weights that feed FP32-class sums.
static qrfs_status check_weight_precision(int32_t precision) {
    if (precision < QRFS_PREC_FP64 || precision > QRFS_PREC_FP16X3)
        return fail(QRFS_ERR_INVALID_ARG, "unknown precision %d", precision);
    return QRFS_OK;
}

qrfs_status qrfs_weights(qrfs_context* ctx, const qrfs_psd* psd, const qrfs_aperture* ap,
                         int64_t n, const double* fx, const double* fy, const double* area,
                         int32_t precision, double* w, void* stream) {
    qrfs_status st = check_psd(psd);
    if (st) return st;
    if (ap && (st = check_ap(ap))) return st;
    if ((st = check_weight_precision(precision))) return st;
    if (n <= 0 || n > QRFS_MAX_POINTS_PER_CALL)
        return fail(QRFS_ERR_INVALID_ARG, "n must be in 1..%lld (got %lld)",
                    (long long)QRFS_MAX_POINTS_PER_CALL, (long long)n);
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(area);
    CHECK_PTR(w);
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    const double c = qrfs::psd_constant(psd->c, psd->wavelength);
    hipError_t e = qrfs::launch_weights(psd->model, c, psd->r0, psd->L0, ap ? 1 : 0,
                                        ap ? ap->D : 0.0, ap ? ap->d : 0.0,
                                        precision != QRFS_PREC_FP64, n, fx, fy, area, w,
                                        (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "weights launch");
    return ok();
}

qrfs_status qrfs_sample_weights(qrfs_context* ctx, qrfs_sampler* s, int64_t n_sets, int64_t K,
                                const qrfs_psd* psd, const qrfs_aperture* ap, int32_t precision,
                                double* fx, double* fy, double* w, void* stream) {
    qrfs_status st = check_sampler(s, K);
    if (st) return st;
    if ((st = check_psd(psd))) return st;
    if (ap && (st = check_ap(ap))) return st;
    if ((st = check_weight_precision(precision))) return st;
    if (K <= 0 || n_sets <= 0)
        return fail(QRFS_ERR_INVALID_ARG, "K and n_sets must be > 0 (got %lld, %lld)",
                    (long long)K, (long long)n_sets);
    if (n_sets > INT64_MAX / K || n_sets * K > QRFS_MAX_POINTS_PER_CALL)
        return fail(QRFS_ERR_INVALID_ARG, "n_sets * K = %lld exceeds %lld points per call",
                    (long long)(n_sets > INT64_MAX / K ? INT64_MAX : n_sets * K),
                    (long long)QRFS_MAX_POINTS_PER_CALL);
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(w);
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    double* area = nullptr;
    if (s->scheme == QRFS_SAMPLER_LEARNED) {  // its cell areas go through the workspace
        if ((st = ensure_workspace(ctx, (size_t)(n_sets * K) * sizeof(double)))) return st;
        area = (double*)ctx->ws;
    }
    const double c = qrfs::psd_constant(psd->c, psd->wavelength);
    hipError_t e =
        sample_weights_any(s, s->index, n_sets, K, psd, c, ap, precision != QRFS_PREC_FP64, fx,
                           fy, area, w, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "sampler / weights launch");
    s->index += (uint64_t)(n_sets * K);
    return ok();
}

qrfs_status qrfs_synthesize_phase(qrfs_context* ctx, int64_t K, const double* fx,
                                  const double* fy, const double* w, int64_t P,
                                  const double* px, const double* py, int64_t R,
                                  int64_t R_block, const qrfs_rng* rng, const double* coef,
                                  int32_t precision, void* phase, void* stream) {
    return sum_entry(ctx, qrfs::BASIS_PHASE, K, fx, fy, w, P, px, py, nullptr, nullptr, R,
                     R_block, rng, coef, precision, phase, stream);
}

qrfs_status qrfs_piston(qrfs_context* ctx, int64_t K, const double* fx, const double* fy,
                        const double* w, int64_t n_ap, const double* cx, const double* cy,
                        const double* apD, const double* apd, int64_t R, int64_t R_block,
                        const qrfs_rng* rng, const double* coef, int32_t precision,
                        void* piston, void* stream) {
    return sum_entry(ctx, qrfs::BASIS_PISTON, K, fx, fy, w, n_ap, cx, cy, apD, apd, R, R_block,
                     rng, coef, precision, piston, stream);
}

qrfs_status qrfs_tilt(qrfs_context* ctx, int64_t K, const double* fx, const double* fy,
                      const double* w, int64_t n_ap, const double* cx, const double* cy,
                      const double* apD, const double* apd, double ux, double uy, int64_t R,
                      int64_t R_block, const qrfs_rng* rng, const double* coef,
                      int32_t precision, void* tilt, void* stream) {
    if (!std::isfinite(ux) || !std::isfinite(uy) || (ux == 0.0 && uy == 0.0))
        return fail(QRFS_ERR_INVALID_ARG, "direction (%g, %g) is zero or not finite", ux, uy);
    const double u[2] = {ux, uy};
    return sum_entry(ctx, qrfs::BASIS_PISTON, K, fx, fy, w, n_ap, cx, cy, apD, apd, R, R_block,
                     rng, coef, precision, tilt, stream, u);
}

qrfs_status qrfs_diff_piston(qrfs_context* ctx, int64_t K, const double* fx, const double* fy,
                             const double* w, int64_t nB, const double* bx, const double* by,
                             int64_t R, int64_t R_block, const qrfs_rng* rng, const double* coef,
                             int32_t precision, void* dp, void* stream) {
    return sum_entry(ctx, qrfs::BASIS_DIFF, K, fx, fy, w, nB, bx, by, nullptr, nullptr, R,
                     R_block, rng, coef, precision, dp, stream);
}

qrfs_status qrfs_diff_piston_structure(qrfs_context* ctx, const qrfs_psd* psd,
                                       const qrfs_aperture* ap, int64_t nB, const double* bx,
                                       const double* by, qrfs_sampler* s, int64_t K, int64_t R,
                                       int64_t R_block, const qrfs_rng* rng, int32_t precision,
                                       double* sf, double* sf_stderr, void* stream) {
    qrfs_status st = check_psd(psd);
    if (st) return st;
    if (!ap) return fail(QRFS_ERR_INVALID_ARG, "aperture is required");
    if ((st = check_ap(ap))) return st;
    if ((st = check_sampler(s, K))) return st;
    if ((st = check_sum_common(K, nB, R, R_block, rng, nullptr, precision))) return st;
    CHECK_PTR(bx);
    CHECK_PTR(by);
    CHECK_PTR(sf);
    if (sf_stderr && !aligned8(sf_stderr))
        return fail(QRFS_ERR_INVALID_ARG, "sf_stderr is not 8-byte aligned");
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);

    const int64_t n_sets = cdiv(R, R_block);
    const int64_t rts = qrfs::sf_row_tiles_per_set(precision, K, R, R_block, nB);
    const qrfs::SfPlan plan = qrfs::sf_plan(precision, K, R, R_block, nB);
    const size_t partial_bytes = align256((size_t)(plan.n_partial_tiles * nB) * 2 * sizeof(double));
    const size_t phi_bytes = align256(plan.phi_floats * sizeof(float));
    const size_t per_set = (size_t)K * 4 * sizeof(double);
    const size_t budget = (size_t)1 << 30;
    int64_t spb = (int64_t)(budget / per_set);
    if (spb < 1) spb = 1;
    if (spb > n_sets) spb = n_sets;
    const size_t arr = align256((size_t)spb * K * sizeof(double));
    if ((st = ensure_workspace(ctx, partial_bytes + phi_bytes + 4 * arr))) return st;
    char* base = (char*)ctx->ws;
    double* partial = (double*)base;
    float* phi = (float*)(base + partial_bytes);
    char* fbase = base + partial_bytes + phi_bytes;
    double* fx = (double*)(fbase);
    double* fy = (double*)(fbase + arr);
    double* area = (double*)(fbase + 2 * arr);
    double* w = (double*)(fbase + 3 * arr);
    hipStream_t stream_ = (hipStream_t)stream;
    const double c = qrfs::psd_constant(psd->c, psd->wavelength);

    for (int64_t s0 = 0; s0 < n_sets; s0 += spb) {
        int64_t s1 = s0 + spb < n_sets ? s0 + spb : n_sets;
        int64_t ns = s1 - s0;
        hipError_t e = sample_weights_any(s, s->index + (uint64_t)(s0 * K), ns, K, psd, c, ap, 0,
                                          fx, fy, area, w, stream_);
        if (e != hipSuccess) return hip_fail(e, "sampler / weights launch");
        qrfs::SumArgs a{};
        a.K = K;
        a.fx = fx;
        a.fy = fy;
        a.w = w;
        a.P = nB;
        a.px = bx;
        a.py = by;
        a.R = R;
        a.R_block = R_block;
        a.seed = rng->seed;
        a.counter = rng->counter;
        a.mode = rng->mode;
        a.coef = nullptr;
        a.out = nullptr;
        a.ksplit = plan.ksplit;
        a.kspan = plan.kspan;
        a.phi_part = phi;
        // absolute set bounds; the batch buffers hold exactly these sets
        a.set0 = s0;
        a.set1 = s1;
        a.partial = partial + s0 * rts * nB * 2;
        e = qrfs::launch_sum(precision, qrfs::BASIS_DIFF, qrfs::EPI_SFSUM, a, stream_);
        if (e != hipSuccess) return hip_fail(e, "structure-function launch");
    }
    hipError_t e =
        plan.ksplit > 1
            ? qrfs::launch_split_sf(phi, plan.ksplit, R, nB, partial, plan.n_partial_tiles, sf,
                                    sf_stderr, stream_)
            : qrfs::launch_reduce_sf(partial, plan.n_partial_tiles, nB, R, sf, sf_stderr, stream_);
    if (e != hipSuccess) return hip_fail(e, "reduction launch");
    s->index += (uint64_t)(n_sets * K);
    return ok();
}

qrfs_status qrfs_point_set_measures(qrfs_context* ctx, int64_t n_sets, int64_t K,
                                    const double* fx, const double* fy, double x0, double y0,
                                    double Lx, double Ly, double r_clash, double* min_dist,
                                    int64_t* n_clash, double* l2_star, void* stream) {
    if (n_sets < 1 || K < 1)
        return fail(QRFS_ERR_INVALID_ARG, "n_sets and K must be >= 1 (got %lld, %lld)",
                    (long long)n_sets, (long long)K);
    if (K > ((int64_t)1 << 24))
        return fail(QRFS_ERR_INVALID_ARG, "K must be <= 2^24 (got %lld)", (long long)K);
    // one block of 256 threads per (set, 256-point tile): at most 2^24
    // blocks keep the launch within 2^32 work-items
    if (n_sets * qrfs::measure_tiles(K) >= ((int64_t)1 << 24))
        return fail(QRFS_ERR_INVALID_ARG, "n_sets * ceil(K/256) must be < 2^24");
    if (!(Lx > 0.0) || !(Ly > 0.0) || !std::isfinite(Lx) || !std::isfinite(Ly) ||
        !std::isfinite(x0) || !std::isfinite(y0))
        return fail(QRFS_ERR_INVALID_ARG, "the unit-square map needs finite x0, y0 and Lx, Ly > 0");
    if (!(r_clash >= 0.0) || !std::isfinite(r_clash))
        return fail(QRFS_ERR_INVALID_ARG, "r_clash must be finite and >= 0 (got %g)", r_clash);
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(min_dist);
    CHECK_PTR(n_clash);
    CHECK_PTR(l2_star);
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    const size_t part_bytes = align256((size_t)(n_sets * qrfs::measure_tiles(K)) * 4 * sizeof(double));
    qrfs_status st = ensure_workspace(ctx, part_bytes);
    if (st) return st;
    hipError_t e = qrfs::launch_point_set_measures(n_sets, K, fx, fy, x0, y0, Lx, Ly, r_clash,
                                                   (double*)ctx->ws, min_dist, n_clash, l2_star,
                                                   (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "point-set measure launch");
    return ok();
}

qrfs_status qrfs_set_sf_expectation(qrfs_context* ctx, int64_t K, const double* fx,
                                    const double* fy, const double* w, int64_t n_sets, int64_t nB,
                                    const double* bx, const double* by, double* S, void* stream) {
    if (K < 1 || n_sets < 1 || nB < 1)
        return fail(QRFS_ERR_INVALID_ARG, "K, n_sets and nB must be >= 1");
    if (n_sets >= ((int64_t)1 << 24))  // one 256-thread block per set
        return fail(QRFS_ERR_INVALID_ARG, "n_sets must be < 2^24");
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(w);
    CHECK_PTR(bx);
    CHECK_PTR(by);
    CHECK_PTR(S);
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    hipError_t e = qrfs::launch_set_sf(n_sets, K, fx, fy, w, nB, bx, by, S, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "per-set structure function launch");
    return ok();
}

qrfs_status qrfs_temporal_sf(qrfs_context* ctx, int64_t R, int64_t M, int32_t precision,
                             const void* pistons, double* sf, double* sf_stderr, void* stream) {
    if (R < 1) return fail(QRFS_ERR_INVALID_ARG, "R must be >= 1 (got %lld)", (long long)R);
    if (M < 1 || M > qrfs::TEMPORAL_MAX_M)
        return fail(QRFS_ERR_INVALID_ARG, "M must be in [1, %d] (got %lld)", qrfs::TEMPORAL_MAX_M,
                    (long long)M);
    if (precision != QRFS_PREC_FP64 && precision != QRFS_PREC_FP32 &&
        precision != QRFS_PREC_SPLIT_BF16 && precision != QRFS_PREC_BF16X6 &&
        precision != QRFS_PREC_FP16X3)
        return fail(QRFS_ERR_INVALID_ARG, "unknown precision %d", precision);
    if (!pistons) return fail(QRFS_ERR_INVALID_ARG, "pistons is NULL");
    if (((uintptr_t)pistons & (precision == QRFS_PREC_FP64 ? 7u : 3u)) != 0)
        return fail(QRFS_ERR_INVALID_ARG, "pistons is misaligned");
    CHECK_PTR(sf);
    if (sf_stderr && !aligned8(sf_stderr))
        return fail(QRFS_ERR_INVALID_ARG, "sf_stderr is not 8-byte aligned");
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    int rows;
    qrfs_status st = temporal_workspace(ctx, R, M, 0, (hipStream_t)stream, &rows);
    if (st) return st;
    const int64_t nb = cdiv(R, rows);
    double* part = (double*)ctx->ws;
    hipStream_t stream_ = (hipStream_t)stream;
    hipError_t e = qrfs::launch_temporal_rows(precision == QRFS_PREC_FP64, false, pistons, R, M,
                                              rows, part, stream_);
    if (e != hipSuccess) return hip_fail(e, "temporal estimator launch");
    e = qrfs::launch_reduce_sf(part, nb, M, R, sf, sf_stderr, stream_);
    if (e != hipSuccess) return hip_fail(e, "reduction launch");
    return ok();
}

qrfs_status qrfs_temporal_piston_structure(qrfs_context* ctx, const qrfs_psd* psd,
                                           const qrfs_aperture* ap, const double* c1,
                                           const double* c2, const double* v, double dt,
                                           int64_t M, qrfs_sampler* s, int64_t K, int64_t R,
                                           int64_t R_block, const qrfs_rng* rng,
                                           int32_t precision, double* sf, double* sf_stderr,
                                           void* stream) {
    qrfs_status st = check_psd(psd);
    if (st) return st;
    if (!ap) return fail(QRFS_ERR_INVALID_ARG, "aperture is required");
    if ((st = check_ap(ap))) return st;
    if ((st = check_sampler(s, K))) return st;
    if (M < 1 || M > qrfs::TEMPORAL_MAX_M)
        return fail(QRFS_ERR_INVALID_ARG, "M must be in [1, %d] (got %lld)", qrfs::TEMPORAL_MAX_M,
                    (long long)M);
    if ((st = check_sum_common(K, 2 * M, R, R_block, rng, nullptr, precision))) return st;
    if (!c1 || !c2 || !v) return fail(QRFS_ERR_INVALID_ARG, "c1, c2 and v are required");
    if (!(dt >= 0.0) || !std::isfinite(dt))
        return fail(QRFS_ERR_INVALID_ARG, "dt must be finite and >= 0");
    for (int i = 0; i < 2; ++i)
        if (!std::isfinite(c1[i]) || !std::isfinite(c2[i]) || !std::isfinite(v[i]))
            return fail(QRFS_ERR_INVALID_ARG, "c1, c2, v must be finite");
    CHECK_PTR(sf);
    if (sf_stderr && !aligned8(sf_stderr))
        return fail(QRFS_ERR_INVALID_ARG, "sf_stderr is not 8-byte aligned");
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);

    const int64_t n_sets = cdiv(R, R_block);
    const int64_t P = 2 * M;
    const bool fp64 = precision == QRFS_PREC_FP64;
    const size_t esize = fp64 ? sizeof(double) : sizeof(float);
    // FP64 series of more than 64 samples use their equal spacing (tiles of
    // 1024 samples: 268 cycles per frequency and tile against 148 per 64
    // points, 32 samples of both telescopes, in the general kernel)
    const bool series = fp64 && M > 64;
    // pieces of whole sets (at most ~1 GiB of frequencies and pistons) whose
    // first realisation is a multiple of the estimator's row blocks (of
    // either size), so the fixed-order reduction sees the same blocks however
    // the sets are cut
    const int64_t q =
        qrfs::TEMPORAL_ROWS_CAPPED / std::gcd(R_block, (int64_t)qrfs::TEMPORAL_ROWS_CAPPED);
    const size_t per_set = (size_t)K * 4 * sizeof(double) + (size_t)R_block * P * esize;
    int64_t spb = (int64_t)(((size_t)1 << 30) / per_set);
    spb = spb / q * q;
    if (spb < q) spb = q;
    if (spb > n_sets) spb = n_sets;
    const size_t pt_bytes = align256((size_t)P * sizeof(double));
    const size_t arr = align256((size_t)spb * K * sizeof(double));
    // such a series keeps the differential pistons only
    const size_t pist_bytes = align256((size_t)spb * R_block * (series ? M : P) * esize);
    const size_t fixed_bytes = 2 * pt_bytes + 4 * arr + pist_bytes;
    int rows_block;
    if ((st = temporal_workspace(ctx, R, M, fixed_bytes, (hipStream_t)stream, &rows_block)))
        return st;
    const int64_t nb = cdiv(R, rows_block);
    const size_t part_bytes = temporal_part_bytes(R, M, rows_block);
    char* base = (char*)ctx->ws;
    double* part = (double*)base;
    double* px = (double*)(base + part_bytes);
    double* py = (double*)(base + part_bytes + pt_bytes);
    char* fbase = base + part_bytes + 2 * pt_bytes;
    double* fx = (double*)fbase;
    double* fy = (double*)(fbase + arr);
    double* area = (double*)(fbase + 2 * arr);
    double* w = (double*)(fbase + 3 * arr);
    void* pist = fbase + 4 * arr;
    hipStream_t stream_ = (hipStream_t)stream;
    const double c = qrfs::psd_constant(psd->c, psd->wavelength);

    hipError_t e = hipSuccess;
    if (!series) {
        e = qrfs::launch_taylor_points(c1, c2, v, dt, M, px, py, stream_);
        if (e != hipSuccess) return hip_fail(e, "point launch");
    }
    for (int64_t s0 = 0; s0 < n_sets; s0 += spb) {
        const int64_t s1 = s0 + spb < n_sets ? s0 + spb : n_sets;
        const int64_t ns = s1 - s0;
        const int64_t r0 = s0 * R_block;
        const int64_t rows = (s1 * R_block < R ? s1 * R_block : R) - r0;
        // equal apertures: the filter of Eq. 7 folds into the weight
        e = sample_weights_any(s, s->index + (uint64_t)(s0 * K), ns, K, psd, c, ap, 0, fx, fy,
                               area, w, stream_);
        if (e != hipSuccess) return hip_fail(e, "sampler / weights launch");
        // the piece as a problem of its own: realisations r0 .. r0 + rows
        if (series) {
            // the samples are equally spaced: rows of 32 of them share the
            // sine and cosine of their first, and p1 - p2 is formed per frequency
            qrfs::SepArgs a{};
            a.K = K;
            a.fx = fx;
            a.fy = fy;
            a.w = w;
            a.R = rows;
            a.R_block = R_block;
            a.P = M;
            a.seed = rng->seed;
            a.counter = rng->counter + (uint64_t)r0;
            a.mode = rng->mode;
            a.V = 32;
            a.ox = c1[0];
            a.oy = c1[1];
            a.sx = -v[0] * dt;
            a.sy = -v[1] * dt;
            a.dx = c2[0] - c1[0];
            a.dy = c2[1] - c1[1];
            a.out = pist;
            e = qrfs::launch_series_diff(a, stream_);
            if (e != hipSuccess) return hip_fail(e, "time-series launch");
        } else {
            qrfs::SumArgs a{};
            a.K = K;
            a.fx = fx;
            a.fy = fy;
            a.w = w;
            a.P = P;
            a.px = px;
            a.py = py;
            a.R = rows;
            a.R_block = R_block;
            a.seed = rng->seed;
            a.counter = rng->counter + (uint64_t)r0;
            a.mode = rng->mode;
            a.coef = nullptr;
            a.out = pist;
            a.partial = nullptr;
            a.ksplit = 1;
            a.kspan = K;
            a.phi_part = nullptr;
            if ((st = run_sum(precision, qrfs::BASIS_PHASE, qrfs::EPI_STORE, a, ns, stream_)))
                return st;
        }
        e = qrfs::launch_temporal_rows(fp64, series, pist, rows, M, rows_block,
                                       part + (r0 / rows_block) * M * 2, stream_);
        if (e != hipSuccess) return hip_fail(e, "temporal estimator launch");
    }
    e = qrfs::launch_reduce_sf(part, nb, M, R, sf, sf_stderr, stream_);
    if (e != hipSuccess) return hip_fail(e, "reduction launch");
    s->index += (uint64_t)(n_sets * K);
    return ok();
}

qrfs_status qrfs_diff_piston_structure_sets(qrfs_context* ctx, int64_t K, const double* fx,
                                            const double* fy, const double* w, int64_t nB,
                                            const double* bx, const double* by, int64_t R,
                                            int64_t R_block, const qrfs_rng* rng,
                                            int32_t precision, double* sf, double* sf_stderr,
                                            void* stream) {
    qrfs_status st = check_sum_common(K, nB, R, R_block, rng, nullptr, precision);
    if (st) return st;
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(w);
    CHECK_PTR(bx);
    CHECK_PTR(by);
    CHECK_PTR(sf);
    if (sf_stderr && !aligned8(sf_stderr))
        return fail(QRFS_ERR_INVALID_ARG, "sf_stderr is not 8-byte aligned");
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    const qrfs::SfPlan plan = qrfs::sf_plan(precision, K, R, R_block, nB);
    const size_t partial_bytes = align256((size_t)(plan.n_partial_tiles * nB) * 2 * sizeof(double));
    const size_t phi_bytes = align256(plan.phi_floats * sizeof(float));
    if ((st = ensure_workspace(ctx, partial_bytes + phi_bytes))) return st;
    st = sf_sets_enqueue(plan, (char*)ctx->ws, K, fx, fy, w, nB, bx, by, R, R_block, rng,
                         precision, sf, sf_stderr, (hipStream_t)stream);
    return st ? st : ok();
}

qrfs_status qrfs_diff_piston_structure_sets_noalloc(qrfs_context* ctx, int64_t K,
                                                    const double* fx, const double* fy,
                                                    const double* w, int64_t nB,
                                                    const double* bx, const double* by,
                                                    int64_t R, int64_t R_block,
                                                    const qrfs_rng* rng, int32_t precision,
                                                    double* sf, double* sf_stderr,
                                                    void* stream) {
    qrfs_status st = check_sum_common(K, nB, R, R_block, rng, nullptr, precision);
    if (st) return st;
    CHECK_PTR(fx);
    CHECK_PTR(fy);
    CHECK_PTR(w);
    CHECK_PTR(bx);
    CHECK_PTR(by);
    CHECK_PTR(sf);
    if (sf_stderr && !aligned8(sf_stderr))
        return fail(QRFS_ERR_INVALID_ARG, "sf_stderr is not 8-byte aligned");
    if (!ctx) return fail(QRFS_ERR_INVALID_ARG, "context is NULL");
    DeviceGuard g(ctx->device);
    if (!g.okay) return fail(QRFS_ERR_DEVICE, "cannot select device %d", ctx->device);
    const qrfs::SfPlan plan = qrfs::sf_plan(precision, K, R, R_block, nB, kScratchBytes);
    const size_t need = qrfs::sf_plan_bytes(plan, nB);
    if (need > kScratchBytes)
        return fail(QRFS_ERR_INVALID_ARG,
                    "needs %zu bytes of scratch; the allocation-free entry point has %zu "
                    "(fewer sets, realisations or baselines per call)",
                    need, kScratchBytes);
    void* base = scratch_ptr(ctx->device);
    if (!base) return fail(QRFS_ERR_UNSUPPORTED, "no static scratch on device %d", ctx->device);
    st = sf_sets_enqueue(plan, (char*)base, K, fx, fy, w, nB, bx, by, R, R_block, rng, precision,
                         sf, sf_stderr, (hipStream_t)stream);
    return st ? st : ok();
}

}  // extern "C"

namespace {
// The sums of qrfs_diff_piston_structure_sets over caller frequency sets,
// with the plan's scratch at `base`: per-tile partials first, then the
// split-K partial sums (every element the later kernels read is written
// first, so the scratch needs no clearing).
qrfs_status sf_sets_enqueue(const qrfs::SfPlan& plan, char* base, int64_t K, const double* fx,
                            const double* fy, const double* w, int64_t nB, const double* bx,
                            const double* by, int64_t R, int64_t R_block, const qrfs_rng* rng,
                            int32_t precision, double* sf, double* sf_stderr, hipStream_t stream) {
    qrfs_status st;
    const int64_t n_sets = cdiv(R, R_block);
    const size_t partial_bytes = align256((size_t)(plan.n_partial_tiles * nB) * 2 * sizeof(double));
    double* partial = (double*)base;
    float* phi = (float*)(base + partial_bytes);
    qrfs::SumArgs a{};
    a.K = K;
    a.fx = fx;
    a.fy = fy;
    a.w = w;
    a.P = nB;
    a.px = bx;
    a.py = by;
    a.R = R;
    a.R_block = R_block;
    a.seed = rng->seed;
    a.counter = rng->counter;
    a.mode = rng->mode;
    a.partial = partial;
    a.ksplit = plan.ksplit;
    a.kspan = plan.kspan;
    a.phi_part = phi;
    if ((st = run_sum(precision, qrfs::BASIS_DIFF, qrfs::EPI_SFSUM, a, n_sets, stream))) return st;
    hipError_t e =
        plan.ksplit > 1
            ? qrfs::launch_split_sf(phi, plan.ksplit, R, nB, partial, plan.n_partial_tiles, sf,
                                    sf_stderr, stream)
            : qrfs::launch_reduce_sf(partial, plan.n_partial_tiles, nB, R, sf, sf_stderr, stream);
    if (e != hipSuccess) return hip_fail(e, "reduction launch");
    return QRFS_OK;
}
}  // namespace
