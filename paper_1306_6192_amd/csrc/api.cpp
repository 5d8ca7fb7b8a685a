// C-ABI of the plain product, operand preparation, comparison reduction and
// diagnostics.  Argument validation happens here, before any HIP call.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <vector>

#include "host.hpp"

namespace mg {

static thread_local char t_err[512] = "";

int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(t_err, sizeof(t_err), fmt, ap);
    va_end(ap);
    return code;
}

void clear_error() { t_err[0] = 0; }

uint64_t now_ns() {
    return (uint64_t)std::chrono::duration_cast<std::chrono::nanoseconds>(
               std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

size_t elem_size(int mode) {
    switch (mode) {
        case GEMM_MODE_F32:
        case GEMM_MODE_F32_SPLIT_BF16X3: return 4;
        case GEMM_MODE_BF16:
        case GEMM_MODE_F16: return 2;
        case GEMM_MODE_F8E4M3: return 1;
        default: return 0;
    }
}

bool mode_known(int mode) { return mode >= 0 && mode < GEMM_NUM_MODES; }

// Largest dimension the kernels index with 32-bit tile arithmetic.
static const int64_t kMaxDim = (int64_t)1 << 30;

static bool overlaps(const void *a, size_t abytes, const void *b, size_t bbytes) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + bbytes && b0 < a0 + abytes;
}

int validate(const gemm_problem_t *p) {
    if (!p) return fail(GEMM_EINVAL, "problem pointer is NULL");
    if (!mode_known(p->mode)) return fail(GEMM_EINVAL, "unknown mode %d", p->mode);
    if (p->flags != 0) return fail(GEMM_EINVAL, "flags must be 0 (got %d)", p->flags);
    if (p->m < 0 || p->n < 0 || p->k < 0)
        return fail(GEMM_EINVAL, "negative dimension (m=%lld n=%lld k=%lld)", (long long)p->m,
                    (long long)p->n, (long long)p->k);
    if (p->m > kMaxDim || p->n > kMaxDim || p->k > kMaxDim)
        return fail(GEMM_EUNSUPPORTED, "dimension above 2^30");
    if (p->lda < std::max<int64_t>(1, p->k))
        return fail(GEMM_EINVAL, "lda=%lld < max(1,k=%lld)", (long long)p->lda, (long long)p->k);
    if (p->ldb < std::max<int64_t>(1, p->n))
        return fail(GEMM_EINVAL, "ldb=%lld < max(1,n=%lld)", (long long)p->ldb, (long long)p->n);
    if (p->ldc < std::max<int64_t>(1, p->n))
        return fail(GEMM_EINVAL, "ldc=%lld < max(1,n=%lld)", (long long)p->ldc, (long long)p->n);
    const bool out_empty = p->m == 0 || p->n == 0;
    if (!out_empty && !p->C) return fail(GEMM_EINVAL, "C is NULL for a non-empty output");
    if (!out_empty && p->k > 0 && (!p->A || !p->B))
        return fail(GEMM_EINVAL, "A or B is NULL for a non-empty product");
    if (p->mode == GEMM_MODE_F8E4M3) {
        if (!(std::isfinite(p->scale_a) && p->scale_a > 0.f && std::isfinite(p->scale_b) &&
              p->scale_b > 0.f))
            return fail(GEMM_EINVAL, "FP8 scales must be finite and > 0");
    }
    if (!out_empty && p->k > 0) {
        const size_t es = elem_size(p->mode);
        const size_t cbytes = ((size_t)(p->m - 1) * p->ldc + p->n) * 4;
        const size_t abytes = ((size_t)(p->m - 1) * p->lda + p->k) * es;
        const size_t bbytes = ((size_t)(p->k - 1) * p->ldb + p->n) * es;
        if (overlaps(p->C, cbytes, p->A, abytes) || overlaps(p->C, cbytes, p->B, bbytes))
            return fail(GEMM_EINVAL, "C overlaps A or B");
    }
    return GEMM_OK;
}

int num_cus() {
    static int cached = -1;
    if (cached > 0) return cached;
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
        cached = n;
    else
        return 256;
    return cached;
}

const KernelCfg *configs(int mode, int *count) {
    if (mode == GEMM_MODE_F32) return f32_configs(count);
    if (mode == GEMM_MODE_F64) return f64_configs(count);
    if (mode == GEMM_MODE_C32) return c32_configs(count);
    return lp_configs(mode, count);
}

int split_grain(int mode) {
    switch (mode) {
        case GEMM_MODE_BF16:
        case GEMM_MODE_F16: return 64;
        case GEMM_MODE_F8E4M3: return 128;
        default: return 32;
    }
}

static bool vec_ok(const void *ptr, int64_t ld, size_t es) {
    return ((uintptr_t)ptr % 16 == 0) && ((ld * (int64_t)es) % 16 == 0);
}

Launch make_launch(const gemm_problem_t &p, const KernelCfg &kc, int split) {
    Launch L;
    TileProblem &P = L.P;
    memset(&P, 0, sizeof(P));
    const size_t es = elem_size(p.mode);
    P.A = p.A;
    P.B = p.B;
    P.C = p.C;
    P.lda = p.lda;
    P.ldb = p.ldb;
    P.ldc = p.ldc;
    P.m = (int32_t)p.m;
    P.n = P.nb = (int32_t)p.n;
    P.k = (int32_t)p.k;
    P.tiles_m = (int32_t)((p.m + kc.bm - 1) / kc.bm);
    P.tiles_n = (int32_t)((p.n + kc.bn - 1) / kc.bn);
    // Split-K boundaries are placed on multiples of the mode's largest k-tile
    // (`grain`), so every configuration of a mode splits k at the same places
    // and sums each element in the same order.
    const int grain = split_grain(p.mode);
    const int ngr = (int)((p.k + grain - 1) / grain);
    split = std::max(1, std::min(split, std::max(1, ngr)));
    int per = (ngr + split - 1) / split;
    if (per < 1) per = 1;
    split = std::max(1, (ngr + per - 1) / per);
    P.splits = split;
    P.kt_per_split = per * (grain / kc.bk);
    P.vec = (vec_ok(p.A, p.lda, es) ? 1 : 0) | (vec_ok(p.B, p.ldb, es) ? 2 : 0) |
            (vec_ok(p.C, p.ldc, 4) ? 4 : 0);
    P.scale = p.mode == GEMM_MODE_F8E4M3 ? p.scale_a * p.scale_b : 1.f;
    P.split_stride = ((int64_t)p.m * p.n + 3) / 4 * 4;
    L.splits = split;
    // a fused configuration adds up to `fused` k ranges in its workgroup
    const bool slabs = split > 1 && split > kc.fused;
    L.nwg = P.tiles_m * P.tiles_n * (kc.fused ? (split + kc.fused - 1) / kc.fused : split);
    L.ws_bytes = slabs ? (int64_t)split * P.split_stride * 4 : 0;
    return L;
}

// The pre-split path's operand copies have an inner dimension of 2 k16 (k
// rounded up to 16), which the tile indexes with 32-bit integers, k-tiles past
// the end included.
bool presplit_shape_ok(int64_t n, int64_t k) {
    const int64_t k16 = (k + 15) / 16 * 16;
    return n % 8 == 0 && n >= 8 && 3 * k16 <= (int64_t)INT32_MAX;
}

bool cfg_eligible(const gemm_problem_t &p, const KernelCfg &kc) {
    if (kc.presplit) return presplit_shape_ok(p.n, p.k);
    if (kc.chunk == 0) return true;
    const int64_t c = kc.chunk;
    return p.k % c == 0 && p.n % c == 0 && p.n >= c && p.lda % c == 0 && p.ldb % c == 0 &&
           (uintptr_t)p.A % 16 == 0 && (uintptr_t)p.B % 16 == 0;
}

// The packed copies (pack.hip) that let a chunked configuration run a problem
// whose operands are not whole 16-byte chunks.
struct PackPlan {
    bool a = false, b = false;       // which operands are copied
    int64_t a_ld = 0, b_ld = 0;      // row strides of the copies, in elements
    int64_t a_bytes = 0, b_bytes = 0;
    int64_t bytes() const { return a_bytes + b_bytes; }
};

// Bytes of the operand copies of the pre-split path (A's hi and lo parts, then
// B's, each 256-byte aligned).
static int64_t presplit_bytes(const gemm_problem_t &p, int64_t *b_off) {
    const int64_t k16 = (p.k + 15) / 16 * 16, n8 = (p.n + 7) / 8 * 8;
    const int64_t a = ((int64_t)p.m * 2 * k16 * 2 + 255) / 256 * 256;
    *b_off = a;
    return a + ((int64_t)2 * k16 * n8 * 2 + 255) / 256 * 256;
}

// The copies pay where each packed element is used often enough and the
// register-staged tile is far behind: for the 16- and 8-bit forms and
// split-BF16x3 from about 192 rows and columns and 512 k (without copies /
// best tile on copies, us: BF16 185x7863x7863 138 / 89, 369x3931x3931 55 / 42,
// 185x1965x3931 24 / 26, 123x3931x3931 25 / 30; E4M3 369x7863x7863 121 / 64;
// split 369x3931x3931 91 / 68; above 2048 rows and columns up to 2.4 times),
// for FP32, whose 4-byte direct loads already take any shape, from about 2048
// (0.9 to 1.09 times below).  Within the range the tuner's points decide.  The
// lines are where the points turn to 192, 512 and 2048, so that all shapes of
// a point run the kind of launch that was measured for it (with lines at 512
// and 2048 themselves the points' shapes just below ran without copies, and
// 537 x 3262 x 5706 on their choice took 264 us; 64 on the choice measured
// with copies).
// Bounded, since the workspace is kept: larger copies are left to the
// register-staged tiles.
static int64_t pack_min(int mode) { return mode == GEMM_MODE_F32 ? 1774 : 157; }
static const int64_t kPackMaxBytes = (int64_t)512 << 20;

static bool pack_plan(const gemm_problem_t &p, const KernelCfg &kc, PackPlan *plan) {
    if ((kc.chunk == 0 && !kc.presplit) || cfg_eligible(p, kc)) return false;
    if (p.m < pack_min(p.mode) || p.n < pack_min(p.mode) || p.k < 444) return false;
    if (kc.presplit) {
        // ragged n: the pre-split copies are made all the same, B's rows
        // padded to eight columns (enqueue_plain makes and sizes them)
        int64_t b_off = 0;
        *plan = PackPlan();
        return presplit_shape_ok((p.n + 7) / 8 * 8, p.k) && presplit_bytes(p, &b_off) <= kPackMaxBytes;
    }
    const int64_t c = kc.chunk, es = 16 / c;
    PackPlan q;
    q.a = p.k % c || p.lda % c || (uintptr_t)p.A % 16;
    q.b = p.n % c || p.ldb % c || (uintptr_t)p.B % 16;
    q.a_ld = q.a ? (p.k + c - 1) / c * c : p.lda;
    q.b_ld = q.b ? (p.n + c - 1) / c * c : p.ldb;
    if (q.a) q.a_bytes = (p.m * q.a_ld * es + 255) / 256 * 256;
    if (q.b) q.b_bytes = (p.k * q.b_ld * es + 255) / 256 * 256;
    if (q.bytes() > kPackMaxBytes) return false;
    *plan = q;
    return true;
}

bool cfg_runs(const gemm_problem_t &p, const KernelCfg &kc) {
    PackPlan plan;
    return cfg_eligible(p, kc) || pack_plan(p, kc, &plan);
}

int effective_cfg(const gemm_problem_t &p, int cfg) {
    int count = 0;
    const KernelCfg *t = configs(p.mode, &count);
    if (!t || cfg < 0 || cfg >= count || cfg_eligible(p, t[cfg])) return cfg;
    // the any-shape form with as many waves along k (every fused configuration
    // has one, so its k ranges stay in one launch without slabs, whatever the
    // operands' strides and alignment; 0: the register-staged tile)
    for (int c = 0; c < count; ++c)
        if (t[c].chunk == 0 && !t[c].presplit && t[c].fused == t[cfg].fused && t[c].bm == t[cfg].bm &&
            t[c].bn == t[cfg].bn)
            return c;
    // no such tile size: the smallest larger one
    int best = 0;
    for (int c = 0; c < count; ++c) {
        const int area = t[c].bm * t[c].bn;
        if (t[c].chunk == 0 && !t[c].presplit && !t[c].fused && area >= t[cfg].bm * t[cfg].bn &&
            area < t[best].bm * t[best].bn)
            best = c;
    }
    return best;
}

// The tuner's choice for a product that cannot run it (chunked or pre-split,
// and no operand copies): the split factor stands, since it fixes the bits, and
// an any-shape configuration takes its place.  The one of the same tile size is
// often far behind: large tiles suit 16-byte direct loads, small ones loads
// through registers.  So up to three tiles per mode, by the 64x64 tiles and k
// ranges per CU (smaller tiles fill more of the chip): `few` below `limit`,
// `most` from 20 on, else `many`; others in the 16- and 8-bit modes where the
// rows start at changing places against the 16-byte boundaries.  Over 200 ragged
// and 210 misaligned products (m, n 16..16384, k 64..16384) they are within 1.04
// to 1.05 of the best any-shape configuration at the same factor (geometric
// means by mode; E4M3 misaligned 1.10), the tile of the same size 1.1 (FP32,
// split-BF16x3) to 2.6.  us, same size / now: E4M3 700x8191x8191 786 / 422,
// 1500x1500x1501 79 / 38, BF16 700x8191x8191 943 / 497, split-BF16x3
// 1500x1500x1501 131 / 74.
struct AnyShape {
    int few, many, most;
    double limit;
};
static const AnyShape kAnyF32 = {24, 25, 25, 20.0}, kAnySplit = {5, 2, 2, 6.0};
static const AnyShape kAny16 = {6, 13, 13, 4.0}, kAny16Ragged = {24, 4, 13, 4.0};
static const AnyShape kAny8 = {6, 11, 11, 4.0}, kAny8Ragged = {14, 4, 11, 3.0};

static int any_shape_cfg(const gemm_problem_t &p, const KernelCfg *t, int cfg, int split) {
    const int same = effective_cfg(p, cfg);
    const int64_t es = (int64_t)elem_size(p.mode);
    const bool ragged_rows = p.lda * es % 16 || p.ldb * es % 16;
    const Launch L = make_launch(p, t[cfg], split);
    // slabs where the choice itself needs none: at most what gemm_plain_noalloc
    // holds, so that it serves the same products
    const bool slabs_fit = L.ws_bytes > 0 || L.splits * L.P.split_stride * 4 <= GEMM_NOALLOC_SCRATCH_BYTES;
    if (t[cfg].fused && !ragged_rows && p.mode != GEMM_MODE_F32_SPLIT_BF16X3) {
        // small tiles with waves along k: the same with loads through registers,
        // but for few of them over a long k, whose ranges are better spread over
        // more workgroups, slabs included (us, in the workgroup / on slabs: FP32
        // 375x320x7552 47 / 30, 338x512x7808 on 176 tiles 47.5 / 50.8; BF16
        // 18x320x2528 18.1 / 11.5, 31x32x512 7.5 / 7.5; E4M3 70x704x4256 21.6 / 12.8)
        const bool few = 2 * (int64_t)L.P.tiles_m * L.P.tiles_n <= num_cus();
        if (!few || p.k < (p.mode == GEMM_MODE_F32 ? 2048 : 1024) || !slabs_fit) return same;
        if (p.mode != GEMM_MODE_F32) return kAny16.few;
        int c = same;
        while (t[c - 1].bm == t[c].bm && t[c - 1].bn == t[c].bn && t[c - 1].chunk == 0) --c;   // fewest waves
        return c;
    }
    if (!slabs_fit) return same;
    const AnyShape &a = p.mode == GEMM_MODE_F32 ? kAnyF32
                        : p.mode == GEMM_MODE_F32_SPLIT_BF16X3 ? kAnySplit
                        : p.mode == GEMM_MODE_F8E4M3 ? (ragged_rows ? kAny8Ragged : kAny8)
                                                     : (ragged_rows ? kAny16Ragged : kAny16);
    const double per_cu = (double)((p.m + 63) / 64) * (double)((p.n + 63) / 64) * L.splits / num_cus();
    return per_cu < a.limit ? a.few : per_cu < 20.0 ? a.many : a.most;
}

void plain_choose(const gemm_problem_t &p, bool pack, int *cfg, int *split) {
    tuner_choose(p.mode, p.m, p.n, p.k, cfg, split);
    int count = 0;
    const KernelCfg *t = configs(p.mode, &count);
    if (!t || *cfg < 0 || *cfg >= count || p.m == 0 || p.n == 0 || p.k == 0) return;
    PackPlan plan;
    if (!cfg_eligible(p, t[*cfg]) && !(pack && pack_plan(p, t[*cfg], &plan))) *cfg = any_shape_cfg(p, t, *cfg, *split);
}

int64_t plain_ws_bytes(const gemm_problem_t &p, int cfg, int split, bool pack) {
    int count = 0;
    const KernelCfg *t = configs(p.mode, &count);
    if (!t || cfg < 0 || cfg >= count || p.m == 0 || p.n == 0 || p.k == 0) return 0;
    PackPlan plan;
    const KernelCfg &kc = pack && pack_plan(p, t[cfg], &plan) ? t[cfg] : t[effective_cfg(p, cfg)];
    int64_t ws = (make_launch(p, kc, split).ws_bytes + 255) / 256 * 256 + plan.bytes();
    if (kc.presplit) {
        int64_t b_off = 0;
        ws += presplit_bytes(p, &b_off);
    }
    return ws;
}

int64_t plain_ws_reported(const gemm_problem_t &p, int cfg, int split, bool pack) {
    const int64_t used = plain_ws_bytes(p, cfg, split, pack);
    int count = 0;
    const KernelCfg *t = configs(p.mode, &count);
    if (!t || cfg < 0 || cfg >= count || p.m == 0 || p.n == 0 || p.k == 0) return used;
    const Launch L = make_launch(p, t[cfg], split);
    const int64_t slabs = L.splits > 1 ? L.splits * L.P.split_stride * 4 : 0;
    return std::max(used, (std::min(slabs, GEMM_NOALLOC_SCRATCH_BYTES) + 255) / 256 * 256);
}

int enqueue_plain(const gemm_problem_t &p, int cfg, int split, void *ws, hipStream_t s, bool pack) {
    if (p.m == 0 || p.n == 0) return GEMM_OK;
    if (p.k == 0) {
        MG_HIP(launch_fill_zero(p.C, p.ldc, (int)p.m, (int)p.n, s));
        return GEMM_OK;
    }
    int count = 0;
    const KernelCfg *t = configs(p.mode, &count);
    if (!t || count == 0) return fail(GEMM_EUNSUPPORTED, "mode %d has no kernels", p.mode);
    if (cfg < 0 || cfg >= count) return fail(GEMM_EINVAL, "config %d out of range [0,%d)", cfg, count);
    PackPlan plan;
    pack = pack && pack_plan(p, t[cfg], &plan);
    if (!pack) cfg = effective_cfg(p, cfg);
    Launch L = make_launch(p, t[cfg], split);
    const bool slabs = L.ws_bytes > 0;
    if (slabs) {
        if (!ws) return fail(GEMM_EINTERNAL, "split-K workspace missing");
        L.P.C = static_cast<float *>(ws);
    }
    if (t[cfg].presplit) {
        // the operands' hi and lo parts after the split-K slabs: 2 k16 elements
        // per row of A and rows of B
        if (!ws) return fail(GEMM_EINTERNAL, "pre-split workspace missing");
        int64_t b_off = 0;
        presplit_bytes(p, &b_off);
        uint8_t *base = static_cast<uint8_t *>(ws) + (L.ws_bytes + 255) / 256 * 256;
        uint16_t *Ap = reinterpret_cast<uint16_t *>(base);
        uint16_t *Bp = reinterpret_cast<uint16_t *>(base + b_off);
        const int64_t k16 = (p.k + 15) / 16 * 16;
        MG_HIP(launch_presplit(static_cast<const float *>(p.A), p.lda, static_cast<const float *>(p.B), p.ldb,
                               (int)p.m, (int)p.n, (int)p.k, Ap, Bp, s));
        L.P.A = Ap;
        L.P.B = Bp;
        L.P.lda = 2 * k16;
        L.P.ldb = L.P.nb = (int32_t)((p.n + 7) / 8 * 8);
        L.P.k = (int32_t)(2 * k16);
        L.P.vec = 3;
    } else if (pack) {
        // the operands' copies after the split-K slabs
        if (!ws) return fail(GEMM_EINTERNAL, "packing workspace missing");
        const int64_t es = (int64_t)elem_size(p.mode);
        uint8_t *Ap = static_cast<uint8_t *>(ws) + (L.ws_bytes + 255) / 256 * 256;
        uint8_t *Bp = Ap + plan.a_bytes;
        MG_HIP(launch_pack(p.A, p.lda * es, p.m, p.k * es, plan.a ? Ap : nullptr, p.B, p.ldb * es, p.k, p.n * es,
                           plan.b ? Bp : nullptr, s));
        if (plan.a) L.P.A = Ap;
        if (plan.b) {
            L.P.B = Bp;
            L.P.nb = (int32_t)plan.b_ld;
        }
        L.P.lda = plan.a_ld;
        L.P.ldb = plan.b_ld;
        L.P.vec |= 3;
    }
    MG_HIP(t[cfg].plain(L.P, L.nwg, s));
    if (slabs)
        MG_HIP(launch_splitk_reduce(static_cast<const float *>(ws), L.P.split_stride, L.splits, L.P.scale,
                                    p.C, p.ldc, (int)p.m, (int)p.n, s));
    return GEMM_OK;
}

// ---------------------------------------------------------------------------
// Device buffers.

int DevBuf::ensure(size_t need, hipStream_t s, bool room) {
    if (need <= bytes) return GEMM_OK;
    const size_t last = bytes;
    if (ptr) {
        MG_HIP(hipStreamSynchronize(s));
        MG_HIP(hipFree(ptr));
        ptr = nullptr;
        bytes = 0;
    }
    const size_t roomy = room ? std::max(need, std::min(2 * last, last + ((size_t)256 << 20))) : need;
    for (size_t want : {roomy, need}) {
        const size_t sz = (std::max<size_t>(want, 1 << 20) + 255) / 256 * 256;
        if (hipMalloc(&ptr, sz) == hipSuccess) {
            bytes = sz;
            return GEMM_OK;
        }
        ptr = nullptr;
        (void)hipGetLastError();
    }
    return fail(GEMM_ENOMEM, "workspace allocation of %zu bytes failed", need);
}

void DevBuf::release() {
    if (ptr) (void)hipFree(ptr);
    ptr = nullptr;
    bytes = 0;
}

struct StreamWs {
    std::mutex mu;   // held by the caller from stream_workspace() to the enqueue of the work that uses a slot
    DevBuf slot[4];
};
static std::mutex g_ws_mu;
static std::map<std::pair<int, hipStream_t>, StreamWs *> g_ws;

static StreamWs *stream_ws(hipStream_t s) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> lk(g_ws_mu);
    StreamWs *&w = g_ws[{dev, s}];
    if (!w) w = new StreamWs();
    return w;
}

// ---------------------------------------------------------------------------
// Buffers of captured work.  A graph may be replayed at any time and on any
// stream, unordered with the calls made on the stream it was captured on, which
// use, grow and free that stream's workspace.  So captured work gets buffers of
// its own: one per (capture, stream, slot), larger ones beside the smaller ones
// that earlier nodes hold, each owned by a user object of the graph, which HIP
// releases with the last of the graph and the executables made of it.
struct CaptureBuf {
    unsigned long long capture;
    hipStream_t stream;
    int slot;              // kStagingSlot: pinned host memory, one per call
    void *ptr = nullptr;
    size_t bytes = 0;
    std::atomic<bool> gone{false};
};
static const int kStagingSlot = -1;
static std::mutex g_capture_mu;
static std::vector<CaptureBuf *> g_capture;
static std::atomic<int> g_capture_gone{0};

// The user object's destructor: it may make no HIP call, so the buffer is only
// marked; free_gone() frees it.
static void capture_gone(void *p) {
    static_cast<CaptureBuf *>(p)->gone.store(true);
    g_capture_gone.fetch_add(1);
}

// Allocating and freeing while a stream is being captured (both enqueue
// nothing) need the relaxed mode.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Free the buffers of graphs that are gone (hipFree waits for the device, so
// for a last replay that is still running).
static void free_gone() {
    if (g_capture_gone.load() == 0) return;
    std::vector<CaptureBuf *> dead;
    {
        std::lock_guard<std::mutex> lk(g_capture_mu);
        const auto keep = std::partition(g_capture.begin(), g_capture.end(), [](CaptureBuf *b) { return !b->gone.load(); });
        dead.assign(keep, g_capture.end());
        g_capture.erase(keep, g_capture.end());
        g_capture_gone.fetch_sub((int)dead.size());
    }
    RelaxedCapture relaxed;
    for (CaptureBuf *b : dead) {
        (void)(b->slot == kStagingSlot ? hipHostFree(b->ptr) : hipFree(b->ptr));
        delete b;
    }
}

static bool capture_of(hipStream_t s, unsigned long long *id, hipGraph_t *graph) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamGetCaptureInfo_v2(s, &st, id, graph, nullptr, nullptr) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusActive;
}

static int capture_buffer(unsigned long long id, hipGraph_t graph, hipStream_t s, int slot, size_t need, void **out) {
    if (slot != kStagingSlot) {
        std::lock_guard<std::mutex> lk(g_capture_mu);
        for (CaptureBuf *b : g_capture)
            if (!b->gone.load() && b->capture == id && b->stream == s && b->slot == slot && b->bytes >= need) {
                *out = b->ptr;
                return GEMM_OK;
            }
    }
    RelaxedCapture relaxed;
    std::unique_ptr<CaptureBuf> b(new CaptureBuf());
    b->capture = id;
    b->stream = s;
    b->slot = slot;
    b->bytes = (std::max<size_t>(need, 65536) + 255) / 256 * 256;
    const hipError_t e = slot == kStagingSlot ? hipHostMalloc(&b->ptr, b->bytes, hipHostMallocDefault)
                                              : hipMalloc(&b->ptr, b->bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(GEMM_ENOMEM, "workspace allocation of %zu bytes failed", b->bytes);
    }
    hipUserObject_t owner = nullptr;
    if (hipUserObjectCreate(&owner, b.get(), capture_gone, 1, hipUserObjectNoDestructorSync) != hipSuccess) {
        (void)hipGetLastError();
        (void)(slot == kStagingSlot ? hipHostFree(b->ptr) : hipFree(b->ptr));
        return fail(GEMM_EHIP, "a captured graph's workspace has no owner");
    }
    // from here on the owner's release marks the buffer and free_gone() frees it
    void *ptr = b->ptr;
    {
        std::lock_guard<std::mutex> lk(g_capture_mu);
        g_capture.push_back(b.release());
    }
    if (hipGraphRetainUserObject(graph, owner, 1, hipGraphUserObjectMove) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipUserObjectRelease(owner, 1);
        return fail(GEMM_EHIP, "a captured graph does not take its workspace");
    }
    *out = ptr;
    return GEMM_OK;
}

int stream_workspace(hipStream_t s, int slot, size_t need, void **out) {
    free_gone();
    unsigned long long id = 0;
    hipGraph_t graph = nullptr;
    if (capture_of(s, &id, &graph)) return capture_buffer(id, graph, s, slot, need, out);
    DevBuf &b = stream_ws(s)->slot[slot];
    const int rc = b.ensure(need, s, true);
    *out = b.ptr;
    return rc;
}

int capture_staging(hipStream_t s, size_t bytes, void **out) {
    *out = nullptr;
    unsigned long long id = 0;
    hipGraph_t graph = nullptr;
    return capture_of(s, &id, &graph) ? capture_buffer(id, graph, s, kStagingSlot, bytes, out) : GEMM_OK;
}

std::unique_lock<std::mutex> lock_stream_workspaces(hipStream_t s) {
    return std::unique_lock<std::mutex>(stream_ws(s)->mu);
}

// ---------------------------------------------------------------------------
// Scratch of gemm_plain_noalloc: split-K partial slabs and split-BF16x3
// operand copies of at most GEMM_NOALLOC_SCRATCH_BYTES, in a device array that
// every GPU the library runs on holds until the process ends.  Host code never
// passes the array's name to a kernel or a copy (on the host it is only a
// stand-in for the symbol): it uses the per-device address
// hipGetSymbolAddress returns, taken once per device with that device
// current.
static __device__ __align__(256) uint8_t scratch[GEMM_NOALLOC_SCRATCH_BYTES];

static const int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxScratchDevices];

int noalloc_scratch(void **out) {
    *out = nullptr;
    int dev = 0;
    MG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxScratchDevices) return fail(GEMM_EUNSUPPORTED, "device %d: at most %d devices", dev,
                                                          kMaxScratchDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return fail(GEMM_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return GEMM_OK;
}

}  // namespace mg

using namespace mg;

extern "C" {

const char *gemm_last_error(void) { return t_err; }

int gemm_version(void) { return 1; }

uint64_t gemm_now_ns(void) { return now_ns(); }

int gemm_num_configs(int32_t mode) {
    clear_error();
    if (mode < 0 || mode >= GEMM_NUM_KERNEL_FAMILIES) return fail(GEMM_EINVAL, "unknown mode %d", mode);
    int count = 0;
    configs(mode, &count);
    return count;
}

int gemm_config_info(int32_t mode, int32_t cfg, int32_t info[6]) {
    clear_error();
    if (mode < 0 || mode >= GEMM_NUM_KERNEL_FAMILIES) return fail(GEMM_EINVAL, "unknown mode %d", mode);
    if (!info) return fail(GEMM_EINVAL, "info is NULL");
    int count = 0;
    const KernelCfg *t = configs(mode, &count);
    if (cfg < 0 || cfg >= count) return fail(GEMM_EINVAL, "config %d out of range", cfg);
    info[0] = t[cfg].bm;
    info[1] = t[cfg].bn;
    info[2] = t[cfg].bk;
    info[3] = t[cfg].waves;
    info[4] = t[cfg].lds_bytes;
    info[5] = t[cfg].mfma_k;
    return GEMM_OK;
}

int gemm_config_chunk(int32_t mode, int32_t cfg) {
    clear_error();
    if (mode < 0 || mode >= GEMM_NUM_KERNEL_FAMILIES) return fail(GEMM_EINVAL, "unknown mode %d", mode);
    int count = 0;
    const KernelCfg *t = configs(mode, &count);
    if (cfg < 0 || cfg >= count) return fail(GEMM_EINVAL, "config %d out of range", cfg);
    return t[cfg].chunk;
}

// `chosen`: (cfg, split) is plain_choose's, not the caller's.
static int plain_common(const gemm_problem_t *p, int cfg, int split, bool chosen, void *stream) {
    int rc = validate(p);
    if (rc != GEMM_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (p->m == 0 || p->n == 0) return GEMM_OK;
    void *ws = nullptr;
    bool pack = true;
    std::unique_lock<std::mutex> ws_lock;
    if (p->k > 0) {
        int count = 0;
        configs(p->mode, &count);
        if (count == 0) return fail(GEMM_EUNSUPPORTED, "mode %d has no kernels", p->mode);
        int64_t need = plain_ws_bytes(*p, cfg, split, true);
        if (need > 0) {
            ws_lock = lock_stream_workspaces(s);
            rc = stream_workspace(s, 0, (size_t)need, &ws);
            if (rc == GEMM_ENOMEM) {
                // without the packed copies (same bits)
                if (chosen) plain_choose(*p, false, &cfg, &split);
                const int64_t less = plain_ws_bytes(*p, cfg, split, false);
                if (less < need) {
                    clear_error();
                    pack = false;
                    rc = less > 0 ? stream_workspace(s, 0, (size_t)less, &ws) : GEMM_OK;
                }
            }
            if (rc != GEMM_OK) return rc;
        }
    }
    return enqueue_plain(*p, cfg, split, ws, s, pack);
}

int gemm_plain(const gemm_problem_t *p, void *stream) {
    clear_error();
    int rc = validate(p);
    if (rc != GEMM_OK) return rc;
    int cfg = 0, split = 1;
    plain_choose(*p, true, &cfg, &split);
    return plain_common(p, cfg, split, true, stream);
}

int gemm_plain_cfg(const gemm_problem_t *p, int32_t cfg, int32_t split_k, void *stream) {
    clear_error();
    if (split_k < 1) return fail(GEMM_EINVAL, "split_k must be >= 1");
    int rc = validate(p);
    if (rc != GEMM_OK) return rc;
    int count = 0;
    configs(p->mode, &count);
    if (count == 0) return fail(GEMM_EUNSUPPORTED, "mode %d has no kernels", p->mode);
    if (cfg < 0 || cfg >= count) return fail(GEMM_EINVAL, "config %d out of range [0,%d)", cfg, count);
    return plain_common(p, cfg, split_k, false, stream);
}

int gemm_plain_workspace_bytes(const gemm_problem_t *p, uint64_t *bytes_out) {
    clear_error();
    if (!bytes_out) return fail(GEMM_EINVAL, "bytes_out is NULL");
    *bytes_out = 0;
    int rc = validate(p);
    if (rc != GEMM_OK) return rc;
    if (p->m == 0 || p->n == 0 || p->k == 0) return GEMM_OK;
    int cfg = 0, split = 1;
    plain_choose(*p, true, &cfg, &split);
    *bytes_out = (uint64_t)plain_ws_reported(*p, cfg, split, true);
    return GEMM_OK;
}

// Allocation-free plain product: gemm_plain's plan, with its workspace in a
// fixed device array instead of the per-stream library workspace.
int gemm_plain_noalloc(const gemm_problem_t *p, void *stream) {
    clear_error();
    int rc = validate(p);
    if (rc != GEMM_OK) return rc;
    if (p->m == 0 || p->n == 0) return GEMM_OK;
    int cfg = 0, split = 1;
    void *ws = nullptr;
    bool pack = true;
    if (p->k > 0) {
        int count = 0;
        configs(p->mode, &count);
        if (count == 0) return fail(GEMM_EUNSUPPORTED, "mode %d has no kernels", p->mode);
        plain_choose(*p, true, &cfg, &split);
        int64_t need = plain_ws_bytes(*p, cfg, split, true);
        if (need > GEMM_NOALLOC_SCRATCH_BYTES) {
            // without the packed copies (same bits)
            pack = false;
            plain_choose(*p, false, &cfg, &split);
            need = plain_ws_bytes(*p, cfg, split, false);
        }
        if (need > GEMM_NOALLOC_SCRATCH_BYTES)
            return fail(GEMM_EINVAL,
                        "this product needs %lld bytes of workspace; gemm_plain_noalloc holds at most %lld "
                        "(use gemm_plain)",
                        (long long)need, (long long)GEMM_NOALLOC_SCRATCH_BYTES);
        if (need > 0) {
            rc = noalloc_scratch(&ws);
            if (rc != GEMM_OK) return rc;
        }
    }
    return enqueue_plain(*p, cfg, split, ws, (hipStream_t)stream, pack);
}

int gemm_convert_f32(const float *x, int64_t count, int32_t to_mode, void *out, void *stream) {
    clear_error();
    if (count < 0) return fail(GEMM_EINVAL, "negative count");
    if (to_mode != GEMM_MODE_BF16 && to_mode != GEMM_MODE_F16)
        return fail(GEMM_EINVAL, "to_mode must be BF16 or F16");
    if (count == 0) return GEMM_OK;
    if (!x || !out) return fail(GEMM_EINVAL, "NULL buffer");
    if (overlaps(x, (size_t)count * 4, out, (size_t)count * 2)) return fail(GEMM_EINVAL, "buffers overlap");
    MG_HIP(launch_convert_f32(x, count, to_mode, out, (hipStream_t)stream));
    return GEMM_OK;
}

int gemm_quantize_e4m3(const float *x, int64_t count, uint8_t *q, float *scale_out, void *stream) {
    clear_error();
    if (count < 0) return fail(GEMM_EINVAL, "negative count");
    if (!scale_out) return fail(GEMM_EINVAL, "scale_out is NULL");
    if (count > 0 && (!x || !q)) return fail(GEMM_EINVAL, "NULL buffer");
    if (count > 0 && overlaps(x, (size_t)count * 4, q, (size_t)count)) return fail(GEMM_EINVAL, "buffers overlap");
    hipStream_t s = (hipStream_t)stream;
    std::unique_lock<std::mutex> ws_lock = lock_stream_workspaces(s);
    void *ws = nullptr;
    int rc = stream_workspace(s, 2, 4096, &ws);
    if (rc != GEMM_OK) return rc;
    MG_HIP(launch_quantize_e4m3(x, count, q, scale_out, static_cast<uint32_t *>(ws), s));
    return GEMM_OK;
}

int gemm_errnorm(const float *C, int64_t ldc, const double *R, int64_t ldr, int64_t m, int64_t n,
                 double *out3, void *stream) {
    clear_error();
    if (m < 0 || n < 0) return fail(GEMM_EINVAL, "negative dimension");
    if (!out3) return fail(GEMM_EINVAL, "out3 is NULL");
    if (ldc < std::max<int64_t>(1, n) || ldr < std::max<int64_t>(1, n)) return fail(GEMM_EINVAL, "bad ld");
    if (m * n > 0 && (!C || !R)) return fail(GEMM_EINVAL, "NULL matrix");
    hipStream_t s = (hipStream_t)stream;
    const int nparts = 2048;
    std::unique_lock<std::mutex> ws_lock = lock_stream_workspaces(s);
    void *ws = nullptr;
    int rc = stream_workspace(s, 2, 4096 + (size_t)nparts * 3 * sizeof(double), &ws);
    if (rc != GEMM_OK) return rc;
    double *partials = reinterpret_cast<double *>(static_cast<char *>(ws) + 4096);
    MG_HIP(launch_errnorm(C, ldc, R, ldr, m, n, out3, partials, nparts, s));
    return GEMM_OK;
}

}  // extern "C"
