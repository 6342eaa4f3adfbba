// Host runtime and C ABI of liblogfx (declared in include/logfx.h).
//
// Validates arguments and masks, picks the exact arithmetic path, owns the
// per-context device scratch (per-tile partial sums, counters, the global
// statistics) and enqueues   pass 1 -> finalize -> pass 2   on the caller's
// stream.  No compute happens on the host.
#include "logfx.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <iterator>
#include <sstream>
#include <string>
#include <type_traits>
#include <vector>

#include "logfx_gate.h"
#include "logfx_internal.h"

using namespace logfx;

namespace {

thread_local std::string g_thread_error;

// Output rows per wave strip of each pass (tiles are kTileWaves strips wide).
struct TileCfg {
    int rows1 = 64;  // pass 1
    int rows2 = 64;  // pass 2
    bool set1 = false, set2 = false;       // by an option or the environment: every call takes them
    bool tuned1 = false, tuned2 = false;   // by the tuner: calls of this class do (call_class)
    int tuned_class = -1;
    // other calls take the heights prepare works out
};

// LOGFX_TILE="rows1,rows2" overrides the defaults (used by the tuner and
// the tests).
TileCfg tile_cfg_from_env() {
    TileCfg t;
    if (const char *s = std::getenv("LOGFX_TILE")) {
        int a, b;
        if (std::sscanf(s, "%d,%d", &a, &b) == 2 && a >= 1 && a <= 1024 && b >= 1 && b <= 1024)
            t.rows1 = a, t.rows2 = b, t.set1 = t.set2 = true;
    }
    return t;
}

}  // namespace

struct logfx_ctx {
    int device = 0;
    std::string err;
    TileCfg tiles;
    bool persistent = false;         // batches: one resident grid walks all tiles
    bool graph = true;               // batches: replay a captured hipGraph
    bool store_z = true;             // pass 1 stores the strengths, pass 2 reads them
    bool pack_log = true;            // integer LoG on packed 16-bit sums where it applies
    void *zmap = nullptr;            // strengths of the images of a call
    long long zcap = 0;              // bytes
    uint8_t *cmap = nullptr;         // 0/1 maps between the levels of a median cascade
    long long ccap = 0;              // bytes
    // device scratch
    unsigned long long *partials = nullptr;   // [cap1][kTileSums]
    long long *counts1 = nullptr;    // [cap1][2]
    int *counts2 = nullptr;          // [cap2][2]
    DevStats *stats = nullptr;       // [capn]
    ImageJob *jobs = nullptr;        // [capn] batch image table
    int *owner1 = nullptr;           // [cap1] image of each pass-1 tile
    int *owner2 = nullptr;           // [cap2] image of each pass-2 tile
    long long cap1 = 0, cap2 = 0, capn = 0;
    // pinned host memory: report mirrors and the staging of the batch tables
    DevStats *h_stats = nullptr;
    int *h_counts2 = nullptr;
    long long h_capn = 0, h_cap2 = 0;
    // batch tables: two pinned staging sets used in turn (a set is rewritten
    // only after the upload from it, two uploads back, has finished), and the
    // tables the device buffers hold, so that an unchanged batch uploads
    // nothing
    struct Staging {
        ImageJob *jobs = nullptr;
        int *own1 = nullptr, *own2 = nullptr;
        long long capn = 0, cap1 = 0, cap2 = 0;
        hipEvent_t done = nullptr;   // the last upload from this set
    } stage[2];
    int stage_next = 0;
    std::vector<ImageJob> tab_jobs;
    std::vector<int> tab_own1, tab_own2;
    bool tab_valid = false;          // jobs / owner1 / owner2 hold tab_*
    // captured batch graph and the launch arguments it was captured with
    hipStream_t capture = nullptr;
    hipGraph_t g = nullptr;
    hipGraphExec_t gexec = nullptr;
    std::vector<unsigned char> gkey;
    // kernel timing: 4 events per timed call (start, after pass 1, after
    // finalize, after pass 2; a graph replay records start and end only),
    // reused across accumulations
    bool timing = false;
    std::vector<hipEvent_t> events;
    long long timed_calls = 0;
    std::vector<char> timed_graph;   // per timed call: 1 if it was a graph replay
    int alloc_count = 0;
    int fail_alloc_at = -1;          // test hook: LOGFX_FAIL_ALLOC=n fails the n-th allocation
    // device address of the static scratch of logfx_extract_noalloc on this
    // context's device (looked up in logfx_create), or the lookup's error
    void *noalloc = nullptr;
    std::string noalloc_err;
    // smoothing gate: parameters, optimiser state and workspaces
    struct Gate {
        float *theta = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;   // [kNParam]
        uint16_t *wbf = nullptr;        // bfloat16 copy of theta
        bool loaded = false;
        long long step = 0;             // AdamW steps since the parameters were set
        uint16_t *act = nullptr, *gact = nullptr;   // activations / gradients of a batch
        float *small = nullptr;         // gap [B][32], logits [B]
        float *partial = nullptr;       // partial weight gradients
        long long capB = 0;
        unsigned long long *cells = nullptr;   // [capImg][2][cells^2]
        uint16_t *feats = nullptr;             // [capImg][3][cells^2]
        int *flags = nullptr;                  // [capImg]
        long long capImg = 0;
        float *h_logits = nullptr;             // pinned report mirrors
        int *h_flags = nullptr;
        long long h_cap = 0, h_capf = 0;
    } gate;
};

namespace {

// LOGFX_LOG=1 (read once): one line per call and every error on stderr.
bool log_on() {
    static const bool on = [] {
        const char *v = std::getenv("LOGFX_LOG");
        return v && *v && std::strcmp(v, "0") != 0;
    }();
    return on;
}

void log_line(const char *fmt, ...) {
    if (!log_on()) return;
    char buf[768];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    std::fprintf(stderr, "[liblogfx] %s\n", buf);
}

int set_err(logfx_ctx *ctx, int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (ctx) ctx->err = buf;
    else g_thread_error = buf;
    log_line("error %d: %s", code, buf);
    return code;
}

int hip_err(logfx_ctx *ctx, hipError_t e, const char *what) {
    return set_err(ctx, e == hipErrorOutOfMemory ? LOGFX_ENOMEM : LOGFX_EDEVICE, "%s: %s", what,
                   hipGetErrorString(e));
}

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) ok = hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard() {
        int cur;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

template <class T>
int dev_alloc(logfx_ctx *ctx, T **p, size_t count) {
    ++ctx->alloc_count;
    if (ctx->fail_alloc_at > 0 && ctx->alloc_count == ctx->fail_alloc_at)
        return set_err(ctx, LOGFX_ENOMEM, "device allocation %d failed (LOGFX_FAIL_ALLOC)",
                       ctx->alloc_count);
    hipError_t e = hipMalloc((void **)p, count * sizeof(T));
    if (e != hipSuccess) {
        *p = nullptr;
        return hip_err(ctx, e, "hipMalloc");
    }
    return LOGFX_OK;
}

// Replace a device buffer by one of `count` elements.
template <class T>
int realloc_dev(logfx_ctx *ctx, T *&p, long long count) {
    (void)hipFree(p);
    p = nullptr;
    return dev_alloc(ctx, &p, (size_t)count);
}

// Grow-only per-context scratch for n1 pass-1 tiles, n2 pass-2 tiles and
// nimg images.
int ensure_scratch(logfx_ctx *ctx, long long n1, long long n2, long long nimg) {
    int rc;
    if (n1 > ctx->cap1 || n2 > ctx->cap2 || nimg > ctx->capn) ctx->tab_valid = false;
    if (n1 > ctx->cap1) {
        ctx->cap1 = 0;
        if ((rc = realloc_dev(ctx, ctx->partials, n1 * kTileSums)) != LOGFX_OK ||
            (rc = realloc_dev(ctx, ctx->counts1, n1 * 2)) != LOGFX_OK ||
            (rc = realloc_dev(ctx, ctx->owner1, n1)) != LOGFX_OK)
            return rc;
        ctx->cap1 = n1;
    }
    if (n2 > ctx->cap2) {
        ctx->cap2 = 0;
        if ((rc = realloc_dev(ctx, ctx->counts2, n2 * 2)) != LOGFX_OK ||
            (rc = realloc_dev(ctx, ctx->owner2, n2)) != LOGFX_OK)
            return rc;
        ctx->cap2 = n2;
    }
    if (nimg > ctx->capn) {
        ctx->capn = 0;
        if ((rc = realloc_dev(ctx, ctx->stats, nimg)) != LOGFX_OK ||
            (rc = realloc_dev(ctx, ctx->jobs, nimg)) != LOGFX_OK)
            return rc;
        ctx->capn = nimg;
    }
    return LOGFX_OK;
}

template <class T>
int grow_host(logfx_ctx *ctx, T *&p, long long &cap, long long n) {
    if (n <= cap) return LOGFX_OK;
    if (p) (void)hipHostFree(p);
    p = nullptr;
    cap = 0;
    hipError_t e = hipHostMalloc((void **)&p, (size_t)n * sizeof(T), hipHostMallocDefault);
    if (e != hipSuccess) return hip_err(ctx, e, "hipHostMalloc");
    cap = n;
    return LOGFX_OK;
}

int ensure_host(logfx_ctx *ctx, long long nimg, long long n2) {
    int rc;
    if ((rc = grow_host(ctx, ctx->h_stats, ctx->h_capn, nimg)) != LOGFX_OK) return rc;
    return grow_host(ctx, ctx->h_counts2, ctx->h_cap2, n2 * 2);
}

// Gate parameters, optimiser state and the bfloat16 copy (allocated once).
int ensure_gate_params(logfx_ctx *ctx) {
    auto &G = ctx->gate;
    if (G.theta) return LOGFX_OK;
    int rc;
    if ((rc = realloc_dev(ctx, G.m, gate::kNParam)) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.v, gate::kNParam)) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.grad, gate::kNParam)) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.wbf, gate::kWbfElems)) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.theta, gate::kNParam)) != LOGFX_OK)
        return rc;
    // the padding of the forward weight layout stays zero
    const hipError_t e = hipMemset(G.wbf, 0, sizeof(uint16_t) * gate::kWbfElems);
    if (e != hipSuccess) {
        (void)hipFree(G.theta);
        G.theta = nullptr;
        return hip_err(ctx, e, "gate parameters");
    }
    return LOGFX_OK;
}

// Grow-only workspace of the network for batches of up to B samples.
int ensure_gate_batch(logfx_ctx *ctx, long long B) {
    auto &G = ctx->gate;
    if (B <= G.capB) return LOGFX_OK;
    G.capB = 0;
    int rc;
    if ((rc = realloc_dev(ctx, G.act, gate::act_elems((int)B))) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.gact, gate::gact_elems((int)B))) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.small, B * (gate::kC3 + 1))) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.partial, gate::partial_elems((int)B))) != LOGFX_OK)
        return rc;
    G.capB = B;
    return LOGFX_OK;
}

// Grow-only per-image gate scratch: cell sums, features, decisions.
int ensure_gate_images(logfx_ctx *ctx, long long n) {
    auto &G = ctx->gate;
    if (n <= G.capImg) return LOGFX_OK;
    G.capImg = 0;
    int rc;
    if ((rc = realloc_dev(ctx, G.cells, n * 2 * gate::kCellCount)) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.feats, n * gate::kFeatC * gate::kCellCount)) != LOGFX_OK ||
        (rc = realloc_dev(ctx, G.flags, n)) != LOGFX_OK)
        return rc;
    G.capImg = n;
    return LOGFX_OK;
}

// The network's buffers for a batch of B <= capB samples.
gate::NetBuffers net_buffers(logfx_ctx *ctx, int B, const uint16_t *feats, const int *idx, const float *labels,
                             float *grad, float *loss) {
    using namespace gate;
    auto &G = ctx->gate;
    NetBuffers n;
    std::memset(&n, 0, sizeof n);
    const long long e1 = (long long)B * kC1 * kH1 * kH1, e2 = (long long)B * kC2 * kH2 * kH2;
    n.x0 = feats;
    n.idx = idx;
    n.w = G.wbf;
    n.theta = G.theta;
    n.a1 = G.act;
    n.a2 = G.act + e1;
    n.a3 = G.act + e1 + e2;
    n.g1 = G.gact;
    n.g2 = G.gact + e1;
    n.gap = G.small;
    n.logits = G.small + (long long)B * kC3;
    n.labels = labels;
    n.grad = grad ? grad : G.grad;
    n.loss = loss;
    n.partial = G.partial;
    n.B = B;
    return n;
}

// Events of timed call number `call` (created on first use).
int timing_events(logfx_ctx *ctx, long long call, hipEvent_t *ev) {
    while ((long long)ctx->events.size() < 4 * (call + 1)) {
        hipEvent_t e;
        hipError_t r = hipEventCreate(&e);
        if (r != hipSuccess) return hip_err(ctx, r, "hipEventCreate");
        ctx->events.push_back(e);
    }
    for (int i = 0; i < 4; ++i) ev[i] = ctx->events[4 * call + i];
    return LOGFX_OK;
}

// ------------------------------------------------------------ mask analysis
struct MaskInfo {
    int size = 0, radius = 0;
    double unit = 1.0;       // grid unit u: taps = k * u
    double k[81];            // integer taps (exact in double)
    double sumabs = 0.0;     // sum |k|
    double sumpos = 0.0;     // sum of the positive k
    double maxabs = 0.0;     // max |k|
};

int analyze_mask(logfx_ctx *ctx, const logfx_mask &m, int which, MaskInfo &mi, bool inexact_ok) {
    if (!m.taps) return set_err(ctx, LOGFX_EINVAL, "mask %d: taps is NULL", which);
    if (m.size < 1 || m.size % 2 == 0 || m.size > 15)
        return set_err(ctx, LOGFX_EINVAL, "mask %d: size %d is not odd in 1..15", which, m.size);
    if (m.size > 2 * kMaxRadius + 1)
        return set_err(ctx, LOGFX_EUNSUPPORTED, "mask %d: size %d > 9 is not supported", which,
                       m.size);
    const int s = m.size, r = s / 2;
    mi.size = s;
    mi.radius = r;
    int min_lsb = 1 << 30;
    bool any = false;
    for (int i = 0; i < s * s; ++i) {
        const float t = m.taps[i];
        if (!std::isfinite(t)) return set_err(ctx, LOGFX_EINVAL, "mask %d: tap %d not finite", which, i);
        if (t == 0.0f) continue;
        any = true;
        int e;
        const double fr = std::frexp((double)t, &e);          // |fr| in [0.5, 1)
        long long M = (long long)std::ldexp(std::fabs(fr), 24);  // 24-bit integer mantissa
        int b = 0;
        while (!(M & 1)) M >>= 1, ++b;
        const int lsb = e - 24 + b;
        if (lsb < min_lsb) min_lsb = lsb;
    }
    mi.unit = any ? std::ldexp(1.0, min_lsb) : 1.0;
    mi.sumabs = mi.sumpos = mi.maxabs = 0.0;
    for (int i = 0; i < s * s; ++i) {
        const double k = (double)m.taps[i] / mi.unit;
        if (std::fabs(k) > 9007199254740992.0 && !inexact_ok)
            return set_err(ctx, LOGFX_EUNSUPPORTED,
                           "mask %d: taps span too many binary orders for exact sums "
                           "(LOGFX_ALLOW_INEXACT runs them with rounded sums)", which);
        mi.k[i] = k;
        mi.sumabs += std::fabs(k);
        if (k > 0.0) mi.sumpos += k;
        if (std::fabs(k) > mi.maxabs) mi.maxabs = std::fabs(k);
    }
    // the eight symmetries of the square grid
    for (int y = 0; y < s; ++y)
        for (int x = 0; x < s; ++x) {
            const float v = m.taps[y * s + x];
            const int ys[4] = {y, s - 1 - y, x, s - 1 - x};
            const int xs[4] = {s - 1 - x, x, y, y};
            for (int q = 0; q < 4; ++q)
                if (m.taps[ys[q] * s + xs[q]] != v)
                    return set_err(ctx, LOGFX_EUNSUPPORTED,
                                   "mask %d is not symmetric under the square's symmetries "
                                   "(asymmetric masks are not supported)", which);
        }
    return LOGFX_OK;
}

// Bound on a crossing's strength in grid units: the largest difference of the
// responses of two of the five pixels, maxpix times the positive part of the
// difference of the mask and the mask moved by their offset, summed.
double strength_bound(const MaskInfo &mi, double maxpix) {
    static const int off[6][2] = {{0, 1}, {1, 0}, {1, 1}, {1, -1}, {0, 2}, {2, 0}};
    const int s = mi.size;
    auto tap = [&](int y, int x) { return y < 0 || y >= s || x < 0 || x >= s ? 0.0 : mi.k[y * s + x]; };
    double most = 0.0;
    for (const auto &o : off) {   // the opposite offsets give the same by symmetry of the mask
        double sum = 0.0;
        for (int y = -2; y < s + 2; ++y)
            for (int x = -2; x < s + 2; ++x) sum += std::max(0.0, tap(y, x) - tap(y - o[0], x - o[1]));
        most = std::max(most, sum);
    }
    return most * maxpix;
}

struct Plan {
    MaskInfo mi[2];
    int order[2];         // kernel mask slot -> user mask index
    int ra = 1, rb = 1;   // kernel radii, ra <= rb
    int path = LOGFX_PATH_INT32;   // the class the caller is told (bound 2^30 on sum|k| maxpix)
    bool i32 = true;      // the LoG runs in exact int32 (every call of that class, and more: check_all)
    double maxpix = 255.0;
    bool std5 = false;    // the 5x5 first deviation stage is on (std5_max >= 0)
    bool inexact = false; // the FP64 LoG sums round (LOGFX_ALLOW_INEXACT)
    bool pk_ok = false;   // the integer LoG may run on packed 16-bit sums (kP1Packed)
    bool mat_ok = false;  // the LoG may run on the matrix cores (kP1Matrix), with these taps
    MatTable mat;
    int ncas = 0;         // further median levels (applied where the first level is)
    int cas[3] = {0, 0, 0};
    int region = 0;       // > 0: the gate decides per region x region square (single images)
    int gx = 1, gy = 1;   // regions per row / per column (powers of two)
    int lgx = 0, lgy = 0; // their log2
};

// The taps of the packed integer LoG (layout in logfx_internal.h): entry
// v(d, c) takes the tap of its orbit, which is the mask's tap at row offset
// d and column offset c (the masks are D4-symmetric).  False when one of
// them, the centre's aside, does not fit int16.
bool fill_packed_taps(const Plan &pl, OrbitTapsI &t) {
    for (int slot = 0; slot < 2; ++slot) {
        const MaskInfo &mi = pl.mi[pl.order[slot]];
        const int r = mi.radius, s = mi.size;
        auto tap = [&](int d, int c) -> double { return d > r || c > r ? 0.0 : mi.k[(r + d) * s + (r + c)]; };
        for (int d = 0; d <= kMaxRadius; ++d)
            for (int m = 0; m < kPkPerRow; ++m) {
                const bool none = m == 0 && d % 2 == 0;
                const double lo = none ? 0.0 : m == 0 ? tap(d, 0) : tap(d, 2 * m - 1);
                const double hi = none ? 0.0 : m == 0 ? tap(d + 1, 0) : tap(d, 2 * m);
                if (!(lo >= -32768.0 && lo <= 32767.0 && hi >= -32768.0 && hi <= 32767.0)) return false;
                t.pk[slot][d * kPkPerRow + m] =
                    (unsigned)(uint16_t)(int16_t)lo | (unsigned)(uint16_t)(int16_t)hi << 16;
            }
    }
    return true;
}

// The taps of the matrix form (layout in logfx_internal.h).  False when one
// does not fit two signed bytes (-32896 .. 32639), or twice that in the
// centre row, whose entry comes twice.
bool fill_matrix_taps(const Plan &pl, MatTable &t) {
    std::memset(&t, 0, sizeof t);
    for (int slot = 0; slot < 2; ++slot) {
        const MaskInfo &mi = pl.mi[pl.order[slot]];
        const int r = mi.radius, s = mi.size;
        for (int e = 0; e < kMatEntries; ++e) {
            const int dy = e < 2 ? 0 : e - 1;
            const bool again = e == 1;   // the centre row's second entry
            if (dy > r) continue;
            for (int dx = -r; dx <= r; ++dx) {
                const double k = mi.k[(r + dy) * s + (r + dx)];
                double v = k;
                if (dy == 0) {
                    v = std::min(std::max(k, -32896.0), 32639.0);
                    if (again) v = k - v;
                }
                if (!(v >= -32896.0 && v <= 32639.0)) return false;
                const int n = (int)v, hi = (n + 128) >> 8, lo = n - 256 * hi;
                unsigned char *row = t.b + ((slot * kMatEntries + e) * 2) * kMatRow + 23 + dx;
                row[0] = (unsigned char)(signed char)hi;
                row[kMatRow] = (unsigned char)(signed char)lo;
            }
        }
    }
    return true;
}

int check_all(logfx_ctx *ctx, const logfx_image *img, const logfx_params *p, Plan &pl) {
    if (!img || !p) return set_err(ctx, LOGFX_EINVAL, "image or params is NULL");
    if (!img->data) return set_err(ctx, LOGFX_EINVAL, "image data is NULL");
    if (img->dtype != LOGFX_U8 && img->dtype != LOGFX_U16)
        return set_err(ctx, LOGFX_EINVAL, "unknown dtype %d", img->dtype);
    if (img->height < 1 || img->width < 1)
        return set_err(ctx, LOGFX_EINVAL, "image is empty (%lld x %lld)", (long long)img->height,
                       (long long)img->width);
    if (img->pitch < img->width)
        return set_err(ctx, LOGFX_EINVAL, "pitch %lld < width %lld", (long long)img->pitch,
                       (long long)img->width);
    const int full = img->dtype == LOGFX_U8 ? 8 : 16;
    const int bits = img->bits == 0 ? full : img->bits;
    if (bits < 1 || bits > full) return set_err(ctx, LOGFX_EINVAL, "bits %d not in 1..%d", bits, full);
    if (!(p->zc_thresh >= 0.0) || !std::isfinite(p->zc_thresh))
        return set_err(ctx, LOGFX_EINVAL, "zc_thresh must be finite and >= 0");
    if (p->std_mode != LOGFX_STD_REL && p->std_mode != LOGFX_STD_ABS)
        return set_err(ctx, LOGFX_EINVAL, "unknown std_mode %d", p->std_mode);
    if (!(p->std_k >= 0.0) || !std::isfinite(p->std_k))
        return set_err(ctx, LOGFX_EINVAL, "std_k must be finite and >= 0");
    if (std::isnan(p->std5_max)) return set_err(ctx, LOGFX_EINVAL, "std5_max is NaN");
    if (p->smooth != LOGFX_SMOOTH_NEVER && p->smooth != LOGFX_SMOOTH_ALWAYS && p->smooth != LOGFX_SMOOTH_GATE)
        return set_err(ctx, LOGFX_EINVAL, "unknown smooth mode %d", p->smooth);
    if (p->median_size != 3 && p->median_size != 5)
        return set_err(ctx, LOGFX_EINVAL, "median_size %d is not 3 or 5", p->median_size);
    if ((p->flags & ~LOGFX_ALLOW_INEXACT) != 0)
        return set_err(ctx, LOGFX_EINVAL, "flags 0x%x: only LOGFX_ALLOW_INEXACT is defined", p->flags);
    for (int i = 0; i < 3; ++i) {
        const int m = p->median_cascade[i];
        if (m != 0 && m != 3 && m != 5)
            return set_err(ctx, LOGFX_EINVAL, "median_cascade[%d] = %d is not 0, 3 or 5", i, m);
        if (m != 0 && i > 0 && p->median_cascade[i - 1] == 0)
            return set_err(ctx, LOGFX_EINVAL, "median_cascade[%d] follows a 0", i);
    }
    int rc;
    for (int j = 0; j < 2; ++j)
        if ((rc = analyze_mask(ctx, p->mask[j], j, pl.mi[j], (p->flags & LOGFX_ALLOW_INEXACT) != 0)) != LOGFX_OK)
            return rc;
    pl.maxpix = std::ldexp(1.0, bits) - 1.0;
    bool int_ok = true, f64_ok = true;
    pl.i32 = true;
    for (int j = 0; j < 2; ++j) {
        const double bound = pl.mi[j].sumabs * pl.maxpix;
        // int32 arithmetic needs every response and partial sum below 2^30 in
        // magnitude (pixels are >= 0, so they lie between minus the sum of
        // the negative taps and the sum of the positive ones, times maxpix;
        // the crossing test adds two of them) and their range, the strength,
        // below 2^31.  A zero-sum mask has half of sum|k| on either side, so
        // it runs in int32 up to twice the bound the class is named by, 12-bit
        // images with the default masks among them (2000^2, whole call with
        // its report: 108 us in FP64, 86 in int32).
        const double pos = pl.mi[j].sumpos * pl.maxpix;
        if (!(pos < 1073741824.0 && bound - pos < 1073741824.0 && bound < 2147483648.0 &&
              pl.mi[j].maxabs < 8388608.0))
            pl.i32 = false;
        // and kFoldRows squares of strengths below 2^64 - 2^48 (those of 2^30 always are)
        if (pl.i32 && bound >= 1073741824.0) {
            const double z = strength_bound(pl.mi[j], pl.maxpix);
            if (!(z * z * kFoldRows < 18446462598732840960.0)) pl.i32 = false;
        }
        if (!(bound < 1073741824.0 && pl.mi[j].maxabs < 8388608.0)) int_ok = false;  // 2^30, 2^23
        if (!(bound < 4503599627370496.0)) f64_ok = false;                              // 2^52
    }
    pl.inexact = !f64_ok;
    if (!f64_ok && !(p->flags & LOGFX_ALLOW_INEXACT))
        return set_err(ctx, LOGFX_EUNSUPPORTED,
                       "mask taps are not exactly summable for %d-bit pixels "
                       "(sum|k| * (2^bits - 1) must stay below 2^52; LOGFX_ALLOW_INEXACT runs "
                       "them with rounded sums)", bits);
    pl.path = int_ok ? LOGFX_PATH_INT32 : LOGFX_PATH_FP64;
    const int r0 = pl.mi[0].radius, r1 = pl.mi[1].radius;
    if (r0 <= r1) pl.order[0] = 0, pl.order[1] = 1;
    else pl.order[0] = 1, pl.order[1] = 0;
    pl.ra = std::max(1, std::min(r0, r1));
    pl.rb = std::max(1, std::max(r0, r1));
    // packed 16-bit sums: every v(d, c) (at most four pixels) below 2^15
    OrbitTapsI probe;
    pl.pk_ok = pl.i32 && pl.maxpix <= 8191.0 && fill_packed_taps(pl, probe);
    pl.mat_ok = !pl.inexact && fill_matrix_taps(pl, pl.mat);
    pl.std5 = p->std5_max >= 0.0;
    if (p->gate_region < 0) return set_err(ctx, LOGFX_EINVAL, "gate_region %d < 0", p->gate_region);
    pl.region = 0;
    pl.gx = pl.gy = 1;
    pl.lgx = pl.lgy = 0;
    if (p->gate_region > 0) {
        const long long R = p->gate_region;
        if (p->smooth != LOGFX_SMOOTH_GATE)
            return set_err(ctx, LOGFX_EINVAL, "gate_region needs smooth = LOGFX_SMOOTH_GATE");
        if (p->median_cascade[0] != 0)
            return set_err(ctx, LOGFX_EINVAL, "gate_region and median_cascade cannot be combined");
        if (R < 128 || R >= (1 << 23))
            return set_err(ctx, LOGFX_EINVAL, "gate_region %lld not in 128 .. 2^23 - 1", R);
        if (img->height % R != 0 || img->width % R != 0)
            return set_err(ctx, LOGFX_EINVAL, "a %lld x %lld image is not a whole number of %lld-pixel regions",
                           (long long)img->height, (long long)img->width, R);
        const long long gx = img->width / R, gy = img->height / R;
        if ((gx & (gx - 1)) != 0 || (gy & (gy - 1)) != 0)
            return set_err(ctx, LOGFX_EINVAL, "%lld x %lld regions: both counts must be powers of two", gy, gx);
        if (gx * gy > LOGFX_GATE_MAX_BATCH)
            return set_err(ctx, LOGFX_EINVAL, "%lld regions: at most %d", gx * gy, LOGFX_GATE_MAX_BATCH);
        pl.region = (int)R;
        pl.gx = (int)gx;
        pl.gy = (int)gy;
        while ((1LL << pl.lgx) < gx) ++pl.lgx;
        while ((1LL << pl.lgy) < gy) ++pl.lgy;
    }
    pl.ncas = 0;
    if (p->smooth != LOGFX_SMOOTH_NEVER)
        while (pl.ncas < 3 && p->median_cascade[pl.ncas] != 0) {
            pl.cas[pl.ncas] = p->median_cascade[pl.ncas];
            ++pl.ncas;
        }
    return LOGFX_OK;
}

template <class Taps, class V>
void fill_taps(const Plan &pl, Taps &t) {
    std::memset(&t, 0, sizeof t);
    for (int slot = 0; slot < 2; ++slot) {
        const MaskInfo &mi = pl.mi[pl.order[slot]];
        const int s = mi.size, r = mi.radius;
        for (int i = 0; i <= r; ++i)
            for (int j = 0; j <= i; ++j) t.k[slot][orbit_index(i, j)] = (V)mi.k[(r + i) * s + (r + j)];
    }
}

// The packed integer form runs when the plan allows it and the context
// does not turn it off (LOGFX_OPT_PACKED_LOG).
bool use_packed(const logfx_ctx *ctx, const Plan &pl) { return pl.pk_ok && ctx->pack_log; }

// The same of the matrix form, on the FP64 path.
bool use_matrix(const logfx_ctx *ctx, const Plan &pl) { return pl.mat_ok && !pl.i32 && ctx->pack_log; }

// Pass-1 strip height of the FP64 path where none was asked for.  Its sums of
// strengths round, strip by strip and tile by tile, in the same order in both
// forms, so the height follows the masks alone: an image's statistics are the
// same bits whichever form runs, in a batch and alone, and in
// logfx_extract_noalloc.  The matrix form works through blocks of 8 rows, the
// strip's and one above and below it: 62.
int fp64_rows(const Plan &pl) { return pl.mat_ok ? 62 : 64; }

// ------------------------------------------------------------ one call
// Tiling of one image in both passes.
struct ImageTiles {
    int tiles_x1, ntiles1, tiles_x2, ntiles2;
};

int check_sides(logfx_ctx *ctx, const logfx_image &img) {
    if (img.height >= (1LL << 30) || img.width >= (1LL << 30))
        return set_err(ctx, LOGFX_EUNSUPPORTED, "image sides must be below 2^30");
    return LOGFX_OK;
}

int tile_image(logfx_ctx *ctx, const logfx_image *img, const Plan &pl, bool storez, int rows1, int rows2,
               ImageTiles &t) {
    TileCfg c;
    c.rows1 = rows1;
    c.rows2 = rows2;
    const long long H = img->height, W = img->width;
    int rc;
    if ((rc = check_sides(ctx, *img)) != LOGFX_OK) return rc;
    const long long tw1 = tile_out_width(kHalo1);
    const long long tw2 = tile_out_width(storez ? (pl.std5 ? kHalo2Z5 : kHalo2Z) : kHalo2);
    const long long tx1 = (W + tw1 - 1) / tw1, ty1 = (H + c.rows1 - 1) / c.rows1;
    const long long tx2 = (W + tw2 - 1) / tw2, ty2 = (H + c.rows2 - 1) / c.rows2;
    if (tx1 * ty1 > (1LL << 30) || tx2 * ty2 > (1LL << 30))
        return set_err(ctx, LOGFX_EUNSUPPORTED, "image too large for one launch");
    if (pass1_lds_bytes(c.rows1, pl.rb) > 65536 || (!storez && lds_bytes(c.rows2, kHalo2, pl.rb) > 65536))
        return set_err(ctx, LOGFX_EUNSUPPORTED, "tile configuration exceeds 64 KiB of LDS");
    t.tiles_x1 = (int)tx1, t.ntiles1 = (int)(tx1 * ty1);
    t.tiles_x2 = (int)tx2, t.ntiles2 = (int)(tx2 * ty2);
    return LOGFX_OK;
}

// For an integer strength c and a threshold thr >= 0: c > thr <=> c > floor(thr).
int int_threshold(double thr) {
    const double f = std::floor(thr);
    return f >= 2147483647.0 ? 2147483647 : (int)f;
}

ImageDesc image_desc(const logfx_image *img) {
    ImageDesc d;
    d.data = img->data;
    d.H = img->height;
    d.W = img->width;
    d.pitch = img->pitch;
    d.dtype = img->dtype;
    return d;
}

// Image i of a launch: its descriptor, output, tiling, first tiles in the
// launch's tile lists and first element in the strength map.
ImageJob make_job(const logfx_image &img, const ImageTiles &t, uint8_t *out, long long zoff, int b1, int b2) {
    ImageJob j;
    std::memset(&j, 0, sizeof j);
    j.zoff = zoff;
    j.img = image_desc(&img);
    j.out = out;
    j.out_pitch = img.width;
    j.tiles_x1 = t.tiles_x1;
    j.tiles_x2 = t.tiles_x2;
    j.ntiles1 = t.ntiles1;
    j.ntiles2 = t.ntiles2;
    j.base1 = b1;
    j.base2 = b2;
    return j;
}

// Everything one call enqueues.
struct Call {
    Plan pl;
    Launch L;
    int n = 1;
    bool storez = false;   // pass 1 stores the strengths in ctx->zmap, pass 2 reads them
    long long px = 0;      // pixels of all images (when the strengths are stored)
    int rows1 = 64, rows2 = 64;   // strip heights of this call
    int cell_slots = 0, cell_rows = 0;   // LDS slots of pass 1's gate cell sums per tile
    std::vector<ImageTiles> tiles;
};

// LDS slots of the gate's per-tile cell sums for pass-1 strips of `rows`
// rows.  A tile's slot of cell (cy, cx) is (cy - its first cell row) x slots
// + (cx - its first cell column), so the slots must cover the span of cell
// indices one tile of tile_out_width(kHalo1) columns and `rows` rows reaches
// in any image -- with CX x CY cells across (kGateCells per region side),
// floor((n - 1) CX / W) + 2 columns for n columns, at most CX (images
// narrower than CX have empty cells between their columns' cells).
void cell_layout(int n, const logfx_image *imgs, const Plan &pl, int rows, long long &slots, long long &crows) {
    const long long CX = (long long)kGateCells * pl.gx, CY = (long long)kGateCells * pl.gy;
    const long long TW = tile_out_width(kHalo1);
    slots = crows = 1;
    for (int i = 0; i < n; ++i) {
        const long long W = imgs[i].width, H = imgs[i].height;
        slots = std::max(slots, std::min(CX, (TW - 1) * CX / W + 2));
        crows = std::max(crows, std::min(CY, (rows - 1) * CY / H + 2));
    }
}

// The tallest strips that calls take by themselves (pass 1 of the integer
// path, the same with the gate's cells, pass 2), and the pixels from which on
// they take these.
constexpr int kTall1 = 48, kTallCells = 62, kTall2 = 64;
constexpr long long kTallPixels = 1LL << 25;

long long call_pixels(int n, const logfx_image *imgs) {
    long long px = 0;
    for (int i = 0; i < n; ++i) px += (long long)imgs[i].height * imgs[i].width;
    return px;
}

// Calls that tuned heights hold for: of the tuned call's path, and within a
// factor of two of its size, which is what the best height depends on.
int call_class(const Plan &pl, int n, const logfx_image *imgs) {
    return 2 * std::ilogb((double)std::min(call_pixels(n, imgs), kTallPixels)) + pl.i32;
}

// Strip height for tiles `tw` columns wide, where none was asked for.  A
// workgroup takes about rows + halo row times, alone on its CU each half as
// long again (`alone`) as with others to fill its waits, so a call takes
// about (rows + halo) max(alone, tiles per CU, rounded up) of them: low strips
// where tall ones leave CUs idle, tall ones where the halo rows add up.
// Pass 1, measured: 512^2 34 us with 64 rows, 12 with 8; 2000^2 45 and 29
// with 24; 4000^2 68 with 61 and 64 with 32; pass 2: 512^2 14.7 and 8.4
// with 8, 2000^2 19.4 and 14.0 with 24, 6000^2 57 with 64 and 83 with 8.
// From 2^25 pixels on, the tallest is within 4 % of the best.  Batches of more
// than 64 images take it too: below that size they wait for the host's work on
// each image (100 of 131 x 257, whole call, 264 us with 64 rows and 261 with
// 12; 100 of 500 x 500, 268 and 286).
int strip_rows(int n, const logfx_image *imgs, long long tw, int most, int step, int halo, double alone) {
    constexpr int kCus = 256;
    if (n > 64 || call_pixels(n, imgs) >= kTallPixels) return most;
    int best = most;
    double cost = 1e300;
    for (int r = most; r >= std::min(most, 6); r -= step) {
        long long tiles = 0;
        for (int i = 0; i < n; ++i) tiles += ((imgs[i].width + tw - 1) / tw) * ((imgs[i].height + r - 1) / r);
        const double c = (r + halo) * std::max(alone, (double)((tiles + kCus - 1) / kCus));
        if (c < cost) cost = c, best = r;
    }
    return best;
}

// Words of the code plane, rounded up so that the plane of low bits after it
// is aligned.
long long zmap_words(long long px) { return (px + 63) / 64 * 64; }
// Device memory for the strengths of `px` pixels (ZMap); false if it cannot
// be had (the call then recomputes the strengths in pass 2).
bool ensure_zmap(logfx_ctx *ctx, long long px, bool i32) {
    const long long bytes = zmap_words(px) * (i32 ? 8 : 16);
    if (bytes <= ctx->zcap) return true;
    (void)hipFree(ctx->zmap);
    ctx->zmap = nullptr;
    ctx->zcap = 0;
    if (hipMalloc(&ctx->zmap, (size_t)bytes) != hipSuccess) {
        ctx->zmap = nullptr;
        (void)hipGetLastError();   // clear the sticky out-of-memory error
        return false;
    }
    ctx->zcap = bytes;
    return true;
}

// Validates the images against the parameters, tiles them and (for a batch)
// uploads the image table and tile owners.
int prepare(logfx_ctx *ctx, int n, const logfx_image *imgs, const logfx_params *p,
            uint8_t *const *outs, bool need_out, bool features, Call &c, hipStream_t s) {
    if (n < 1 || !imgs) return set_err(ctx, LOGFX_EINVAL, "no images");
    int rc = check_all(ctx, &imgs[0], p, c.pl);
    if (rc != LOGFX_OK) return rc;
    // every image, before any of their sizes is used
    const int bits0 = imgs[0].bits == 0 ? (imgs[0].dtype == LOGFX_U8 ? 8 : 16) : imgs[0].bits;
    for (int i = 0; i < n; ++i) {
        if (i > 0) {
            Plan tmp;
            if ((rc = check_all(ctx, &imgs[i], p, tmp)) != LOGFX_OK) return rc;
            const int bi = imgs[i].bits == 0 ? (imgs[i].dtype == LOGFX_U8 ? 8 : 16) : imgs[i].bits;
            if (imgs[i].dtype != imgs[0].dtype || bi != bits0)
                return set_err(ctx, LOGFX_EINVAL, "image %d: all images of a batch must share "
                                                  "dtype and bits", i);
        }
        if ((rc = check_sides(ctx, imgs[i])) != LOGFX_OK) return rc;
        if (need_out && (!outs || !outs[i])) return set_err(ctx, LOGFX_EINVAL, "output %d is NULL", i);
    }
    // Integer path: up to 48 rows, for which five workgroups' LDS fit a CU
    // (8192^2: 196 us with 48 rows, 213 with 64, 199 with 43).  With the
    // gate's cells, whose sums leave the tile at its end, the tallest that
    // four workgroups' allows (32 of 2048^2: 454 with 48, 449 with 61).
    const bool tuned = call_class(c.pl, n, imgs) == ctx->tiles.tuned_class;
    const bool keep1 = ctx->tiles.set1 || (ctx->tiles.tuned1 && tuned);
    const bool keep2 = ctx->tiles.set2 || (ctx->tiles.tuned2 && tuned);
    c.rows1 = keep1      ? ctx->tiles.rows1
              : c.pl.i32 ? strip_rows(n, imgs, tile_out_width(kHalo1), features ? kTallCells : kTall1, 4, 6, 1.7)
                         : fp64_rows(c.pl);
    if (features) {
        // pass 1 keeps a slot per (cell row, cell column) a tile spans in
        // LDS beside the tile (the matrix form: beside its rings and
        // responses, whichever form runs, so that both take one height):
        // lower the strip height where they would not fit in 64 KiB
        // together (only images of a few hundred pixels with cells of a
        // pixel or two come near it)
        const size_t mat = c.pl.mat_ok && !c.pl.i32 ? kMatLdsBytes : 0;
        long long slots = 1, crows = 1;
        for (; c.rows1 > 1; --c.rows1) {
            cell_layout(n, imgs, c.pl, c.rows1, slots, crows);
            if (std::max(mat, pass1_lds_bytes(c.rows1, c.pl.rb)) + 2 * sizeof(unsigned) * slots * crows <= 65536) break;
        }
        cell_layout(n, imgs, c.pl, c.rows1, slots, crows);
        c.cell_slots = (int)slots;
        c.cell_rows = (int)crows;
    }
    if (n > 1 && c.pl.region > 0) return set_err(ctx, LOGFX_EINVAL, "gate_region applies to single-image calls");
    // strengths are stored between the passes when the context allows it and
    // the memory for them can be had; the 5x5 first stage and the median
    // cascade are built on the stored strengths only, so they always ask
    // for them (and the cascade for a byte per pixel between its levels);
    // so is the per-region gate
    c.storez = false;
    const bool need_z = c.pl.std5 || c.pl.ncas > 0 || c.pl.region > 0;
    if (need_out && (ctx->store_z || need_z)) {
        const long long px = c.px = call_pixels(n, imgs);
        c.storez = ensure_zmap(ctx, px, c.pl.i32);
        if (!c.storez && need_z)
            return set_err(ctx, LOGFX_ENOMEM, "the 5x5 first deviation stage, the median cascade and the "
                                              "per-region gate need %lld bytes of device memory for the "
                                              "crossing strengths",
                           px * (c.pl.i32 ? 8 : 16));
        if (c.pl.ncas > 0 && px > ctx->ccap) {
            (void)hipFree(ctx->cmap);
            ctx->cmap = nullptr;
            ctx->ccap = 0;
            if (hipMalloc(&ctx->cmap, (size_t)px) != hipSuccess) {
                ctx->cmap = nullptr;
                (void)hipGetLastError();
                return set_err(ctx, LOGFX_ENOMEM, "the median cascade needs %lld bytes of device memory", px);
            }
            ctx->ccap = px;
        }
    }
    c.rows2 = keep2      ? ctx->tiles.rows2
              : c.storez ? strip_rows(n, imgs, tile_out_width(c.pl.std5 ? kHalo2Z5 : kHalo2Z), kTall2, 8, 4, 1.5)
                         : kTall2;
    c.n = n;
    c.tiles.resize(n);
    long long t1 = 0, t2 = 0;
    for (int i = 0; i < n; ++i) {
        if ((rc = tile_image(ctx, &imgs[i], c.pl, c.storez, c.rows1, c.rows2, c.tiles[i])) != LOGFX_OK) return rc;
        t1 += c.tiles[i].ntiles1;
        t2 += c.tiles[i].ntiles2;
    }
    if (t1 >= (1LL << 31) || t2 >= (1LL << 31))
        return set_err(ctx, LOGFX_EUNSUPPORTED, "too many tiles for one launch");
    if ((rc = ensure_scratch(ctx, t1, t2, n)) != LOGFX_OK) return rc;
    std::memset(&c.L, 0, sizeof c.L);
    c.L.nimg = n;
    c.L.total1 = (int)t1;
    c.L.total2 = (int)t2;
    long long zoff = 0;
    auto job = [&](int i, int b1, int b2) {
        const ImageJob j = make_job(imgs[i], c.tiles[i], outs ? outs[i] : nullptr, zoff, b1, b2);
        zoff += imgs[i].height * imgs[i].width;
        return j;
    };
    if (n == 1) {
        c.L.one = job(0, 0, 0);
        return LOGFX_OK;
    }
    // batch: the image table and the tile owners; uploaded on the call's
    // stream only when they differ from what the device buffers hold
    std::vector<ImageJob> jobs((size_t)n);
    std::vector<int> own1((size_t)t1), own2((size_t)t2);
    int b1 = 0, b2 = 0;
    for (int i = 0; i < n; ++i) {
        jobs[i] = job(i, b1, b2);
        for (int k = 0; k < c.tiles[i].ntiles1; ++k) own1[b1 + k] = i;
        for (int k = 0; k < c.tiles[i].ntiles2; ++k) own2[b2 + k] = i;
        b1 += c.tiles[i].ntiles1;
        b2 += c.tiles[i].ntiles2;
    }
    const bool same = ctx->tab_valid && ctx->tab_jobs.size() == jobs.size() && ctx->tab_own1 == own1 &&
                      ctx->tab_own2 == own2 &&
                      std::memcmp(ctx->tab_jobs.data(), jobs.data(), sizeof(ImageJob) * jobs.size()) == 0;
    if (!same) {
        auto &S = ctx->stage[ctx->stage_next];
        hipError_t e;
        if (S.done && (e = hipEventSynchronize(S.done)) != hipSuccess) return hip_err(ctx, e, "hipEventSynchronize");
        if ((rc = grow_host(ctx, S.jobs, S.capn, n)) != LOGFX_OK || (rc = grow_host(ctx, S.own1, S.cap1, t1)) != LOGFX_OK ||
            (rc = grow_host(ctx, S.own2, S.cap2, t2)) != LOGFX_OK)
            return rc;
        std::memcpy(S.jobs, jobs.data(), sizeof(ImageJob) * n);
        std::memcpy(S.own1, own1.data(), sizeof(int) * t1);
        std::memcpy(S.own2, own2.data(), sizeof(int) * t2);
        ctx->tab_valid = false;
        if ((e = hipMemcpyAsync(ctx->jobs, S.jobs, sizeof(ImageJob) * n, hipMemcpyHostToDevice, s)) != hipSuccess ||
            (e = hipMemcpyAsync(ctx->owner1, S.own1, sizeof(int) * t1, hipMemcpyHostToDevice, s)) != hipSuccess ||
            (e = hipMemcpyAsync(ctx->owner2, S.own2, sizeof(int) * t2, hipMemcpyHostToDevice, s)) != hipSuccess)
            return hip_err(ctx, e, "table upload");
        if (!S.done && (e = hipEventCreateWithFlags(&S.done, hipEventDisableTiming)) != hipSuccess)
            return hip_err(ctx, e, "hipEventCreate");
        if ((e = hipEventRecord(S.done, s)) != hipSuccess) return hip_err(ctx, e, "hipEventRecord");
        ctx->stage_next ^= 1;
        ctx->tab_jobs.swap(jobs);
        ctx->tab_own1.swap(own1);
        ctx->tab_own2.swap(own2);
        ctx->tab_valid = true;
    }
    c.L.jobs = ctx->jobs;
    c.L.owner1 = ctx->owner1;
    c.L.owner2 = ctx->owner2;
    return LOGFX_OK;
}

// The three launches of one call, built once so that a graph replay can
// compare them with the captured ones.
struct Launches {
    union {
        Pass1Args<OrbitTapsI> i;
        Pass1Args<OrbitTapsD> d;
    } p1;
    union {
        Pass2Args<OrbitTapsI> i;
        Pass2Args<OrbitTapsD> d;
    } p2;
    FinalizeArgs fin;
    bool fused;                    // pass 2 does the finalize
    int grid1, grid2;
    int ra, rb;
    bool i32;                      // exact int32 LoG, else FP64
    bool packed;                   // pass 1 on packed 16-bit sums (integer path)
    bool matrix;                   // pass 1 on the matrix cores (FP64 path), with these taps
    MatTable table;
    bool dbg;
    bool storez;
    // median cascade: further levels after pass 2 (pass 2 writes the
    // scratch map when their number is odd, so the last level ends in the
    // caller's outputs)
    int ncas;
    LevelArgs lev[3];
    int halo2;
    // smoothing gate
    bool features;                 // pass 1 sums the cells; the features are finished after it
    bool gated;                    // the network decides the median per image before pass 2
    unsigned long long *cells;
    uint16_t *feats;
    double maxval;
    gate::NetBuffers net;
    int *flags;
    uint8_t *decisions;            // optional copy of the decisions (logfx_gate)
    int nsets;                     // feature sets / decisions: images x regions
    int gx, gy;                    // regions per image row / column (1, 1: whole images)
};

// How far a call runs.
enum Until { UNTIL_PASS1 = 0, UNTIL_FEATURES = 1, UNTIL_DECISION = 2, UNTIL_OUTPUT = 3 };

template <class Taps, class V>
void fill_args(const Call &c, logfx_ctx *ctx, const logfx_params *p, double *const L[2],
               double *const Z[2], Pass1Args<Taps> &a1, Pass2Args<Taps> &a2, bool &dbg, bool packed) {
    std::memset(&a1, 0, sizeof a1);
    std::memset(&a2, 0, sizeof a2);
    a1.L = a2.L = c.L;
    fill_taps<Taps, V>(c.pl, a1.taps);
    fill_taps<Taps, V>(c.pl, a2.taps);
    if constexpr (std::is_same<Taps, OrbitTapsI>::value)
        if (packed) fill_packed_taps(c.pl, a1.taps);
    dbg = false;
    for (int slot = 0; slot < 2; ++slot) {
        const int u = c.pl.order[slot];
        a1.zc_thr[slot] = a2.zc_thr[slot] = p->zc_thresh / c.pl.mi[u].unit;
        a1.zc_thr_i[slot] = a2.zc_thr_i[slot] = int_threshold(a1.zc_thr[slot]);
        a1.unit[slot] = c.pl.mi[u].unit;
        a1.dbgL[slot] = L ? L[u] : nullptr;
        a1.dbgZ[slot] = Z ? Z[u] : nullptr;
        dbg = dbg || a1.dbgL[slot] || a1.dbgZ[slot];
    }
    a1.rows = c.rows1;
    a1.partials = ctx->partials;
    a1.counts = ctx->counts1;
    a2.rows = c.rows2;
    a2.stats = ctx->stats;
    a2.counts = ctx->counts2;
    a2.smooth = p->smooth != LOGFX_SMOOTH_NEVER;   // GATE without a gate falls back to ALWAYS
    if (c.storez) {
        // the split form where the strengths, at most sum|k| maxpix, are
        // exact integers of at most kZSplitBits bits
        ZMap &z = a1.z;
        int bits[2];
        for (int slot = 0; slot < 2; ++slot) {
            const MaskInfo &mi = c.pl.mi[c.pl.order[slot]];
            bits[slot] = std::ilogb(std::max(1.0, mi.sumabs * c.pl.maxpix)) + 1;
            z.shift[slot] = std::max(0, bits[slot] - 16);
        }
        z.split = !c.pl.inexact && std::max(bits[0], bits[1]) <= kZSplitBits;
        if (!z.split) z.shift[0] = z.shift[1] = 0;
        z.hi = ctx->zmap;
        z.lo = static_cast<char *>(ctx->zmap) + zmap_words(c.px) * 4;
        a2.z = z;
    }
    a2.median_size = p->median_size;
    a1.cells_lx = kGateCellsLog2 + c.pl.lgx;
    a1.cells_ly = kGateCellsLog2 + c.pl.lgy;
    a2.std5 = c.pl.std5 && c.storez;
    a2.zfloor = c.pl.inexact ? std::ldexp(1.0f, -120) : 0.0f;
    for (int slot = 0; slot < 2; ++slot) {
        const double t = a2.std5 ? p->std5_max / c.pl.mi[c.pl.order[slot]].unit : 0.0;
        a2.thr600[slot] = 600.0 * t * t;   // s5 > t <=> 25 sum z^2 - (sum z)^2 > 600 t^2 (t >= 0)
        const double zmax = c.pl.mi[c.pl.order[slot]].sumabs * c.pl.maxpix;
        a2.zscale[slot] = c.pl.inexact && zmax > 0.0 ? std::ldexp(1.0, std::min(0, 51 - std::ilogb(zmax))) : 1.0;
    }
}

hipError_t launch_all(const Launches &k, hipStream_t s, hipEvent_t *ev, int until) {
    hipError_t e;
    const bool i32 = k.i32;
    const int mode = (k.dbg ? kP1Maps : 0) | (k.features ? kP1Cells : 0) | (k.storez ? kP1StoreZ : 0) |
                     (k.matrix ? kP1Matrix : k.packed ? kP1Packed : 0);
    if (k.features && (e = gate::launch_zero_cells(k.cells, k.nsets, s)) != hipSuccess) return e;
    e = i32 ? launch_pass1_i(k.ra, k.rb, k.p1.i, mode, k.grid1, s)
            : launch_pass1_d(k.ra, k.rb, k.p1.d, k.table, mode, k.grid1, s);
    if (e != hipSuccess || until == UNTIL_PASS1) return e;
    if (until < UNTIL_OUTPUT) {   // the gate alone: no thresholds needed
        if ((e = gate::launch_finish_features(k.fin.L, k.cells, k.maxval, k.feats, k.gx, k.gy, s)) != hipSuccess) return e;
        if (until == UNTIL_FEATURES) return hipSuccess;
        return gate::launch_forward(k.net, s, k.flags, k.decisions);
    }
    if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
    if (!k.fused && (e = launch_finalize(k.fin, s)) != hipSuccess) return e;
    if (k.gated) {
        if ((e = gate::launch_finish_features(k.fin.L, k.cells, k.maxval, k.feats, k.gx, k.gy, s)) != hipSuccess ||
            (e = gate::launch_forward(k.net, s, k.flags, k.decisions)) != hipSuccess)
            return e;
    }
    if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
    if (k.storez) {
        e = i32 ? launch_pass2z_i(k.p2.i, k.grid2, s) : launch_pass2z_d(k.p2.d, k.grid2, s);
        for (int i = 0; i < k.ncas && e == hipSuccess; ++i) e = launch_median_level(k.lev[i], k.halo2, s);
        return e;
    }
    return i32 ? launch_pass2_i(k.ra, k.rb, k.p2.i, k.grid2, s)
               : launch_pass2_d(k.ra, k.rb, k.p2.d, k.grid2, s);
}

// Every cell of the gate's feature grid must hold fewer than 2^32 pixels.
int check_cells(logfx_ctx *ctx, int n, const logfx_image *imgs, const Plan &pl) {
    for (int i = 0; i < n; ++i) {
        const long long ch = (imgs[i].height / pl.gy + gate::kCells - 1) / gate::kCells;
        const long long cw = (imgs[i].width / pl.gx + gate::kCells - 1) / gate::kCells;
        if (ch * cw >= (1LL << 32))
            return set_err(ctx, LOGFX_EUNSUPPORTED, "image %d: gate cells of more than 2^32 pixels", i);
    }
    if (n > LOGFX_GATE_MAX_BATCH)
        return set_err(ctx, LOGFX_EUNSUPPORTED, "the gate takes at most %d images per call", LOGFX_GATE_MAX_BATCH);
    return LOGFX_OK;
}

// gate: 0 none, 1 features only (into feats), 2 features + network
// (decisions in the context's flags).
int build_launches(logfx_ctx *ctx, const Call &c, const logfx_params *p, double *const L[2],
                   double *const Z[2], Launches &k, int gate = 0, uint16_t *feats = nullptr) {
    std::memset(&k, 0, sizeof k);
    k.i32 = c.pl.i32;
    k.ra = c.pl.ra;
    k.rb = c.pl.rb;
    k.storez = c.storez;
    k.packed = use_packed(ctx, c.pl);
    if (k.i32) fill_args<OrbitTapsI, int>(c, ctx, p, L, Z, k.p1.i, k.p2.i, k.dbg, k.packed);
    else fill_args<OrbitTapsD, double>(c, ctx, p, L, Z, k.p1.d, k.p2.d, k.dbg, false);
    k.matrix = use_matrix(ctx, c.pl) && !k.dbg;
    if (k.matrix) {
        MatArgs &m = k.p1.d.mat;
        k.table = c.pl.mat;
        for (int slot = 0; slot < 2; ++slot) {
            // the planes hold the pixels' bytes less 128
            const MaskInfo &mi = c.pl.mi[c.pl.order[slot]];
            const double sum = 2.0 * mi.sumpos - mi.sumabs, off = 128.0 * 257.0 * sum;
            m.sum |= off != 0.0;
            m.kd[slot] = off;
        }
    }
    k.gx = c.pl.gx;
    k.gy = c.pl.gy;
    k.nsets = c.n * c.pl.gx * c.pl.gy;
    if (gate > 0) {
        auto &G = ctx->gate;
        int rc;
        if ((rc = ensure_gate_images(ctx, k.nsets)) != LOGFX_OK) return rc;
        k.features = true;
        k.cells = G.cells;
        k.feats = feats ? feats : G.feats;
        k.maxval = c.pl.maxpix;
        if (k.i32)
            k.p1.i.cells = G.cells, k.p1.i.cell_slots = c.cell_slots, k.p1.i.cell_rows = c.cell_rows;
        else
            k.p1.d.cells = G.cells, k.p1.d.cell_slots = c.cell_slots, k.p1.d.cell_rows = c.cell_rows;
        if (gate > 1) {
            if ((rc = ensure_gate_batch(ctx, k.nsets)) != LOGFX_OK) return rc;
            k.gated = true;
            k.net = net_buffers(ctx, k.nsets, k.feats, nullptr, nullptr, nullptr, nullptr);
            k.flags = G.flags;
            if (k.i32) {
                k.p2.i.med_flags = G.flags;
                k.p2.i.region = c.pl.region;
                k.p2.i.reg_gx = c.pl.gx;
            } else {
                k.p2.d.med_flags = G.flags;
                k.p2.d.region = c.pl.region;
                k.p2.d.reg_gx = c.pl.gx;
            }
        }
    }
    k.halo2 = c.pl.std5 ? kHalo2Z5 : kHalo2Z;
    k.ncas = c.storez ? c.pl.ncas : 0;
    if (k.ncas > 0) {
        // level i reads the scratch map iff an odd number of levels remain
        uint8_t *first = k.ncas % 2 ? ctx->cmap : nullptr;
        if (k.i32) k.p2.i.out_map = first;
        else k.p2.d.out_map = first;
        for (int i = 0; i < k.ncas; ++i) {
            LevelArgs &l = k.lev[i];
            l.L = c.L;
            l.rows = c.rows2;
            l.median_size = c.pl.cas[i];
            l.from_scratch = (k.ncas - i) % 2;
            l.scratch = ctx->cmap;
            l.med_flags = k.gated ? ctx->gate.flags : nullptr;
            l.counts = i == k.ncas - 1 ? ctx->counts2 : nullptr;
        }
    }
    k.fin.L = c.L;
    k.fin.partials = ctx->partials;
    k.fin.exact = k.i32;
    k.fin.counts = ctx->counts1;
    k.fin.std_mode = p->std_mode;
    k.fin.std_k = p->std_k;
    for (int slot = 0; slot < 2; ++slot) k.fin.abs_thr[slot] = p->std_k / c.pl.mi[c.pl.order[slot]].unit;
    k.fin.stats = ctx->stats;
    k.fused = c.n == 1 && k.storez && !k.gated && c.L.total1 <= kFuseTiles;
    if (k.i32) k.p2.i.fin = k.fin, k.p2.i.fused = k.fused;
    else k.p2.d.fin = k.fin, k.p2.d.fused = k.fused;
    k.grid1 = c.L.total1;
    k.grid2 = c.L.total2;
    if (c.n > 1 && ctx->persistent && !k.dbg) {
        // a persistent launch: as many workgroups as fit on the device
        int m1 = 0, m2 = 0;
        const bool i32 = k.i32;
        const int mode = (k.storez ? kP1StoreZ : 0) | (k.matrix ? kP1Matrix : k.packed ? kP1Packed : 0);
        hipError_t e = i32 ? launch_pass1_i(k.ra, k.rb, k.p1.i, mode, 0, nullptr, &m1)
                           : launch_pass1_d(k.ra, k.rb, k.p1.d, k.table, mode, 0, nullptr, &m1);
        if (e == hipSuccess && k.storez)
            e = i32 ? launch_pass2z_i(k.p2.i, 0, nullptr, &m2) : launch_pass2z_d(k.p2.d, 0, nullptr, &m2);
        else if (e == hipSuccess)
            e = i32 ? launch_pass2_i(k.ra, k.rb, k.p2.i, 0, nullptr, &m2)
                    : launch_pass2_d(k.ra, k.rb, k.p2.d, 0, nullptr, &m2);
        if (e != hipSuccess) return hip_err(ctx, e, "occupancy query");
        if (m1 > 0) k.grid1 = std::min(k.grid1, m1);
        if (m2 > 0) k.grid2 = std::min(k.grid2, m2);
    }
    return LOGFX_OK;
}

// Replays the context's graph when the launches equal the captured ones,
// else captures a new graph first.
int graph_launch(logfx_ctx *ctx, const Launches &k, hipStream_t s) {
    const unsigned char *kb = reinterpret_cast<const unsigned char *>(&k);
    hipError_t e;
    if (!ctx->gexec || ctx->gkey.size() != sizeof k || std::memcmp(ctx->gkey.data(), kb, sizeof k) != 0) {
        if (ctx->gexec) (void)hipGraphExecDestroy(ctx->gexec);
        if (ctx->g) (void)hipGraphDestroy(ctx->g);
        ctx->gexec = nullptr;
        ctx->g = nullptr;
        ctx->gkey.clear();
        if (!ctx->capture && (e = hipStreamCreateWithFlags(&ctx->capture, hipStreamNonBlocking)) != hipSuccess)
            return hip_err(ctx, e, "hipStreamCreate");
        if ((e = hipStreamBeginCapture(ctx->capture, hipStreamCaptureModeThreadLocal)) != hipSuccess)
            return hip_err(ctx, e, "hipStreamBeginCapture");
        hipError_t le = launch_all(k, ctx->capture, nullptr, UNTIL_OUTPUT);
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(ctx->capture, &g);
        if (le != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return hip_err(ctx, le, "captured launch");
        }
        if (e != hipSuccess) return hip_err(ctx, e, "hipStreamEndCapture");
        hipGraphExec_t x = nullptr;
        if ((e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0)) != hipSuccess) {
            (void)hipGraphDestroy(g);
            return hip_err(ctx, e, "hipGraphInstantiate");
        }
        ctx->g = g;
        ctx->gexec = x;
        ctx->gkey.assign(kb, kb + sizeof k);
    }
    if ((e = hipGraphLaunch(ctx->gexec, s)) != hipSuccess) return hip_err(ctx, e, "hipGraphLaunch");
    return LOGFX_OK;
}

int fill_reports(logfx_ctx *ctx, const Call &c, const logfx_params *p, const Launches &k, logfx_report *reps,
                 hipStream_t s) {
    int rc;
    if ((rc = ensure_host(ctx, c.n, c.L.total2)) != LOGFX_OK) return rc;
    auto &G = ctx->gate;
    hipError_t e;
    if (k.gated) {
        if ((rc = grow_host(ctx, G.h_logits, G.h_cap, k.nsets)) != LOGFX_OK ||
            (rc = grow_host(ctx, G.h_flags, G.h_capf, k.nsets)) != LOGFX_OK)
            return rc;
        if ((e = hipMemcpyAsync(G.h_logits, k.net.logits, sizeof(float) * k.nsets, hipMemcpyDeviceToHost, s)) !=
                hipSuccess ||
            (e = hipMemcpyAsync(G.h_flags, k.flags, sizeof(int) * k.nsets, hipMemcpyDeviceToHost, s)) != hipSuccess)
            return hip_err(ctx, e, "report copy");
    }
    if ((e = hipMemcpyAsync(ctx->h_stats, ctx->stats, sizeof(DevStats) * c.n, hipMemcpyDeviceToHost, s)) !=
            hipSuccess ||
        (e = hipMemcpyAsync(ctx->h_counts2, ctx->counts2, sizeof(int) * 2 * (size_t)c.L.total2,
                            hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return hip_err(ctx, e, "report copy");
    long long b2 = 0;
    for (int i = 0; i < c.n; ++i) {
        logfx_report &r = reps[i];
        std::memset(&r, 0, sizeof r);
        const ImageJob &j = c.n == 1 ? c.L.one : ctx->tab_jobs[i];
        r.pixels = j.img.H * j.img.W;
        for (int slot = 0; slot < 2; ++slot) {
            const int u = c.pl.order[slot];
            const double unit = c.pl.mi[u].unit;
            r.sigma_g[u] = ctx->h_stats[i].sigma[slot] * unit;
            r.thresh[u] = ctx->h_stats[i].thresh[slot] * unit;
            r.zc_count[u] = ctx->h_stats[i].zc[slot];
        }
        for (int t = 0; t < c.tiles[i].ntiles2; ++t) {
            r.extracted += ctx->h_counts2[2 * (b2 + t)];
            r.output += ctx->h_counts2[2 * (b2 + t) + 1];
        }
        b2 += c.tiles[i].ntiles2;
        r.path = c.pl.path;
        r.inexact = c.pl.inexact ? 1 : 0;
        r.smoothed = p->smooth != LOGFX_SMOOTH_NEVER;
        if (k.gated && c.pl.region > 0) {   // one image: the flags of its regions
            r.gated = 1;
            r.regions = k.nsets;
            for (int q = 0; q < k.nsets; ++q) r.regions_smoothed += G.h_flags[q] != 0;
            r.smoothed = r.regions_smoothed > 0;
        } else if (k.gated) {
            r.gated = 1;
            r.smoothed = G.h_flags[i] != 0;
            r.gate_logit = G.h_logits[i];
        } else if (p->smooth == LOGFX_SMOOTH_GATE) {
            r.gate_fallback = 1;
        }
    }
    return LOGFX_OK;
}

int run(logfx_ctx *ctx, int n, const logfx_image *imgs, const logfx_params *p, uint8_t *const *outs,
        double *const maps_L[2], double *const maps_Z[2], logfx_report *reps, void *stream) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    const bool maps = maps_L != nullptr;
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return set_err(ctx, LOGFX_EDEVICE, "cannot select device %d", ctx->device);
    hipStream_t s = (hipStream_t)stream;
    Call c;
    const bool gated = !maps && p && p->smooth == LOGFX_SMOOTH_GATE && ctx->gate.loaded;
    int rc = prepare(ctx, n, imgs, p, outs, !maps, gated, c, s);
    if (rc != LOGFX_OK) return rc;
    if (gated && (rc = check_cells(ctx, n, imgs, c.pl)) != LOGFX_OK) return rc;
    Launches k;
    if ((rc = build_launches(ctx, c, p, maps_L, maps_Z, k, gated ? 2 : 0)) != LOGFX_OK) return rc;
    hipError_t e;
    const bool use_graph = n > 1 && ctx->graph && !maps;
    if (log_on())
        log_line("%s: %d image(s), first %lld x %lld, %s path, radii %d/%d, tiles %d/%d (rows %d/%d), %s, smooth %d%s%s",
             maps ? "extract_maps" : (n > 1 ? "extract_batch" : "extract"), n, (long long)imgs[0].height,
             (long long)imgs[0].width,
             !c.pl.i32 ? k.matrix ? "fp64 (matrix)" : "fp64" : k.packed ? "int32 (packed)" : "int32", c.pl.ra, c.pl.rb,
             c.L.total1, c.L.total2, c.rows1, c.rows2, c.storez ? "stored strengths" : "recomputed strengths",
             p->smooth, gated ? " (gated)" : "", use_graph ? ", graph" : "");
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    const bool timed = ctx->timing && !maps;
    if (timed) {
        if ((rc = timing_events(ctx, ctx->timed_calls, ev)) != LOGFX_OK) return rc;
        if ((e = hipEventRecord(ev[0], s)) != hipSuccess) return hip_err(ctx, e, "hipEventRecord");
    }
    if (use_graph) {
        if ((rc = graph_launch(ctx, k, s)) != LOGFX_OK) return rc;
    } else if ((e = launch_all(k, s, timed ? ev : nullptr, maps ? UNTIL_PASS1 : UNTIL_OUTPUT)) != hipSuccess) {
        return hip_err(ctx, e, "kernel launch");
    }
    if (maps) return LOGFX_OK;
    if (timed) {
        if ((e = hipEventRecord(ev[3], s)) != hipSuccess) return hip_err(ctx, e, "hipEventRecord");
        ctx->timed_graph.resize(ctx->timed_calls + 1);
        ctx->timed_graph[ctx->timed_calls] = use_graph;
        ++ctx->timed_calls;
    }
    if (reps) return fill_reports(ctx, c, p, k, reps, s);
    return LOGFX_OK;
}

// Features, or features and decisions, of n images (no pass 2).
int run_gate(logfx_ctx *ctx, int n, const logfx_image *imgs, const logfx_params *p, uint16_t *feats,
             float *logits, uint8_t *decisions, int until, void *stream) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return set_err(ctx, LOGFX_EDEVICE, "cannot select device %d", ctx->device);
    if (until == UNTIL_DECISION && !ctx->gate.loaded)
        return set_err(ctx, LOGFX_EINVAL, "the gate has no parameters (logfx_gate_set_params / logfx_gate_load)");
    if (until == UNTIL_FEATURES && !feats) return set_err(ctx, LOGFX_EINVAL, "feats is NULL");
    hipStream_t s = (hipStream_t)stream;
    Call c;
    int rc = prepare(ctx, n, imgs, p, nullptr, false, true, c, s);
    if (rc != LOGFX_OK) return rc;
    if ((rc = check_cells(ctx, n, imgs, c.pl)) != LOGFX_OK) return rc;
    Launches k;
    if ((rc = build_launches(ctx, c, p, nullptr, nullptr, k, until == UNTIL_FEATURES ? 1 : 2, feats)) != LOGFX_OK)
        return rc;
    k.decisions = decisions;
    hipError_t e;
    if ((e = launch_all(k, s, nullptr, until)) != hipSuccess) return hip_err(ctx, e, "kernel launch");
    if (logits && (e = hipMemcpyAsync(logits, k.net.logits, sizeof(float) * k.nsets, hipMemcpyDeviceToDevice, s)) !=
                      hipSuccess)
        return hip_err(ctx, e, "logit copy");
    return LOGFX_OK;
}

// Checks shared by the network calls.
int gate_batch_args(logfx_ctx *ctx, int B, const uint16_t *feats) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (B < 1 || B > LOGFX_GATE_MAX_BATCH)
        return set_err(ctx, LOGFX_EINVAL, "batch %d not in 1..%d", B, LOGFX_GATE_MAX_BATCH);
    if (!feats) return set_err(ctx, LOGFX_EINVAL, "feats is NULL");
    if (!ctx->gate.loaded)
        return set_err(ctx, LOGFX_EINVAL, "the gate has no parameters (logfx_gate_set_params / logfx_gate_load)");
    return LOGFX_OK;
}


// ------------------------------------------------------------ autotuner
// Key of a tuned configuration: device architecture, arithmetic path, mask
// radii, pixel type, smoothing, whether the call is a batch and its size.
std::string tune_key(logfx_ctx *ctx, const Call &c, const logfx_params *p, const logfx_image *imgs) {
    hipDeviceProp_t prop;
    std::string arch = "unknown";
    if (hipGetDeviceProperties(&prop, ctx->device) == hipSuccess) {
        arch = prop.gcnArchName;
        const size_t colon = arch.find(':');
        if (colon != std::string::npos) arch.resize(colon);
    }
    std::ostringstream k;
    k << arch << "|" << (!c.pl.i32 ? "fp64" : use_packed(ctx, c.pl) ? "int32pk" : "int32")
      << "|r" << c.pl.ra << c.pl.rb
      << "|" << (imgs[0].dtype == LOGFX_U8 ? "u8" : "u16") << "|med"
      << (p->smooth != LOGFX_SMOOTH_NEVER ? p->median_size : 0) << (p->smooth == LOGFX_SMOOTH_GATE ? "g" : "")
      << "|" << (c.n > 1 ? "batch" : "single") << (c.pl.std5 ? "|s5" : "") << "|px" << call_class(c.pl, c.n, imgs) / 2;
    for (int i = 0; i < c.pl.ncas; ++i) k << (i == 0 ? "|c" : "") << c.pl.cas[i];
    return k.str();
}

// The cache is a text file of JSON objects, one per line:
// {"key": "...", "rows1": R1, "rows2": R2, "persistent": P, "ms": T, "auto1": A1, "auto2": A2}
// where A = 1 leaves the pass the heights that calls take by themselves.
struct Tuned {
    logfx_tune_result r;
    int auto1, auto2;
};
bool cache_lookup(const char *path, const std::string &key, Tuned &t) {
    std::ifstream f(path);
    std::string line;
    bool found = false;
    while (std::getline(f, line)) {
        const std::string tag = "\"key\": \"" + key + "\"";
        if (line.find(tag) == std::string::npos) continue;
        int r1, r2, pe, a1, a2;
        double ms;
        const size_t at = line.find("\"rows1\"");
        if (at == std::string::npos) continue;
        if (std::sscanf(line.c_str() + at,
                        "\"rows1\": %d, \"rows2\": %d, \"persistent\": %d, \"ms\": %lf, \"auto1\": %d, \"auto2\": %d",
                        &r1, &r2, &pe, &ms, &a1, &a2) == 6 &&
            r1 >= 1 && r1 <= 1024 && r2 >= 1 && r2 <= 1024) {
            t.r.rows1 = r1, t.r.rows2 = r2, t.r.persistent = pe, t.r.ms = ms;
            t.auto1 = a1, t.auto2 = a2;
            found = true;   // the last entry for a key wins
        }
    }
    return found;
}

void cache_store(const char *path, const std::string &key, const Tuned &t) {
    std::ofstream f(path, std::ios::app);
    char buf[512];
    std::snprintf(buf, sizeof buf,
                  "{\"key\": \"%s\", \"rows1\": %d, \"rows2\": %d, \"persistent\": %d, \"ms\": %.6f, "
                  "\"auto1\": %d, \"auto2\": %d}\n",
                  key.c_str(), t.r.rows1, t.r.rows2, t.r.persistent, t.r.ms, t.auto1, t.auto2);
    f << buf;
}


// FNV-1a, 64-bit: the checksum of a training-state file.
uint64_t fnv1a64(const void *data, size_t n, uint64_t h = 1469598103934665603ull) {
    const unsigned char *p = static_cast<const unsigned char *>(data);
    for (size_t i = 0; i < n; ++i) {
        h ^= p[i];
        h *= 1099511628211ull;
    }
    return h;
}

// Training state read from a LOGFXGS1 file: parameters, AdamW moments, step.
struct GateState {
    std::vector<float> theta, m, v;
    int64_t step = 0;
};

// Reads a file written by logfx_gate_save_state; checks the header, the
// sizes and the checksum before anything reaches the context.
int read_gate_state(logfx_ctx *ctx, const char *path, GateState &st) {
    std::ifstream f(path, std::ios::binary);
    if (!f) return set_err(ctx, LOGFX_EINVAL, "cannot open %s", path);
    std::vector<char> bytes((std::istreambuf_iterator<char>(f)), std::istreambuf_iterator<char>());
    const size_t n = gate::kNParam, body = 8 + 8 + 8 + 3 * n * sizeof(float);
    if (bytes.size() != body + 8 || std::memcmp(bytes.data(), "LOGFXGS1", 8) != 0)
        return set_err(ctx, LOGFX_EINVAL, "%s is not a gate training-state file of %d parameters", path,
                       gate::kNParam);
    int32_t hdr[2];
    std::memcpy(hdr, bytes.data() + 8, sizeof hdr);
    uint64_t sum;
    std::memcpy(&sum, bytes.data() + body, sizeof sum);
    if (hdr[0] != gate::kNParam || hdr[1] != 1)
        return set_err(ctx, LOGFX_EINVAL, "%s: %d parameters, version %d (expected %d, 1)", path, hdr[0], hdr[1],
                       gate::kNParam);
    if (fnv1a64(bytes.data(), body) != sum) return set_err(ctx, LOGFX_EINVAL, "%s: checksum mismatch", path);
    std::memcpy(&st.step, bytes.data() + 16, sizeof st.step);
    if (st.step < 0) return set_err(ctx, LOGFX_EINVAL, "%s: negative step count", path);
    st.theta.resize(n);
    st.m.resize(n);
    st.v.resize(n);
    const char *q = bytes.data() + 24;
    std::memcpy(st.theta.data(), q, n * sizeof(float));
    std::memcpy(st.m.data(), q + n * sizeof(float), n * sizeof(float));
    std::memcpy(st.v.data(), q + 2 * n * sizeof(float), n * sizeof(float));
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(st.theta[i]) || !std::isfinite(st.m[i]) || !std::isfinite(st.v[i]) || st.v[i] < 0.0f)
            return set_err(ctx, LOGFX_EINVAL, "%s: value %zu is not a valid parameter or moment", path, i);
    return LOGFX_OK;
}

}  // namespace

// ===================================================================== ABI
extern "C" {

const char *logfx_version(void) { return "liblogfx 0.2 (gfx950)"; }

const char *logfx_last_error(const logfx_ctx *ctx) {
    return ctx ? ctx->err.c_str() : g_thread_error.c_str();
}

int logfx_create(logfx_ctx **out, int device) {
    if (!out) return set_err(nullptr, LOGFX_EINVAL, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || n == 0)
        return set_err(nullptr, LOGFX_EDEVICE, "no HIP device available (%s)",
                       e == hipSuccess ? "0 devices" : hipGetErrorString(e));
    if (device < 0 || device >= n)
        return set_err(nullptr, LOGFX_EINVAL, "device %d not in 0..%d", device, n - 1);
    logfx_ctx *ctx = new (std::nothrow) logfx_ctx;
    if (!ctx) return set_err(nullptr, LOGFX_ENOMEM, "out of host memory");
    ctx->device = device;
    ctx->tiles = tile_cfg_from_env();
    if (const char *f = std::getenv("LOGFX_FAIL_ALLOC")) ctx->fail_alloc_at = std::atoi(f);
    {   // the static scratch of logfx_extract_noalloc, with the device current
        DeviceGuard g(device);
        void *p = nullptr;
        const hipError_t se = g.ok ? noalloc_scratch(device, &p) : hipErrorInvalidDevice;
        if (se == hipSuccess) ctx->noalloc = p;
        else ctx->noalloc_err = hipGetErrorString(se);
    }
    *out = ctx;
    return LOGFX_OK;
}

int logfx_destroy(logfx_ctx *ctx) {
    if (!ctx) return LOGFX_OK;
    {
        DeviceGuard g(ctx->device);
        if (ctx->gexec) (void)hipGraphExecDestroy(ctx->gexec);
        if (ctx->g) (void)hipGraphDestroy(ctx->g);
        if (ctx->capture) (void)hipStreamDestroy(ctx->capture);
        for (auto &S : ctx->stage) {
            if (S.done) {
                (void)hipEventSynchronize(S.done);
                (void)hipEventDestroy(S.done);
            }
            if (S.jobs) (void)hipHostFree(S.jobs);
            if (S.own1) (void)hipHostFree(S.own1);
            if (S.own2) (void)hipHostFree(S.own2);
        }
        (void)hipFree(ctx->zmap);
        (void)hipFree(ctx->cmap);
        (void)hipFree(ctx->partials);
        (void)hipFree(ctx->counts1);
        (void)hipFree(ctx->counts2);
        (void)hipFree(ctx->stats);
        (void)hipFree(ctx->jobs);
        (void)hipFree(ctx->owner1);
        (void)hipFree(ctx->owner2);
        if (ctx->h_stats) (void)hipHostFree(ctx->h_stats);
        if (ctx->h_counts2) (void)hipHostFree(ctx->h_counts2);
        for (hipEvent_t ev : ctx->events) (void)hipEventDestroy(ev);
        auto &G = ctx->gate;
        for (void *q : {(void *)G.theta, (void *)G.m, (void *)G.v, (void *)G.grad, (void *)G.wbf, (void *)G.act,
                        (void *)G.gact, (void *)G.small, (void *)G.partial, (void *)G.cells, (void *)G.feats,
                        (void *)G.flags})
            (void)hipFree(q);
        if (G.h_logits) (void)hipHostFree(G.h_logits);
        if (G.h_flags) (void)hipHostFree(G.h_flags);
    }
    delete ctx;
    return LOGFX_OK;
}

int logfx_make_log_mask(int32_t size, double sigma, int32_t grid_bits, float *taps_out,
                        double *unit_out) {
    if (!taps_out) return set_err(nullptr, LOGFX_EINVAL, "taps_out is NULL");
    if (size < 1 || size % 2 == 0 || size > 15)
        return set_err(nullptr, LOGFX_EINVAL, "size %d is not odd in 1..15", size);
    if (!(sigma > 0.0) || !std::isfinite(sigma))
        return set_err(nullptr, LOGFX_EINVAL, "sigma must be finite and > 0");
    if (grid_bits < 2 || grid_bits > 23)
        return set_err(nullptr, LOGFX_EINVAL, "grid_bits %d not in 2..23", grid_bits);
    const int r = size / 2, n = size * size;
    double v[225];
    double total = 0.0;
    // eq. (1) sampled at integer offsets
    for (int y = -r; y <= r; ++y)
        for (int x = -r; x <= r; ++x) {
            const double q = (double)(x * x + y * y) / (2.0 * sigma * sigma);
            const double val = -1.0 / (M_PI * sigma * sigma * sigma * sigma) * (1.0 - q) * std::exp(-q);
            v[(y + r) * size + (x + r)] = val;
            total += val;
        }
    const double mean = total / n;
    double peak = 0.0;
    for (int i = 0; i < n; ++i) {
        v[i] -= mean;
        peak = std::max(peak, std::fabs(v[i]));
    }
    if (!(peak > 0.0)) return set_err(nullptr, LOGFX_EINVAL, "degenerate mask");
    int e;
    std::frexp(peak, &e);
    const double u = std::ldexp(1.0, e - grid_bits);
    long long k[225], sum = 0;
    for (int i = 0; i < n; ++i) {
        k[i] = (long long)std::nearbyint(v[i] / u);
        sum += k[i];
    }
    k[r * size + r] -= sum;  // exact zero sum
    for (int i = 0; i < n; ++i) taps_out[i] = (float)((double)k[i] * u);
    if (unit_out) *unit_out = u;
    return LOGFX_OK;
}

int logfx_check_params(const logfx_image *img, const logfx_params *p, int32_t *path_out) {
    Plan pl;
    int rc = check_all(nullptr, img, p, pl);
    if (rc == LOGFX_OK && path_out) *path_out = pl.path;
    return rc;
}

int logfx_extract(logfx_ctx *ctx, const logfx_image *img, const logfx_params *p, uint8_t *out,
                  logfx_report *rep, void *stream) {
    if (!img) return set_err(ctx, LOGFX_EINVAL, "image is NULL");
    uint8_t *outs[1] = {out};
    return run(ctx, 1, img, p, outs, nullptr, nullptr, rep, stream);
}

int logfx_extract_noalloc(logfx_ctx *ctx, const logfx_image *img, const logfx_params *p, uint8_t *out,
                          void *stream) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!img) return set_err(ctx, LOGFX_EINVAL, "image is NULL");
    if (!out) return set_err(ctx, LOGFX_EINVAL, "output 0 is NULL");
    Call c;   // c.tiles stays empty: this path allocates nothing, host or device
    c.rows1 = ctx->tiles.rows1;
    c.rows2 = ctx->tiles.rows2;
    int rc = check_all(ctx, img, p, c.pl);
    if (rc != LOGFX_OK) return rc;
    if (c.pl.std5 || c.pl.ncas > 0 || c.pl.region > 0)
        return set_err(ctx, LOGFX_EINVAL, "the 5x5 first stage, the median cascade and the per-region gate "
                                          "need context memory (logfx_extract runs them)");
    if (p->smooth == LOGFX_SMOOTH_GATE && ctx->gate.loaded)
        return set_err(ctx, LOGFX_EINVAL, "the gate needs context memory (logfx_extract runs it)");
    ImageTiles t;
    if ((rc = tile_image(ctx, img, c.pl, false, c.rows1, c.rows2, t)) != LOGFX_OK) return rc;
    if (t.ntiles1 > kNoAllocMaxTiles || t.ntiles2 > kNoAllocMaxTiles)
        return set_err(ctx, LOGFX_EINVAL, "a %lld x %lld image needs %d pass-1 and %d pass-2 tiles; the static "
                                          "scratch holds %lld per pass", (long long)img->height,
                       (long long)img->width, t.ntiles1, t.ntiles2, kNoAllocMaxTiles);
    if (!c.pl.i32 && !ctx->tiles.set1 && !(ctx->tiles.tuned1 && call_class(c.pl, 1, img) == ctx->tiles.tuned_class)) {
        // logfx_extract's height, for its statistics: at most twice the tiles
        c.rows1 = fp64_rows(c.pl);
        static_assert(kNoAllocMaxTiles1 >= 2 * kNoAllocMaxTiles, "ceil(H / 62) <= 2 ceil(H / 96)");
        if ((rc = tile_image(ctx, img, c.pl, false, c.rows1, c.rows2, t)) != LOGFX_OK) return rc;
    }
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return set_err(ctx, LOGFX_EDEVICE, "cannot select device %d", ctx->device);
    if (!ctx->noalloc)
        return set_err(ctx, LOGFX_EDEVICE, "the static scratch of device %d is not available: %s", ctx->device,
                       ctx->noalloc_err.c_str());
    c.n = 1;
    c.storez = false;
    std::memset(&c.L, 0, sizeof c.L);
    c.L.nimg = 1;
    c.L.total1 = t.ntiles1;
    c.L.total2 = t.ntiles2;
    c.L.one = make_job(*img, t, out, 0, 0, 0);
    Launches k;
    if ((rc = build_launches(ctx, c, p, nullptr, nullptr, k, 0)) != LOGFX_OK) return rc;
    // the sums, counts and statistics in the static array
    unsigned char *base = static_cast<unsigned char *>(ctx->noalloc);
    unsigned long long *partials = reinterpret_cast<unsigned long long *>(base + kNoAllocPartialsOff);
    long long *counts1 = reinterpret_cast<long long *>(base + kNoAllocCounts1Off);
    int *counts2 = reinterpret_cast<int *>(base + kNoAllocCounts2Off);
    DevStats *stats = reinterpret_cast<DevStats *>(base + kNoAllocStatsOff);
    if (k.i32) {
        k.p1.i.partials = partials, k.p1.i.counts = counts1;
        k.p2.i.stats = stats, k.p2.i.counts = counts2;
    } else {
        k.p1.d.partials = partials, k.p1.d.counts = counts1;
        k.p2.d.stats = stats, k.p2.d.counts = counts2;
    }
    k.fin.partials = partials;
    k.fin.counts = counts1;
    k.fin.stats = stats;
    const hipError_t e = launch_all(k, (hipStream_t)stream, nullptr, UNTIL_OUTPUT);
    if (e != hipSuccess) return hip_err(ctx, e, "kernel launch");
    return LOGFX_OK;
}

int logfx_extract_batch(logfx_ctx *ctx, int32_t n, const logfx_image *imgs, const logfx_params *p,
                        uint8_t *const *outs, logfx_report *reps, void *stream) {
    return run(ctx, n, imgs, p, outs, nullptr, nullptr, reps, stream);
}

int logfx_extract_maps(logfx_ctx *ctx, const logfx_image *img, const logfx_params *p, double *L1,
                       double *L2, double *Z1, double *Z2, void *stream) {
    double *L[2] = {L1, L2}, *Z[2] = {Z1, Z2};
    if (!img) return set_err(ctx, LOGFX_EINVAL, "image is NULL");
    return run(ctx, 1, img, p, nullptr, L, Z, nullptr, stream);
}

int logfx_set_option(logfx_ctx *ctx, int32_t option, int64_t value) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    switch (option) {
    case LOGFX_OPT_ROWS1:
    case LOGFX_OPT_ROWS2:
        if (value < 1 || value > 1024) return set_err(ctx, LOGFX_EINVAL, "rows %lld not in 1..1024", (long long)value);
        (option == LOGFX_OPT_ROWS1 ? ctx->tiles.rows1 : ctx->tiles.rows2) = (int)value;
        (option == LOGFX_OPT_ROWS1 ? ctx->tiles.set1 : ctx->tiles.set2) = true;
        return LOGFX_OK;
    case LOGFX_OPT_PERSISTENT: ctx->persistent = value != 0; return LOGFX_OK;
    case LOGFX_OPT_GRAPH: ctx->graph = value != 0; return LOGFX_OK;
    case LOGFX_OPT_STORE_Z: ctx->store_z = value != 0; return LOGFX_OK;
    case LOGFX_OPT_PACKED_LOG: ctx->pack_log = value != 0; return LOGFX_OK;
    default: return set_err(ctx, LOGFX_EINVAL, "unknown option %d", option);
    }
}

int logfx_get_option(logfx_ctx *ctx, int32_t option, int64_t *value) {
    if (!ctx || !value) return set_err(ctx, LOGFX_EINVAL, "ctx or value is NULL");
    switch (option) {
    case LOGFX_OPT_ROWS1: *value = ctx->tiles.rows1; return LOGFX_OK;
    case LOGFX_OPT_ROWS2: *value = ctx->tiles.rows2; return LOGFX_OK;
    case LOGFX_OPT_PERSISTENT: *value = ctx->persistent; return LOGFX_OK;
    case LOGFX_OPT_GRAPH: *value = ctx->graph; return LOGFX_OK;
    case LOGFX_OPT_STORE_Z: *value = ctx->store_z; return LOGFX_OK;
    case LOGFX_OPT_PACKED_LOG: *value = ctx->pack_log; return LOGFX_OK;
    default: return set_err(ctx, LOGFX_EINVAL, "unknown option %d", option);
    }
}

int logfx_timing_enable(logfx_ctx *ctx, int on) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->timing = on != 0;
    ctx->timed_calls = 0;
    return LOGFX_OK;
}

int logfx_timing_read(logfx_ctx *ctx, double *ms_out, int64_t *calls_out) {
    if (!ctx || !ms_out) return set_err(ctx, LOGFX_EINVAL, "ctx or ms_out is NULL");
    for (int k = 0; k < 4; ++k) ms_out[k] = 0.0;
    DeviceGuard dg(ctx->device);
    for (long long c = 0; c < ctx->timed_calls; ++c) {
        hipEvent_t *ev = &ctx->events[4 * c];
        hipError_t e = hipEventSynchronize(ev[3]);
        if (e != hipSuccess) return hip_err(ctx, e, "hipEventSynchronize");
        float ms = 0.0f;
        if (!ctx->timed_graph[c]) {
            for (int k = 0; k < 3; ++k) {
                if ((e = hipEventElapsedTime(&ms, ev[k], ev[k + 1])) != hipSuccess)
                    return hip_err(ctx, e, "hipEventElapsedTime");
                ms_out[k] += ms;
            }
        }
        if ((e = hipEventElapsedTime(&ms, ev[0], ev[3])) != hipSuccess)
            return hip_err(ctx, e, "hipEventElapsedTime");
        ms_out[3] += ms;
    }
    if (calls_out) *calls_out = ctx->timed_calls;
    ctx->timed_calls = 0;
    return LOGFX_OK;
}

int logfx_gate_features(logfx_ctx *ctx, int32_t n, const logfx_image *imgs, const logfx_params *p,
                        uint16_t *feats, void *stream) {
    return run_gate(ctx, n, imgs, p, feats, nullptr, nullptr, UNTIL_FEATURES, stream);
}

int logfx_gate(logfx_ctx *ctx, int32_t n, const logfx_image *imgs, const logfx_params *p, float *logits,
               uint8_t *decisions, void *stream) {
    return run_gate(ctx, n, imgs, p, nullptr, logits, decisions, UNTIL_DECISION, stream);
}

int logfx_gate_set_params(logfx_ctx *ctx, const float *theta, int64_t n) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!theta) return set_err(ctx, LOGFX_EINVAL, "theta is NULL");
    if (n != gate::kNParam) return set_err(ctx, LOGFX_EINVAL, "%lld parameters, the gate has %d", (long long)n, gate::kNParam);
    for (int64_t i = 0; i < n; ++i)
        if (!std::isfinite(theta[i])) return set_err(ctx, LOGFX_EINVAL, "parameter %lld is not finite", (long long)i);
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return set_err(ctx, LOGFX_EDEVICE, "cannot select device %d", ctx->device);
    int rc;
    if ((rc = ensure_gate_params(ctx)) != LOGFX_OK) return rc;
    auto &G = ctx->gate;
    const size_t bytes = sizeof(float) * gate::kNParam;
    hipError_t e;
    if ((e = hipMemcpy(G.theta, theta, bytes, hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemset(G.m, 0, bytes)) != hipSuccess || (e = hipMemset(G.v, 0, bytes)) != hipSuccess ||
        (e = gate::launch_params_to_bf16(G.theta, G.wbf, nullptr)) != hipSuccess ||
        (e = hipDeviceSynchronize()) != hipSuccess)
        return hip_err(ctx, e, "gate parameters");
    G.step = 0;
    G.loaded = true;
    return LOGFX_OK;
}

int logfx_gate_get_params(logfx_ctx *ctx, float *theta, int64_t n) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!theta) return set_err(ctx, LOGFX_EINVAL, "theta is NULL");
    if (n != gate::kNParam) return set_err(ctx, LOGFX_EINVAL, "%lld parameters, the gate has %d", (long long)n, gate::kNParam);
    if (!ctx->gate.loaded) return set_err(ctx, LOGFX_EINVAL, "the gate has no parameters");
    DeviceGuard dg(ctx->device);
    hipError_t e;
    if ((e = hipDeviceSynchronize()) != hipSuccess ||
        (e = hipMemcpy(theta, ctx->gate.theta, sizeof(float) * gate::kNParam, hipMemcpyDeviceToHost)) != hipSuccess)
        return hip_err(ctx, e, "gate parameters");
    return LOGFX_OK;
}

int logfx_gate_load(logfx_ctx *ctx, const char *path) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!path) return set_err(ctx, LOGFX_EINVAL, "path is NULL");
    std::ifstream f(path, std::ios::binary);
    if (!f) return set_err(ctx, LOGFX_EINVAL, "cannot open %s", path);
    char magic[8];
    f.read(magic, 8);
    if (f && std::memcmp(magic, "LOGFXGS1", 8) == 0) {   // a training-state file: its parameters
        f.close();
        GateState st;
        const int rc = read_gate_state(ctx, path, st);
        if (rc != LOGFX_OK) return rc;
        return logfx_gate_set_params(ctx, st.theta.data(), gate::kNParam);
    }
    int32_t hdr[2];
    std::vector<float> theta(gate::kNParam);
    f.read(reinterpret_cast<char *>(hdr), sizeof hdr);
    if (!f || std::memcmp(magic, "LOGFXGT1", 8) != 0 || hdr[0] != gate::kNParam || hdr[1] != 0)
        return set_err(ctx, LOGFX_EINVAL, "%s is not a gate parameter file of %d values", path, gate::kNParam);
    f.read(reinterpret_cast<char *>(theta.data()), sizeof(float) * gate::kNParam);
    if (!f) return set_err(ctx, LOGFX_EINVAL, "%s is truncated", path);
    return logfx_gate_set_params(ctx, theta.data(), gate::kNParam);
}

int logfx_gate_save(logfx_ctx *ctx, const char *path) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    if (!path) return set_err(ctx, LOGFX_EINVAL, "path is NULL");
    std::vector<float> theta(gate::kNParam);
    int rc = logfx_gate_get_params(ctx, theta.data(), gate::kNParam);
    if (rc != LOGFX_OK) return rc;
    std::ofstream f(path, std::ios::binary | std::ios::trunc);
    const int32_t hdr[2] = {gate::kNParam, 0};
    f.write("LOGFXGT1", 8);
    f.write(reinterpret_cast<const char *>(hdr), sizeof hdr);
    f.write(reinterpret_cast<const char *>(theta.data()), sizeof(float) * gate::kNParam);
    if (!f) return set_err(ctx, LOGFX_EINVAL, "cannot write %s", path);
    return LOGFX_OK;
}

int logfx_gate_save_state(logfx_ctx *ctx, const char *path) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!path) return set_err(ctx, LOGFX_EINVAL, "path is NULL");
    auto &G = ctx->gate;
    if (!G.loaded) return set_err(ctx, LOGFX_EINVAL, "the gate has no parameters");
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return set_err(ctx, LOGFX_EDEVICE, "cannot select device %d", ctx->device);
    const size_t n = gate::kNParam, vb = n * sizeof(float), body = 24 + 3 * vb;
    std::vector<char> bytes(body + 8);
    std::memcpy(bytes.data(), "LOGFXGS1", 8);
    const int32_t hdr[2] = {gate::kNParam, 1};
    std::memcpy(bytes.data() + 8, hdr, sizeof hdr);
    const int64_t step = G.step;
    std::memcpy(bytes.data() + 16, &step, sizeof step);
    hipError_t e;
    if ((e = hipDeviceSynchronize()) != hipSuccess ||
        (e = hipMemcpy(bytes.data() + 24, G.theta, vb, hipMemcpyDeviceToHost)) != hipSuccess ||
        (e = hipMemcpy(bytes.data() + 24 + vb, G.m, vb, hipMemcpyDeviceToHost)) != hipSuccess ||
        (e = hipMemcpy(bytes.data() + 24 + 2 * vb, G.v, vb, hipMemcpyDeviceToHost)) != hipSuccess)
        return hip_err(ctx, e, "gate state");
    const uint64_t sum = fnv1a64(bytes.data(), body);
    std::memcpy(bytes.data() + body, &sum, sizeof sum);
    std::ofstream f(path, std::ios::binary | std::ios::trunc);
    f.write(bytes.data(), (std::streamsize)bytes.size());
    if (!f) return set_err(ctx, LOGFX_EINVAL, "cannot write %s", path);
    return LOGFX_OK;
}

int logfx_gate_load_state(logfx_ctx *ctx, const char *path) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!path) return set_err(ctx, LOGFX_EINVAL, "path is NULL");
    GateState st;
    int rc = read_gate_state(ctx, path, st);
    if (rc != LOGFX_OK) return rc;
    if ((rc = logfx_gate_set_params(ctx, st.theta.data(), gate::kNParam)) != LOGFX_OK) return rc;
    auto &G = ctx->gate;
    DeviceGuard dg(ctx->device);
    const size_t vb = gate::kNParam * sizeof(float);
    hipError_t e;
    if ((e = hipMemcpy(G.m, st.m.data(), vb, hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(G.v, st.v.data(), vb, hipMemcpyHostToDevice)) != hipSuccess) {
        G.loaded = false;
        return hip_err(ctx, e, "gate state");
    }
    G.step = st.step;
    return LOGFX_OK;
}

int logfx_gate_forward(logfx_ctx *ctx, int32_t B, const uint16_t *feats, const int32_t *idx, float *logits,
                       void *stream) {
    int rc = gate_batch_args(ctx, B, feats);
    if (rc != LOGFX_OK) return rc;
    if (!logits) return set_err(ctx, LOGFX_EINVAL, "logits is NULL");
    DeviceGuard dg(ctx->device);
    hipStream_t s = (hipStream_t)stream;
    if ((rc = ensure_gate_batch(ctx, B)) != LOGFX_OK) return rc;
    const gate::NetBuffers n = net_buffers(ctx, B, feats, idx, nullptr, nullptr, nullptr);
    hipError_t e;
    if ((e = gate::launch_forward(n, s)) != hipSuccess ||
        (e = hipMemcpyAsync(logits, n.logits, sizeof(float) * B, hipMemcpyDeviceToDevice, s)) != hipSuccess)
        return hip_err(ctx, e, "gate forward");
    return LOGFX_OK;
}

int logfx_gate_backward(logfx_ctx *ctx, int32_t B, const uint16_t *feats, const int32_t *idx, const float *labels,
                        float *grad, float *loss, void *stream) {
    int rc = gate_batch_args(ctx, B, feats);
    if (rc != LOGFX_OK) return rc;
    if (!labels) return set_err(ctx, LOGFX_EINVAL, "labels is NULL");
    DeviceGuard dg(ctx->device);
    hipStream_t s = (hipStream_t)stream;
    if ((rc = ensure_gate_batch(ctx, B)) != LOGFX_OK) return rc;
    const gate::NetBuffers n = net_buffers(ctx, B, feats, idx, labels, grad, loss);
    hipError_t e;
    if ((e = gate::launch_forward(n, s)) != hipSuccess || (e = gate::launch_backward(n, s)) != hipSuccess)
        return hip_err(ctx, e, "gate backward");
    return LOGFX_OK;
}

int logfx_gate_step(logfx_ctx *ctx, const float *grad, double lr, void *stream) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    ctx->err.clear();
    if (!ctx->gate.loaded) return set_err(ctx, LOGFX_EINVAL, "the gate has no parameters");
    if (!(lr >= 0.0) || !std::isfinite(lr)) return set_err(ctx, LOGFX_EINVAL, "lr must be finite and >= 0");
    DeviceGuard dg(ctx->device);
    auto &G = ctx->gate;
    const long long t = ++G.step;
    gate::AdamArgs a;
    std::memset(&a, 0, sizeof a);
    a.theta = G.theta;
    a.m = G.m;
    a.v = G.v;
    a.grad = grad ? grad : G.grad;
    a.wbf = G.wbf;
    a.lr = (float)lr;
    a.beta1 = 0.9f;
    a.beta2 = 0.999f;
    a.eps = 1e-8f;
    a.wd = 1e-4f;
    a.bc1 = (float)(1.0 - std::pow(0.9, (double)t));
    a.bc2 = (float)(1.0 - std::pow(0.999, (double)t));
    a.n = gate::kNParam;
    hipError_t e = gate::launch_adamw(a, (hipStream_t)stream);
    if (e != hipSuccess) return hip_err(ctx, e, "gate step");
    return LOGFX_OK;
}

int logfx_tune(logfx_ctx *ctx, int32_t n, const logfx_image *imgs, const logfx_params *p,
               uint8_t *const *outs, int32_t reps, const char *cache_path, logfx_tune_result *res,
               void *stream) {
    if (!ctx) return set_err(nullptr, LOGFX_EINVAL, "ctx is NULL");
    if (reps < 1 || reps > 1000) return set_err(ctx, LOGFX_EINVAL, "reps %d not in 1..1000", reps);
    ctx->err.clear();
    hipStream_t s = (hipStream_t)stream;
    DeviceGuard dg(ctx->device);
    Call c;
    const TileCfg saved = ctx->tiles;
    const bool gated = p && p->smooth == LOGFX_SMOOTH_GATE && ctx->gate.loaded;
    ctx->tiles = TileCfg();   // c takes the heights that calls take by themselves
    int rc = prepare(ctx, n, imgs, p, outs, true, gated, c, s);
    ctx->tiles = saved;
    if (rc != LOGFX_OK) return rc;
    const std::string key = tune_key(ctx, c, p, imgs);
    Tuned best;
    std::memset(&best, 0, sizeof best);
    if (!cache_path) cache_path = std::getenv("LOGFX_TUNE_CACHE");   // may stay NULL
    if (cache_path && !*cache_path) cache_path = nullptr;
    // the heights `t` leaves in force
    auto chosen = [&](const Tuned &t) {
        TileCfg g;
        g.rows1 = t.r.rows1, g.rows2 = t.r.rows2;
        g.tuned1 = !t.auto1, g.tuned2 = !t.auto2;
        g.tuned_class = call_class(c.pl, n, imgs);
        return g;
    };
    if (cache_path && cache_lookup(cache_path, key, best)) {
        best.r.from_cache = 1;
    } else {
        const bool saved_p = ctx->persistent, saved_g = ctx->graph, saved_t = ctx->timing;
        ctx->graph = false;   // direct launches, so that each kernel is timed on its own
        const int cand[] = {32, 40, 48, 56, 64, 96};
        constexpr int ncand = sizeof cand / sizeof cand[0];
        // the candidates are timed round-robin, twice, and each keeps its
        // faster round: one pass over them in order favours whichever runs
        // first (the clock drops as the device warms up)
        constexpr int kRounds = 2;
        // time one configuration: the sums of pass-1, pass-2 and whole-call milliseconds
        auto measure = [&](double ms[4]) -> int {
            int r;
            if ((r = run(ctx, n, imgs, p, outs, nullptr, nullptr, nullptr, stream)) != LOGFX_OK) return r;
            ctx->timing = true;
            ctx->timed_calls = 0;
            for (int i = 0; i < reps; ++i)
                if ((r = run(ctx, n, imgs, p, outs, nullptr, nullptr, nullptr, stream)) != LOGFX_OK) return r;
            int64_t calls;
            return logfx_timing_read(ctx, ms, &calls);
        };
        // candidate ncand: the heights that calls take by themselves
        double t1[ncand + 1], t2[ncand + 1];
        for (int i = 0; i <= ncand; ++i) t1[i] = t2[i] = 1e300;
        for (int round = 0; round < kRounds && rc == LOGFX_OK; ++round)
            for (int i = 0; i <= ncand; ++i) {
                TileCfg g;
                bool use1 = true, use2 = true;
                if (i < ncand) {
                    g.set1 = use1 = pass1_lds_bytes(cand[i], c.pl.rb) <= 65536;
                    g.set2 = use2 = lds_bytes(cand[i], kHalo2, c.pl.rb) <= 65536;
                    if (!use1 && !use2) continue;
                    if (use1) g.rows1 = cand[i];
                    if (use2) g.rows2 = cand[i];
                }
                ctx->tiles = g;
                double ms[4];
                if ((rc = measure(ms)) != LOGFX_OK) break;
                if (use1) t1[i] = std::min(t1[i], ms[0]);
                if (use2) t2[i] = std::min(t2[i], ms[2]);
            }
        // reported where these win: their height, or the tallest of those
        // that go by the size
        const bool tall = call_pixels(n, imgs) >= kTallPixels;
        best.auto1 = best.auto2 = 1;
        best.r.rows1 = !c.pl.i32 || tall ? c.rows1 : gated ? kTallCells : kTall1;
        best.r.rows2 = !c.storez || tall ? c.rows2 : kTall2;
        double best1 = t1[ncand], best2 = t2[ncand];
        for (int i = 0; i < ncand; ++i) {
            if (t1[i] < best1) best1 = t1[i], best.r.rows1 = cand[i], best.auto1 = 0;
            if (t2[i] < best2) best2 = t2[i], best.r.rows2 = cand[i], best.auto2 = 0;
        }
        ctx->tiles = chosen(best);
        int pe = 0;
        double bestms = 0.0;
        if (rc == LOGFX_OK) {
            // batches: one workgroup per tile or a persistent grid, also
            // round-robin
            double tp[2] = {1e300, 1e300};
            for (int round = 0; round < kRounds && rc == LOGFX_OK; ++round)
                for (int q = 0; q < (n > 1 ? 2 : 1) && rc == LOGFX_OK; ++q) {
                    double ms[4];
                    ctx->persistent = q == 1;
                    if ((rc = measure(ms)) == LOGFX_OK) tp[q] = std::min(tp[q], ms[3]);
                }
            pe = tp[1] < tp[0] ? 1 : 0;
            bestms = tp[pe];
        }
        ctx->timing = saved_t;
        ctx->timed_calls = 0;
        ctx->graph = saved_g;
        ctx->persistent = saved_p;
        if (rc != LOGFX_OK) {
            ctx->tiles = saved;
            return rc;
        }
        best.r.persistent = pe, best.r.ms = bestms / reps;
        best.r.from_cache = 0;
        if (cache_path) cache_store(cache_path, key, best);
    }
    ctx->tiles = chosen(best);
    ctx->persistent = best.r.persistent != 0;
    if (res) *res = best.r;
    return LOGFX_OK;
}

}  // extern "C"
