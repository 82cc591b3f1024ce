// Host side of the C ABI declared in include/gbd.h.
#include "../../include/gbd.h"
#include "gbd_internal.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

using namespace gbd;

// Segment partials of gbd_plan_eval_noalloc: a static device array, so that
// entry point allocates nothing.  Each GPU the library runs on holds its own
// copy until the process ends.  Host code never passes `scratch` itself to a
// kernel (on the host it names a stand-in, not device memory): gbd_ctx_create
// takes each device's address with hipGetSymbolAddress once, with that
// device current, and every use goes through that address.
static __device__ __align__(256) unsigned char scratch[GBD_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_dev[kMaxDevices];  // per device: the address of its `scratch`
}  // namespace

// grow-only device buffer
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
};

struct BatchWork {
    DevBuf rec, l5, e0t, tab1, tab2, e0, e0part, part, flags, point, row_sums, terms;
    uint32_t *host_flags = nullptr;  // pinned: the point evaluation's status
    void *stage = nullptr;           // pinned staging of the batch tables
    size_t stage_bytes = 0;
    hipEvent_t stage_ev = nullptr;   // after the last copy from stage
    bool stage_pending = false;      // stage_ev recorded and not yet waited for
    double *metrics = nullptr;       // pinned: the finalising kernel writes the metrics here
    int64_t metrics_cap = 0;
    int64_t n_metrics = 0;           // of a started batch (0: none to collect)
};

// autotuner cache key: (kind, precision, log2 N bucket, log2 M bucket)
struct TuneKey {
    int kind, precision, ln, lm;
    bool operator<(const TuneKey &o) const {
        if (kind != o.kind) return kind < o.kind;
        if (precision != o.precision) return precision < o.precision;
        if (ln != o.ln) return ln < o.ln;
        return lm < o.lm;
    }
};
struct TuneVal {
    int rows, waves, seg_scale_pct;  // segments = auto count * pct / 100
    double ms;
};

// Device blocks of beamlet handles, by power-of-two size class (4 KiB and
// up): a freed handle's block waits in its class for the next handle of the
// same context instead of going back to the driver (hipMalloc and hipFree
// take tens of microseconds each, and a parameter sweep creates and frees
// thousands of handles).  A reused block is written by an upload on the
// context stream, after every kernel that read its previous contents there
// (gbd_ctx_set_stream waits for the old stream first).  At most
// kPoolCacheBytes wait; the pool frees them once the context and every handle
// drawn from it are gone.
constexpr size_t kPoolCacheBytes = (size_t)4 << 30;
struct DevPool {
    std::mutex mu;
    std::map<size_t, std::vector<void *>> cached;
    size_t cached_bytes = 0;
    ~DevPool() {
        for (auto &kv : cached)
            for (void *p : kv.second) (void)hipFree(p);
    }
    static size_t size_class(size_t bytes) {
        size_t c = 4096;
        while (c < bytes) c <<= 1;
        return c;
    }
    // a block of size class cls on the current device
    hipError_t get(size_t cls, void **p) {
        {
            std::lock_guard<std::mutex> lock(mu);
            auto it = cached.find(cls);
            if (it != cached.end() && !it->second.empty()) {
                *p = it->second.back();
                it->second.pop_back();
                cached_bytes -= cls;
                return hipSuccess;
            }
        }
        return hipMalloc(p, cls);
    }
    void put(void *p, size_t cls) {
        {
            std::lock_guard<std::mutex> lock(mu);
            if (cached_bytes + cls <= kPoolCacheBytes) {
                cached[cls].push_back(p);
                cached_bytes += cls;
                return;
            }
        }
        (void)hipFree(p);
    }
};

struct gbd_ctx_s {
    int device;
    std::shared_ptr<DevPool> pool;  // beamlet handles' device blocks
    // pinned staging of beamlet uploads: rewritten once the previous upload's
    // copy has run (up_ev), so a handle's creation does not wait for its own
    void *up_stage = nullptr;
    size_t up_bytes = 0;
    hipEvent_t up_ev = nullptr;
    bool up_pending = false;
    hipStream_t stream;
    int cus;
    gbd_plan_s *own_plan;  // plan used by gbd_eval
    BatchWork batch;
    std::map<TuneKey, TuneVal> tuned;
    // kernel timing (gbd_ctx_set_kernel_timing): recorded event pairs, and
    // spare pairs for reuse
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> timed, spare_events;
};

struct gbd_beamlets_s {
    gbd_ctx_s *ctx;
    BeamletsDev dev;
    void *mem;
    size_t mem_class;               // mem's size class in pool
    std::shared_ptr<DevPool> pool;  // where mem returns (kept alive past the context)
    bool higher_order;  // some beamlet has a nonzero Hermite-Gaussian order
    bool one_matrix;    // one matrix and one waist for all: abcd0, w00
    double abcd0[16], w00;
};

struct gbd_plane_s {
    PlaneGeom g;
};

struct gbd_plan_s {
    gbd_ctx_s *ctx;
    int64_t capacity;
    int64_t n;
    PlaneGeom pl;
    bool ready;
    uint32_t flags;  // FLAG_STEEP / FLAG_CROSS / FLAG_HG of the last setup (which mixed forms apply)
    Rec64 *r64;
    Rec32 *r32;
    RecSq64 *q64;  // FP64 sigma^(k^2) tables of the FP64 rotor form
    RecHG64 *h64;  // Hermite-Gaussian factors, allocated at the first setup of higher-order beamlets
    RecHG32 *h32;
    RecCut64 *c64;  // truncation factors, allocated at the first setup of truncated beamlets
    RecCut32 *c32;
    int64_t n_cut;  // truncated beamlets of the last setup (the last n_cut records)
    int32_t rows;   // row chunks of the last setup's beamlets (0: no table)
    int32_t *row_start;  // the last setup's chunk table
    int64_t row_cap;     // chunks it holds, allocated at the first setup of beamlets with a table
    uint32_t *status_dev;   // two (flags, peak) word pairs used by alternate setups; each setup clears the other
    int status_parity;      // the pair the next setup uses
    bool status_zeroed;     // both words cleared (once, before the first setup)
    uint64_t *status_post;  // coherent host memory: the last setup's status words and sequence number
    uint32_t status_seq;    // the last launched setup's sequence number
    int sep_scale;          // FP16 separable form: accumulators hold the field times 2^sep_scale
    uint32_t sep_key;       // the status key sep_scale came from
    void *scratch;
    size_t scratch_bytes;
    // a captured evaluation's graph writes the scratch it was captured with at
    // every replay: once outgrown it is kept (here) until the plan is freed
    bool scratch_captured;
    std::vector<void *> held;
    uint32_t *status_cur;  // the last launched setup's status pair (null: none launched)
    bool spec_ok;  // the last setup succeeded: gbd_eval may launch the next evaluation before reading the status
};

// plan_eval_impl under a guard: the configuration writes the output without
// the guarded reduction (no partials) or product by rows, so it cannot run before the status
constexpr int kNoSpeculation = 1;

// the setup flags that select how an evaluation runs
constexpr uint32_t kFormFlags = FLAG_STEEP | FLAG_CROSS | FLAG_HG | FLAG_ROWS | FLAG_CROSS1 | FLAG_CROSS2 |
                               FLAG_CUT0 | FLAG_CUT1 | FLAG_CUT2 | FLAG_CUT3;

struct gbd_mlp_s {
    gbd_ctx_s *ctx;
    int n_in, width, depth, max_batch, mode;
    int64_t P;
    std::vector<int64_t> woff, boff;  // per layer (depth hidden + head): W and b offsets in the flat vector
    float *mem;                       // one allocation holding everything below
    float *params, *grads, *m, *v;
    float *Z, *H;                     // [depth][max_batch][width]
    float *dz0, *dz1;                 // [max_batch][width]
    float *xb, *yb, *yhat, *g, *loss;
    uint16_t *xt;                     // BF16 inputs, transposed (the two-kernel path)
    uint16_t *wf, *wb;                // its BF16 operands of the weights (MlpNet), or null
    int64_t step;
};

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what) {
    return fail(e == hipErrorOutOfMemory ? GBD_ENOMEM : GBD_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(call, what)                    \
    do {                                       \
        hipError_t e_ = (call);                \
        if (e_ != hipSuccess) return hip_fail(e_, what); \
    } while (0)

// Ray-transfer matrices must be symplectic: M^T J M = J with
// J = [[0, I], [-I, 0]] (equivalent to the block relations of Sec. 2.1).
// The checks below run over every beamlet of a handle with matrices of its
// own (12,720 traced ones: 1.0 ms a handle with J's zeros multiplied out,
// element-wise finite tests and packing, 0.44 ms as here).
constexpr double kJ[4][4] = {{0, 0, 1, 0}, {0, 0, 0, 1}, {-1, 0, 0, 0}, {0, -1, 0, 0}};
// the four products of (M^T J M)_rc with a nonzero entry of J (m finite)
inline void symplectic_terms(const double *m, int r, int c, double (&t)[4]) {
    t[0] = m[r] * m[8 + c];
    t[1] = m[4 + r] * m[12 + c];
    t[2] = -m[8 + r] * m[c];
    t[3] = -m[12 + r] * m[4 + c];
}
bool symplectic(const double *m, double tol = 1e-10) {
    bool bad = false;
    for (int r = 0; r < 4; r++)
        for (int c = 0; c < 4; c++) {
            double t[4];
            symplectic_terms(m, r, c, t);
            const double v = ((t[0] + t[1]) + t[2]) + t[3];
            const double mag = ((fabs(t[0]) + fabs(t[1])) + fabs(t[2])) + fabs(t[3]);
            bad |= fabs(v - kJ[r][c]) > tol * (mag + fabs(kJ[r][c]));
        }
    return !bad;
}

// Traced (finite-difference) matrices: a block can vanish (A at a focus), so
// entry-wise relative residuals are ill-posed.  Balance with the symplectic
// similarity diag(1/s, 1/s, s, s) M diag(s, s, 1/s, 1/s), s^2 = sqrt(|B| / |C|)
// (Frobenius norms), which leaves A and D and scales B, C to equal norms, and
// bound max |M'^T J M' - J| by tol * max(1, max |M'|)^2.
bool symplectic_balanced(const double *m, double tol) {
    double nb = 0.0, nc = 0.0;
    for (int r = 0; r < 2; r++)
        for (int c = 0; c < 2; c++) {
            nb += m[4 * r + c + 2] * m[4 * r + c + 2];
            nc += m[4 * (r + 2) + c] * m[4 * (r + 2) + c];
        }
    const double s2 = (nb > 0.0 && nc > 0.0) ? sqrt(sqrt(nb) / sqrt(nc)) : 1.0;
    double b[16], big = 1.0, zero = 0.0;
    for (int r = 0; r < 4; r++)
        for (int c = 0; c < 4; c++) {
            double v = m[4 * r + c];
            if (r < 2 && c >= 2) v /= s2;
            if (r >= 2 && c < 2) v *= s2;
            b[4 * r + c] = v;
            big = fabs(v) > big ? fabs(v) : big;
            zero += 0.0 * v;
        }
    if (!(zero == 0.0)) return false;  // balanced out of range
    const double lim = tol * big * big;
    bool good = true;
    for (int r = 0; r < 4; r++)
        for (int c = 0; c < 4; c++) {
            double t[4];
            symplectic_terms(b, r, c, t);
            good &= fabs(((t[0] + t[1]) + t[2]) + t[3] - kJ[r][c]) <= lim;
        }
    return good;
}

// The row chunks (BeamletsDev::row_start) of n whole beamlets in stored order
// (perm[i] the caller's index of the i-th): consecutive beamlets whose inputs
// can give the same y factor, i.e. equal y, y slope and waist under one
// shared matrix, kRowLen at most; whether they do is checked on the device.
// Higher orders: a row's beamlets are first put in order of their y order
// (stable), which the y factor depends on.  Empty if the rows are too short
// to gain: the product over the chunks replaces one over the beamlets, at
// least kRowGain times as many.
constexpr int64_t kRowMinBeamlets = 64, kRowGain = 4;
std::vector<int32_t> row_chunks(int64_t n, std::vector<int64_t> &perm, const double *r1, const double *th1,
                                const double *w0, int64_t n_w0, const int32_t *order) {
    std::vector<int32_t> start;
    if (n < kRowMinBeamlets || n > 0x7fffffff) return start;
    const size_t most = (size_t)(n / kRowGain);
    start.reserve(std::min<size_t>(most, 1024) + 1);
    auto cut = [&](int64_t i, int64_t e) {  // beamlets [i, e) into chunks; false: too many
        for (; i < e; i += kRowLen) {
            if (start.size() >= most) return false;
            start.push_back((int32_t)i);
        }
        return true;
    };
    int64_t j = perm[0];  // the run's first beamlet
    for (int64_t i = 0, e; i < n; i = e) {
        const double y = r1[2 * j + 1], th = th1 ? th1[2 * j + 1] : 0.0, w = n_w0 == 1 ? 0.0 : w0[j];
        for (e = i + 1; e < n; e++) {
            j = perm[e];
            if (r1[2 * j + 1] != y || (th1 && th1[2 * j + 1] != th) || (n_w0 != 1 && w0[j] != w)) break;
        }
        if (!order) {
            if (!cut(i, e)) return std::vector<int32_t>();
            continue;
        }
        // by the y order, stable (beamlets with orders have no edges: perm is the identity)
        int64_t n1 = 0, n2 = 0;
        for (int64_t k = i; k < e; k++) {
            n1 += order[2 * k + 1] == 1;
            n2 += order[2 * k + 1] == 2;
        }
        const int64_t b2 = e - n2, b1 = b2 - n1;
        int64_t at0 = i, at1 = b1, at2 = b2;  // no array: a counter stored and read back would be a chain
        for (int64_t k = i; k < e; k++) {
            const int32_t o = order[2 * k + 1];
            perm[o == 0 ? at0 : o == 1 ? at1 : at2] = k;
            at0 += o == 0;
            at1 += o == 1;
            at2 += o == 2;
        }
        if (!cut(i, b1) || !cut(b1, b2) || !cut(b2, e)) return std::vector<int32_t>();
    }
    start.push_back((int32_t)n);
    return start;
}

bool finite_all(const double *p, int64_t count) {
    // a set exponent carries into the top bit; no early exit, so the loop vectorises
    constexpr uint64_t kExp = 0x7ff0000000000000ull, kOne = 0x0010000000000000ull;
    uint64_t top = 0;
    for (int64_t i = 0; i < count; i++) {
        uint64_t w;
        memcpy(&w, p + i, sizeof w);
        top |= (w & kExp) + kOne;
    }
    return (top >> 63) == 0;
}

int ensure_device(gbd_ctx_s *ctx) {
    HIP_TRY(hipSetDevice(ctx->device), "hipSetDevice");
    return GBD_OK;
}

struct Shape {
    int rows, waves, nseg, form;
    bool half;  // mixed separable form in FP16 hi/lo halves (else FP32 MFMA)
    bool cross = false;  // the rotor's sum by the cross form (launch_eval_cross)
};

// mixed kernel form (0 direct, 1 stepped, 2 rotor, 3 separable): requested
// or automatic.  The stepped and rotor forms need a well-sampled grid (no
// FLAG_STEEP), the separable form phasors without cross terms (no
// FLAG_CROSS); a request that does not apply falls back to the automatic
// choice among the others.
int pick_form(int precision, uint32_t flags, const gbd_eval_opts *o, bool allow_sep = true) {
    const bool steep = (flags & FLAG_STEEP) != 0;
    if (precision != GBD_MIXED) {
        // FP64: direct, rotor (needs a well-sampled grid) or separable (needs
        // phasors and higher-order factors without cross terms).  A request
        // that does not apply falls back to the automatic choice among the
        // others.
        const bool sep64 = allow_sep && !(flags & FLAG_CROSS);
        const bool rot64 = !steep;
        const int v = o ? (o->variant == 5 ? 4 : o->variant) : 0;
        if (v == 1) return 0;
        if (v == 3 && rot64) return 2;
        if (v == 4 && sep64) return 3;
        return sep64 ? 3 : rot64 ? 2 : 0;
    }
    const bool sep = allow_sep && !(flags & FLAG_CROSS);
    const int v = o ? (o->variant == 5 ? 4 : o->variant) : 0;  // 5: the separable form on FP32 MFMA
    if (v == 1) return 0;
    // higher-order beamlets: the stepped form does not carry their factor
    if (v == 2) return (steep || (flags & FLAG_HG)) ? 0 : 1;
    if (v == 3) return steep ? 0 : 2;
    return sep ? 3 : steep ? 0 : 2;
}

// the variant a resolved form reports (gbd_eval_opts.variant)
int form_variant(int precision, int form, bool half = false) {
    return (precision == GBD_MIXED && form == 3 && !half) ? 5 : form + 1;
}

int ilog2(int64_t v) {
    int r = 0;
    while (v > 1) {
        v >>= 1;
        r++;
    }
    return r;
}

// cache kinds: single evaluations in a VALU form, batched sweeps, single
// evaluations in the separable form (only the segment count applies; the sum
// by rows has none), single evaluations of planes that the cross form takes
// at its shape (a kind of their own: the rotor form's best shape on strong
// cross terms would switch it off)
constexpr int kTuneEval = 0, kTuneBatch = 1, kTuneSep = 2, kTuneCross = 3;
TuneKey tune_key(int kind, int precision, int64_t n, int64_t m) { return TuneKey{kind, precision, ilog2(n), ilog2(m)}; }

// Fewest segments a form allows: the mixed separable form sums a segment in
// plain FP32 on the matrix cores, at most kSepMaxSegLen beamlets per sum.
int64_t min_segments(int precision, int form, int64_t n) {
    return (form == 3 && precision == GBD_MIXED) ? (n + kSepMaxSegLen - 1) / kSepMaxSegLen : 1;
}

// The cross form takes over the rotor form's sums where every cross term is
// weak (the setup's flags), at the rotor's default shape (32 rows, 4
// wavefronts) and at two segments or more: one segment asked for is the
// batched sweep's arithmetic, the rotor recurrence.  Below kCrossMinPairs
// the rotor form is as fast (448 beamlets on 64 x 90 pixels 18 us against 24;
// 1,264 on 64 x 90 31 against 27, 12,892 on 1024^2 2,640 against 560).
constexpr int64_t kCrossMinPairs = 3000000;
bool cross_applies(int precision, int form, uint32_t flags, int64_t n, int64_t m) {
    return precision == GBD_MIXED && form == 2 && (flags & FLAG_CROSS) && !(flags & (FLAG_HG | FLAG_CROSS2)) &&
           n * m >= kCrossMinPairs;
}

// Beamlets of a plain FP32 sum of the cross form at most, so that its error
// stays below the rotor form's, which compensates its sums every 128 (12,892
// beamlets on 1024^2 pixels, rotor 5.5e-7: 4.5e-7 at 640, 5.1e-7 at 768, 5.9e-7 at
// 1,024; 15,856 on 323 x 433, 5.4e-7: 5.0e-7 at 566, 6.2e-7 at 755; 100,668 on 512^2
// 1.3e-6 at 3,146 and 5.6e-6 at 14,381).  Over 90 drawn planes the errors meet
// between 500 and 760 beamlets, so automatic counts cut the sums short where
// that costs little, the partials growing with the plane; with these limits none
// of 230 drawn planes of up to 128 across on 1024^2 was further off, of 200
// larger ones 6, by 2 to 16 %, at 600 to 645.  On fewer than 128 rows the rotor form runs 16 rows and is nearer
// (1,804 on 127^2: 2.9e-7; the cross form 2.6e-7 at 320, 4.2e-7 at 640).
// kCrossSegLen: what a count of the caller's own may leave, and one lowered to
// a fixed buffer, which is held to the field of the same count given.
constexpr int64_t kCrossSegLen = 656, kCrossSegLenLow = 320;
int64_t cross_longest(int64_t n, const PlaneGeom &pl) {
    const int64_t m = (int64_t)pl.nx * pl.ny;
    return pl.ny < 128 ? kCrossSegLenLow : m < 100000 ? 480 : m < 500000 ? 496 : n < 6144 ? 576 : kCrossSegLen;
}

// Scratch that a form takes over its general form's at most: beyond it the
// general form runs, whose scratch does not grow with the beamlets (cross
// form: 8 bytes per pixel and `longest` beamlets).
constexpr int64_t kFormScratch = (int64_t)4 << 30;

// Its automatic segment count: one workgroup per CU at a time, each pass of 16
// beamlets about 2.4 us and three passes' worth of start-up, 16 bytes per
// pixel and segment through memory for the partials; segments of 64 ...
// `longest` beamlets.  0: too long sums or too much scratch.
int64_t cross_segments(int cus, int64_t tiles, int64_t n, int64_t m, int64_t longest) {
    int64_t best = 0;
    double best_t = 1e300;
    const int64_t least = std::max<int64_t>(2, (n + longest - 1) / longest), most = std::max<int64_t>(least, n / 64);
    for (int64_t seg = least; seg <= most && seg <= 2048 && seg * m * 8 <= kFormScratch; seg++) {
        const double rounds = (double)((tiles * seg + cus - 1) / cus);
        const double t = rounds * (double)((n / seg + 15) / 16 + 3) * 2.4e-6 + (double)seg * (double)m * 16.0 / 5e12;
        if (t < best_t) {
            best_t = t;
            best = seg;
        }
    }
    return best;
}

// Bytes of the row sums and y factors of an evaluation by rows.
size_t row_scratch(int64_t rows, const PlaneGeom &pl, int precision) {
    return (size_t)rows * ((size_t)pl.nx + (size_t)pl.ny) * (precision == GBD_FP64 ? 16 : 8);
}

// Whether the sum by rows of n beamlets in `rows` chunks takes less time than
// the products by beamlet.  Its product has a workgroup per 32 x 32 pixels,
// each through all chunks (0.030 us a chunk, FP64 0.046, up to a round of
// workgroups over the CUs), the other splits the beamlets over the chip
// whatever the plane: short runs on small planes are better off there.
// Microseconds, mixed, by rows / by beamlet, of runs of 4 and of 16: 10,000
// on 64^2 79 / 39, 31 / 39; 100,000 on 64^2 642 / 114, 183 / 115; 1,000 on 64^2
// 23 / 32, 18 / 32; 100,000 on 300^2 700 / 442, 205 / 440; 10,000 on 1024^2 236 /
// 256, 79 / 254.  FP64, whose products by beamlet are slower: 10,000 on 64^2
// 123 / 73, 43 / 75, but 144 / 248 on 300^2 at runs of 4.
bool rows_pay(int precision, int cus, int64_t n, int64_t rows, const PlaneGeom &pl) {
    if (rows <= 0 || row_scratch(rows, pl, precision) > (size_t)kFormScratch) return false;
    const bool mixed = precision == GBD_MIXED;
    auto tiles = [&](int64_t wx, int64_t wy) { return ((pl.nx + wx - 1) / wx) * ((pl.ny + wy - 1) / wy); };
    const double rounds = (double)tiles(kRowTilePx, kRowTilePx) / cus;
    const double product = (double)rows * std::max(mixed ? 0.030 : 0.046, (mixed ? 0.0225 : 0.037) * rounds);
    const double sums = (double)n * pl.nx / (mixed ? 1.05e6 : 5.3e5);
    const double by_beamlet = mixed ? (double)n * (256 * 128 * tiles(256, 128)) / 4.9e7 + 14.0
                                    : (double)n * (128 * 128 * tiles(128, 128)) / 6.9e6 + 44.0;
    return product + sums <= by_beamlet;
}

// Workgroup tile of a separable shape in pixels.
void sep_wg_tile(const Shape &s, int &px, int &py) {
    if (s.half) {
        px = kSepHWavesX * kSepHTile;
        py = kSepHWavesY * kSepHTile;
    } else {
        px = kSepTileX * kSepWavesX;
        py = s.rows * (s.waves / kSepWavesX);
    }
}

// Most segments an automatic count takes: at least 256 beamlets each, or
// down to `shortest` while the partial sums (elem bytes per pixel and
// segment) stay within 64 MiB, where their traffic is small against a chip
// left idle (rotor form, 4 wavefronts: 448 beamlets on 64 x 90 pixels 174 us
// in one segment, 14 in 32; 1,264 on 300^2 202 us in 4, 62 in 46; FP64, 3,228
// on 512^2 505 us in 12, 398 in 16) and the allocation-free evaluation's
// buffer holds them.
int64_t most_segments(int64_t n, int64_t shortest, const PlaneGeom &pl, int64_t elem) {
    const int64_t fit = GBD_NOALLOC_SCRATCH_BYTES / std::max<int64_t>(1, (int64_t)pl.nx * pl.ny * elem);
    return std::max<int64_t>(1, std::max<int64_t>(n / 256, std::min<int64_t>(n / shortest, fit)));
}

// An automatic count lowered to a whole number of workgroups per CU where the
// fullest CU then holds at least 5 % fewer beamlets: a few workgroups over a
// multiple of the CUs cost most of another round (9 x 29 workgroups on 256
// CUs: FP64 separable, 8,021 beamlets on 300 x 257, 354 us, in 28 segments
// 190; FP16 halves, 6 x 43, 84, in 42 53; rotor FP64, 1,804 on 409 x 275,
// 21 x 37 186, in 36 158; a truncated rim of 128 across on 300^2, all in all
// 159, then 121).
int64_t whole_rounds(int64_t seg, int64_t tiles, int64_t cus) {
    const int64_t rounds = tiles * seg / cus;
    const int64_t low = rounds * cus / tiles;
    return low >= 1 && 20 * rounds * seg < 19 * (rounds + (tiles * seg % cus != 0)) * low ? low : seg;
}

// Launch shape and mixed form.  32 rows per lane is a rotor-form shape: where
// the form resolves to direct or stepped it runs 16.
// general: the forms that hold for any records with these form flags only (no
// cross form).
Shape choose_shape(const gbd_ctx_s *ctx, int precision, int64_t n, const PlaneGeom &pl, uint32_t flags,
                   const gbd_eval_opts *o, bool general = false) {
    Shape s;
    s.form = pick_form(precision, flags, o);
    // the mixed separable form runs on FP16 MFMA in hi/lo halves unless the
    // FP32 one is requested (variant 5); the setup bounds higher-order
    // factors with their axis polynomials for the FP16 scaling
    s.half = s.form == 3 && precision == GBD_MIXED && !(o && o->variant == 5);
    if (s.form == 3) {
        // separable form: fixed 64 x 32 pixel tile per wavefront (s.rows is
        // the tile height), 2 x 4 wavefronts per workgroup (s.waves), or in
        // FP16 halves 64 x 64 per wavefront, 4 x 2 wavefronts; the row and
        // wavefront options of the other forms do not apply
        const bool mixed = precision == GBD_MIXED;
        s.rows = s.half ? kSepHTile : mixed ? kSepTileY : kSepRows64;
        s.waves = s.half ? kSepHWavesX * kSepHWavesY : kSepWavesX * (mixed ? kSepWavesY : kSep64WavesY);
        int wgx, wgy;
        sep_wg_tile(s, wgx, wgy);
        s.nseg = (o && o->segments > 0) ? o->segments : 0;
        // the MFMA accumulators sum a segment in plain FP32: its error grows
        // with the segment's length (823,592 beamlets on 64^2 pixels: 1.6e-7
        // at 3,217 per segment, 6.1e-7 at 12,868, 3.4e-6 at 51,474, 1.4e-5
        // at 205,898), so mixed-precision segments hold at most 16,384
        // beamlets, whatever the count's source (automatic, tuned or explicit)
        const int64_t min_seg = min_segments(precision, s.form, n);
        if (s.nseg <= 0) {
            // one round of workgroups, 8 wavefronts per CU (the register
            // budget allows two wavefronts per SIMD; a partial second round
            // leaves CUs idle: on 512^2 pixels, 16 tiles, 16 segments ran
            // 0.78 ms, 32 0.79 ms; with the earlier four-product form's
            // 256 x 128 workgroup tiles 16 segments ran 1.78 ms, 32 0.91 ms,
            // 48 1.22 ms)
            const int64_t tiles =
                std::max<int64_t>(1, (int64_t)((pl.nx + wgx - 1) / wgx) * ((pl.ny + wgy - 1) / wgy));
            const int64_t per_cu = 8 / s.waves;
            int64_t seg = ((int64_t)ctx->cus * per_cu + tiles - 1) / tiles;
            auto it = ctx->tuned.find(tune_key(kTuneSep, precision, n, (int64_t)pl.nx * pl.ny));
            if (it != ctx->tuned.end()) seg = std::max<int64_t>(1, seg * it->second.seg_scale_pct / 100);
            seg = whole_rounds(std::min<int64_t>(seg, most_segments(n, 64, pl, mixed ? 8 : 16)), tiles, ctx->cus);
            s.nseg = (int)std::max<int64_t>(1, std::min<int64_t>(seg, 1024));
        }
        // the cap wins over the 1024-segment limit (above 16.7 M beamlets)
        if (s.nseg < min_seg) s.nseg = (int)std::min<int64_t>(min_seg, 0x7fffffff);
        return s;
    }
    // rotor form: 32 rows per lane where the grid fills a 4-wave tile
    const bool cross = !general && cross_applies(precision, s.form, flags, n, (int64_t)pl.nx * pl.ny);
    s.rows = (s.form == 2 && (pl.ny >= 128 || cross)) ? 32 : (precision != GBD_MIXED && s.form == 0) ? 4 : 16;
    s.waves = 4;
    s.nseg = 0;
    int seg_pct = 100;
    const bool user = o && (o->rows_per_lane || o->waves || o->segments);
    if (!user) {
        auto it = ctx->tuned.find(tune_key(cross ? kTuneCross : kTuneEval, precision, n, (int64_t)pl.nx * pl.ny));
        if (it != ctx->tuned.end()) {
            s.rows = it->second.rows;
            s.waves = it->second.waves;
            seg_pct = it->second.seg_scale_pct;
        }
    }
    if (o) {
        if (o->rows_per_lane) s.rows = o->rows_per_lane;
        if (o->waves) s.waves = o->waves;
        if (o->segments) s.nseg = o->segments;
    }
    if (s.rows == 32 && s.form != 2) s.rows = 16;
    if (precision != GBD_MIXED && s.form == 0 && s.rows > 8) s.rows = 8;  // FP64 direct form: up to 8 rows
    // FP64 rotor form with higher-order factors: up to 16 rows (registers)
    if (precision != GBD_MIXED && s.form == 2 && (flags & FLAG_HG) && s.rows > 16) s.rows = 16;
    if (cross && s.rows == 32 && s.waves == 4) {
        int64_t seg = s.nseg;
        const int64_t longest = seg > 0 ? kCrossSegLen : cross_longest(n, pl);
        const int64_t M = (int64_t)pl.nx * pl.ny;
        if (seg <= 0) {
            const int64_t tiles = std::max<int64_t>(1, (int64_t)((pl.nx + kCrossTile - 1) / kCrossTile) *
                                                           ((pl.ny + kCrossTile - 1) / kCrossTile));
            seg = cross_segments(ctx->cus, tiles, n, M, longest);
            if (seg)
                seg = std::max<int64_t>(std::max<int64_t>(2, (n + longest - 1) / longest),
                                        std::min<int64_t>(seg * seg_pct / 100, kFormScratch / (M * 8)));
        } else if (seg * longest < n) {
            seg = 0;
        }
        if (seg >= 2 && n >= 4) {
            s.cross = true;
            s.nseg = (int)seg;
        } else if (pl.ny < 128 && !(o && o->rows_per_lane)) {
            s.rows = 16;  // the rotor form's own
        }
    }
    if (s.nseg <= 0) {
        // enough workgroups to keep every SIMD of every CU busy ~6 waves deep
        const int64_t tx = (pl.nx + 63) / 64;
        const int64_t ty = (pl.ny + s.waves * s.rows - 1) / (s.waves * s.rows);
        const int64_t tiles = std::max<int64_t>(1, tx * ty);
        const int64_t target_blocks = (int64_t)ctx->cus * 4 * 6 / s.waves;
        int64_t seg = (target_blocks + tiles - 1) / tiles;
        seg = std::max<int64_t>(1, seg * seg_pct / 100);
        seg = whole_rounds(std::min<int64_t>(seg, most_segments(n, 8, pl, 16)), tiles, ctx->cus);
        s.nseg = (int)std::max<int64_t>(1, std::min<int64_t>(seg, 1024));
    }
    return s;
}

bool valid_shape(int rows, int waves, int precision = GBD_MIXED) {
    const bool r = rows == 1 || rows == 2 || rows == 4 || rows == 8 || rows == 16 || rows == 32;
    (void)precision;
    return r && (waves == 1 || waves == 2 || waves == 4);
}

EvalGeom make_geom(const PlaneGeom &pl, int64_t n, const Shape &s) {
    EvalGeom g;
    g.nx = pl.nx;
    g.ny = pl.ny;
    g.dx = pl.dx;
    g.dy = pl.dy;
    g.a0 = -0.5 * (pl.nx - 1) * pl.dx;
    g.b0 = -0.5 * (pl.ny - 1) * pl.dy;
    if (s.cross) {
        g.tiles_x = (pl.nx + kCrossTile - 1) / kCrossTile;
        g.tiles_y = (pl.ny + kCrossTile - 1) / kCrossTile;
    } else if (s.form == 3) {
        int wgx, wgy;
        sep_wg_tile(s, wgx, wgy);
        g.tiles_x = (pl.nx + wgx - 1) / wgx;
        g.tiles_y = (pl.ny + wgy - 1) / wgy;
    } else {
        g.tiles_x = (pl.nx + 63) / 64;
        g.tiles_y = (pl.ny + s.waves * s.rows - 1) / (s.waves * s.rows);
    }
    g.n = n;
    int64_t nseg = std::max<int64_t>(1, std::min<int64_t>(s.nseg, std::max<int64_t>(1, n)));
    g.seg_len = (n + nseg - 1) / nseg;
    if (g.seg_len == 0) g.seg_len = 1;
    g.nseg = (int32_t)((n + g.seg_len - 1) / g.seg_len);
    if (g.nseg < 1) g.nseg = 1;
    g.work = g.tiles_x * g.tiles_y * g.nseg;
    return g;
}

// Weideman's coefficients for the Faddeeva function (FaddeevaCoef): a_n,
// n = 1..N, are the Fourier coefficients of the even, 2 pi-periodic
// F(theta) = e^(-s^2) (L^2 + s^2), s = L tan(theta / 2), taken by the
// midpoint rule (spectrally accurate for a smooth periodic integrand).
void weideman(int N, double *L, double *a) {
    *L = std::sqrt(N / std::sqrt(2.0));
    const int K = 4096;
    const double pi = 3.14159265358979323846;
    for (int n = 1; n <= N; n++) {
        double acc = 0.0;
        for (int i = 0; i < K; i++) {
            const double th = -pi + (i + 0.5) * 2.0 * pi / K;
            const double t = *L * std::tan(0.5 * th);
            acc += std::exp(-t * t) * (*L * *L + t * t) * std::cos(n * th);
        }
        a[n - 1] = acc / K;
    }
}

const FaddeevaCoef &faddeeva_coef() {
    static const FaddeevaCoef fc = [] {
        FaddeevaCoef f{};
        weideman(kFaddeevaN64, &f.L64, f.a64);
        double L32, a32[kFaddeevaN32];
        weideman(kFaddeevaN32, &L32, a32);
        f.L32 = (float)L32;
        for (int i = 0; i < kFaddeevaN32; i++) f.a32[i] = (float)a32[i];
        return f;
    }();
    return fc;
}

constexpr int kCutWaves = 2;  // workgroups a CU holds of the column form (240 registers a lane): one round of them

// The truncated-beamlet kernel's column form (launch_eval_cut's level) where
// its polynomials reach; pixel by pixel where the direct form is asked for.
int cut_level(int precision, uint32_t flags, const gbd_eval_opts *o) {
    if (o && o->variant == 1) return 0;
    if (precision == GBD_MIXED && !(flags & FLAG_CUT0)) return 4;
    return !(flags & FLAG_CUT1) ? 3 : !(flags & FLAG_CUT2) ? 2 : !(flags & FLAG_CUT3) ? 1 : 0;
}

// Launch geometry of the truncated-beamlet kernel: 64-column tiles of
// 4 wavefronts x the level's rows, segments for 2 wavefronts per SIMD (pixel
// by pixel ~6), each of at least 8 beamlets while the partials are small
// (most_segments), else 32.  Level 4 takes segments of one tile, with partials
// of 64 MiB at most, or is lowered to 3 (2,028 on 512 x 512: the
// kernel 300 us in 16 segments of 32 rows, 430 in 8 of 16).
EvalGeom cut_geom(const gbd_ctx_s *ctx, int precision, int &level, const PlaneGeom &pl, int64_t n_cut,
                  int64_t max_seg = 1024) {
    const int64_t one = (n_cut + kCutOneTile - 1) / kCutOneTile;
    if (level == 4 && one > std::min<int64_t>(max_seg, most_segments(n_cut, kCutOneTile, pl, 16) + 1)) level = 3;
    Shape s;
    s.form = 0;
    s.half = false;
    s.waves = 4;
    s.rows = level == 4 ? 2 * kCutRows : level > 1 ? kCutRows : level == 1 ? kCutRows / 2 : precision == GBD_MIXED ? kCutRows32 : kCutRows64;
    const int64_t tx = (pl.nx + 63) / 64;
    const int64_t ty = (pl.ny + s.waves * s.rows - 1) / (s.waves * s.rows);
    const int64_t tiles = std::max<int64_t>(1, tx * ty);
    int64_t seg = ((int64_t)ctx->cus * (level ? kCutWaves : 6) + tiles - 1) / tiles;
    seg = whole_rounds(std::min<int64_t>(seg, std::max<int64_t>(n_cut / 32, most_segments(n_cut, 8, pl, 16))), tiles,
                       ctx->cus);
    if (level == 4) seg = std::max<int64_t>(seg, one);
    s.nseg = (int)std::max<int64_t>(1, std::min<int64_t>(seg, max_seg));
    return make_geom(pl, n_cut, s);
}

// Whether launches on the context's stream are being captured into a graph.
bool captures(const gbd_ctx_s *ctx) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &st) != hipSuccess) {
        (void)hipGetLastError();  // the null stream, while another one is captured
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

// Bytes of partial sums of an evaluation in the general forms.
size_t general_scratch(const gbd_ctx_s *ctx, const gbd_plan_s *plan, int precision, const gbd_eval_opts *opts) {
    const int64_t n = plan->n - plan->n_cut;
    const Shape s = choose_shape(ctx, precision, n, plan->pl, plan->flags, opts, true);
    int level = 0;
    const int64_t seg = (n > 0 ? make_geom(plan->pl, n, s).nseg : 0) +
                        (plan->n_cut > 0 ? cut_geom(ctx, precision, level, plan->pl, plan->n_cut).nseg : 0);
    return (size_t)seg * (size_t)plan->pl.nx * (size_t)plan->pl.ny * 16;
}

// fixed: a caller-provided partial-sum buffer of fixed_bytes (the static
// buffer of gbd_plan_eval_noalloc), used instead of the plan's grow-only one;
// then nothing is allocated and an automatic segment count is lowered to fit.
// guard (gbd_eval's launch ahead of the setup status): the output is
// written only by the guarded reduction or product by rows, or nothing is launched and the call
// returns kNoSpeculation; guard->check_key is set when the form's FP16 scale
// depends on the key.
// post_req (with post set): a setup status still to be posted, by the
// separable form's evaluation kernel at its start, else by status_post_kernel
// ahead of this evaluation's first kernel; post is cleared once a launch has
// taken it (a call that launches nothing leaves it set).
// dense: not by rows.
int plan_eval_impl(gbd_ctx_s *ctx, gbd_plan_s *plan, int precision, void *out, int64_t out_bytes,
                   const gbd_eval_opts *opts, void *fixed = nullptr, size_t fixed_bytes = 0,
                   EvalGuard *guard = nullptr, StatusPost *post_req = nullptr, bool dense = false) {
    if (!plan->ready && !guard) return fail(GBD_EINVAL, "gbd_plan_eval: plan has no valid setup");
    if (precision != GBD_FP64 && precision != GBD_MIXED) return fail(GBD_EINVAL, "precision must be GBD_FP64 or GBD_MIXED");
    const int64_t M = (int64_t)plan->pl.nx * plan->pl.ny;
    const int64_t elem = precision == GBD_FP64 ? 16 : 8;
    if (M == 0) return GBD_OK;
    if (!out) return fail(GBD_EINVAL, "field_out is NULL");
    if (out_bytes < M * elem)
        return fail(GBD_ERANGE, "field_out holds %lld bytes, %lld needed", (long long)out_bytes, (long long)(M * elem));
    if (opts && (opts->variant < 0 || opts->variant > 5)) return fail(GBD_EINVAL, "variant must be 0 ... 5");
    // rows_per_lane and waves do not apply to the separable form (its tile is
    // fixed; gbd_plan_shape reports it, and handing that shape back is fine)
    const bool sep_form = pick_form(precision, plan->flags, opts) == 3;
    if (opts && opts->rows_per_lane && !sep_form &&
        !valid_shape(opts->rows_per_lane, opts->waves ? opts->waves : 4, precision))
        return fail(GBD_EINVAL, "unsupported rows_per_lane %d / waves %d", opts->rows_per_lane, opts->waves);
    // A captured evaluation is replayed over whatever records later setups
    // leave in the plan: it takes the general forms, not those that rest on
    // this setup's row chunks, small cross terms or slow edge terms.
    const bool general = !guard && captures(ctx);
    Shape s = choose_shape(ctx, precision, plan->n - plan->n_cut, plan->pl, plan->flags, opts, general);
    if (s.form != 3 && !valid_shape(s.rows, s.waves, precision))
        return fail(GBD_EINVAL, "unsupported rows_per_lane %d / waves %d", s.rows, s.waves);
    int rc = ensure_device(ctx);
    if (rc) return rc;
    if (guard && plan->n == 0) return kNoSpeculation;
    if (plan->n == 0) {
        if (fixed)
            HIP_TRY(launch_fill_zero(out, (size_t)(M * elem), ctx->stream), "zero fill launch");
        else
            HIP_TRY(hipMemsetAsync(out, 0, (size_t)(M * elem), ctx->stream), "hipMemsetAsync");
        return GBD_OK;
    }
    // the whole beamlets [0, n_main) in the chosen form; truncated ones
    // [n_main, n) by their own kernel into the following segments
    const int64_t n_main = plan->n - plan->n_cut;
    // the mixed separable form's partials are compact (float2) and come first
    // (of the cross form too)
    bool compact = n_main > 0 && (s.form == 3 || s.cross) && precision == GBD_MIXED;
    EvalGeom g{}, gc{};
    int32_t nseg_main = 0, nseg_cut = 0;
    int level = general ? 0 : cut_level(precision, plan->flags, opts);
    if (plan->n_cut > 0) {
        gc = cut_geom(ctx, precision, level, plan->pl, plan->n_cut);
        nseg_cut = gc.nseg;
    }
    // The separable form by rows wherever the beamlets come in row chunks
    // (row_chunks; the setup found their y factors equal) that pay and FP32 MFMA in
    // Gauss's form is not asked for: one segment, written by the product (with
    // truncated beamlets into the first partial).  Segment counts do not apply.
    // The fixed buffer has to hold the row sums beside any partials.
    const bool rows_route = !general && !dense && s.form == 3 && n_main > 0 && (precision == GBD_FP64 || s.half) &&
                            rows_pay(precision, ctx->cus, n_main, plan->rows, plan->pl);
    bool by_rows = rows_route && !(plan->flags & FLAG_ROWS);
    const size_t row_bytes = by_rows ? row_scratch(plan->rows, plan->pl, precision) : 0;
    auto row_offset = [&](int64_t nc) -> size_t {  // where the row sums start, with nc truncated segments
        const size_t part = nc == 0 ? 0 : reduce_wide_offset(compact ? 1 : 0, M) + (size_t)(nc + (compact ? 0 : 1)) * M * 16;
        return (part + 255) & ~(size_t)255;
    };
    // a count given by the caller is refused by its own form's limits, by rows or not
    const bool given = opts && opts->segments > 0;
    if (n_main > 0) {
        g = make_geom(plan->pl, n_main, s);
        nseg_main = g.nseg;
    }
    // partial bytes of nm main and nc truncated segments (none when one
    // segment writes the output directly)
    // (the cross form's count as the rotor form's, whose shape it reports)
    const size_t per_cut = (size_t)M * 16;
    auto need_of = [&](int64_t nm, int64_t nc) -> size_t {
        if (nm + nc <= 1 && nc == 0) return 0;
        return compact && !s.cross ? reduce_wide_offset((int32_t)nm, M) + (size_t)nc * per_cut : (size_t)(nm + nc) * per_cut;
    };
    auto refuse_segments = [&] {
        return fail(GBD_ERANGE, "%d segments of %lld pixels need %zu bytes of partial sums; the static buffer holds %zu",
                    (int)(nseg_main + nseg_cut), (long long)M, need_of(nseg_main, nseg_cut), fixed_bytes);
    };
    auto grid_too_large = [](const EvalGeom &q) {
        return (int64_t)q.tiles_x * q.tiles_y * q.nseg > (int64_t)0x7fffffff - 8;
    };
    if (by_rows && given) {
        if (grid_too_large(g)) return fail(GBD_ERANGE, "grid too large");
        if (fixed && need_of(nseg_main, nseg_cut) > fixed_bytes) return refuse_segments();
    }
    if (fixed && by_rows) {
        while (nseg_cut > 1 && row_offset(nseg_cut) + row_bytes > fixed_bytes) {
            gc = cut_geom(ctx, precision, level, plan->pl, plan->n_cut, nseg_cut - 1);
            nseg_cut = gc.nseg;
        }
        by_rows = row_offset(nseg_cut) + row_bytes <= fixed_bytes;
        if (!by_rows && plan->n_cut > 0) {
            gc = cut_geom(ctx, precision, level, plan->pl, plan->n_cut);
            nseg_cut = gc.nseg;
        }
    }
    if (guard) {
        // the flags that this evaluation's route depends on
        guard->mask = FLAG_STEEP | FLAG_CROSS | FLAG_HG;
        if (rows_route) guard->mask |= FLAG_ROWS;
        if (cross_applies(precision, s.form, plan->flags & ~(uint32_t)FLAG_CROSS2, n_main, M))
            guard->mask |= FLAG_CROSS1 | FLAG_CROSS2;
        if (plan->n_cut > 0) guard->mask |= FLAG_CUT0 | FLAG_CUT1 | FLAG_CUT2 | FLAG_CUT3;
        guard->flags = plan->flags & guard->mask;
    }
    if (by_rows) {
        s.nseg = 1;
        g = make_geom(plan->pl, n_main, s);
        nseg_main = g.nseg;
    }
    // Sums of the cross form too long for it once the count is lowered to what
    // the fixed buffer holds: the rotor form's, compensated, shape and all.
    auto rotor_instead = [&] {
        s = choose_shape(ctx, precision, n_main, plan->pl, plan->flags, opts, true);
        compact = false;
        g = make_geom(plan->pl, n_main, s);
        nseg_main = g.nseg;
    };
    if (fixed && s.cross && !given) {
        const size_t per = (size_t)M * 16;
        const int64_t room = (int64_t)(fixed_bytes / per);
        if (nseg_main + nseg_cut > room) {
            const int64_t left = room - std::min<int64_t>(nseg_cut, (int64_t)(fixed_bytes / 2 / per));
            if (left < 2 || std::min<int64_t>(left, nseg_main) * (plan->pl.ny < 128 ? kCrossSegLenLow : kCrossSegLen) < n_main)
                rotor_instead();
        }
    }
    if (fixed && !by_rows) {
        const bool small = compact && !s.cross;
        const size_t per_main = (size_t)M * (small ? 8 : 16);
        if (need_of(nseg_main, nseg_cut) > fixed_bytes) {
            if (given) return refuse_segments();
            if (nseg_cut > 0) {  // truncated beamlets: at most half the buffer
                const int64_t max_cut = (int64_t)((fixed_bytes / 2) / per_cut);
                if (max_cut < 1)
                    return fail(GBD_ERANGE, "%lld pixels: one segment of partial sums (%zu bytes) exceeds half the "
                                "static buffer (%zu bytes)", (long long)M, per_cut, fixed_bytes);
                if (nseg_cut > max_cut) {
                    gc = cut_geom(ctx, precision, level, plan->pl, plan->n_cut, max_cut);
                    nseg_cut = gc.nseg;
                }
            }
            if (n_main > 0) {
                const size_t used = (size_t)nseg_cut * per_cut + (small ? 16 : 0);
                int64_t max_main = used < fixed_bytes ? (int64_t)((fixed_bytes - used) / per_main) : 0;
                if (nseg_cut == 0 && max_main < 2) max_main = 1;  // one segment: no partials
                const int64_t floor_seg = min_segments(precision, s.form, n_main);
                if (max_main < std::max<int64_t>(floor_seg, 1))
                    return fail(GBD_ERANGE, "%lld beamlets on %lld pixels need at least %lld segments of partial sums; "
                                "the static buffer (%zu bytes) holds %lld", (long long)n_main, (long long)M,
                                (long long)std::max<int64_t>(floor_seg, 1), fixed_bytes, (long long)max_main);
                if (nseg_main > max_main) {
                    s.nseg = (int)max_main;
                    g = make_geom(plan->pl, n_main, s);
                    nseg_main = g.nseg;
                }
            }
            if (need_of(nseg_main, nseg_cut) > fixed_bytes)
                return fail(GBD_ERANGE, "partial sums need %zu bytes; the static buffer holds %zu",
                            need_of(nseg_main, nseg_cut), fixed_bytes);
        }
    }
    if ((n_main > 0 && grid_too_large(g)) || (nseg_cut > 0 && grid_too_large(gc)))
        return fail(GBD_ERANGE, "grid too large");
    const int32_t total = nseg_main + nseg_cut;
    const bool reduce = total > 1 || nseg_cut > 0;
    if (guard && !reduce && !by_rows) return kNoSpeculation;
    StatusPost sp;  // the post handed to the separable form's kernel
    if (post_req && post_req->post) {
        if (n_main > 0 && (s.form == 3 || s.cross)) {
            sp = *post_req;
        } else {
            HIP_TRY(launch_status_post(*post_req, ctx->stream), "status post launch");
            post_req->post = nullptr;
        }
    }
    const int32_t nseg2 = compact ? nseg_main : 0;
    void *partial = fixed ? fixed : plan->scratch;
    if ((reduce || by_rows) && !fixed) {
        size_t need = by_rows ? row_offset(nseg_cut) + row_bytes
                              : (size_t)total * (size_t)M * 16;  // bounds the compact layout too
        // a caller's plan has its evaluation captured after a first one that
        // allocates: enough for the general forms too
        if ((by_rows || s.cross || (nseg_cut > 0 && level)) && plan != ctx->own_plan)
            need = std::max(need, general_scratch(ctx, plan, precision, opts));
        if (need > plan->scratch_bytes) {
            if (plan->scratch && plan->scratch_captured)
                plan->held.push_back(plan->scratch);
            else if (plan->scratch)
                (void)hipFree(plan->scratch);
            plan->scratch = nullptr;
            plan->scratch_bytes = 0;
            plan->scratch_captured = false;
            HIP_TRY(hipMalloc(&plan->scratch, need), "hipMalloc(segment partials)");
            plan->scratch_bytes = need;
        }
        plan->scratch_captured |= general;
        partial = plan->scratch;
    }
    if (n_main > 0) {
        const void *rec = precision == GBD_FP64 ? (const void *)plan->r64 : (const void *)plan->r32;
        const bool hg = (plan->flags & FLAG_HG) != 0;
        const void *hrec = !hg ? nullptr : precision == GBD_FP64 ? (const void *)plan->h64 : (const void *)plan->h32;
        EvalGeom gl = g;
        if (reduce && !by_rows) gl.nseg = std::max<int32_t>(total, 2);  // segment partials, never the output
        const bool stamped = s.form == 3 || s.cross;  // the launch's events take the kernel's own times
        if (s.form == 2 && !s.cross)
            HIP_TRY(launch_sigma(gl, plan->r64, precision == GBD_FP64 ? plan->q64 : nullptr,
                                 precision == GBD_FP64 ? nullptr : plan->r32, ctx->stream),
                    "sigma table kernel launch");
        std::pair<hipEvent_t, hipEvent_t> tev{nullptr, nullptr};
        if (ctx->timing && !fixed) {  // the allocation-free path records none
            if (!ctx->spare_events.empty()) {
                tev = ctx->spare_events.back();
                ctx->spare_events.pop_back();
            } else {
                // timing only (read after a later synchronisation): no
                // system-scope fence, whose cache writeback would stall the
                // stream between the kernels
                HIP_TRY(hipEventCreateWithFlags(&tev.first, hipEventDisableSystemFence), "hipEventCreate");
                const hipError_t e = hipEventCreateWithFlags(&tev.second, hipEventDisableSystemFence);
                if (e != hipSuccess) {
                    (void)hipEventDestroy(tev.first);
                    return hip_fail(e, "hipEventCreate");
                }
            }
            ctx->timed.push_back(tev);
            // the matrix forms' launches take the kernel's own times; the
            // others are bracketed by event records
            if (!stamped) HIP_TRY(hipEventRecord(tev.first, ctx->stream), "hipEventRecord");
        }
        if (by_rows) {
            const RowGeom rg{plan->pl.nx, plan->pl.ny, g.dx, g.dy, g.a0, g.b0, plan->rows};
            void *sums = static_cast<char *>(partial) + row_offset(nseg_cut);
            void *dst = reduce ? partial : out;
            // with a reduction behind it the product writes a partial, which needs no guard
            EvalGuard gd;
            if (guard && !reduce) {
                guard->check_key = 0;  // the scale is read on the device
                gd = *guard;
            }
            if (precision == GBD_FP64)
                HIP_TRY(launch_rows64(rg, plan->row_start, plan->r64, static_cast<const RecHG64 *>(hrec),
                                      static_cast<double2 *>(sums),
                                      static_cast<double2 *>(dst), gd, ctx->stream, tev.first, tev.second, sp),
                        "row kernels launch");
            else
                HIP_TRY(launch_rows32(rg, plan->row_start, plan->r32, static_cast<const RecHG32 *>(hrec),
                                      plan->status_cur, static_cast<float2 *>(sums),
                                      static_cast<float2 *>(dst), gd, ctx->stream, tev.first, tev.second, sp),
                        "row kernels launch");
        } else if (s.cross)
            HIP_TRY(launch_eval_cross((plan->flags & FLAG_CROSS1) ? 2 : 1, gl, plan->r32, plan->status_cur,
                                      static_cast<float2 *>(partial), ctx->stream, tev.first, tev.second, sp),
                    "eval kernel launch");
        else if (s.form == 3 && precision == GBD_FP64)
            HIP_TRY(launch_eval_sep64(gl, plan->r64, static_cast<const RecHG64 *>(hrec),
                                      static_cast<double2 *>(partial), static_cast<double2 *>(out), ctx->stream,
                                      tev.first, tev.second, sp),
                    "eval kernel launch");
        else if (s.form == 3 && s.half)
            HIP_TRY(launch_eval_seph(gl, plan->r32, static_cast<const RecHG32 *>(hrec), plan->sep_scale,
                                     general ? plan->status_dev : nullptr, static_cast<float2 *>(partial),
                                     static_cast<float2 *>(out), ctx->stream, tev.first, tev.second, sp),
                    "eval kernel launch");
        else if (s.form == 3)
            HIP_TRY(launch_eval_sep(gl, plan->r32, static_cast<const RecHG32 *>(hrec),
                                    static_cast<float2 *>(partial), static_cast<float2 *>(out), ctx->stream,
                                    tev.first, tev.second, sp),
                    "eval kernel launch");
        else
            HIP_TRY(launch_eval(precision, s.rows, s.waves, s.form, gl, rec, hrec, plan->q64, partial, out,
                                ctx->stream),
                    "eval kernel launch");
        if (tev.second && !stamped) HIP_TRY(hipEventRecord(tev.second, ctx->stream), "hipEventRecord");
        if (post_req) post_req->post = nullptr;  // posted by the kernel just launched (form 3), or above
    }
    if (nseg_cut > 0) {
        const void *rec = precision == GBD_FP64 ? (const void *)(plan->r64 + n_main) : (const void *)(plan->r32 + n_main);
        const void *crec = precision == GBD_FP64 ? (const void *)plan->c64 : (const void *)plan->c32;
        void *wide = static_cast<char *>(partial) + reduce_wide_offset(nseg2, M);
        HIP_TRY(launch_eval_cut(precision, level, gc, rec, crec, faddeeva_coef(), nseg_main - nseg2, wide, ctx->stream),
                "truncated-beamlet kernel launch");
    }
    if (reduce) {
        EvalGeom gr = n_main > 0 ? g : gc;
        gr.nseg = total;
        EvalGuard gd;
        if (guard) {
            guard->check_key = s.form == 3 && s.half && !by_rows;  // the FP16 form's scale came from the key
            gd = *guard;
        }
        HIP_TRY(launch_reduce(precision, gr, nseg2, partial, out, ctx->stream, gd), "reduce kernel launch");
    }
    return GBD_OK;
}

// Whether the beamlets meet the plane at one distance with one curvature: the
// setup then takes these from the host (gbd_terms.h).
bool shares_terms(const gbd_beamlets_s *b, const gbd_plane_s *p) {
    return b->one_matrix && p->g.n[0] == 0.0 && p->g.n[1] == 0.0;
}

// The post of the last launched setup's status.
StatusPost pending_post(const gbd_plan_s *plan) {
    StatusPost sp;
    sp.status = plan->status_cur;
    sp.post = plan->status_post;
    sp.seq = plan->status_seq;
    return sp;
}

// The setup in two halves: plan_setup_launch enqueues the setup kernel and
// the post of its status pair (status_post_kernel; with post false the
// caller has the post made, as gbd_eval does by its evaluation kernel), and
// plan_setup_finish waits for the post and takes the status.
int plan_setup_launch(gbd_ctx_s *ctx, gbd_plan_s *plan, gbd_beamlets_s *b, gbd_plane_s *p, bool post = true) {
    if (b->dev.n > plan->capacity)
        return fail(GBD_ERANGE, "plan capacity %lld < %lld beamlets", (long long)plan->capacity, (long long)b->dev.n);
    int rc = ensure_device(ctx);
    if (rc) return rc;
    plan->ready = false;
    plan->spec_ok = false;
    plan->status_cur = nullptr;
    plan->n = b->dev.n;
    plan->pl = p->g;
    plan->n_cut = b->dev.n_cut;
    if (b->dev.n_cut > 0 && (!plan->c64 || !plan->c32)) {
        const size_t cap = (size_t)std::max<int64_t>(1, plan->capacity);
        if (!plan->c64) HIP_TRY(hipMalloc(&plan->c64, cap * sizeof(RecCut64)), "hipMalloc(truncation records)");
        if (!plan->c32) HIP_TRY(hipMalloc(&plan->c32, cap * sizeof(RecCut32)), "hipMalloc(truncation records)");
    }
    if (b->dev.order && (!plan->h64 || !plan->h32)) {
        const size_t cap = (size_t)std::max<int64_t>(1, plan->capacity);
        if (!plan->h64) HIP_TRY(hipMalloc(&plan->h64, cap * sizeof(RecHG64)), "hipMalloc(Hermite-Gaussian records)");
        if (!plan->h32) HIP_TRY(hipMalloc(&plan->h32, cap * sizeof(RecHG32)), "hipMalloc(Hermite-Gaussian records)");
    }
    plan->rows = b->dev.rows;
    if (plan->rows > plan->row_cap) {
        // for any beamlets the plan takes (at most one chunk per kRowGain beamlets)
        const int64_t cap = std::max<int64_t>(plan->rows, plan->capacity / kRowGain);
        if (plan->row_start) (void)hipFree(plan->row_start);
        plan->row_start = nullptr;
        plan->row_cap = 0;
        HIP_TRY(hipMalloc(&plan->row_start, (size_t)(cap + 1) * sizeof(int32_t)), "hipMalloc(row chunks)");
        plan->row_cap = cap;
    }
    if (b->dev.n > 0) {
        // the axial term l0 / lambda is common to every beamlet: reduce it once
        const double g0 = b->dev.l0 / b->dev.lam;
        const double gturns = g0 - nearbyint(g0);
        if (!plan->status_zeroed) {
            HIP_TRY(hipMemsetAsync(plan->status_dev, 0, 4 * sizeof(uint32_t), ctx->stream), "hipMemsetAsync(status)");
            plan->status_zeroed = true;
        }
        const bool hg = b->dev.order != nullptr;
        const bool cut = b->dev.n_cut > 0;
        uint32_t *status = plan->status_dev + 2 * plan->status_parity;
        uint32_t *status_next = plan->status_dev + 2 * (plan->status_parity ^ 1);
        MatrixTerms mt;
        const bool shared = shares_terms(b, p);
        if (shared)
            mt = matrix_terms(b->abcd0, (p->g.n[2] * p->g.O[2]) / p->g.n[2], b->dev.lam, b->w00);
        HIP_TRY(launch_setup(b->dev, p->g, gturns, shared ? &mt : nullptr, plan->r64, plan->r32, hg ? plan->h64 : nullptr,
                             hg ? plan->h32 : nullptr, cut ? plan->c64 : nullptr, cut ? plan->c32 : nullptr,
                             status, status_next, plan->row_start, ctx->stream),
                "setup kernel launch");
        plan->status_parity ^= 1;
        plan->status_seq++;
        plan->status_cur = status;
        if (post) HIP_TRY(launch_status_post(pending_post(plan), ctx->stream), "status post launch");
    }
    return GBD_OK;
}

int plan_setup_finish(gbd_ctx_s *ctx, gbd_plan_s *plan) {
    plan->flags = 0;
    if (plan->status_cur) {
        // poll the posted word for this setup's sequence number: busy at
        // first, then yielding; after a second (a stream with long work queued
        // ahead) wait for the stream, after which the post is visible
        const uint32_t seq = plan->status_seq;
        const volatile uint64_t *post = plan->status_post;
        uint64_t w = *post;
        const auto t0 = std::chrono::steady_clock::now();
        for (uint32_t spins = 0; (uint32_t)(w >> 32) != seq; w = *post) {
            if (++spins < 4096) continue;
            const auto dt = std::chrono::steady_clock::now() - t0;
            if (dt > std::chrono::seconds(1)) {
                HIP_TRY(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");
                w = *post;
                if ((uint32_t)(w >> 32) != seq) return fail(GBD_EHIP, "the setup status was not posted");
                break;
            }
            if (dt > std::chrono::microseconds(200)) std::this_thread::yield();
        }
        const uint32_t st = (uint32_t)w & 0xffffu;
        // FP16 separable form: largest term 2^P over the grid -> scale 2^(2 kSepHalfExp - P)
        const uint32_t key = ((uint32_t)w >> 16) & 0xfffu;
        plan->sep_key = key;
        plan->sep_scale = seph_scale(key);
        if (st & FLAG_PARALLEL) return fail(GBD_EPARALLEL, "a base ray is parallel to the detector plane");
        if (st & FLAG_BRANCH)
            return fail(GBD_EBRANCH, "an eigenvalue of A + B Q1^-1 lies off the principal branch (inverting system)");
        if (st & FLAG_NONFINITE) return fail(GBD_EINVAL, "non-finite beamlet parameters after propagation");
        if (st & FLAG_HG_TILT)
            return fail(GBD_EINVAL, "higher-order and truncated beamlets need a detector plane normal to the axis");
        plan->flags = st & kFormFlags;
    }
    plan->ready = true;
    plan->spec_ok = plan->status_cur != nullptr;
    return GBD_OK;
}

int plan_setup_impl(gbd_ctx_s *ctx, gbd_plan_s *plan, gbd_beamlets_s *b, gbd_plane_s *p) {
    const int rc = plan_setup_launch(ctx, plan, b, p);
    return rc ? rc : plan_setup_finish(ctx, plan);
}

void plan_destroy(gbd_plan_s *plan) {
    if (!plan) return;
    if (plan->r64) (void)hipFree(plan->r64);
    if (plan->r32) (void)hipFree(plan->r32);
    if (plan->q64) (void)hipFree(plan->q64);
    if (plan->h64) (void)hipFree(plan->h64);
    if (plan->h32) (void)hipFree(plan->h32);
    if (plan->c64) (void)hipFree(plan->c64);
    if (plan->c32) (void)hipFree(plan->c32);
    if (plan->row_start) (void)hipFree(plan->row_start);
    if (plan->status_dev) (void)hipFree(plan->status_dev);
    if (plan->scratch) (void)hipFree(plan->scratch);
    for (void *p : plan->held) (void)hipFree(p);
    if (plan->status_post) {
        // a post still in flight writes this memory: let the device finish first
        (void)hipDeviceSynchronize();
        (void)hipHostFree(plan->status_post);
    }
    delete plan;
}

int plan_new(gbd_ctx_s *ctx, int64_t capacity, gbd_plan_s **out) {
    gbd_plan_s *p = new (std::nothrow) gbd_plan_s();
    if (!p) return fail(GBD_ENOMEM, "host allocation failed");
    p->ctx = ctx;
    p->capacity = capacity;
    const size_t cap = (size_t)std::max<int64_t>(1, capacity);
    hipError_t e = hipMalloc(&p->r64, cap * sizeof(Rec64));
    if (e == hipSuccess) e = hipMalloc(&p->r32, cap * sizeof(Rec32));
    if (e == hipSuccess) e = hipMalloc(&p->q64, cap * sizeof(RecSq64));
    if (e == hipSuccess) e = hipMalloc(&p->status_dev, 4 * sizeof(uint32_t));
    if (e == hipSuccess) e = hipHostMalloc(&p->status_post, sizeof(uint64_t), hipHostMallocCoherent);
    if (e == hipSuccess) *p->status_post = 0;
    if (e != hipSuccess) {
        plan_destroy(p);
        return hip_fail(e, "plan allocation");
    }
    *out = p;
    return GBD_OK;
}

int grow(DevBuf &b, size_t bytes, const char *what) {
    if (bytes <= b.bytes) return GBD_OK;
    if (b.p) (void)hipFree(b.p);
    b.p = nullptr;
    b.bytes = 0;
    bytes = std::max<size_t>(bytes, 256);
    hipError_t e = hipMalloc(&b.p, bytes);
    if (e != hipSuccess) return hip_fail(e, what);
    b.bytes = bytes;
    return GBD_OK;
}

void batch_free(BatchWork &w) {
    DevBuf *all[] = {&w.rec,    &w.l5,   &w.e0t,     &w.tab1,  &w.tab2, &w.e0,
                     &w.e0part, &w.part, &w.flags, &w.point, &w.row_sums, &w.terms};
    if (w.stage_ev) {
        (void)hipEventSynchronize(w.stage_ev);
        (void)hipEventDestroy(w.stage_ev);
    }
    for (DevBuf *b : all)
        if (b->p) (void)hipFree(b->p);
    if (w.host_flags) (void)hipHostFree(w.host_flags);
    if (w.stage) (void)hipHostFree(w.stage);
    if (w.metrics) {
        // a batch not collected may still write them: let the device finish first
        (void)hipDeviceSynchronize();
        (void)hipHostFree(w.metrics);
    }
    w = BatchWork();
}

}  // namespace

extern "C" {

const char *gbd_last_error(void) { return g_err.c_str(); }

int gbd_ctx_create(gbd_ctx_t *out, int device, void *hip_stream) {
    if (!out) return fail(GBD_EINVAL, "out is NULL");
    int count = 0;
    HIP_TRY(hipGetDeviceCount(&count), "hipGetDeviceCount");
    if (device < 0 || device >= count) return fail(GBD_EINVAL, "device %d out of range (%d devices)", device, count);
    HIP_TRY(hipSetDevice(device), "hipSetDevice");
    if (device >= kMaxDevices) return fail(GBD_EINVAL, "device %d: at most %d devices", device, kMaxDevices);
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_dev[device]) {
            void *ptr = nullptr;
            HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(static partial buffer)");
            if (!ptr) return fail(GBD_EHIP, "hipGetSymbolAddress(static partial buffer) returned NULL");
            g_scratch_dev[device] = ptr;
        }
    }
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device), "hipDeviceGetAttribute");
    gbd_ctx_s *c = new (std::nothrow) gbd_ctx_s();
    if (!c) return fail(GBD_ENOMEM, "host allocation failed");
    c->pool = std::make_shared<DevPool>();
    c->device = device;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->cus = cus > 0 ? cus : 256;
    c->own_plan = nullptr;
    *out = c;
    return GBD_OK;
}

int gbd_ctx_set_stream(gbd_ctx_t ctx, void *hip_stream) {
    if (!ctx) return fail(GBD_EINVAL, "ctx is NULL");
    hipStream_t next = static_cast<hipStream_t>(hip_stream);
    if (next != ctx->stream) {
        // pooled blocks are reused in stream order: drain the old stream first
        HIP_TRY(hipSetDevice(ctx->device), "hipSetDevice");
        HIP_TRY(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");
    }
    ctx->stream = next;
    return GBD_OK;
}

void gbd_ctx_destroy(gbd_ctx_t ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    if (ctx->up_ev) {
        (void)hipEventSynchronize(ctx->up_ev);
        (void)hipEventDestroy(ctx->up_ev);
    }
    if (ctx->up_stage) (void)hipHostFree(ctx->up_stage);
    plan_destroy(ctx->own_plan);
    batch_free(ctx->batch);
    for (auto *v : {&ctx->timed, &ctx->spare_events})
        for (auto &ev : *v) {
            (void)hipEventDestroy(ev.first);
            (void)hipEventDestroy(ev.second);
        }
    delete ctx;
}

int gbd_ctx_set_kernel_timing(gbd_ctx_t ctx, int enable) {
    if (!ctx) return fail(GBD_EINVAL, "ctx is NULL");
    ctx->timing = enable != 0;
    return GBD_OK;
}

int gbd_ctx_kernel_times(gbd_ctx_t ctx, float *ms_out, int32_t cap, int32_t *n) {
    if (!ctx || !n || (cap > 0 && !ms_out)) return fail(GBD_EINVAL, "NULL argument");
    if (cap < 0) return fail(GBD_EINVAL, "negative capacity");
    int rc = ensure_device(ctx);
    if (rc) return rc;
    int32_t k = 0;
    hipError_t first_err = hipSuccess;
    for (auto &ev : ctx->timed) {
        float ms = 0.0f;
        hipError_t e = hipEventSynchronize(ev.second);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev.first, ev.second);
        if (e != hipSuccess && first_err == hipSuccess) first_err = e;
        if (k < cap) ms_out[k] = ms;
        k++;
        ctx->spare_events.push_back(ev);
    }
    ctx->timed.clear();
    *n = k;
    if (first_err != hipSuccess) return hip_fail(first_err, "kernel timing events");
    return GBD_OK;
}

static int beamlets_impl(gbd_ctx_t ctx, gbd_beamlets_t *out, int64_t n, double lambda, double l0, const double *r1,
                  const double *th1, const double *w0, int64_t n_w0, const double *amp, const double *path,
                  const double *abcd, int64_t n_abcd, const double *base, double sympl_tol,
                  const int32_t *order = nullptr, const double *edge = nullptr) {
    if (!ctx || !out) return fail(GBD_EINVAL, "ctx/out is NULL");
    if (!(sympl_tol > 0.0 && sympl_tol <= 1e-3)) return fail(GBD_EINVAL, "sympl_tol must be in (0, 1e-3]");
    if (n < 0) return fail(GBD_EINVAL, "n < 0");
    if (!(lambda > 0.0) || !std::isfinite(lambda)) return fail(GBD_EINVAL, "lambda must be finite and > 0");
    if (!std::isfinite(l0)) return fail(GBD_EINVAL, "l0 must be finite");
    if (n > 0) {
        if (!r1 || !w0 || !abcd) return fail(GBD_EINVAL, "r1, w0 and abcd are required");
        if (!(n_w0 == 1 || n_w0 == n)) return fail(GBD_EINVAL, "n_w0 must be 1 or n");
        if (!(n_abcd == 1 || n_abcd == n)) return fail(GBD_EINVAL, "n_abcd must be 1 or n");
        if (!finite_all(r1, 2 * n) || (th1 && !finite_all(th1, 2 * n)) || (amp && !finite_all(amp, 2 * n)) ||
            (path && !finite_all(path, n)) || !finite_all(abcd, 16 * n_abcd) || (base && !finite_all(base, 5 * n)))
            return fail(GBD_EINVAL, "non-finite input");
        for (int64_t i = 0; i < n_w0; i++)
            if (!(w0[i] > 0.0) || !std::isfinite(w0[i])) return fail(GBD_EINVAL, "w0[%lld] must be finite and > 0", (long long)i);
        for (int64_t i = 0; i < n_abcd; i++)
            if (!(base ? symplectic_balanced(abcd + 16 * i, sympl_tol) : symplectic(abcd + 16 * i, sympl_tol)))
                return fail(GBD_ENOTSYMPLECTIC, "abcd[%lld] is not symplectic", (long long)i);
        if (order)
            for (int64_t i = 0; i < 2 * n; i++)
                if (order[i] < 0 || order[i] > 2)
                    return fail(GBD_EINVAL, "order[%lld][%lld] = %d is outside 0 ... 2", (long long)(i / 2),
                                (long long)(i % 2), order[i]);
        if (edge) {
            if (!finite_all(edge, 3 * n)) return fail(GBD_EINVAL, "non-finite edge");
            for (int64_t i = 0; i < n; i++) {
                const double ex = edge[3 * i], ey = edge[3 * i + 1];
                if ((ex != 0.0 || ey != 0.0) && !(std::fabs(ex * ex + ey * ey - 1.0) <= 1e-12))
                    return fail(GBD_EINVAL, "edge[%lld]: the normal (e_x, e_y) must have unit length", (long long)i);
            }
        }
    } else {
        n_w0 = 1;
        n_abcd = 1;
        base = nullptr;
        order = nullptr;
        edge = nullptr;
    }
    // truncated beamlets are stored last (stable order otherwise): the
    // evaluation gives them a kernel of their own
    std::vector<int64_t> perm((size_t)std::max<int64_t>(n, 0));
    int64_t n_cut = 0;
    {
        size_t at = 0;
        for (int64_t i = 0; i < n; i++)
            if (!edge || (edge[3 * i] == 0.0 && edge[3 * i + 1] == 0.0)) perm[at++] = i;
        for (int64_t i = 0; i < n; i++)
            if (edge && (edge[3 * i] != 0.0 || edge[3 * i + 1] != 0.0)) {
                perm[at++] = i;
                n_cut++;
            }
    }
    std::vector<int32_t> chunks;
    if (n_abcd == 1 && !base) chunks = row_chunks(n - n_cut, perm, r1, th1, w0, n_w0, order);
    const int64_t n_rows = chunks.empty() ? 0 : (int64_t)chunks.size() - 1;
    bool higher = false;
    if (order)
        for (int64_t i = 0; i < 2 * n && !higher; i++) higher = order[i] != 0;
    int rc = ensure_device(ctx);
    if (rc) return rc;
    // one device block: r1, th1, amp [n][2]; w0 [n_w0]; path [n]; abcd [n_abcd][16]; base [n][5];
    // edge [n][3]; orders [n][2] int32; the row chunks' starts int32 and their bits
    const size_t nn = (size_t)std::max<int64_t>(n, 1);
    const size_t off_r1 = 0, off_th1 = off_r1 + 2 * nn, off_amp = off_th1 + 2 * nn, off_w0 = off_amp + 2 * nn,
                 off_path = off_w0 + (size_t)n_w0, off_abcd = off_path + nn, off_base = off_abcd + 16 * (size_t)n_abcd,
                 off_edge = off_base + (base ? 5 * nn : 0), off_order = off_edge + (edge ? 3 * nn : 0),
                 off_rows = off_order + (order ? nn : 0),
                 off_bits = off_rows + (n_rows ? ((size_t)n_rows + 2) / 2 : 0),
                 total = off_bits + (n_rows ? ((size_t)(n - n_cut) + 63) / 64 : 0);
    const size_t bytes = total * sizeof(double);
    if (!ctx->up_ev) HIP_TRY(hipEventCreateWithFlags(&ctx->up_ev, hipEventDisableTiming), "hipEventCreate");
    if (ctx->up_pending) HIP_TRY(hipEventSynchronize(ctx->up_ev), "hipEventSynchronize");
    ctx->up_pending = false;
    if (bytes > ctx->up_bytes) {
        if (ctx->up_stage) (void)hipHostFree(ctx->up_stage);
        ctx->up_stage = nullptr;
        ctx->up_bytes = 0;
        const size_t want = std::max<size_t>(bytes, (size_t)1 << 20);
        HIP_TRY(hipHostMalloc(&ctx->up_stage, want, hipHostMallocDefault), "hipHostMalloc(beamlet staging)");
        ctx->up_bytes = want;
    }
    double *host = static_cast<double *>(ctx->up_stage);
    bool in_order = n > 0;  // stored as the caller has them: whole arrays are copied
    for (int64_t i = 0; i < n; i++) in_order &= perm[i] == i;
    // the n rows of one array, in stored order (no source: zeros)
    auto put_rows = [&](auto *dst, auto width, const auto *src) {
        constexpr int W = decltype(width)::value;
        if (!src)
            memset(dst, 0, (size_t)n * W * sizeof *dst);
        else if (in_order)
            memcpy(dst, src, (size_t)n * W * sizeof *dst);
        else
            for (int64_t i = 0; i < n; i++) memcpy(dst + W * i, src + W * perm[i], W * sizeof *dst);
    };
    using std::integral_constant;
    if (n > 0) {
        put_rows(&host[off_r1], integral_constant<int, 2>(), r1);
        put_rows(&host[off_th1], integral_constant<int, 2>(), th1);
        if (amp)
            put_rows(&host[off_amp], integral_constant<int, 2>(), amp);
        else
            for (int64_t i = 0; i < n; i++) {
                host[off_amp + 2 * i] = 1.0;
                host[off_amp + 2 * i + 1] = 0.0;
            }
        if (n_w0 == 1 || order)  // orders reorder beamlets of one waist only (row_chunks)
            memcpy(&host[off_w0], w0, (size_t)n_w0 * sizeof(double));
        else
            put_rows(&host[off_w0], integral_constant<int, 1>(), w0);
        put_rows(&host[off_path], integral_constant<int, 1>(), path);
        if (n_abcd == 1)
            memcpy(&host[off_abcd], abcd, 16 * sizeof(double));
        else
            put_rows(&host[off_abcd], integral_constant<int, 16>(), abcd);
        if (base) put_rows(&host[off_base], integral_constant<int, 5>(), base);
        if (edge) put_rows(&host[off_edge], integral_constant<int, 3>(), edge);
        if (order) put_rows(reinterpret_cast<int32_t *>(&host[off_order]), integral_constant<int, 2>(), order);
        memset(&host[off_rows], 0, (total - off_rows) * sizeof(double));
    } else {
        memset(host, 0, bytes);
        host[off_w0] = 1.0;
        for (int i = 0; i < 4; i++) host[off_abcd + 5 * i] = 1.0;
    }
    if (n_rows) {
        memcpy(&host[off_rows], chunks.data(), chunks.size() * sizeof(int32_t));
        uint32_t *bits = reinterpret_cast<uint32_t *>(&host[off_bits]);
        for (int64_t c = 0; c < n_rows; c++) bits[chunks[c] >> 5] |= 1u << (chunks[c] & 31);
    }
    void *mem = nullptr;
    const size_t cls = DevPool::size_class(total * sizeof(double));
    HIP_TRY(ctx->pool->get(cls, &mem), "hipMalloc(beamlets)");
    hipError_t e = hipMemcpyAsync(mem, host, bytes, hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) e = hipEventRecord(ctx->up_ev, ctx->stream);
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(ctx->stream);
        ctx->pool->put(mem, cls);
        return hip_fail(e, "beamlet upload");
    }
    ctx->up_pending = true;
    gbd_beamlets_s *b = new (std::nothrow) gbd_beamlets_s();
    if (!b) {
        ctx->pool->put(mem, cls);
        return fail(GBD_ENOMEM, "host allocation failed");
    }
    double *d = static_cast<double *>(mem);
    b->ctx = ctx;
    b->mem = mem;
    b->mem_class = cls;
    b->pool = ctx->pool;
    b->dev.n = n;
    b->dev.n_w0 = n_w0;
    b->dev.n_abcd = n_abcd;
    b->dev.lam = lambda;
    b->dev.l0 = l0;
    b->dev.r1 = d + off_r1;
    b->dev.th1 = d + off_th1;
    b->dev.amp = d + off_amp;
    b->dev.w0 = d + off_w0;
    b->dev.path = d + off_path;
    b->dev.abcd = d + off_abcd;
    b->dev.base = base ? d + off_base : nullptr;
    b->dev.order = order ? reinterpret_cast<const int32_t *>(d + off_order) : nullptr;
    b->dev.edge = edge ? d + off_edge : nullptr;
    b->dev.n_cut = n_cut;
    b->dev.row_start = n_rows ? reinterpret_cast<const int32_t *>(d + off_rows) : nullptr;
    b->dev.row_bits = n_rows ? reinterpret_cast<const uint32_t *>(d + off_bits) : nullptr;
    b->dev.rows = (int32_t)n_rows;
    b->higher_order = higher;
    bool one = n > 0 && n_abcd == 1 && !base;
    for (int64_t i = 1; i < n_w0 && one; i++) one = w0[i] == w0[0];
    b->one_matrix = one;
    if (b->one_matrix) {
        memcpy(b->abcd0, abcd, sizeof b->abcd0);
        b->w00 = w0[0];
    }
    *out = b;
    return GBD_OK;
}

int gbd_beamlets(gbd_ctx_t ctx, gbd_beamlets_t *out, int64_t n, double lambda, double l0, const double *r1,
                 const double *th1, const double *w0, int64_t n_w0, const double *amp, const double *path,
                 const double *abcd, int64_t n_abcd) {
    return beamlets_impl(ctx, out, n, lambda, l0, r1, th1, w0, n_w0, amp, path, abcd, n_abcd, nullptr, 1e-10);
}

int gbd_beamlets_traced(gbd_ctx_t ctx, gbd_beamlets_t *out, int64_t n, double lambda, double l0, const double *r1,
                        const double *th1, const double *w0, int64_t n_w0, const double *amp, const double *path,
                        const double *abcd, const double *base, double sympl_tol) {
    if (n > 0 && !base) return fail(GBD_EINVAL, "base is NULL");
    return beamlets_impl(ctx, out, n, lambda, l0, r1, th1, w0, n_w0, amp, path, abcd, n, base, sympl_tol);
}

int gbd_beamlets_hg(gbd_ctx_t ctx, gbd_beamlets_t *out, int64_t n, double lambda, double l0, const double *r1,
                    const double *th1, const double *w0, int64_t n_w0, const double *amp, const double *path,
                    const double *abcd, int64_t n_abcd, const int32_t *order) {
    if (n > 0 && !order) return fail(GBD_EINVAL, "order is NULL");
    return beamlets_impl(ctx, out, n, lambda, l0, r1, th1, w0, n_w0, amp, path, abcd, n_abcd, nullptr, 1e-10, order);
}

int gbd_beamlets_truncated(gbd_ctx_t ctx, gbd_beamlets_t *out, int64_t n, double lambda, double l0,
                           const double *r1, const double *th1, const double *w0, int64_t n_w0, const double *amp,
                           const double *path, const double *abcd, int64_t n_abcd, const double *edge) {
    if (n > 0 && !edge) return fail(GBD_EINVAL, "edge is NULL");
    return beamlets_impl(ctx, out, n, lambda, l0, r1, th1, w0, n_w0, amp, path, abcd, n_abcd, nullptr, 1e-10,
                         nullptr, edge);
}

int gbd_trace(gbd_ctx_t ctx, int32_t n_mirrors, const double *mirrors, double z_in, double z_out, double l0,
              int64_t n, const double *r1, const double *th1, double dr, double dth, double *base_out,
              double *abcd_out, int32_t *flags_out) {
    if (!ctx) return fail(GBD_EINVAL, "ctx is NULL");
    if (n_mirrors < 0 || n_mirrors > kMaxMirrors) return fail(GBD_EINVAL, "n_mirrors must be in [0, %d]", kMaxMirrors);
    if (n < 0) return fail(GBD_EINVAL, "n < 0");
    if (!(dr > 0.0) || !(dth > 0.0) || !std::isfinite(dr) || !std::isfinite(dth))
        return fail(GBD_EINVAL, "dr and dth must be finite and > 0");
    if (!std::isfinite(z_in) || !std::isfinite(z_out) || !std::isfinite(l0)) return fail(GBD_EINVAL, "non-finite plane");
    if (n_mirrors > 0 && !mirrors) return fail(GBD_EINVAL, "mirrors is NULL");
    if (n > 0 && (!r1 || !base_out || !abcd_out || !flags_out)) return fail(GBD_EINVAL, "NULL array");
    TraceSystem S;
    S.n = n_mirrors;
    S.z_in = z_in;
    S.z_out = z_out;
    S.l0 = l0;
    for (int i = 0; i < n_mirrors; i++) {
        const double *e = mirrors + 5 * i;
        if (!finite_all(e, 5)) return fail(GBD_EINVAL, "non-finite mirror %d", i);
        S.m[i] = TraceMirror{e[0], e[1] == 0.0 ? 0.0 : 1.0 / e[1], e[2], e[3], e[4]};
    }
    if (n > 0 && (!finite_all(r1, 2 * n) || (th1 && !finite_all(th1, 2 * n))))
        return fail(GBD_EINVAL, "non-finite ray");
    if (n == 0) return GBD_OK;
    int rc = ensure_device(ctx);
    if (rc) return rc;
    // device block: r1 [n][2], th1 [n][2], base [n][5], abcd [n][16], flags [n] (int32)
    const size_t nd = (size_t)n;
    const size_t off_th = 2 * nd, off_base = 4 * nd, off_abcd = 9 * nd, off_flags = 25 * nd;
    void *mem = nullptr;  // a pooled block: returned after the synchronisation below
    const size_t cls = DevPool::size_class(off_flags * sizeof(double) + nd * sizeof(int32_t));
    HIP_TRY(ctx->pool->get(cls, &mem), "hipMalloc(trace)");
    double *d = static_cast<double *>(mem);
    int32_t *dflags = reinterpret_cast<int32_t *>(d + off_flags);
    hipError_t e = hipMemcpyAsync(d, r1, 2 * nd * sizeof(double), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess && th1) e = hipMemcpyAsync(d + off_th, th1, 2 * nd * sizeof(double), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess)
        e = launch_trace(S, n, d, th1 ? d + off_th : nullptr, dr, dth, d + off_base, d + off_abcd, dflags, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(base_out, d + off_base, 5 * nd * sizeof(double), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(abcd_out, d + off_abcd, 16 * nd * sizeof(double), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(flags_out, dflags, nd * sizeof(int32_t), hipMemcpyDeviceToHost, ctx->stream);
    const hipError_t es = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = es;
    ctx->pool->put(mem, cls);
    if (e != hipSuccess) return hip_fail(e, "trace");
    return GBD_OK;
}

void gbd_beamlets_free(gbd_beamlets_t b) {
    if (!b) return;
    if (b->mem) b->pool->put(b->mem, b->mem_class);
    delete b;
}

int gbd_plane(gbd_ctx_t ctx, gbd_plane_t *out, const double origin[3], const double normal[3], const double xhint[3],
              int32_t nx, int32_t ny, double dx, double dy) {
    if (!ctx || !out || !origin || !normal || !xhint) return fail(GBD_EINVAL, "NULL argument");
    if (nx < 0 || ny < 0) return fail(GBD_EINVAL, "nx, ny must be >= 0");
    if (!(dx > 0.0) || !(dy > 0.0) || !std::isfinite(dx) || !std::isfinite(dy)) return fail(GBD_EINVAL, "dx, dy must be finite and > 0");
    if (!finite_all(origin, 3) || !finite_all(normal, 3) || !finite_all(xhint, 3)) return fail(GBD_EINVAL, "non-finite plane");
    PlaneGeom g;
    const double nn = sqrt(normal[0] * normal[0] + normal[1] * normal[1] + normal[2] * normal[2]);
    if (!(nn > 0.0)) return fail(GBD_EINVAL, "normal has zero length");
    for (int i = 0; i < 3; i++) {
        g.O[i] = origin[i];
        g.n[i] = normal[i] / nn;
    }
    // e1: xhint with its normal component removed (Gram-Schmidt); e2 = n x e1
    const double hn = xhint[0] * g.n[0] + xhint[1] * g.n[1] + xhint[2] * g.n[2];
    double e1[3];
    for (int i = 0; i < 3; i++) e1[i] = xhint[i] - hn * g.n[i];
    const double el = sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
    const double hl = sqrt(xhint[0] * xhint[0] + xhint[1] * xhint[1] + xhint[2] * xhint[2]);
    if (!(el > 1e-9 * hl)) return fail(GBD_EINVAL, "xhint is parallel to the normal");
    for (int i = 0; i < 3; i++) g.e1[i] = e1[i] / el;
    g.e2[0] = g.n[1] * g.e1[2] - g.n[2] * g.e1[1];
    g.e2[1] = g.n[2] * g.e1[0] - g.n[0] * g.e1[2];
    g.e2[2] = g.n[0] * g.e1[1] - g.n[1] * g.e1[0];
    g.nx = nx;
    g.ny = ny;
    g.dx = dx;
    g.dy = dy;
    gbd_plane_s *p = new (std::nothrow) gbd_plane_s();
    if (!p) return fail(GBD_ENOMEM, "host allocation failed");
    p->g = g;
    *out = p;
    return GBD_OK;
}

void gbd_plane_free(gbd_plane_t p) { delete p; }

int gbd_plan_create(gbd_ctx_t ctx, gbd_plan_t *out, int64_t capacity) {
    if (!ctx || !out) return fail(GBD_EINVAL, "ctx/out is NULL");
    if (capacity < 0) return fail(GBD_EINVAL, "capacity < 0");
    int rc = ensure_device(ctx);
    if (rc) return rc;
    return plan_new(ctx, capacity, out);
}

int gbd_plan_setup(gbd_ctx_t ctx, gbd_plan_t plan, gbd_beamlets_t b, gbd_plane_t p) {
    if (!ctx || !plan || !b || !p) return fail(GBD_EINVAL, "NULL argument");
    if (b->ctx != ctx) return fail(GBD_EINVAL, "the beamlets belong to another context");
    return plan_setup_impl(ctx, plan, b, p);
}

int gbd_plan_eval(gbd_ctx_t ctx, gbd_plan_t plan, int precision, void *field_out, int64_t out_bytes,
                  const gbd_eval_opts *opts) {
    if (!ctx || !plan) return fail(GBD_EINVAL, "NULL argument");
    return plan_eval_impl(ctx, plan, precision, field_out, out_bytes, opts);
}

int gbd_plan_eval_noalloc(gbd_ctx_t ctx, gbd_plan_t plan, int precision, void *field_out, int64_t out_bytes,
                          const gbd_eval_opts *opts) {
    if (!ctx || !plan) return fail(GBD_EINVAL, "NULL argument");
    void *buf = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        buf = g_scratch_dev[ctx->device];
    }
    if (!buf) return fail(GBD_EHIP, "device %d has no static partial buffer address", ctx->device);
    return plan_eval_impl(ctx, plan, precision, field_out, out_bytes, opts, buf, (size_t)GBD_NOALLOC_SCRATCH_BYTES);
}

void gbd_plan_free(gbd_plan_t plan) { plan_destroy(plan); }

int gbd_issue_probe(gbd_ctx_t ctx, int32_t cls, int32_t iters, double *ms_out, double *wave_instructions_out) {
    if (!ctx || !ms_out || !wave_instructions_out) return fail(GBD_EINVAL, "NULL argument");
    if (cls < 0 || cls > 9) return fail(GBD_EINVAL, "class must be 0 ... 9");
    if (iters < 1) return fail(GBD_EINVAL, "iters must be >= 1");
    int rc = ensure_device(ctx);
    if (rc) return rc;
    const int blocks = ctx->cus * 8;
    float *sink = nullptr;
    HIP_TRY(hipMalloc(&sink, (size_t)blocks * 256 * sizeof(float)), "hipMalloc(probe)");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = launch_issue_probe(cls, blocks, iters, sink, ctx->stream);
    if (e == hipSuccess) e = hipEventRecord(e0, ctx->stream);
    if (e == hipSuccess) e = launch_issue_probe(cls, blocks, iters, sink, ctx->stream);
    if (e == hipSuccess) e = hipEventRecord(e1, ctx->stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(sink);
    if (e != hipSuccess) return hip_fail(e, "issue probe");
    const double waves = (double)blocks * 4.0;
    *ms_out = ms;
    // class 9 counts its MFMA instructions
    *wave_instructions_out = waves * (double)iters * ((cls <= 3 || cls == 7 || cls == 8) ? 16.0 : 4.0);
    return GBD_OK;
}

int gbd_plan_shape(gbd_ctx_t ctx, gbd_plan_t plan, int precision, const gbd_eval_opts *opts, gbd_eval_opts *resolved) {
    if (!ctx || !plan || !resolved) return fail(GBD_EINVAL, "NULL argument");
    Shape s = choose_shape(ctx, precision, plan->n - plan->n_cut, plan->pl, plan->flags, opts);
    EvalGeom g = make_geom(plan->pl, plan->n - plan->n_cut, s);
    resolved->rows_per_lane = s.rows;
    resolved->waves = s.waves;
    resolved->segments = g.nseg;
    resolved->variant = form_variant(precision, s.form, s.half);
    return GBD_OK;
}

int gbd_eval(gbd_ctx_t ctx, gbd_beamlets_t b, gbd_plane_t p, int precision, void *field_out, int64_t out_bytes,
             const gbd_eval_opts *opts) {
    if (!ctx || !b || !p) return fail(GBD_EINVAL, "NULL argument");
    if (b->ctx != ctx) return fail(GBD_EINVAL, "the beamlets belong to another context");
    if (precision != GBD_FP64 && precision != GBD_MIXED) return fail(GBD_EINVAL, "precision must be GBD_FP64 or GBD_MIXED");
    const int64_t M = (int64_t)p->g.nx * p->g.ny;
    const int64_t elem = precision == GBD_FP64 ? 16 : 8;
    if (M > 0 && !field_out) return fail(GBD_EINVAL, "field_out is NULL");
    if (M > 0 && out_bytes < M * elem)
        return fail(GBD_ERANGE, "field_out holds %lld bytes, %lld needed", (long long)out_bytes, (long long)(M * elem));
    if (!ctx->own_plan || ctx->own_plan->capacity < b->dev.n) {
        plan_destroy(ctx->own_plan);
        ctx->own_plan = nullptr;
        int rc = ensure_device(ctx);
        if (rc) return rc;
        rc = plan_new(ctx, std::max<int64_t>(b->dev.n, 1024), &ctx->own_plan);
        if (rc) return rc;
    }
    gbd_plan_s *plan = ctx->own_plan;
    if (!plan->spec_ok) {
        int rc = plan_setup_impl(ctx, plan, b, p);
        if (rc) return rc;
        return plan_eval_impl(ctx, plan, precision, field_out, out_bytes, opts);
    }
    // The last setup of this plan succeeded: launch the evaluation right
    // behind this setup with its flags and FP16 scale, before the host has
    // read the new status, so no host round trip separates the two kernels.
    // The reduction writes the output only if the status has no error and
    // the same key and route flags (EvalGuard); otherwise it writes nothing and,
    // for a mere change of form or scale, the evaluation runs again below.
    const uint32_t pflags = plan->flags;
    const uint32_t pkey = plan->sep_key;
    const int pscale = plan->sep_scale;
    int rc = plan_setup_launch(ctx, plan, b, p, false);
    if (rc) return rc;
    if (!plan->status_cur)  // no beamlets: nothing was launched
        return (rc = plan_setup_finish(ctx, plan)) ? rc : plan_eval_impl(ctx, plan, precision, field_out, out_bytes, opts);
    plan->flags = pflags;
    plan->sep_key = pkey;
    plan->sep_scale = pscale;
    EvalGuard guard;
    guard.status = plan->status_cur;
    guard.key = pkey;
    const size_t timed_before = ctx->timed.size();
    // the setup status is posted by the separable form's kernel at its start
    // (one kernel launch fewer), else by its own kernel
    StatusPost post_req = pending_post(plan);
    const int ahead = plan_eval_impl(ctx, plan, precision, field_out, out_bytes, opts, nullptr, 0, &guard, &post_req);
    if (post_req.post) HIP_TRY(launch_status_post(post_req, ctx->stream), "status post launch");
    rc = plan_setup_finish(ctx, plan);
    if (!rc && ahead == GBD_OK && (plan->flags & guard.mask) == guard.flags &&
        (!guard.check_key || plan->sep_key == pkey))
        return GBD_OK;
    // the launch ahead wrote nothing: drop its timing pair, if any
    while (ctx->timed.size() > timed_before) {
        ctx->spare_events.push_back(ctx->timed.back());
        ctx->timed.pop_back();
    }
    if (rc) return rc;  // a setup error (the guard kept the output untouched)
    if (ahead != GBD_OK && ahead != kNoSpeculation) return ahead;
    // evaluate with the status just read
    return plan_eval_impl(ctx, plan, precision, field_out, out_bytes, opts);
}

int gbd_autotune(gbd_ctx_t ctx, gbd_plan_t plan, int precision, int32_t reps, gbd_eval_opts *best, double *best_ms) {
    if (!ctx || !plan) return fail(GBD_EINVAL, "NULL argument");
    if (!plan->ready) return fail(GBD_EINVAL, "gbd_autotune: plan has no valid setup");
    if (precision != GBD_FP64 && precision != GBD_MIXED) return fail(GBD_EINVAL, "precision must be GBD_FP64 or GBD_MIXED");
    if (reps < 1) reps = 1;
    const int64_t M = (int64_t)plan->pl.nx * plan->pl.ny;
    if (M == 0 || plan->n == 0) return fail(GBD_EINVAL, "nothing to tune (empty plan)");
    int rc = ensure_device(ctx);
    if (rc) return rc;
    void *out = nullptr;
    const int64_t out_bytes = M * (precision == GBD_FP64 ? 16 : 8);
    HIP_TRY(hipMalloc(&out, (size_t)out_bytes), "hipMalloc(autotune output)");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t he = hipEventCreate(&e0);
    if (he == hipSuccess) he = hipEventCreate(&e1);
    TuneVal bestv{0, 0, 100, 1e300};
    static const int rows_c[] = {2, 4, 8, 16, 32}, waves_c[] = {1, 2, 4}, pct_c[] = {50, 100, 200, 400};
    const int64_t n_main = plan->n - plan->n_cut;  // the beamlets choose_shape sizes the form for
    // the separable form has a fixed tile: only its segment count is tuned
    const bool sep = pick_form(precision, plan->flags, nullptr) == 3;
    const int kind = sep ? kTuneSep
                     : cross_applies(precision, pick_form(precision, plan->flags, nullptr), plan->flags, n_main, M) ? kTuneCross
                                                                                                                  : kTuneEval;
    const int n_rows = sep ? 1
                           : precision == GBD_MIXED ? ((plan->flags & FLAG_STEEP) ? 4 : 5)
                           : (plan->flags & FLAG_STEEP) ? 3
                           : (plan->flags & FLAG_HG)    ? 4
                                                        : 5;
    const int n_waves = sep ? 1 : 3;
    // milliseconds per evaluation (rc, he: errors)
    auto timed = [&](bool dense) {
        rc = plan_eval_impl(ctx, plan, precision, out, out_bytes, nullptr, nullptr, 0, nullptr, nullptr, dense);
        float f = 0.f;  // after a warm-up / scratch growth
        if (rc == GBD_OK) he = hipEventRecord(e0, ctx->stream);
        for (int r = 0; r < reps && rc == GBD_OK && he == hipSuccess; r++)
            rc = plan_eval_impl(ctx, plan, precision, out, out_bytes, nullptr, nullptr, 0, nullptr, nullptr, dense);
        if (rc == GBD_OK && he == hipSuccess) he = hipEventRecord(e1, ctx->stream);
        if (rc == GBD_OK && he == hipSuccess) he = hipEventSynchronize(e1);
        if (rc == GBD_OK && he == hipSuccess) he = hipEventElapsedTime(&f, e0, e1);
        return (double)f / reps;
    };
    // a plan that goes by rows has no segments: the counts are those of the
    // product by beamlets, which captured evaluations and beamlets in no rows
    // of the same size take
    for (int ri = 0; ri < n_rows && he == hipSuccess && rc == GBD_OK; ri++)
        for (int wi = 0; wi < n_waves && he == hipSuccess && rc == GBD_OK; wi++)
            for (int pi = 0; pi < 4 && he == hipSuccess && rc == GBD_OK; pi++) {
                // a candidate is addressed through the cache so that choose_shape
                // resolves its segment count exactly as a tuned call would
                const TuneKey key = tune_key(kind, precision, n_main, M);
                const auto saved = ctx->tuned.find(key) != ctx->tuned.end() ? ctx->tuned[key] : TuneVal{0, 0, 0, -1};
                ctx->tuned[key] = TuneVal{sep ? 0 : rows_c[ri], sep ? 0 : waves_c[wi], pct_c[pi], 0.0};
                const double ms = timed(sep);
                if (saved.ms < 0)
                    ctx->tuned.erase(key);
                else
                    ctx->tuned[key] = saved;
                if (rc == GBD_OK && he == hipSuccess && ms < bestv.ms)
                    bestv = TuneVal{sep ? 0 : rows_c[ri], sep ? 0 : waves_c[wi], pct_c[pi], ms};
            }
    // what the plan's evaluations take
    double ms = bestv.ms;
    if (sep && plan->rows > 0 && rc == GBD_OK && he == hipSuccess) ms = std::min(ms, timed(false));
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(out);
    if (rc) return rc;
    if (he != hipSuccess) return hip_fail(he, "autotune timing");
    ctx->tuned[tune_key(kind, precision, n_main, M)] = bestv;
    if (best) {
        const Shape s = choose_shape(ctx, precision, n_main, plan->pl, plan->flags, nullptr);
        const EvalGeom g = make_geom(plan->pl, n_main, s);
        *best = gbd_eval_opts{s.rows, s.waves, g.nseg, form_variant(precision, s.form, s.half)};
    }
    if (best_ms) *best_ms = ms;
    return GBD_OK;
}

int gbd_autotune_save(gbd_ctx_t ctx, const char *path) {
    if (!ctx || !path) return fail(GBD_EINVAL, "NULL argument");
    FILE *f = fopen(path, "w");
    if (!f) return fail(GBD_EINVAL, "cannot write %s", path);
    fprintf(f, "# kind precision log2N log2M rows waves seg_pct ms\n");
    for (const auto &kv : ctx->tuned)
        fprintf(f, "%d %d %d %d %d %d %d %.6f\n", kv.first.kind, kv.first.precision, kv.first.ln, kv.first.lm,
                kv.second.rows, kv.second.waves, kv.second.seg_scale_pct, kv.second.ms);
    fclose(f);
    return GBD_OK;
}

int gbd_autotune_load(gbd_ctx_t ctx, const char *path) {
    if (!ctx || !path) return fail(GBD_EINVAL, "NULL argument");
    FILE *f = fopen(path, "r");
    if (!f) return fail(GBD_EINVAL, "cannot read %s", path);
    char line[256];
    int loaded = 0;
    while (fgets(line, sizeof line, f)) {
        if (line[0] == '#') continue;
        TuneKey k;
        TuneVal v;
        if (sscanf(line, "%d %d %d %d %d %d %d %lf", &k.kind, &k.precision, &k.ln, &k.lm, &v.rows, &v.waves,
                   &v.seg_scale_pct, &v.ms) == 8 &&
            (k.kind == kTuneSep ? v.rows == 0 && v.waves == 0
                                : (k.kind == kTuneEval || k.kind == kTuneBatch || k.kind == kTuneCross) &&
                                      valid_shape(v.rows, v.waves, k.precision)) &&
            v.seg_scale_pct > 0 && v.seg_scale_pct <= 10000) {
            ctx->tuned[k] = v;
            loaded++;
        }
    }
    fclose(f);
    return loaded;
}

int gbd_eval_point(gbd_ctx_t ctx, gbd_beamlets_t b, gbd_plane_t p, void *field_out, int64_t out_bytes) {
    if (!ctx || !b || !p) return fail(GBD_EINVAL, "NULL argument");
    if (b->ctx != ctx) return fail(GBD_EINVAL, "the beamlets belong to another context");
    if (b->higher_order || b->dev.n_cut > 0)
        return fail(GBD_EINVAL, "point evaluation takes whole fundamental Gaussian beamlets only");
    const int64_t M = (int64_t)p->g.nx * p->g.ny;
    if (M == 0) return GBD_OK;
    if (!field_out) return fail(GBD_EINVAL, "field_out is NULL");
    if (out_bytes < M * 16)
        return fail(GBD_ERANGE, "field_out holds %lld bytes, %lld needed", (long long)out_bytes, (long long)(M * 16));
    int rc = ensure_device(ctx);
    if (rc) return rc;
    BatchWork &w = ctx->batch;
    if ((rc = grow(w.point, (size_t)std::max<int64_t>(b->dev.n, 1) * sizeof(RecPt), "point records")) ||
        (rc = grow(w.flags, 4 * sizeof(uint32_t), "flags")))
        return rc;
    if (!w.host_flags) HIP_TRY(hipHostMalloc(&w.host_flags, 4 * sizeof(uint32_t), hipHostMallocDefault), "hipHostMalloc");
    const double g0 = b->dev.l0 / b->dev.lam;
    uint32_t *flags = static_cast<uint32_t *>(w.flags.p);
    HIP_TRY(hipMemsetAsync(flags + 3, 0, sizeof(uint32_t), ctx->stream), "hipMemsetAsync");
    HIP_TRY(launch_point(b->dev, p->g, g0 - nearbyint(g0), static_cast<RecPt *>(w.point.p),
                         static_cast<double2 *>(field_out), flags + 3, ctx->stream),
            "point evaluation launch");
    HIP_TRY(hipMemcpyAsync(w.host_flags + 3, flags + 3, sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->stream),
            "status copy");
    HIP_TRY(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");
    if (w.host_flags[3] & FLAG_BRANCH)
        return fail(GBD_EBRANCH, "an eigenvalue left the principal branch at some pixel (field_out is not valid)");
    return GBD_OK;
}

int gbd_airy(gbd_ctx_t ctx, gbd_plane_t p, double D, double f, double lambda, float *out, int64_t out_bytes) {
    if (!ctx || !p) return fail(GBD_EINVAL, "NULL argument");
    if (!(D > 0.0) || !(f > 0.0) || !(lambda > 0.0) || !std::isfinite(D) || !std::isfinite(f) || !std::isfinite(lambda))
        return fail(GBD_EINVAL, "D, f and lambda must be finite and > 0");
    const int64_t M = (int64_t)p->g.nx * p->g.ny;
    if (M == 0) return GBD_OK;
    if (!out) return fail(GBD_EINVAL, "out is NULL");
    if (out_bytes < M * 4) return fail(GBD_ERANGE, "out holds %lld bytes, %lld needed", (long long)out_bytes, (long long)(M * 4));
    int rc = ensure_device(ctx);
    if (rc) return rc;
    const double vscale = M_PI * D / (lambda * f);
    HIP_TRY(launch_airy(p->g.nx, p->g.ny, p->g.dx, p->g.dy, vscale, out, ctx->stream), "airy kernel launch");
    return GBD_OK;
}

int gbd_eval_batch_start(gbd_ctx_t ctx, int32_t n_inst, const gbd_beamlets_t *bs, const gbd_plane_t *ps, const float *airy,
                   int64_t airy_bytes, const double *zone_edges, int32_t n_zones, void *fields_out, int64_t fields_bytes, const gbd_eval_opts *opts) {
    if (!ctx) return fail(GBD_EINVAL, "ctx is NULL");
    ctx->batch.n_metrics = 0;
    if (n_inst < 0) return fail(GBD_EINVAL, "n_inst < 0");
    if (n_inst == 0) return GBD_OK;
    if (!bs || !ps) return fail(GBD_EINVAL, "beamlets/planes arrays are NULL");
    if (n_zones < 0 || n_zones > kMaxZones) return fail(GBD_EINVAL, "n_zones must be in [0, %d]", kMaxZones);
    if (n_zones > 0) {
        if (!zone_edges) return fail(GBD_EINVAL, "zone_edges is NULL");
        for (int z = 0; z <= n_zones; z++)
            if (!(zone_edges[z] >= 0.0) || !std::isfinite(zone_edges[z]) || (z > 0 && zone_edges[z] < zone_edges[z - 1]))
                return fail(GBD_EINVAL, "zone_edges must be finite, >= 0 and non-decreasing");
    }
    if (opts && (opts->variant < 0 || opts->variant > 5)) return fail(GBD_EINVAL, "variant must be 0 ... 5");
    int rows = 32, waves = 4;  // 32 rows: rotor form; 16 where the form resolves otherwise
    int64_t pairs = 0, n_max = 0;
    for (int32_t i = 0; i < n_inst; i++) {
        if (!bs[i] || !ps[i]) return fail(GBD_EINVAL, "instance %d has a NULL handle", i);
        if (bs[i]->ctx != ctx) return fail(GBD_EINVAL, "instance %d: the beamlets belong to another context", i);
        if (bs[i]->higher_order || bs[i]->dev.n_cut > 0)
            return fail(GBD_EINVAL, "instance %d: the batched sweep takes whole fundamental Gaussian beamlets only", i);
        pairs += bs[i]->dev.n * ((int64_t)ps[i]->g.nx * ps[i]->g.ny);
        n_max = std::max<int64_t>(n_max, bs[i]->dev.n);
    }
    if (!(opts && (opts->rows_per_lane || opts->waves))) {
        auto it = ctx->tuned.find(tune_key(kTuneBatch, GBD_MIXED, pairs, n_inst));
        if (it != ctx->tuned.end()) {
            rows = it->second.rows;
            waves = it->second.waves;
        }
    }
    if (opts) {
        if (opts->rows_per_lane) rows = opts->rows_per_lane;
        if (opts->waves) waves = opts->waves;
    }
    if (!valid_shape(rows, waves)) return fail(GBD_EINVAL, "unsupported batch rows_per_lane %d / waves %d", rows, waves);
    // work items per instance for a given tile height; the count at 16 rows
    // bounds the one at 32 (the row count is final once the form is known)
    auto tiles_of = [&](const PlaneGeom &g, int r) -> int64_t {
        return (int64_t)((g.nx + 63) / 64) * ((g.ny + waves * r - 1) / (waves * r));
    };
    int64_t total = 0, field_elems = 0, n_items = 0, row_tiles = 0, setup_blocks = 0, row_blocks = 0;
    for (int32_t i = 0; i < n_inst; i++) {
        const PlaneGeom &g = ps[i]->g;
        if (airy) {
            if (g.nx != ps[0]->g.nx || g.ny != ps[0]->g.ny)
                return fail(GBD_EINVAL, "instances sharing a reference irradiance need equal grids (instance %d)", i);
            if (airy_bytes < (int64_t)g.nx * g.ny * 4) return fail(GBD_ERANGE, "reference irradiance too small");
        }
        total += bs[i]->dev.n;
        field_elems += (int64_t)g.nx * g.ny;
        n_items += tiles_of(g, std::min(rows, 16));
        row_tiles += (int64_t)((g.nx + kRowTilePx - 1) / kRowTilePx) * ((g.ny + kRowTilePx - 1) / kRowTilePx);
        setup_blocks += batch_setup_blocks(bs[i]->dev);
        row_blocks += (int64_t)bs[i]->dev.rows * ((g.nx + 63) / 64);
    }
    if (fields_out && fields_bytes < field_elems * 8)
        return fail(GBD_ERANGE, "fields_out holds %lld bytes, %lld needed", (long long)fields_bytes,
                    (long long)(field_elems * 8));
    if (n_items > 0x3fffffff || row_tiles > 0x0fffffff || setup_blocks > 0x3fffffff || row_blocks > 0x3fffffff) return fail(GBD_ERANGE, "too many work items");
    if (total / kE0Chunk + n_inst > 0x3fffffff) return fail(GBD_ERANGE, "too many beamlets in the batch");
    int rc = ensure_device(ctx);
    if (rc) return rc;

    // per-beamlet setup of every instance; the status decides the mixed form.
    // The host tables pass through one pinned staging buffer:
    //   [BatchInst x n | offs x (n + 1) | blks x (n + 1)]   uploaded before the setup (tab1)
    //   [status x 4 | peaks x n | row flags x n]            read back after it
    //   [BatchEval x n | items | e0map | row lists]         uploaded before the evaluation (tab2)
    // each table part in one copy to a device buffer of the same layout.  The
    // host rewrites the buffer only once the stream has passed the previous
    // call's copies from it (stage_ev).
    const int PS = 2 + 2 * n_zones;
    BatchWork &w = ctx->batch;
    const int64_t max_chunks = total / kE0Chunk + n_inst;  // normalisation chunks, at most
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t t1_offs = al(n_inst * sizeof(BatchInst));
    const size_t t1_blks = t1_offs + al((n_inst + 1) * sizeof(int64_t));
    const size_t t1_bytes = t1_blks + al((n_inst + 1) * sizeof(int32_t));
    const size_t n_words = 4 + 2 * (size_t)n_inst;
    const size_t rb_bytes = al(n_words * sizeof(uint32_t));
    const size_t t2_items = al(n_inst * sizeof(BatchEval));
    const size_t t2_e0map = t2_items + al((size_t)std::max<int64_t>(2 * n_items, 2) * sizeof(int32_t));
    const size_t t2_rows = t2_e0map + al((size_t)max_chunks * sizeof(int32_t));
    const size_t t2_bytes = t2_rows + al(4 * (size_t)n_inst * sizeof(int32_t));
    if ((rc = grow(w.rec, (size_t)std::max<int64_t>(total, 1) * sizeof(Rec32), "batch records")) ||
        (rc = grow(w.l5, (size_t)std::max<int64_t>(total, 1) * sizeof(double), "batch records")) ||
        (airy && (rc = grow(w.e0t, (size_t)std::max<int64_t>(total, 1) * sizeof(double2), "batch normalisation"))) ||
        (airy && (rc = grow(w.e0part, (size_t)max_chunks * sizeof(double2), "batch normalisation"))) ||
        (rc = grow(w.tab1, t1_bytes, "batch table")) || (rc = grow(w.tab2, t2_bytes, "batch table")) ||
        (rc = grow(w.e0, n_inst * sizeof(double2), "batch normalisation")) ||
        (rc = grow(w.terms, n_inst * sizeof(MatrixTerms), "batch matrix terms")) ||
        (rc = grow(w.part, (size_t)std::max<int64_t>(n_items + row_tiles, 1) * PS * sizeof(double), "batch partials")) ||
        (rc = grow(w.flags, rb_bytes, "batch flags")))
        return rc;
    hipStream_t st = ctx->stream;
    if (!w.stage_ev) HIP_TRY(hipEventCreateWithFlags(&w.stage_ev, hipEventDisableTiming), "hipEventCreate");
    if (w.stage_pending) HIP_TRY(hipEventSynchronize(w.stage_ev), "hipEventSynchronize");
    w.stage_pending = false;
    if (airy && (int64_t)n_inst * (2 + n_zones) > w.metrics_cap) {
        HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");  // a batch not collected may still write them
        if (w.metrics) (void)hipHostFree(w.metrics);
        w.metrics = nullptr;
        w.metrics_cap = 0;
        const int64_t cap = std::max<int64_t>((int64_t)n_inst * (2 + n_zones), 1024);
        HIP_TRY(hipHostMalloc(&w.metrics, (size_t)cap * sizeof(double), hipHostMallocDefault), "hipHostMalloc(metrics)");
        w.metrics_cap = cap;
    }
    const size_t stage_bytes = t1_bytes + rb_bytes + t2_bytes;
    if (stage_bytes > w.stage_bytes) {
        if (w.stage) (void)hipHostFree(w.stage);
        w.stage = nullptr;
        w.stage_bytes = 0;
        HIP_TRY(hipHostMalloc(&w.stage, stage_bytes, hipHostMallocDefault), "hipHostMalloc(batch staging)");
        w.stage_bytes = stage_bytes;
    }
    char *h1 = static_cast<char *>(w.stage), *hrb = h1 + t1_bytes, *h2 = hrb + rb_bytes;
    char *d1 = static_cast<char *>(w.tab1.p), *d2 = static_cast<char *>(w.tab2.p);
    BatchInst *inst = reinterpret_cast<BatchInst *>(h1);
    int64_t *offs = reinterpret_cast<int64_t *>(h1 + t1_offs);
    int32_t *blks = reinterpret_cast<int32_t *>(h1 + t1_blks);
    offs[0] = 0;
    blks[0] = 0;
    for (int32_t i = 0; i < n_inst; i++) {
        const BeamletsDev &b = bs[i]->dev;
        offs[i + 1] = offs[i] + b.n;
        blks[i + 1] = blks[i] + (int32_t)batch_setup_blocks(b);
        const double g0 = b.l0 / b.lam;
        inst[i].b = b;
        inst[i].pl = ps[i]->g;
        inst[i].rec_off = offs[i];
        inst[i].gturns = g0 - nearbyint(g0);
        inst[i].shared = shares_terms(bs[i], ps[i]) ? 1 : 0;
    }
    const BatchInst *dinst = reinterpret_cast<const BatchInst *>(d1);
    const int64_t *doffs = reinterpret_cast<const int64_t *>(d1 + t1_offs);
    HIP_TRY(hipMemcpyAsync(d1, h1, t1_bytes, hipMemcpyHostToDevice, st), "table upload");
    HIP_TRY(hipEventRecord(w.stage_ev, st), "hipEventRecord");
    w.stage_pending = true;
    // [0] status, [1] first bad instance, [2] queue head, [4 ...] per-instance peaks, then row flags
    uint32_t *flags = static_cast<uint32_t *>(w.flags.p);
    HIP_TRY(launch_batch_clear(flags, dinst, static_cast<MatrixTerms *>(w.terms.p), n_inst, st), "batch clear launch");
    HIP_TRY(launch_batch_setup(dinst, doffs, reinterpret_cast<const int32_t *>(d1 + t1_blks), n_inst, blks[n_inst],
                               static_cast<Rec32 *>(w.rec.p), static_cast<double *>(w.l5.p),
                               airy ? static_cast<double2 *>(w.e0t.p) : nullptr, flags,
                               reinterpret_cast<int32_t *>(flags + 1), flags + 4, flags + 4 + n_inst,
                               static_cast<const MatrixTerms *>(w.terms.p), st),
            "batch setup launch");
    HIP_TRY(hipMemcpyAsync(hrb, flags, n_words * sizeof(uint32_t), hipMemcpyDeviceToHost, st), "status copy");
    HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
    w.stage_pending = false;
    const uint32_t *hflags = reinterpret_cast<const uint32_t *>(hrb), *peaks = hflags + 4, *rowbad = peaks + n_inst;
    const uint32_t stat = hflags[0];
    const int32_t bad = (int32_t)hflags[1];
    if (stat & FLAG_PARALLEL) return fail(GBD_EPARALLEL, "instance %d: a base ray is parallel to the plane", bad);
    if (stat & FLAG_BRANCH) return fail(GBD_EBRANCH, "instance %d: an eigenvalue left the principal branch", bad);
    if (stat & FLAG_NONFINITE) return fail(GBD_EINVAL, "instance %d: non-finite beamlet parameters", bad);
    // an item sums all of its instance's beamlets; the separable form does so
    // in one plain FP32 sum per pixel, so it applies only while every
    // instance fits one segment of the single evaluation (kSepMaxSegLen);
    // the rotor form folds 128-beamlet tile sums and stays accurate at any N
    const int form = pick_form(GBD_MIXED, stat, opts, n_max <= kSepMaxSegLen);
    // the separable form in FP16 halves unless FP32 MFMA is requested (variant 5)
    const bool half = form == 3 && !(opts && opts->variant == 5);
    if (rows == 32 && form != 2) rows = 16;  // 32 rows is a rotor-form shape
    if (form == 2)
        HIP_TRY(launch_batch_sigma(dinst, doffs, n_inst, total, static_cast<const double *>(w.l5.p),
                                   static_cast<Rec32 *>(w.rec.p), st),
                "rotor table launch");

    // evaluation tables; the work list takes instances largest first (LPT),
    // each instance's tiles contiguous and in order
    BatchEval *ev = reinterpret_cast<BatchEval *>(h2);
    int32_t *items = reinterpret_cast<int32_t *>(h2 + t2_items);
    int32_t *e0map = reinterpret_cast<int32_t *>(h2 + t2_e0map);  // normalisation chunk -> instance
    // each instance whose beamlets come in row chunks goes by rows, as a single evaluation of it does
    int32_t *sum_inst = reinterpret_cast<int32_t *>(h2 + t2_rows), *sum_first = sum_inst + n_inst,
            *prod_inst = sum_first + n_inst, *prod_first = prod_inst + n_inst;
    // in groups, one after the other, whose sums share one buffer of kFormScratch at most
    struct RowGroup {
        BatchRows br{};
        int32_t begin, end;  // instances
        int32_t list = 0;    // its first entry of the lists
        int32_t sum_blocks = 0;
    };
    std::vector<RowGroup> groups;
    int64_t sum_off = 0, sum_most = 0;
    int32_t n_rows = 0;
    int64_t foff = 0;
    int32_t n_chunks = 0;
    for (int32_t i = 0; i < n_inst; i++) {
        const PlaneGeom &g = ps[i]->g;
        BatchEval &e = ev[i];
        e = BatchEval();
        e.rec_off = offs[i];
        e.n = bs[i]->dev.n;
        e.nx = g.nx;
        e.ny = g.ny;
        const BeamletsDev &b = bs[i]->dev;
        if (half && !rowbad[i] && (int64_t)g.nx * g.ny > 0 && rows_pay(GBD_MIXED, ctx->cus, b.n, b.rows, g)) {
            const int64_t elems = (int64_t)b.rows * (g.nx + g.ny);
            if (groups.empty() || (sum_off + elems) * (int64_t)sizeof(float2) > kFormScratch) {
                groups.push_back(RowGroup{BatchRows{}, i, i, n_rows, 0});
                sum_off = 0;
            }
            RowGroup &G = groups.back();
            e.rows = b.rows;
            e.row_start = b.row_start;
            e.sum_off = sum_off;
            sum_off += elems;
            sum_most = std::max(sum_most, sum_off);
            sum_inst[n_rows] = i;
            sum_first[n_rows++] = G.sum_blocks;
            const int cols = g.nx > 64 ? 128 : 64;
            G.sum_blocks += b.rows * ((g.nx + cols - 1) / cols);
            G.br.n++;
            G.end = i + 1;
            e.tiles_x = (g.nx + kRowTilePx - 1) / kRowTilePx;
            e.tiles_y = (g.ny + kRowTilePx - 1) / kRowTilePx;
        } else if (form == 3) {  // separable form: the single evaluation's workgroup tiles
            Shape sh;
            sh.form = 3;
            sh.half = half;
            sh.rows = kSepTileY;
            sh.waves = kSepWavesX * kSepWavesY;
            int wgx, wgy;
            sep_wg_tile(sh, wgx, wgy);
            e.tiles_x = (g.nx + wgx - 1) / wgx;
            e.tiles_y = (g.ny + wgy - 1) / wgy;
        } else {
            e.tiles_x = (g.nx + 63) / 64;
            e.tiles_y = (g.ny + waves * rows - 1) / (waves * rows);
        }
        e.dx = g.dx;
        e.dy = g.dy;
        e.a0 = -0.5 * (g.nx - 1) * g.dx;
        e.b0 = -0.5 * (g.ny - 1) * g.dy;
        e.field_off = foff;
        foff += (int64_t)g.nx * g.ny;
        e.scale = peaks[i] ? 2 * kSepHalfExp - ((int)peaks[i] - 2048) : 0;  // as a single evaluation's setup
        e.e0_off = n_chunks;
        e.e0_chunks = (int32_t)((e.n + kE0Chunk - 1) / kE0Chunk);
        for (int32_t c = 0; c < e.e0_chunks; c++) e0map[n_chunks++] = i;
    }
    std::vector<int32_t> order(n_inst);
    for (int32_t i = 0; i < n_inst; i++) order[i] = i;
    // an instance's cost: its pairs, by rows its (chunk, pixel) products
    auto cost = [&](int32_t i) { return (ev[i].rows ? ev[i].rows : ev[i].n) * ((int64_t)ev[i].nx * ev[i].ny); };
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return cost(x) > cost(y); });
    // by rows: the k-th largest to XCD 0 ... 7, 7 ... 0, 0 ...
    for (RowGroup &G : groups) {
        BatchRows &br = G.br;
        std::vector<int32_t> list[kXcds];
        int32_t k = 0;
        for (int32_t i : order)
            if (ev[i].rows && i >= G.begin && i < G.end) {
                const int32_t r = k++ % (2 * kXcds);
                list[r < kXcds ? r : 2 * kXcds - 1 - r].push_back(i);
            }
        int32_t at = 0;
        for (int x = 0; x < kXcds; x++) {
            br.prod_list[x] = at;
            for (int32_t i : list[x]) {
                prod_inst[G.list + at] = i;
                prod_first[G.list + at++] = br.prod_tiles[x];
                br.prod_tiles[x] += ev[i].tiles_x * ev[i].tiles_y;
            }
        }
        br.prod_list[kXcds] = at;
    }
    int64_t n_it = 0, n_part = 0;
    for (int32_t k = 0; k < n_inst; k++) {
        const int32_t i = order[k];
        if (ev[i].rows) continue;
        ev[i].item_off = n_it;
        const int32_t tiles = ev[i].tiles_x * ev[i].tiles_y;
        for (int32_t t = 0; t < tiles; t++) {
            items[2 * n_it] = i;
            items[2 * n_it + 1] = t;
            n_it++;
        }
    }
    n_items = n_it;
    n_part = n_it;  // the partials of instances by rows follow those of the work list
    for (int32_t i = 0; i < n_inst; i++)
        if (ev[i].rows) {
            ev[i].item_off = n_part;
            n_part += (int64_t)ev[i].tiles_x * ev[i].tiles_y;
        }
    if ((rc = grow(w.row_sums, (size_t)std::max<int64_t>(sum_most, 1) * sizeof(float2), "batch row sums"))) return rc;
    // the tables up to the last part in use (the work list is empty when every instance goes by rows)
    const size_t t2_used = n_rows ? t2_bytes : t2_e0map + (size_t)n_chunks * sizeof(int32_t);
    HIP_TRY(hipMemcpyAsync(d2, h2, t2_used, hipMemcpyHostToDevice, st), "table upload");
    HIP_TRY(hipEventRecord(w.stage_ev, st), "hipEventRecord");
    w.stage_pending = true;

    BatchArgs a;
    a.inst = reinterpret_cast<const BatchEval *>(d2);
    a.n_inst = n_inst;
    a.items = reinterpret_cast<const int32_t *>(d2 + t2_items);
    a.n_items = (int32_t)n_items;
    a.rec = static_cast<const Rec32 *>(w.rec.p);
    a.e0 = static_cast<const double2 *>(w.e0.p);
    a.airy = airy;
    a.fields = static_cast<float2 *>(fields_out);
    a.part = static_cast<double *>(w.part.p);
    a.counter = flags + 2;
    a.n_zones = n_zones;
    for (int z = 0; z <= kMaxZones; z++)
        a.zone_r2[z] = (z <= n_zones && n_zones > 0) ? zone_edges[z] * zone_edges[z] : 0.0;
    if (airy)
        HIP_TRY(launch_batch_e0(a.inst, n_inst, reinterpret_cast<const int32_t *>(d2 + t2_e0map), n_chunks,
                                static_cast<const double2 *>(w.e0t.p), static_cast<double2 *>(w.e0part.p),
                                static_cast<double2 *>(w.e0.p), st),
                "normalisation launch");
    for (RowGroup &G : groups) {
        const int32_t *lists = reinterpret_cast<const int32_t *>(d2 + t2_rows) + G.list;
        G.br.sum_inst = lists;
        G.br.sum_first = lists + n_inst;
        G.br.prod_inst = lists + 2 * n_inst;
        G.br.prod_first = lists + 3 * n_inst;
        G.br.peaks = flags + 4;
        G.br.sums = static_cast<float2 *>(w.row_sums.p);
        HIP_TRY(launch_batch_rows(a, G.br, G.sum_blocks, st), "batch row launch");
    }
    HIP_TRY(launch_batch_eval(rows, waves, form, half, ctx->cus, a, st), "batch eval launch");
    if (airy) {
        HIP_TRY(launch_batch_finalize(a.inst, n_inst, a.part, n_zones, w.metrics, st),
                "finalize launch");
        w.n_metrics = (int64_t)n_inst * (2 + n_zones);
    }
    return GBD_OK;
}

int gbd_eval_batch_finish(gbd_ctx_t ctx, double *metrics_out, int64_t count) {
    if (!ctx || !metrics_out) return fail(GBD_EINVAL, "NULL argument");
    BatchWork &w = ctx->batch;
    if (w.n_metrics == 0) return fail(GBD_EINVAL, "no batch was started with a reference irradiance");
    if (count != w.n_metrics)
        return fail(GBD_ERANGE, "metrics_out holds %lld values, the batch has %lld", (long long)count, (long long)w.n_metrics);
    const int rc = ensure_device(ctx);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(ctx->stream), "hipStreamSynchronize");  // (a stream left since has been drained)
    w.stage_pending = false;
    memcpy(metrics_out, w.metrics, (size_t)count * sizeof(double));
    w.n_metrics = 0;
    return GBD_OK;
}

int gbd_eval_batch(gbd_ctx_t ctx, int32_t n_inst, const gbd_beamlets_t *bs, const gbd_plane_t *ps, const float *airy,
                   int64_t airy_bytes, const double *zone_edges, int32_t n_zones, double *metrics_out,
                   void *fields_out, int64_t fields_bytes, const gbd_eval_opts *opts) {
    if (ctx && n_inst > 0) {
        if (metrics_out && !airy) return fail(GBD_EINVAL, "metrics need the reference irradiance");
        if (airy && !metrics_out) return fail(GBD_EINVAL, "metrics_out is NULL");
    }
    const int rc = gbd_eval_batch_start(ctx, n_inst, bs, ps, airy, airy_bytes, zone_edges, n_zones, fields_out,
                                        fields_bytes, opts);
    if (rc || n_inst == 0 || !airy) return rc;
    return gbd_eval_batch_finish(ctx, metrics_out, (int64_t)n_inst * (2 + n_zones));
}

int gbd_autotune_batch(gbd_ctx_t ctx, int32_t n_inst, const gbd_beamlets_t *bs, const gbd_plane_t *ps,
                       const float *airy, int64_t airy_bytes, int32_t reps, gbd_eval_opts *best, double *best_ms) {
    if (!ctx || n_inst <= 0 || !bs || !ps || !airy) return fail(GBD_EINVAL, "bad argument");
    if (reps < 1) reps = 1;
    int64_t pairs = 0;
    for (int32_t i = 0; i < n_inst; i++) {
        if (!bs[i] || !ps[i]) return fail(GBD_EINVAL, "instance %d has a NULL handle", i);
        pairs += bs[i]->dev.n * ((int64_t)ps[i]->g.nx * ps[i]->g.ny);
    }
    std::vector<double> metrics((size_t)n_inst * 2);
    static const int rows_c[] = {2, 4, 8, 16, 32}, waves_c[] = {1, 2, 4};
    TuneVal bestv{0, 0, 100, 1e300};
    for (int ri = 0; ri < 5; ri++)
        for (int wi = 0; wi < 3; wi++) {
            gbd_eval_opts o{rows_c[ri], waves_c[wi], 0, 0};
            int rc = gbd_eval_batch(ctx, n_inst, bs, ps, airy, airy_bytes, nullptr, 0, metrics.data(), nullptr, 0, &o);
            if (rc) return rc;
            const auto t0 = std::chrono::steady_clock::now();
            for (int r = 0; r < reps; r++) {
                rc = gbd_eval_batch(ctx, n_inst, bs, ps, airy, airy_bytes, nullptr, 0, metrics.data(), nullptr, 0, &o);
                if (rc) return rc;
            }
            const double ms =
                std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count() / reps;
            if (ms < bestv.ms) bestv = TuneVal{rows_c[ri], waves_c[wi], 100, ms};
        }
    ctx->tuned[tune_key(kTuneBatch, GBD_MIXED, pairs, n_inst)] = bestv;
    if (best) *best = gbd_eval_opts{bestv.rows, bestv.waves, 0, 0};
    if (best_ms) *best_ms = bestv.ms;
    return GBD_OK;
}

int gbd_mlp_create(gbd_ctx_t ctx, gbd_mlp_t *out, int32_t n_in, int32_t width, int32_t depth, int32_t max_batch,
                   int mode) {
    if (!ctx || !out) return fail(GBD_EINVAL, "NULL argument");
    if (n_in < 1 || n_in > 64 || width < 1 || width > 1024 || depth < 1 || depth > 8 || max_batch < 1 ||
        max_batch > 65536)
        return fail(GBD_EINVAL, "unsupported network shape (n_in %d, width %d, depth %d, max_batch %d)", n_in, width,
                    depth, max_batch);
    if (mode != GBD_MLP_FP32 && mode != GBD_MLP_BF16) return fail(GBD_EINVAL, "mode must be GBD_MLP_FP32 or GBD_MLP_BF16");
    int rc = ensure_device(ctx);
    if (rc) return rc;
    gbd_mlp_s *m = new (std::nothrow) gbd_mlp_s();
    if (!m) return fail(GBD_ENOMEM, "host allocation failed");
    m->ctx = ctx;
    m->n_in = n_in;
    m->width = width;
    m->depth = depth;
    m->max_batch = max_batch;
    m->mode = mode;
    int64_t k = 0, prev = n_in;
    for (int l = 0; l <= depth; l++) {
        const int64_t o = (l < depth) ? width : 1;
        m->woff.push_back(k);
        k += o * prev;
        m->boff.push_back(k);
        k += o;
        prev = width;
    }
    m->P = k;
    // activations in rows of a batch rounded up to 16, on 16-byte boundaries
    // (the two-kernel path keeps BF16 transposes in H's place)
    const int64_t mb = ((int64_t)max_batch + 15) / 16 * 16, P4 = (m->P + 3) / 4 * 4;
    const int64_t act = (int64_t)depth * mb * width, bw = mb * width;
    const bool fused = mlp_fused(mode == GBD_MLP_BF16, width, depth);
    const int64_t pack = fused ? depth * mlp_pack_layer(width) : 0;  // BF16 values, forward and transposed
    const int64_t total = 4 * P4 + 2 * act + 2 * bw + mb * (n_in + 3 + (n_in + 1) / 2) + pack + 1;
    hipError_t e = hipMalloc(&m->mem, (size_t)total * sizeof(float));
    if (e != hipSuccess) {
        delete m;
        return hip_fail(e, "hipMalloc(mlp)");
    }
    float *q = m->mem;
    m->params = q; q += P4;
    m->grads = q; q += P4;
    m->m = q; q += P4;
    m->v = q; q += P4;
    if (fused) {
        m->wf = reinterpret_cast<uint16_t *>(q); q += pack / 2;
        m->wb = reinterpret_cast<uint16_t *>(q); q += pack / 2;
    }
    m->Z = q; q += act;
    m->H = q; q += act;
    m->dz0 = q; q += bw;
    m->dz1 = q; q += bw;
    m->xb = q; q += mb * n_in;
    m->yb = q; q += mb;
    m->yhat = q; q += mb;
    m->g = q; q += mb;
    m->xt = reinterpret_cast<uint16_t *>(q); q += mb * ((n_in + 1) / 2);
    m->loss = q;
    e = hipMemsetAsync(m->mem, 0, (size_t)total * sizeof(float), ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        (void)hipFree(m->mem);
        delete m;
        return hip_fail(e, "mlp init");
    }
    *out = m;
    return GBD_OK;
}

void gbd_mlp_free(gbd_mlp_t m) {
    if (!m) return;
    if (m->mem) (void)hipFree(m->mem);
    delete m;
}

int64_t gbd_mlp_num_params(gbd_mlp_t m) { return m ? m->P : (int64_t)fail(GBD_EINVAL, "NULL argument"); }

// The two-kernel path's view of a batch (mlp_fused)
static MlpNet mlp_net(gbd_mlp_t m, const float *x, const float *target, const int32_t *rows, int B, float *yhat) {
    MlpNet n{};
    n.n_in = m->n_in;
    n.W = m->width;
    n.D = m->depth;
    n.B = B;
    n.bt = (B + 15) / 16 * 16;
    n.params = m->params;
    for (int l = 0; l <= m->depth && l <= kMlpFusedDepth; l++) {
        n.woff[l] = m->woff[l];
        n.boff[l] = m->boff[l];
    }
    n.x = x;
    n.y = target;
    n.rows = rows;
    n.yhat = yhat;
    n.dz = m->Z;
    n.hlast = m->dz0;
    n.g = m->g;
    n.yb = m->yb;
    n.dzt = reinterpret_cast<uint16_t *>(m->H);
    n.ht = n.dzt + (int64_t)m->depth * m->width * n.bt;
    n.xt = m->xt;
    n.wf = m->wf;
    n.wb = m->wb;
    return n;
}

int gbd_mlp_set_params(gbd_mlp_t m, const float *params, int64_t n) {
    if (!m || !params) return fail(GBD_EINVAL, "NULL argument");
    if (n != m->P) return fail(GBD_EINVAL, "expected %lld parameters, got %lld", (long long)m->P, (long long)n);
    for (int64_t i = 0; i < n; i++)
        if (!std::isfinite(params[i])) return fail(GBD_EINVAL, "non-finite parameter %lld", (long long)i);
    int rc = ensure_device(m->ctx);
    if (rc) return rc;
    hipStream_t st = m->ctx->stream;
    HIP_TRY(hipMemcpyAsync(m->params, params, n * sizeof(float), hipMemcpyHostToDevice, st), "parameter upload");
    HIP_TRY(hipMemsetAsync(m->m, 0, n * sizeof(float), st), "optimiser reset");
    HIP_TRY(hipMemsetAsync(m->v, 0, n * sizeof(float), st), "optimiser reset");
    HIP_TRY(launch_mlp_pack(mlp_net(m, nullptr, nullptr, nullptr, 0, nullptr), st), "weight packing launch");
    HIP_TRY(hipStreamSynchronize(st), "hipStreamSynchronize");
    m->step = 0;
    return GBD_OK;
}

static int mlp_copy_out(gbd_mlp_t m, const float *src, float *dst, int64_t n) {
    if (!m || !dst) return fail(GBD_EINVAL, "NULL argument");
    if (n != m->P) return fail(GBD_EINVAL, "expected %lld values, got %lld", (long long)m->P, (long long)n);
    int rc = ensure_device(m->ctx);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(dst, src, n * sizeof(float), hipMemcpyDeviceToHost, m->ctx->stream), "download");
    HIP_TRY(hipStreamSynchronize(m->ctx->stream), "hipStreamSynchronize");
    return GBD_OK;
}

int gbd_mlp_get_params(gbd_mlp_t m, float *params, int64_t n) { return mlp_copy_out(m, m ? m->params : nullptr, params, n); }
int gbd_mlp_get_grads(gbd_mlp_t m, float *grads, int64_t n) { return mlp_copy_out(m, m ? m->grads : nullptr, grads, n); }

// forward over the batch already gathered into m->xb; leaves Z, H, yhat
static int mlp_forward_impl(gbd_mlp_t m, int B) {
    hipStream_t st = m->ctx->stream;
    const int W = m->width;
    const float *in = m->xb;
    int fan = m->n_in;
    for (int l = 0; l < m->depth; l++) {
        MlpGemm g{};
        g.M = B;
        g.N = W;
        g.K = fan;
        g.A = in;
        g.sam = fan;
        g.sak = 1;
        g.B = m->params + m->woff[l];
        g.sbk = 1;
        g.sbn = fan;
        g.bias = m->params + m->boff[l];
        g.C = m->Z + (int64_t)l * m->max_batch * W;
        g.H = m->H + (int64_t)l * m->max_batch * W;
        g.epi = 0;
        HIP_TRY(launch_mlp_gemm(m->mode == GBD_MLP_BF16, g, st), "mlp forward launch");
        in = g.H;
        fan = W;
    }
    HIP_TRY(launch_mlp_head_forward(in, m->params + m->woff[m->depth], m->params + m->boff[m->depth], B, W, m->yhat, st),
            "mlp head launch");
    return GBD_OK;
}

// Gradients of one batch (and, with adam.on, the step) by the two-kernel path
static int mlp_fused_backward(gbd_mlp_t m, const float *x, const float *target, const int32_t *rows, int B,
                              float *loss, float *loss_sum, const MlpAdam &adam) {
    const MlpNet n = mlp_net(m, x, target, rows, B, m->yhat);
    HIP_TRY(launch_mlp_rows(n, true, m->ctx->stream), "mlp rows launch");
    HIP_TRY(launch_mlp_grads(n, m->grads, loss, loss_sum, adam, m->ctx->stream), "mlp gradient launch");
    return GBD_OK;
}

int gbd_mlp_forward(gbd_mlp_t m, const float *x, const int32_t *rows, int32_t batch, float *y) {
    if (!m || !x || !y) return fail(GBD_EINVAL, "NULL argument");
    if (batch < 0 || batch > m->max_batch) return fail(GBD_ERANGE, "batch %d outside [0, %d]", batch, m->max_batch);
    if (batch == 0) return GBD_OK;
    int rc = ensure_device(m->ctx);
    if (rc) return rc;
    hipStream_t st = m->ctx->stream;
    if (mlp_fused(m->mode == GBD_MLP_BF16, m->width, m->depth)) {
        HIP_TRY(launch_mlp_rows(mlp_net(m, x, nullptr, rows, batch, y), false, st), "mlp rows launch");
        return GBD_OK;
    }
    HIP_TRY(launch_mlp_gather(x, nullptr, rows, batch, m->n_in, m->xb, nullptr, st), "mlp gather launch");
    rc = mlp_forward_impl(m, batch);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(y, m->yhat, batch * sizeof(float), hipMemcpyDeviceToDevice, st), "mlp output copy");
    return GBD_OK;
}

int gbd_mlp_backward(gbd_mlp_t m, const float *x, const float *target, const int32_t *rows, int32_t batch,
                     float *loss_dev) {
    if (!m || !x || !target) return fail(GBD_EINVAL, "NULL argument");
    if (batch < 1 || batch > m->max_batch) return fail(GBD_ERANGE, "batch %d outside [1, %d]", batch, m->max_batch);
    int rc = ensure_device(m->ctx);
    if (rc) return rc;
    hipStream_t st = m->ctx->stream;
    const int W = m->width, B = batch, D = m->depth;
    if (mlp_fused(m->mode == GBD_MLP_BF16, W, D))
        return mlp_fused_backward(m, x, target, rows, B, loss_dev ? loss_dev : m->loss, nullptr, MlpAdam{});
    HIP_TRY(launch_mlp_gather(x, target, rows, B, m->n_in, m->xb, m->yb, st), "mlp gather launch");
    rc = mlp_forward_impl(m, B);
    if (rc) return rc;
    const int64_t stride = (int64_t)m->max_batch * W;
    const float *Hlast = m->H + (int64_t)(D - 1) * stride;
    const float *Zlast = m->Z + (int64_t)(D - 1) * stride;
    // head: loss, its gradient, head weights' gradient, dZ of the last hidden layer
    HIP_TRY(launch_mlp_head_backward(m->yhat, m->yb, Hlast, m->params + m->woff[D], Zlast, B, W, m->g, m->loss,
                                     m->grads + m->woff[D], m->dz0, st),
            "mlp head backward launch");
    float *dz = m->dz0, *dz_next = m->dz1;
    for (int l = D - 1; l >= 0; l--) {
        const int fan = (l == 0) ? m->n_in : W;
        const float *Hprev = (l == 0) ? m->xb : m->H + (int64_t)(l - 1) * stride;
        // dW_l[o][i] = sum_b dZ[b][o] Hprev[b][i]
        MlpGemm gw{};
        gw.M = W;
        gw.N = fan;
        gw.K = B;
        gw.A = dz;
        gw.sam = 1;
        gw.sak = W;
        gw.B = Hprev;
        gw.sbk = fan;
        gw.sbn = 1;
        gw.C = m->grads + m->woff[l];
        gw.epi = 2;
        HIP_TRY(launch_mlp_gemm(m->mode == GBD_MLP_BF16, gw, st), "mlp weight-gradient launch");
        HIP_TRY(launch_mlp_colsum(dz, B, W, m->grads + m->boff[l], st), "mlp bias-gradient launch");
        if (l > 0) {
            // dZ_{l-1}[b][i] = (sum_o dZ[b][o] W_l[o][i]) SiLU'(Z_{l-1}[b][i])
            MlpGemm gh{};
            gh.M = B;
            gh.N = W;
            gh.K = W;
            gh.A = dz;
            gh.sam = W;
            gh.sak = 1;
            gh.B = m->params + m->woff[l];
            gh.sbk = W;
            gh.sbn = 1;
            gh.zmul = m->Z + (int64_t)(l - 1) * stride;
            gh.C = dz_next;
            gh.epi = 1;
            HIP_TRY(launch_mlp_gemm(m->mode == GBD_MLP_BF16, gh, st), "mlp backward launch");
            std::swap(dz, dz_next);
        }
    }
    if (loss_dev) HIP_TRY(hipMemcpyAsync(loss_dev, m->loss, sizeof(float), hipMemcpyDeviceToDevice, st), "loss copy");
    return GBD_OK;
}

static bool adamw_args_ok(float lr, float beta1, float beta2, float eps, float weight_decay) {
    return lr >= 0.0f && beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps >= 0.0f &&
           weight_decay >= 0.0f;
}

int gbd_mlp_adamw(gbd_mlp_t m, float lr, float beta1, float beta2, float eps, float weight_decay) {
    if (!m) return fail(GBD_EINVAL, "NULL argument");
    if (!adamw_args_ok(lr, beta1, beta2, eps, weight_decay)) return fail(GBD_EINVAL, "invalid AdamW hyper-parameters");
    int rc = ensure_device(m->ctx);
    if (rc) return rc;
    m->step++;
    const float c1 = 1.0f - powf(beta1, (float)m->step), c2 = 1.0f - powf(beta2, (float)m->step);
    HIP_TRY(launch_mlp_adamw(mlp_net(m, nullptr, nullptr, nullptr, 0, nullptr), m->grads, m->m, m->v, m->P, lr, beta1,
                             beta2, eps, weight_decay, c1, c2, m->ctx->stream),
            "adamw launch");
    return GBD_OK;
}

int gbd_mlp_train(gbd_mlp_t m, const float *x, const float *target, const int32_t *rows, int32_t steps, int32_t batch,
                  const float *lr_host, float beta1, float beta2, float eps, float weight_decay, float *loss_sum_dev) {
    if (!m || !x || !target || !rows || !lr_host) return fail(GBD_EINVAL, "NULL argument");
    if (steps < 0) return fail(GBD_EINVAL, "negative step count %d", steps);
    if (batch < 1 || batch > m->max_batch) return fail(GBD_ERANGE, "batch %d outside [1, %d]", batch, m->max_batch);
    // every step's arguments are checked before the first one runs
    for (int32_t s = 0; s < steps; s++)
        if (!adamw_args_ok(lr_host[s], beta1, beta2, eps, weight_decay))
            return fail(GBD_EINVAL, "invalid AdamW hyper-parameters (step %d)", s);
    const bool fused = mlp_fused(m->mode == GBD_MLP_BF16, m->width, m->depth);
    if (fused && steps > 0) {
        const int rc = ensure_device(m->ctx);
        if (rc) return rc;
    }
    for (int32_t s = 0; s < steps && fused; s++) {
        m->step++;
        const float c1 = 1.0f - powf(beta1, (float)m->step), c2 = 1.0f - powf(beta2, (float)m->step);
        const MlpAdam adam{1, m->m, m->v, lr_host[s], beta1, beta2, eps, weight_decay, c1, c2};
        const int rc = mlp_fused_backward(m, x, target, rows + (int64_t)s * batch, batch, m->loss, loss_sum_dev, adam);
        if (rc) return rc;
    }
    for (int32_t s = 0; s < steps && !fused; s++) {
        int rc = gbd_mlp_backward(m, x, target, rows + (int64_t)s * batch, batch, nullptr);
        if (rc) return rc;
        if (loss_sum_dev) HIP_TRY(launch_mlp_accum(loss_sum_dev, m->loss, m->ctx->stream), "loss sum launch");
        rc = gbd_mlp_adamw(m, lr_host[s], beta1, beta2, eps, weight_decay);
        if (rc) return rc;
    }
    return GBD_OK;
}

}  // extern "C"
