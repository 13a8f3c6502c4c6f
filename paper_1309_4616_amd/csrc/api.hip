// C ABI and host driver of the hot path.
//
// phi_action / expeuler_step follow the interpolation scheme of Sec. II-C and
// Sec. III-C of the paper: map the spectral interval [a, b] of A to [-2, 2]
// (c = (a+b)/2, gamma = (b-a)/4), take s substeps of length delta = tau/s
// with delta (b - a) <= l_max, and on each substep apply the Newton form of
// the Leja interpolant of phi_k(delta A) to a start vector r:
//
//   w_0 = r,  p = d_0 w_0,
//   w_{j+1} = ((A - cI)/gamma - xi_j I) w_j,  p += d_{j+1} w_{j+1},
//
// stopping after the first m >= 2 with t_{m-1} + t_m <= tol ||p||, where
// t_j = |d_j| ||w_j||.  Substeps of phi_1 use y' = A y + v, y(0) = 0, so
// y(t) = t phi_1(tA) v and y_{l+1} = y_l + delta phi_1(delta A)(A y_l + v).
// The exponential Euler step of eq. (2), for u' = A u + g(u), equals
// u + tau phi_1(tau A)(A u + g(u)); with substeps y_0 = u,
// y_{l+1} = y_l + delta phi_1(delta A)(A y_l + g(u)), u_new = y_s.
// A substep that has not met the stop test after m_max products doubles s
// and restarts the call (up to max_retries times).
//
// Each product is one fused sweep (sweep.hip).  The stop test runs on the
// device, so the host enqueues products ahead and reads a 64-byte status
// record back to pinned memory only to decide when to stop enqueueing.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <functional>
#include <string>

#include "expi_internal.h"
#include "leja.h"

namespace expi {

// pair2d.hip: the pair sweep of 2D constant-coefficient stencils (same
// arguments, partials and finalize as the 3D one)
bool pair2d_supported(const Op& op, int tw);
bool pair2d_rows_valid(int rows);
hipError_t launch_pair2d(const Op& op, int tw, PairArgs a, hipStream_t s, hipEvent_t after_sweep, bool finalize,
                         int mode, int cus, int rows, int* nparts = nullptr);
int device_cus();

namespace {

thread_local std::string tl_error = "no error";

// A pair sweep exists for the operator (3D or 2D stencil kernel).
bool pair_any_supported(const Op& op, int tw) { return pair_supported(op, tw) || pair2d_supported(op, tw); }
// ... and the operator's setting allows it
bool pairs_on(const Op& op, int tw) { return op.use_pairs != 0 && pair_any_supported(op, tw); }
// The pair sweep of the operator's dimension.  A 2D operator's use_pairs
// above 1 is the rows per tile of its pair sweep (expi_op_set_pairs).
hipError_t launch_pair_op(const Op& op, int tw, const PairArgs& a, hipStream_t s, hipEvent_t after_sweep = nullptr,
                          bool finalize = true, int mode = PAIR_NEWTON, int rows = -1, int* nparts = nullptr) {
    if (op.dim == 2) {
        if (rows < 0) rows = op.use_pairs > 1 ? op.use_pairs : 0;
        return launch_pair2d(op, tw, a, s, after_sweep, finalize, mode, device_cus(), rows, nparts);
    }
    return launch_pair(op, tw, a, s, after_sweep, finalize, mode, nparts);
}

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess) {                                                         \
            set_error(std::string(#expr) + ": " + hipGetErrorString(e_));               \
            return EXPI_EHIP;                                                           \
        }                                                                               \
    } while (0)

int fail(int code, const std::string& msg) {
    set_error(msg);
    return code;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct WsLayout {
    size_t state, partials, w0, w1, p, y, total;
};

WsLayout layout(const Op& op, int dtype) {
    WsLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += align256(bytes);
        return o;
    };
    // complex operators: every vector holds (re, im) pairs
    const size_t n = (size_t)op.size * (op.kind == 2 ? 2 : 1);
    const size_t tw = (dtype == EXPI_F32) ? 4 : 8;
    L.state = take(256);
    L.partials = take(partials_bytes(op));
    L.w0 = take(n * tw);
    L.w1 = take(n * tw);
    L.p = take(n * tw);
    L.y = take(n * 8);
    L.total = off;
    return L;
}

// ---- pinned read-back slots (per host thread) -----------------------------
constexpr int kSlots = 64;

struct HostCtx {
    int device = -1;
    NewtonState* pinned = nullptr;
    NewtonState* pinned_dev = nullptr;   // device address of `pinned`
    hipEvent_t ev[kSlots];
    bool inflight[kSlots];
    int next = 0;
    hipEvent_t tev[2 * kMaxLeja];   // timing events around Newton products
    bool have_tev = false;
};
thread_local HostCtx tl_ctx;

int ctx_init() {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (tl_ctx.device == dev && tl_ctx.pinned) return EXPI_OK;
    // coherent: the finalize kernels write the slots directly
    HIP_TRY(hipHostMalloc((void**)&tl_ctx.pinned, kSlots * sizeof(NewtonState), hipHostMallocCoherent));
    HIP_TRY(hipHostGetDevicePointer((void**)&tl_ctx.pinned_dev, tl_ctx.pinned, 0));
    for (int i = 0; i < kSlots; ++i) {
        HIP_TRY(hipEventCreateWithFlags(&tl_ctx.ev[i], hipEventDisableTiming));
        tl_ctx.inflight[i] = false;
    }
    tl_ctx.device = dev;
    tl_ctx.next = 0;
    tl_ctx.have_tev = false;
    return EXPI_OK;
}

int timing_events() {
    if (tl_ctx.have_tev) return EXPI_OK;
    // timing only: no system-scope fence (cache writeback and invalidate)
    // at each record, which would slow the work that follows it
    for (int i = 0; i < 2 * kMaxLeja; ++i)
        HIP_TRY(hipEventCreateWithFlags(&tl_ctx.tev[i], hipEventDisableSystemFence));
    tl_ctx.have_tev = true;
    return EXPI_OK;
}

// The next free slot (waits for its previous use to end).
int reserve_slot(int* slot_out) {
    const int slot = tl_ctx.next;
    tl_ctx.next = (tl_ctx.next + 1) % kSlots;
    if (tl_ctx.inflight[slot]) {
        HIP_TRY(hipEventSynchronize(tl_ctx.ev[slot]));
        tl_ctx.inflight[slot] = false;
    }
    *slot_out = slot;
    return EXPI_OK;
}

int readback(const NewtonState* st, hipStream_t s, int* slot_out) {
    int slot;
    int rc = reserve_slot(&slot);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(&tl_ctx.pinned[slot], st, sizeof(NewtonState), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipEventRecord(tl_ctx.ev[slot], s));
    tl_ctx.inflight[slot] = true;
    *slot_out = slot;
    return EXPI_OK;
}

// A batch whose last finalize kernel writes the state into a slot (device
// address tl_ctx.pinned_dev + slot): the slot is marked (done = -1, a value
// no kernel writes) before the launches and an event follows them.  A slot
// still marked when it is read (no finalize ran) is filled by a plain copy
// (wait_slot).
int mirror_begin(int* slot_out) {
    int slot;
    int rc = reserve_slot(&slot);
    if (rc) return rc;
    tl_ctx.pinned[slot].done = -1;
    *slot_out = slot;
    return EXPI_OK;
}

int mirror_end(int slot, hipStream_t s) {
    HIP_TRY(hipEventRecord(tl_ctx.ev[slot], s));
    tl_ctx.inflight[slot] = true;
    return EXPI_OK;
}

int wait_slot(int slot, NewtonState* out, const NewtonState* st = nullptr) {
    HIP_TRY(hipEventSynchronize(tl_ctx.ev[slot]));
    tl_ctx.inflight[slot] = false;
    std::memcpy(out, &tl_ctx.pinned[slot], sizeof(NewtonState));
    if (out->done == -1 && st) HIP_TRY(hipMemcpy(out, st, sizeof(NewtonState), hipMemcpyDeviceToHost));
    return EXPI_OK;
}

// ---- parameters ------------------------------------------------------------
struct Params {
    double l_max = 100.0;
    int m_max = 100;
    int max_retries = 4;
    bool have_interval = false;
    int profile = 0;        // 0 off, 1 every launch, 2 one launch per Newton loop
    double ia = 0, ib = 0;
    const float* selector = nullptr;
    int hidden = 0;
    bool pairs = true;
    int fuse_start = 0;
    double sel_l_max = 500.0;      // largest delta (b - a) a predicted substep count may give
    float* sel_features = nullptr;
};

int read_params(const expi_params* p, Params* out) {
    Params q;
    if (p) {
        q.l_max = p->l_max;
        q.m_max = p->m_max;
        q.max_retries = p->max_retries;
        q.have_interval = p->have_interval != 0;
        q.profile = p->profile;
        q.ia = p->interval_a;
        q.ib = p->interval_b;
        q.selector = static_cast<const float*>(p->selector);
        q.hidden = p->selector_hidden;
        q.pairs = p->no_pairs == 0;
        q.fuse_start = p->fuse_start;
        if (p->selector_l_max != 0.0) q.sel_l_max = p->selector_l_max;
        q.sel_features = static_cast<float*>(p->selector_features);
    }
    if (!(q.sel_l_max > 0) || !std::isfinite(q.sel_l_max))
        return fail(EXPI_EINVAL, "params.selector_l_max must be positive and finite (or 0)");
    if (q.fuse_start < 0 || q.fuse_start > 2) return fail(EXPI_EINVAL, "params.fuse_start must be 0, 1 or 2");
    if (q.profile < 0 || q.profile > 2) return fail(EXPI_EINVAL, "params.profile must be 0, 1 or 2");
    if (q.selector && (q.hidden < 1 || q.hidden > 256))
        return fail(EXPI_EINVAL, "params.selector_hidden must be in [1, 256]");
    if (!(q.l_max > 0) || !std::isfinite(q.l_max)) return fail(EXPI_EINVAL, "params.l_max must be positive and finite");
    if (q.m_max < 2 || q.m_max >= kMaxLeja) return fail(EXPI_EINVAL, "params.m_max must be in [2, 255]");
    if (q.max_retries < 0 || q.max_retries > 30) return fail(EXPI_EINVAL, "params.max_retries must be in [0, 30]");
    if (q.have_interval && !(std::isfinite(q.ia) && std::isfinite(q.ib) && q.ia < q.ib))
        return fail(EXPI_EINVAL, "params interval must satisfy a < b, both finite");
    *out = q;
    return EXPI_OK;
}

bool overlap(const void* a, size_t abytes, const void* b, size_t bbytes) {
    const char* pa = static_cast<const char*>(a);
    const char* pb = static_cast<const char*>(b);
    return pa < pb + bbytes && pb < pa + abytes;
}

// ---- interval ----------------------------------------------------------------
int op_interval(Op& op, double* a, double* b, char* ws, hipStream_t s) {
    {
        std::lock_guard<std::mutex> lock(op.mu);
        if (op.have_interval) {
            *a = op.ia;
            *b = op.ib;
            return EXPI_OK;
        }
    }
    int rc = ctx_init();
    if (rc) return rc;
    const WsLayout L = layout(op, EXPI_F64);
    NewtonState* st = reinterpret_cast<NewtonState*>(ws + L.state);
    HIP_TRY(launch_reset(st, s));
    SweepArgs args{};
    args.st = st;
    args.partials = reinterpret_cast<double*>(ws + L.partials);
    HIP_TRY(launch_sweep(op, EPI_GERSH, 0, 0, args, s));
    int slot;
    rc = readback(st, s, &slot);
    if (rc) return rc;
    NewtonState h;
    rc = wait_slot(slot, &h);
    if (rc) return rc;
    if (!std::isfinite(h.gmin) || !std::isfinite(h.gmax))
        return fail(EXPI_ENONFINITE, "Gershgorin interval is not finite (operator entries inf/NaN?)");
    std::lock_guard<std::mutex> lock(op.mu);
    op.ia = h.gmin;
    op.ib = h.gmax;
    op.have_interval = true;
    *a = op.ia;
    *b = op.ib;
    return EXPI_OK;
}

// ---- divided differences (cached per key) --------------------------------------
typedef std::tuple<int, double, double, double, int> DdKey;

std::vector<double> get_dd(Op& op, const DdKey& key) {
    {
        std::lock_guard<std::mutex> lock(op.mu);
        auto it = op.dd_cache.find(key);
        if (it != op.dd_cache.end()) return it->second;
    }
    std::vector<double> d(std::get<4>(key));
    divided_differences(std::get<0>(key), std::get<1>(key), std::get<2>(key), std::get<3>(key),
                        (int)d.size(), d.data());
    std::lock_guard<std::mutex> lock(op.mu);
    if (op.dd_cache.size() > 64) op.dd_cache.clear();
    op.dd_cache.emplace(key, d);
    return d;
}

// The complex ones, kept as real parts then imaginary parts.
void get_dd_skew(Op& op, int k, const DdKey& key, std::vector<double>* re, std::vector<double>* im) {
    const int count = std::get<4>(key);
    std::vector<double> d;
    {
        std::lock_guard<std::mutex> lock(op.mu);
        auto it = op.dd_cache.find(key);
        if (it != op.dd_cache.end()) d = it->second;
    }
    if (d.empty()) {
        d.resize(2 * (size_t)count);
        divided_differences_skew(k, std::get<1>(key), std::get<2>(key), std::get<3>(key), count, d.data(),
                                 d.data() + count);
        std::lock_guard<std::mutex> lock(op.mu);
        if (op.dd_cache.size() > 64) op.dd_cache.clear();
        op.dd_cache.emplace(key, d);
    }
    re->assign(d.begin(), d.begin() + count);
    im->assign(d.begin() + count, d.end());
}

int get_hint(Op& op, const DdKey& key) {
    std::lock_guard<std::mutex> lock(op.mu);
    auto it = op.degree_hint.find(key);
    return it == op.degree_hint.end() ? 0 : it->second;
}

void set_hint(Op& op, const DdKey& key, int m) {
    std::lock_guard<std::mutex> lock(op.mu);
    if (op.degree_hint.size() > 1024) op.degree_hint.clear();
    op.degree_hint[key] = m;
}

// Degrees differ from substep to substep of a call (later ones start from
// smoother vectors), from tolerance to tolerance and with the storage type, so
// each has a record of its own; the substep shares the key through the
// coefficient count, which is at most kMaxLeja.
DegreeKey degree_key(DdKey key, int l, double tol, int tw) {
    std::get<4>(key) += (kMaxLeja + 1) * (1 + std::min(l, 63));
    return DegreeKey(key, tol, tw);
}

// The lowest degree seen lately.  Tests are deferred no further than that: a
// loop that stops before them is run again, about twice its work, so inputs
// whose degree goes up and down must not cause it each time.  With degrees in
// random order a loop is lower than all of the last 16 or more at most once in
// 17; the tested launches between the lowest and the usual degree cost one
// stop test each.
constexpr int kDegreeWindow = 16;
// Loops that have to be seen first.  After c degrees in random order the next
// is lower than all of them once in c + 1 times: from 4 on, the loops run twice
// (1.3 of the next 12, at less than their time once more) cost no more than the
// deferred tests give on small operators (9% of a call), and a degree known
// from one other vector costs nothing.
constexpr int kDegreeLoops = 4;
// In chains a loop run twice takes about what it took once in pairs or single
// products (2000 x 1500, degree 17 after rough vectors of 25: 277 us against
// 262), so two are enough there.
constexpr int kChainLoops = 2;

DegreeWindow get_degrees(Op& op, const DegreeKey& key) {
    std::lock_guard<std::mutex> lock(op.mu);
    auto it = op.degrees.find(key);
    return it == op.degrees.end() ? DegreeWindow() : it->second;
}

void add_degree(Op& op, const DegreeKey& key, int m) {
    std::lock_guard<std::mutex> lock(op.mu);
    if (op.degrees.size() > 1024) op.degrees.clear();
    DegreeWindow& w = op.degrees[key];
    w.last = m;
    w.low = w.low ? std::min(w.low, m) : m;
    w.next = w.count ? std::min(w.next, m) : m;
    w.loops = std::min(w.loops + 1, kDegreeLoops);
    if (++w.count >= kDegreeWindow) {
        w.low = w.next;
        w.count = 0;
    }
}

// ---- one Newton loop -----------------------------------------------------------
struct LoopOut {
    int m = 0;
    int done = 0;
    double err = 0;
    int timed = 0;        // products covered by the timed launches (profile mode)
    double ms = 0;        // their summed device time
    int pairs_timed = 0;  // pair sweeps among them
    double pair_ms = 0;   // and their device time
    int pair_launches = 0, single_launches = 0;   // launches that did work
    double rnorm = 0;     // ||r||
    double hist[kHist] = {0, 0, 0, 0, 0};
    int pred_m = 0, pred_s = 0;
    int restart_s = 0;    // learned mode: restart the step with this many substeps
    int fallback = 0;     // learned mode: the prediction fell short
    int finalized = 0;    // products followed by a norm reduction and stop test
    double fix = 0;       // p holds d_{m+1} w_{m+1} too many (pair stopped at its first product)
    const void* fix_w = nullptr;   // where w_{m+1} is
    bool updated = false;          // the caller's update is already in the stream
    bool redo = false;             // the loop stopped at m, earlier than the deferred tests can take p
                                   // back to: run it again with Ctx::known = this
    int abandoned = 0;             // with redo: products that ran
};

struct Ctx {
    Op* op;
    int tw;                 // storage code of w, p: 0 double, 1 float
    char* ws;
    WsLayout L;
    NewtonState* st;
    double* partials;
    hipStream_t s;
    const double* xi;
    std::vector<double> d;
    double c, gamma, tol;
    int m_max;
    DdKey key;
    int profile;            // Params::profile
    const float* selector;
    int hidden;
    double ia, ib, tau;
    bool pairs;             // fuse consecutive products into pair sweeps
    // learned mode: a degree predicted earlier for this step (skip the
    // probe and the network), and whether the probe's prediction may change
    // the substep count: a prediction in [s_min, s_cur) ends the loop
    // (LoopOut::restart_s) so the caller can restart with fewer substeps
    int fixed_m = 0;
    bool decide_s = false;
    int s_cur = 1, s_min = 1;
    float* features = nullptr;   // device float[8]: features of the prediction
    std::vector<double> di;      // imaginary parts of d (complex operators; else empty)
    // stop tests of several launches at once where the degree is known from
    // an earlier loop, and chains of products on 2D stencils; `spare` is
    // workspace this loop may use for partials besides its own region
    bool defer = false;
    // what the loop's first run found (LoopOut::redo): the same products up to
    // that degree without tests
    const LoopOut* known = nullptr;
    bool chains = false;
    bool resident = false;   // the whole loop in one workgroup
    char* spare = nullptr;
    size_t spare_bytes = 0;
    int substep = 0;
};

// Bytes of partials a single product into vectors of storage code tw writes at
// most (stencils: with two points per lane or, where vectors are unaligned,
// one, whose rows may be laid out differently).
size_t single_partials(const Op& op, int tw) {
    Tiles t = product_tiles(op, tw, tw);
    int grid = make_geom(op, t).grid;
    if (op.kind == 0) {
        t.vec = 1;
        grid = std::max(grid, make_geom(op, t).grid);
    }
    return (size_t)grid * 4 * sizeof(double);
}

// The same of a launch of one Newton product or of a pair.
size_t newton_partials(const Ctx& C, bool two) {
    if (!two) return single_partials(*C.op, C.tw);
    return C.op->dim == 2 ? pair2d_partials(*C.op, PAIR_NEWTON) : (size_t)pair_geom(*C.op, device_cus()).grid * 32;
}

// Partials of launches whose tests are deferred: each needs a place of its
// own, taken from the workspace's partials region, then from `spare`.
struct TestPlan {
    TestArgs t{};
    const Ctx& C;
    size_t used = 0, used_spare = 0, cap;
    size_t room;           // the larger of the two: what one launch may take
    int products = 0;
    bool untested;         // launches only write their partials somewhere
    explicit TestPlan(const Ctx& c) : C(c), cap(partials_bytes(*c.op)), room(std::max(cap, c.spare_bytes)) {
        t.st = c.st;
        t.tol = c.tol;
        t.roff = -1;
        untested = c.known != nullptr;
    }
    // Room for the sums of two launches at least: the tests of one by itself
    // cost more than its finalize kernel (700^2 FP32, Euler step of two
    // substeps, where nothing is spare: 455 us against 440).
    bool holds_two() const {
        const size_t bytes = align256(newton_partials(C, C.pairs));
        return cap / bytes + C.spare_bytes / bytes >= 2;
    }
    // a place for `bytes` of partials (null: none left)
    double* place(size_t bytes, int n) {
        bytes = align256(bytes);
        if (untested) used = used_spare = 0;
        if (t.launches >= kMaxTestLaunches || products + n > kMaxTestProducts) return nullptr;
        if (used + bytes <= cap) {
            used += bytes;
            return reinterpret_cast<double*>(reinterpret_cast<char*>(C.partials) + used - bytes);
        }
        if (used_spare + bytes <= C.spare_bytes) {
            used_spare += bytes;
            return reinterpret_cast<double*>(C.spare + used_spare - bytes);
        }
        return nullptr;
    }
    void add(const double* part, int nparts, int stride, int off, int n) {
        if (untested) return;
        t.l[t.launches++] = TestLaunch{part, nparts, stride, off, n};
        products += n;
    }
    // the next places may overwrite these (their tests are in the stream)
    void clear() {
        t.launches = 0;
        products = 0;
        used = used_spare = 0;
    }
};

// Estimate of the degree from the divided differences alone: where their
// two-term sum falls below the tolerance for terms of the start vector's
// norm.  Rough inputs stop near it, smooth ones earlier.
int estimate_degree(const std::vector<double>& d, double tol, int m_max) {
    for (int m = 2; m <= m_max; ++m)
        if (std::fabs(d[m - 1]) + std::fabs(d[m]) <= tol * std::fabs(d[0])) return m;
    return m_max;
}

// First product reads `src` (storage code tin) and writes w_1 to w0 and p to
// `p`.  Later products read the buffer holding the latest w and write the
// other one: a single product j writes w_{j+1}, a pair sweep at j writes
// w_{j+2} (w_{j+1} stays on chip).
// start_u: an Euler step's first substep with its start vector fused into
// the first pair sweep (PAIR_START): `src` is then u (FP64) and r is never
// stored.
//
// spec: the caller's update, enqueued after each status read-back of the
// plain loop when it runs one batch at a time (a degree hint is known); it
// must run only if the loop has stopped (launch_update_st).  The host then
// needs no round trip between the stop and the update: out->updated tells
// that the update after the deciding read-back is in the stream.
int newton_loop(Ctx& C, const void* src, int tin, void* p, LoopOut* out, bool start_u = false,
                const std::function<hipError_t()>* spec = nullptr) {
    const std::vector<double>& d = C.d;
    if (C.resident && tin == 0) {
        // the whole loop in one launch
        ResidentArgs r{};
        r.x = static_cast<const double*>(src);
        r.p = static_cast<double*>(p);
        r.st = C.st;
        r.tol = C.tol;
        r.m_max = C.m_max;
        for (int q = 0; q <= C.m_max; ++q) r.d[q] = d[q];
        for (int q = 0; q < C.m_max; ++q) r.beta[q] = -(C.c / C.gamma + C.xi[q]);
        int slot;
        int rc = mirror_begin(&slot);
        if (rc) return rc;
        r.mirror = tl_ctx.pinned_dev + slot;
        HIP_TRY(launch_resident2d(*C.op, r, 1.0 / C.gamma, C.s));
        rc = mirror_end(slot, C.s);
        if (rc) return rc;
        if (spec) HIP_TRY((*spec)());
        NewtonState h;
        rc = wait_slot(slot, &h, C.st);
        if (rc) return rc;
        out->m = h.m;
        out->done = h.done;
        out->err = h.err;
        out->rnorm = h.rnorm;
        for (int q = 0; q < kHist; ++q) out->hist[q] = h.hist[q];
        out->finalized = h.m;
        out->updated = spec && h.done == 1;
        out->pair_launches = h.m / 2;   // products counted two by two
        out->single_launches = h.m % 2;
        if (h.done == 1) set_hint(*C.op, C.key, h.m);
        return EXPI_OK;
    }
    void* w[2] = {C.ws + C.L.w0, C.ws + C.L.w1};
    // tolerance of the stop tests of the launches enqueued next; 0 makes a
    // finalize record the norms and the latest term t_m without stopping
    // (the test t_{m-1} + t_m <= 0 holds only for an exactly zero sum)
    double tol_now = C.tol;
    SweepArgs a{};
    a.st = C.st;
    a.partials = C.partials;
    a.tol = C.tol;
    a.alpha = 1.0 / C.gamma;
    a.p = p;
    a.x = src;
    a.out = w[0];
    a.j = 0;
    a.beta = -(C.c / C.gamma + C.xi[0]);
    a.d0 = d[0];
    a.d1 = d[1];
    if (!C.di.empty()) {
        a.d0i = C.di[0];
        a.d1i = C.di[1];
    }
    a.guard = 0;
    int cur = 0;   // w[cur] holds the latest w

    struct Launch {
        int j, n;        // first product index, products covered
        const void* out;
        bool timed;      // events recorded around it
    };
    std::vector<Launch> log;
    // profile 1: time every launch from product 1 on; 2: only the first one
    bool sampled = false;
    auto timing = [&]() {
        if (C.profile == 1) return true;
        if (C.profile == 2 && !sampled) return sampled = true;
        return false;
    };

    // Products 0 and 1 in one pair sweep when the start vector has the
    // storage type and alignment the pair sweep reads (w_2 goes to w[0]:
    // `src` may be w[1]).  Otherwise product 0 alone.
    const bool first_pair = C.pairs && C.m_max >= 3 && tin == C.tw && (((uintptr_t)src & 15) == 0);
    // With a known degree, the products up to the last launch before it run
    // without a test each (their norms are kept) and are tested together:
    // jd is where the tested launches begin.  expected: the lowest degree this
    // substep stopped at lately; no test at or past it is deferred.  Without
    // one that is sure (kDegreeLoops, kChainLoops), chains of products are tested each, up
    // to where the loop is expected to stop or to half the estimated degree.
    // group: the degree the launches are laid out for, that of the last time.
    // A stop at the first product of a
    // pair leaves a rounding of the extra term in p, and pairs and single
    // products sum their norms in different orders, so 3D pairs are laid out
    // for the degree of the last loop of this length, whichever substep it
    // was, and only their tests are deferred.
    const DegreeKey degree_of = degree_key(C.key, C.substep, C.tol, C.tw);
    const DegreeWindow seen = get_degrees(*C.op, degree_of);
    const bool sure = seen.loops >= (C.chains ? kChainLoops : kDegreeLoops);
    const int expected = seen.low, own_degree = seen.last;
    const int last_degree = get_hint(*C.op, C.key);
    const int group = (own_degree >= 2 && (C.chains || !C.pairs)) ? own_degree : last_degree;
    const bool defer_on = C.defer && !C.profile && !C.selector;
    const bool chain_first = defer_on && C.chains && !start_u && tin == C.tw && C.m_max >= 6;
    const bool known = C.known != nullptr;
    TestPlan plan(C);
    int jd = 0;
    bool each = false;   // a test after every chain
    if (known) {
        jd = C.known->m;
    } else if (defer_on && expected >= 2 && group >= 2 && (C.chains || (sure && plan.holds_two()))) {
        const int open = (start_u || !(first_pair || chain_first)) ? 1 : 2;
        const int end = std::min(group, C.m_max);
        jd = end - ((C.pairs && (C.chains || (end - open) % 2 == 0)) ? 2 : 1);
        if (expected < end) jd = std::min(jd, C.pairs ? open + (expected - 1 - open) / 2 * 2 : expected - 1);
        // (without chains of 5, chains take an even count)
        if (C.chains && !chain2d_length(*C.op, 5) && (jd - (open == 2 ? 0 : 1)) % 2 != 0) --jd;
        each = !sure;
    } else if (defer_on && C.chains) {
        each = true;
        jd = estimate_degree(d, C.tol, C.m_max) / 2;
    }
    const bool guessed = each && expected < 2;   // no loop seen
    if (each) {
        // products 0 and 1 with tests (nearly constant vectors stop there),
        // then chains, of four where the degree is a guess, and of two where
        // those replace single products
        if (jd < (C.pairs ? 6 : 4)) jd = 0;
        else if (!C.pairs) jd = jd / 2 * 2;
        else if (guessed) jd = 2 + (jd - 2) / 4 * 4;
        each = jd > 0;
    }
    std::vector<int> tested;   // products that had run at each of the deferred tests
    int finalized = 0;
    int j = 0;
    auto mod = [&](int q) { return C.di.empty() ? std::fabs(d[q]) : std::hypot(d[q], C.di[q]); };
    // the tests of the launches collected so far
    auto flush = [&]() -> int {
        if (plan.t.launches == 0) return EXPI_OK;
        int m = plan.t.m0;
        int dof = 0;
        if (plan.t.roff >= 0) plan.t.d[dof++] = mod(0);
        for (int q = 0; q < plan.products; ++q) plan.t.d[dof + q] = mod(m + q);
        plan.t.dfix = d[m + plan.products - 1];
        HIP_TRY(launch_tests(plan.t, C.s));
        tested.push_back(m + plan.products - 1);
        // (the first value of a fused start is the start vector's norm)
        finalized += plan.products - (m == 0 ? 1 : 0);
        plan.t.m0 = m + plan.products;
        plan.t.roff = -1;
        plan.t.cont = 1;
        plan.clear();
        return EXPI_OK;
    };
    // products j .. j+n-1 as one chain (j = 0: from the start vector), tested
    // by the next flush; false in *ok when its partials have no place
    auto chain = [&](int j, int n, bool* ok) -> int {
        double* part = plan.place(chain2d_partials(*C.op, n, device_cus(), plan.room), n);
        *ok = part != nullptr;
        if (!part) return EXPI_OK;
        if (plan.t.launches == 0) plan.t.m0 = j + 1;
        ChainArgs b{};
        b.first = j == 0;
        b.x = b.first ? src : w[cur];
        b.out = b.first ? w[0] : w[cur ^ 1];
        b.p = p;
        b.partials = part;
        b.st = C.st;
        b.alpha = 1.0 / C.gamma;
        b.d0 = d[0];
        for (int q = 0; q < n; ++q) {
            b.beta[q] = -(C.c / C.gamma + C.xi[j + q]);
            b.d[q] = d[j + q + 1];
        }
        b.guard = plan.t.cont;
        int np = 0;
        HIP_TRY(launch_chain2d(*C.op, C.tw, n, b, device_cus(), plan.room, &np, C.s));
        if (b.first) plan.t.roff = 0;
        else cur ^= 1;
        plan.add(part, np, 16, 1, n);
        // (FP32 sums keep the bits of single products: such a stop runs again)
        plan.t.pair_last = n == 2 && (C.pairs || C.tw == 0);
        plan.t.outbuf = cur;
        log.push_back({j, n, w[cur], false});
        return EXPI_OK;
    };
    // Products 0 and 1 as a chain of two where the loop is laid out in chains
    // (a pair sweep that is tested by itself is no chain: it takes 424 us at
    // 8192^2 FP64, a chain of two 467; the two round alike).
    const bool chain_open = chain_first && (known ? jd >= 2 : jd >= 4 && !each);
    if (!chain_open && chain_first && (each ? !first_pair : first_pair && jd > 2)) {
        bool ok = true;
        int rc = chain(0, 2, &ok);
        if (rc) return rc;
        if (!ok) return fail(EXPI_EHIP, "internal: no room for a chain's partials");
        j = 2;
        if (each) rc = flush();
        if (rc) return rc;
    } else if (!chain_open) {
        double* part0 = C.partials;
        bool fin0 = true;
        if (known || (jd > 2 && !each)) {
            // the opening launch joins the deferred tests
            part0 = plan.place(!(start_u || first_pair) ? single_partials(*C.op, C.tw)
                               : C.op->dim == 2         ? pair2d_partials(*C.op, PAIR_FIRST)
                                                        : (size_t)pair_geom(*C.op, device_cus()).grid * 64,
                               2);
            fin0 = part0 == nullptr;
            if (!part0) part0 = C.partials;
        }
        a.partials = part0;
        int np = 0;
        if (start_u) {
            // r and product 0 in one pair sweep (j = -1: its tests are those at
            // m = 0 and m = 1, and neither can stop)
            PairArgs b{};
            b.x = src;
            b.out = w[0];
            b.p = p;
            b.partials = part0;
            b.st = C.st;
            b.alpha = 1.0 / C.gamma;
            b.sigma = 1.0;
            b.beta2 = -(C.c / C.gamma + C.xi[0]);
            b.d1 = d[0];
            b.d2 = d[1];
            b.tol = C.tol;
            b.j = -1;
            b.guard = 0;
            HIP_TRY(launch_pair(*C.op, C.tw, b, C.s, nullptr, fin0, PAIR_START, &np));
            log.push_back({-1, 2, w[0], false});
            j = 1;
            if (!fin0) plan.add(part0, np, 4, 0, 2);
            else finalized = 1;
        } else if (first_pair) {
            PairArgs b{};
            b.x = src;
            b.out = w[0];
            b.p = p;
            b.partials = part0;
            b.st = C.st;
            b.alpha = 1.0 / C.gamma;
            b.beta1 = -(C.c / C.gamma + C.xi[0]);
            b.beta2 = -(C.c / C.gamma + C.xi[1]);
            b.d0 = d[0];
            b.d1 = d[1];
            b.d2 = d[2];
            b.tol = C.tol;
            b.j = 0;
            b.guard = 0;
            HIP_TRY(launch_pair_op(*C.op, C.tw, b, C.s, nullptr, fin0, PAIR_FIRST, -1, &np));
            log.push_back({0, 2, w[0], false});
            j = 2;
            plan.t.m0 = 1;
            plan.t.roff = 0;
            if (!fin0) plan.add(part0, np, 8, 1, 2);
            else finalized = 2;
        } else {
            HIP_TRY(launch_sweep(*C.op, EPI_FIRST, tin, C.tw, a, C.s, nullptr, fin0, &np));
            log.push_back({0, 1, w[0], false});
            j = 1;
            plan.t.m0 = 1;
            plan.t.roff = 0;
            if (!fin0) plan.add(part0, np, 4, 1, 1);
            else finalized = 1;
        }
        a.partials = C.partials;
        if (fin0) {
            // tested already: deferred launches, if any, go on from its state
            plan.clear();
            plan.t.m0 = j + 1;
            plan.t.roff = -1;
            plan.t.cont = 1;
            if (!each) jd = 0;
        }
    }

    // single product j (j >= 1); `fin` adds the norm reduction and stop test
    // (with `part`, the launch leaves its norms there for the deferred tests)
    auto single = [&](int j, bool fin, double* part = nullptr) -> int {
        int np = 0;
        a.partials = part ? part : C.partials;
        a.x = w[cur];
        a.out = w[cur ^ 1];
        a.j = j;
        a.beta = -(C.c / C.gamma + C.xi[j]);
        a.d1 = d[j + 1];
        if (!C.di.empty()) a.d1i = C.di[j + 1];
        a.guard = (part && !plan.t.cont) ? 0 : 1;
        a.tol = tol_now;
        const bool tm = timing();
        if (tm) HIP_TRY(hipEventRecord(tl_ctx.tev[2 * j], C.s));
        HIP_TRY(launch_sweep(*C.op, EPI_NEWTON, C.tw, C.tw, a, C.s, tm ? tl_ctx.tev[2 * j + 1] : nullptr,
                             fin && !part, &np));
        if (part) {
            plan.add(part, np, 4, 1, 1);
            plan.t.pair_last = 0;
        }
        log.push_back({j, 1, w[cur ^ 1], tm});
        cur ^= 1;
        if (fin && !part) ++finalized;
        return EXPI_OK;
    };
    // products j and j+1 in one pair sweep
    auto pair = [&](int j, bool fin, double* part = nullptr) -> int {
        int np = 0;
        PairArgs b{};
        b.x = w[cur];
        b.out = w[cur ^ 1];
        b.p = p;
        b.partials = part ? part : C.partials;
        b.st = C.st;
        b.alpha = 1.0 / C.gamma;
        b.beta1 = -(C.c / C.gamma + C.xi[j]);
        b.beta2 = -(C.c / C.gamma + C.xi[j + 1]);
        b.d1 = d[j + 1];
        b.d2 = d[j + 2];
        b.tol = tol_now;
        b.j = j;
        b.guard = (part && !plan.t.cont) ? 0 : 1;
        b.outbuf = cur ^ 1;
        const bool tm = timing();
        if (tm) HIP_TRY(hipEventRecord(tl_ctx.tev[2 * j], C.s));
        HIP_TRY(launch_pair_op(*C.op, C.tw, b, C.s, tm ? tl_ctx.tev[2 * j + 1] : nullptr,
                               fin && !part, PAIR_NEWTON, -1, &np));
        if (part) {
            plan.add(part, np, 4, 0, 2);
            plan.t.pair_last = 1;
            plan.t.outbuf = cur ^ 1;
        }
        log.push_back({j, 2, w[cur ^ 1], tm});
        cur ^= 1;
        if (fin && !part) finalized += 2;
        return EXPI_OK;
    };
    // `count` products from j on (pairs where allowed), advancing j; the
    // finalize of the last launch writes the state into `mirror` if given.
    // fin = false: no norm reductions, except that the last launch records
    // its norms and terms (a finalize with tol 0, which cannot stop on
    // finite values), so that the next test's t_{m-1} is the term of the
    // product just before it, not that of the last tested one.
    auto advance = [&](int& j, int count, bool fin, NewtonState* mirror = nullptr) -> int {
        const int end = j + count;
        while (j < end) {
            int rc;
            const bool two = C.pairs && end - j >= 2;
            const bool last = j + (two ? 2 : 1) == end;
            if (last) set_state_mirror(mirror);
            const bool record = !fin && last;
            if (record) tol_now = 0.0;
            if (two) {
                rc = pair(j, fin || record);
                j += 2;
            } else {
                rc = single(j, fin || record);
                j += 1;
            }
            tol_now = C.tol;
            set_state_mirror(nullptr);
            if (rc) return rc;
        }
        return EXPI_OK;
    };
    auto sync_state = [&](NewtonState* st) -> int {
        int slot;
        int rc = readback(C.st, C.s, &slot);
        if (rc) return rc;
        return wait_slot(slot, st);
    };

    if (each && j == 1) {
        const int rc = single(1, true);
        if (rc) return rc;
        j = 2;
    }
    // the deferred part: products up to jd
    while (j < jd) {
        int rc;
        bool ok = true;
        const int left = jd - j;
        if (C.chains) {
            // (const coefficient: 6, then 5 or 4 so that what is left is no
            // single product, and a pair for a remainder of 2; else 4 and 2)
            int n = 0;
            const bool six = !guessed && chain2d_length(*C.op, 6);
            if (six && left >= 6 && left != 8 && left != 7 && left != 9) n = 6;
            else if (six && (left == 5 || left == 7 || left == 9)) n = 5;
            else if (left >= 4) n = 4;
            else if (left >= 2 && (j > 0 || known)) n = 2;
            if (n) {
                rc = chain(j, n, &ok);
                if (rc) return rc;
                if (ok) j += n;
                if (ok && each) rc = flush();
                if (rc) return rc;
                if (ok) continue;
                // no place left: test what there is, which frees all places
                if (plan.t.launches == 0) break;
                rc = flush();
                if (rc) return rc;
                continue;
            }
        }
        if (each) break;
        const bool two = C.pairs && left >= 2;
        double* part = plan.place(newton_partials(C, two), two ? 2 : 1);
        if (!part) {
            if (plan.t.launches == 0) break;
            rc = flush();
            if (rc) return rc;
            continue;
        }
        rc = two ? pair(j, false, part) : single(j, false, part);
        if (rc) return rc;
        j += two ? 2 : 1;
    }
    // (an empty plan has room for any launch, so a chain that opens the loop
    // has run: the launches below go on from it)
    if (j == 0) return fail(EXPI_EHIP, "internal: the opening chain was not launched");
    {
        const int rc = flush();
        if (rc) return rc;
    }
    a.partials = C.partials;

    // launches that began before the stop did work (the opening ones always
    // do); later ones returned at once
    auto count_launches = [&](int m) {
        for (const Launch& L : log) {
            if (L.j >= m && L.j > 0) continue;
            // (a chain counts its products two by two)
            if (L.n >= 2) out->pair_launches += L.n / 2;
            else ++out->single_launches;
        }
    };
    auto learn = [&](int m) {
        set_hint(*C.op, C.key, m);
        add_degree(*C.op, degree_of, m);
    };
    if (known) {
        if (j != jd) return fail(EXPI_EHIP, "internal: products missing from a loop run again");
        HIP_TRY(launch_accept(C.st, C.s));
        *out = *C.known;
        out->redo = false;
        learn(jd);
        count_launches(jd);
        return EXPI_OK;
    }

    NewtonState last{};
    bool finished = false;
    bool learned_tail = false;
    bool have_pred = false;
    int pred = 0;
    if (C.selector && C.m_max >= 6 && C.fixed_m > 0) {
        // learned mode with the degree already predicted for this step
        pred = C.fixed_m;
        have_pred = true;
        out->pred_m = pred;
    } else if (C.selector && C.m_max >= 6 && (C.decide_s || get_hint(*C.op, C.key) < 2)) {
        // (the network is consulted where it can change something: where a
        // shorter substep count is allowed, or where the plain loop has no
        // degree from an earlier loop with the same substep length)
        // Learned mode: four products with stop tests give the features; the
        // network predicts the substep count and the degree m; products up to
        // m skip the norm reductions except the last two, whose two-term stop
        // test judges the prediction.  If it is not met the plain loop below
        // continues.  Products up to 3 (at least) with stop tests (t_0..t_4
        // are recorded by the tests); pair sweeps where allowed, so that a
        // loop opened by the start-vector pair runs products 1-2 and 3-4 as
        // pairs
        while (j < 4) {
            const int rc = C.pairs ? pair(j, true) : single(j, true);
            if (rc) return rc;
            j += C.pairs ? 2 : 1;
        }
        HIP_TRY(launch_selector(C.selector, C.hidden, C.st, C.ia, C.ib, C.tau, C.m_max, C.features, C.s));
        int rc = sync_state(&last);
        if (rc) return rc;
        out->pred_m = last.pred_m;
        out->pred_s = last.pred_s;
        if (last.done) {
            finished = true;
        } else {
            pred = last.pred_m;
            have_pred = true;
            const int sh = std::min(std::max(last.pred_s, C.s_min), C.s_cur);
            if (C.decide_s && sh < C.s_cur) {
                // fewer, longer substeps: the caller restarts the step
                out->restart_s = sh;
                out->finalized = finalized;
                out->m = last.m;
                return EXPI_OK;
            }
        }
    }
    if (have_pred) {
        {
            int rc;
            const int mh = std::min(std::max(pred, j + 1), C.m_max);
            // products up to mh - 2 without stop tests (the last of them
            // records t_{mh-2}), then the last two with tests (one pair
            // sweep tests after each of its two products)
            if (mh - 2 > j) {
                rc = advance(j, mh - 2 - j, false);
                if (rc) return rc;
            }
            // the last two with tests; as in the plain loop, their state
            // comes back through a pinned slot and the update (guarded by
            // the stop flag) is enqueued before the host waits for it
            int slot;
            rc = mirror_begin(&slot);
            if (rc) return rc;
            rc = advance(j, mh - j, true, tl_ctx.pinned_dev + slot);
            if (rc) return rc;
            rc = mirror_end(slot, C.s);
            if (rc) return rc;
            if (spec) HIP_TRY((*spec)());
            rc = wait_slot(slot, &last, C.st);
            if (rc) return rc;
            if (last.done) finished = true;
            else out->fallback = 1;
            out->updated = spec && last.done == 1;
        }
        learned_tail = true;
    }

    if (!finished) {
        const int hint = learned_tail ? 0 : group;
        // With a degree hint (or after a prediction) the first batch ends at
        // the expected stop and later batches are one launch; without one,
        // batches of 4 then 2 products run one batch ahead of the status
        // read-back.
        const int step = C.pairs ? 2 : 1;
        int chunk = learned_tail ? step : (hint >= 2 ? std::max(hint - j, 1) : 4);
        const bool ahead = !learned_tail && hint < 2;
        std::deque<int> pending;
        while (!finished) {
            if (j < C.m_max) {
                const int cnt = std::min(chunk, C.m_max - j);
                int slot;
                int rc = mirror_begin(&slot);
                if (rc) return rc;
                rc = advance(j, cnt, true, tl_ctx.pinned_dev + slot);
                if (rc) return rc;
                rc = mirror_end(slot, C.s);
                if (rc) return rc;
                pending.push_back(slot);
                if (spec && !ahead) HIP_TRY((*spec)());
                chunk = ahead ? 2 : step;
            }
            const size_t keep = ahead ? 1 : 0;
            while (!pending.empty() && (pending.size() > keep || j >= C.m_max)) {
                int rc = wait_slot(pending.front(), &last, C.st);
                if (rc) return rc;
                pending.pop_front();
                if (last.done) {
                    finished = true;
                    break;
                }
            }
            if (!finished && pending.empty() && j >= C.m_max) finished = true;
        }
        out->updated = spec && !ahead && last.done == 1;
    }
    out->m = last.m;
    out->done = last.done;
    out->err = last.err;
    out->rnorm = last.rnorm;
    for (int q = 0; q < kHist; ++q) out->hist[q] = last.hist[q];
    out->finalized = finalized;
    if (last.done == 3) {
        // the launches past the tests that found the stop did nothing
        out->redo = true;
        out->done = 1;
        for (int q : tested)
            if (out->abandoned < last.m) out->abandoned = q;
        out->finalized = out->abandoned;
        return EXPI_OK;
    }
    if (last.done == 1 && last.fix != 0.0) {
        // the pair sweep at m - 1 wrote w_{m+1}
        for (const Launch& L : log)
            if (L.n == 2 && L.j == last.m - 1) out->fix_w = L.out;
        if (!out->fix_w) return fail(EXPI_EHIP, "internal: no pair sweep for the stop at m");
        out->fix = last.fix;
    }
    if (last.done == 1) learn(last.m);
    if (last.done != 2) count_launches(last.m);
    if (C.profile && last.done != 2) {
        // launches that began before the stop did work and precede the read-back
        for (const Launch& L : log) {
            if (!L.timed || L.j >= last.m) continue;
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, tl_ctx.tev[2 * L.j], tl_ctx.tev[2 * L.j + 1]));
            out->ms += ms;
            out->timed += L.n;
            if (L.n == 2) {
                out->pair_ms += ms;
                out->pairs_timed += 1;
            }
        }
    }
    return EXPI_OK;
}

void stats_add(expi_stats* st, const LoopOut& lo) {
    if (st->newton_steps == 0 && st->matvecs <= 1) {
        // features of the first substep's loop
        st->rnorm = lo.rnorm;
        for (int q = 0; q < kHist; ++q) st->t_first[q] = lo.hist[q];
        st->pred_degree = lo.pred_m;
        st->pred_substeps = lo.pred_s;
    }
    st->fallback += lo.fallback;
    st->finalized += lo.finalized;
    st->newton_steps += lo.m;
    st->matvecs += lo.m;
    st->degree_max = std::max(st->degree_max, lo.m);
    st->degree_last = lo.m;
    st->err_est = std::max(st->err_est, lo.err);
    st->timed_products += lo.timed;
    st->newton_ms += lo.ms;
    st->timed_pairs += lo.pairs_timed;
    st->pair_ms += lo.pair_ms;
    st->pair_launches += lo.pair_launches;
    st->single_launches += lo.single_launches;
}

int common_setup(Op& op, double tau, double tol, int dtype, const Params& P, char* ws,
                 hipStream_t s, double* ia, double* ib) {
    (void)tau;
    (void)tol;
    (void)dtype;
    int rc = ctx_init();
    if (rc) return rc;
    if (P.profile) {
        rc = timing_events();
        if (rc) return rc;
    }
    if (P.have_interval) {
        *ia = P.ia;
        *ib = P.ib;
    } else {
        rc = op_interval(op, ia, ib, ws, s);
        if (rc) return rc;
    }
    if (!(*ia < *ib))
        return fail(EXPI_EINVAL, "degenerate spectral interval (a >= b); pass one in params");
    return EXPI_OK;
}

int substep_count(double tau, double a, double b, double l_max) {
    const double q = std::ceil(tau * (b - a) / l_max);
    if (!(q >= 1.0)) return 1;
    if (q > 1e8) return 100000000;
    return (int)q;
}

int validate_call(const expi_op* op, double tau, double tol, int dtype, void* ws, size_t ws_bytes) {
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    if (!(tau >= 0) || !std::isfinite(tau)) return fail(EXPI_EINVAL, "tau must be finite and >= 0");
    if (!(tol > 0) || !std::isfinite(tol)) return fail(EXPI_EINVAL, "tol must be finite and > 0");
    if (dtype != EXPI_F64 && dtype != EXPI_F32) return fail(EXPI_EINVAL, "dtype must be EXPI_F64 or EXPI_F32");
    if (!ws) return fail(EXPI_EWORKSPACE, "workspace is NULL");
    if (((uintptr_t)ws & 255) != 0) return fail(EXPI_EWORKSPACE, "workspace must be 256-byte aligned");
    if (reinterpret_cast<const Op*>(op)->kind == 2 && dtype != EXPI_F64)
        return fail(EXPI_EINVAL, "complex operators run in FP64 only");
    const size_t need = layout(*reinterpret_cast<const Op*>(op), dtype).total;
    if (ws_bytes < need)
        return fail(EXPI_EWORKSPACE, "workspace too small: need " + std::to_string(need) + " bytes");
    return EXPI_OK;
}

}  // namespace

void set_error(const std::string& msg) { tl_error = msg; }

// ---- phi_action -------------------------------------------------------------------
// y_slot: whether the layout's y slot is free for this call.
static int run_phi(Op& op, int k, double tau, const double* v, double* y, double tol, int dtype,
                   const Params& P, char* ws, expi_stats* st, hipStream_t s, bool y_slot = true) {
    double ia, ib;
    int rc = common_setup(op, tau, tol, dtype, P, ws, s, &ia, &ib);
    if (rc) return rc;
    const double c = 0.5 * (ia + ib), gamma = 0.25 * (ib - ia);
    const int count = P.m_max + 1;
    const double* xi = leja_points(count);
    const int tw = (dtype == EXPI_F32) ? 1 : 0;
    const WsLayout L = layout(op, dtype);
    const int64_t n = op.size;
    int sub = substep_count(tau, ia, ib, P.l_max);
    Ctx C{&op, tw, ws, L, reinterpret_cast<NewtonState*>(ws + L.state),
          reinterpret_cast<double*>(ws + L.partials), s, xi, {}, c, gamma, tol, P.m_max, {},
          P.profile, P.selector, P.hidden, ia, ib, tau, P.pairs && pairs_on(op, tw)};
    expi_stats acc{};
    for (int attempt = 0; attempt <= P.max_retries; ++attempt) {
        const double delta = tau / sub;
        C.key = DdKey(k, delta, c, gamma, count);
        C.d = get_dd(op, C.key);
        const int rerun = acc.rerun_products;
        acc = expi_stats{};
        acc.rerun_products = rerun;
        acc.substeps = sub;
        acc.retries = attempt;
        acc.interval_a = ia;
        acc.interval_b = ib;
        // (a loop in one workgroup writes the whole record itself)
        C.chains = P.pairs && op.use_pairs != 0 && chain2d_supported(op, tw);
        C.resident = C.chains && !P.profile && !P.selector && resident2d_supported(op, tw, P.m_max);
        if (!C.resident) HIP_TRY(launch_reset(C.st, s));
        bool ok = true;
        LoopOut stop;   // a loop to be run again
        for (int l = 0; l < sub && ok; ++l) {
            // p goes straight into y when y is the result and has p's type
            const bool p_in_y = (sub == 1 && tw == 0);
            void* p = p_in_y ? (void*)y : (void*)(ws + L.p);
            const void* src;
            int tin;
            // phi_k, k >= 2, over several substeps: z_l = y(l delta)/tau^k is
            // kept in y; the substep is sum_{j<k} w_j/j! + phi_k(delta A) w_k
            // with w_0 = z_l, w_j = delta A w_{j-1} + c_j v,
            // c_j = s^-j (l/s)^(k-j)/(k-j)!.  At l = 0 every w_j but w_k is
            // zero and w_k = s^-k v, so the loop runs on v and p is scaled.
            const bool phik_sub = (k >= 2 && sub > 1);
            double pscale = (k == 1) ? 1.0 / sub : 1.0;
            if (phik_sub && l == 0) {
                src = v;
                tin = 0;
                pscale = std::pow((double)sub, -(double)k);
            } else if (phik_sub) {
                // w_k lands in w1 (the loop's start vector); w_{k-1} in w0,
                // which the loop's first product overwrites after reading w1
                const void* prev = y;
                int tprev = 0;
                double fact = 1.0;   // j!
                for (int jj = 1; jj <= k; ++jj) {
                    fact *= jj;
                    void* buf = ((k - jj) % 2 == 0) ? (void*)(ws + L.w1) : (void*)(ws + L.w0);
                    double kf = 1.0;   // (k - jj)!
                    for (int q = 2; q <= k - jj; ++q) kf *= q;
                    SweepArgs a{};
                    a.x = prev;
                    a.out = buf;
                    a.g = v;
                    a.gmode = G_VEC_SCALED;
                    a.gscale = std::pow((double)sub, -(double)jj) *
                               std::pow((double)l / sub, (double)(k - jj)) / kf;
                    a.sigma = delta;
                    HIP_TRY(launch_sweep(op, EPI_START, tprev, tw, a, s));
                    acc.matvecs += 1;
                    // y <- y + w_j / j! for j < k
                    if (jj < k) HIP_TRY(launch_update(n, y, y, buf, tw, 1.0 / fact, C.st, 0, s));
                    prev = buf;
                    tprev = tw;
                }
                src = ws + L.w1;
                tin = tw;
            } else if (k == 1 && l > 0) {
                // r = A y_l + v with y_l = tau * y' (y' = y_l / tau is kept in y)
                SweepArgs a{};
                a.x = y;
                a.out = ws + L.w1;
                a.g = v;
                a.gmode = G_VEC;
                a.sigma = tau;
                HIP_TRY(launch_sweep(op, EPI_START, 0, tw, a, s));
                acc.matvecs += 1;
                src = ws + L.w1;
                tin = tw;
            } else if (k != 1 && l > 0) {
                src = y;   // previous substep's result, copied into y below
                tin = 0;
            } else {
                src = v;
                tin = 0;
            }
            LoopOut lo;
            C.pairs = P.pairs && pairs_on(op, tw) && (((uintptr_t)p & 15) == 0);
            C.spare = y_slot ? ws + L.y : nullptr;
            C.spare_bytes = y_slot ? (size_t)n * 8 : 0;
            // (a substep of phi_k, k >= 2, adds to y while it forms its start
            // vector, so it cannot be run again)
            C.defer = !(phik_sub && l > 0);
            C.substep = l;
            C.known = stop.redo ? &stop : nullptr;
            // the update of this substep, enqueued ahead of the status
            // read-back where it always runs (p_in_y needs one only for a fix)
            const double* yin = ((k == 1 || phik_sub) && l > 0) ? y : nullptr;
            const double scale = pscale;
            const std::function<hipError_t()> spec = [&]() {
                return launch_update_st(n, y, yin, p, tw, scale, C.st, ws + L.w0, ws + L.w1, s);
            };
            rc = newton_loop(C, src, tin, p, &lo, false, p_in_y ? nullptr : &spec);
            if (rc) return rc;
            if (lo.redo) {
                // the same substep up to the degree found
                const int start = k == 1 && l > 0 ? 1 : 0;   // (its start vector is formed again)
                acc.matvecs -= start;
                acc.rerun_products += lo.abandoned + start;
                stop = lo;
                --l;
                continue;
            }
            stop.redo = false;
            stats_add(&acc, lo);
            if (lo.done == 2) return fail(EXPI_ENONFINITE, "a norm became inf/NaN (non-finite input?)");
            if (lo.done != 1) {
                ok = false;
                break;
            }
            if (!p_in_y) {
                // k = 1: y' <- y' + p / s (y' = 0 before the first substep);
                // k >= 2 over substeps: z <- z + p (l > 0) or s^-k p (l = 0);
                // otherwise e^{delta A} (or phi_k, single substep) applied: y <- p
                if (!lo.updated)
                    HIP_TRY(launch_update(n, y, yin, p, tw, scale, C.st, 1, s, lo.fix_w, lo.fix));
            } else if (lo.fix != 0.0) {
                // y holds p: remove the one term too many in place
                HIP_TRY(launch_update(n, y, nullptr, y, 0, 1.0, C.st, 1, s, lo.fix_w, lo.fix));
            }
        }
        acc.converged = ok ? 1 : 0;
        if (ok) {
            if (st) *st = acc;
            return EXPI_OK;
        }
        sub *= 2;
    }
    if (st) *st = acc;
    return fail(EXPI_ENOTCONV, "no convergence within m_max products after all substep doublings");
}

static int run_expeuler(Op& op, int nonlin, double tau, double* u, double tol, int dtype,
                        const Params& P, char* ws, expi_stats* st, hipStream_t s) {
    double ia, ib;
    int rc = common_setup(op, tau, tol, dtype, P, ws, s, &ia, &ib);
    if (rc) return rc;
    const double c = 0.5 * (ia + ib), gamma = 0.25 * (ib - ia);
    const int count = P.m_max + 1;
    const double* xi = leja_points(count);
    const int tw = (dtype == EXPI_F32) ? 1 : 0;
    const WsLayout L = layout(op, dtype);
    const int64_t n = op.size;
    int sub = substep_count(tau, ia, ib, P.l_max);
    Ctx C{&op, tw, ws, L, reinterpret_cast<NewtonState*>(ws + L.state),
          reinterpret_cast<double*>(ws + L.partials), s, xi, {}, c, gamma, tol, P.m_max, {},
          P.profile, P.selector, P.hidden, ia, ib, tau, P.pairs && pairs_on(op, tw)};
    double* yb = reinterpret_cast<double*>(ws + L.y);
    void* p = ws + L.p;
    expi_stats acc{};
    // learned mode: the probe of the first loop may predict fewer substeps
    // (at least ceil(tau (b - a) / sel_l_max)); the step then restarts with
    // them and the predicted degree.  If that fails, the plain method redoes
    // the step with the original substep count.
    const int s_plain = sub;
    const int s_min = std::max(1, substep_count(tau, ia, ib, P.sel_l_max));
    C.features = P.sel_features;
    bool learned_sub = false;     // running the predicted substep count
    int wasted_mv = 0, wasted_newton = 0, wasted_fin = 0, pred_s = 0, pred_m = 0, fallbacks = 0;
    // products spent on an abandoned probe or a failed prediction count too
    auto finish = [&](expi_stats& a) {
        a.matvecs += wasted_mv;
        a.newton_steps += wasted_newton;
        a.finalized += wasted_fin;
        a.fallback += fallbacks;
        if (pred_s) {
            a.pred_substeps = pred_s;
            a.pred_degree = pred_m;
        }
    };
    for (int attempt = 0; attempt <= P.max_retries; ++attempt) {
        const double delta = tau / sub;
        C.key = DdKey(1, delta, c, gamma, count);
        C.d = get_dd(op, C.key);
        C.s_cur = sub;
        C.s_min = s_min;
        C.decide_s = C.selector && attempt == 0 && !learned_sub && s_min < sub;
        C.fixed_m = learned_sub ? pred_m : 0;
        // substeps longer than l_max (only the learned count makes them):
        // the stop test's tolerance scales by l_max / (delta (b - a)), since
        // the two-term estimate of the remainder is looser on long substeps
        const double len = delta * (ib - ia);
        C.tol = (learned_sub && len > P.l_max) ? tol * (P.l_max / len) : tol;
        const int rerun = acc.rerun_products;
        acc = expi_stats{};
        acc.rerun_products = rerun;
        acc.substeps = sub;
        acc.retries = attempt;
        acc.interval_a = ia;
        acc.interval_b = ib;
        HIP_TRY(launch_reset(C.st, s));
        bool ok = true;
        LoopOut stop;   // a loop to be run again
        int restart = 0;
        for (int l = 0; l < sub && ok; ++l) {
            // r = A y_l + g(u), y_0 = u: its own sweep, or (first substep)
            // the first half of the loop's first pair sweep.  The fused form
            // saves a sweep when the degree m is odd and costs one (a single
            // product at the end) when it is even; the degree the last step
            // with this step size stopped at decides.
            const int hint = get_hint(op, C.key);
            // (the fused start vector forms u - u^3 only)
            const bool fuse = l == 0 && nonlin == EXPI_G_CUBIC && op.bdata == EXPI_BDATA_NONE &&
                              C.pairs && C.m_max >= 3 &&
                              pair_start_supported(op) &&
                              (((uintptr_t)u & 15) == 0) &&
                              (P.fuse_start == 2 || (P.fuse_start == 0 && hint >= 3 && hint % 2 == 1));
            acc.matvecs += 1;
            // y_{l+1} = y_l + delta p; the last substep writes u
            const double* yin = (l == 0) ? u : yb;
            double* yout = (l == sub - 1) ? u : yb;
            const std::function<hipError_t()> spec = [&]() {
                return launch_update_st(n, yout, yin, p, tw, delta, C.st, ws + L.w0, ws + L.w1, s);
            };
            LoopOut lo;
            C.chains = P.pairs && op.use_pairs != 0 && chain2d_supported(op, tw);
            C.resident = C.chains && !P.profile && !P.selector && resident2d_supported(op, tw, P.m_max);
            C.spare = sub == 1 ? ws + L.y : nullptr;   // y_l lives there otherwise
            C.spare_bytes = sub == 1 ? (size_t)n * 8 : 0;
            C.defer = true;
            C.substep = l;
            C.known = stop.redo ? &stop : nullptr;
            if (fuse) {
                rc = newton_loop(C, u, 0, p, &lo, true, &spec);
                acc.fused_starts += 1;
            } else {
                SweepArgs a{};
                a.x = (l == 0) ? (const void*)u : (const void*)yb;
                a.out = ws + L.w1;
                a.g = u;
                a.gmode = (l == 0) ? G_CUBIC_SELF : G_CUBIC_OF;
                a.gkind = nonlin;
                a.bdata = op.bdata;   // u' = A_0 u + b_f + g(u)
                a.sigma = 1.0;
                HIP_TRY(launch_sweep(op, EPI_START, 0, tw, a, s));
                rc = newton_loop(C, ws + L.w1, tw, p, &lo, false, &spec);
            }
            if (rc) return rc;
            if (lo.redo) {
                // the same substep up to the degree found
                acc.matvecs -= 1;
                acc.rerun_products += lo.abandoned + 1;
                if (fuse) acc.fused_starts -= 1;
                stop = lo;
                --l;
                continue;
            }
            if (lo.restart_s) {
                // the probe predicts fewer substeps: its products are spent
                restart = lo.restart_s;
                pred_s = lo.restart_s;
                pred_m = lo.pred_m;
                wasted_mv = acc.matvecs + lo.m;
                wasted_newton = lo.m;
                wasted_fin = lo.finalized;
                break;
            }
            stop.redo = false;
            stats_add(&acc, lo);
            if (lo.done == 2) return fail(EXPI_ENONFINITE, "a norm became inf/NaN (non-finite input?)");
            if (lo.done != 1) {
                ok = false;
                break;
            }
            if (!lo.updated) HIP_TRY(launch_update(n, yout, yin, p, tw, delta, C.st, 1, s, lo.fix_w, lo.fix));
        }
        if (restart) {
            // not a retry: the step starts again with the predicted count
            sub = restart;
            learned_sub = true;
            --attempt;
            continue;
        }
        acc.converged = ok ? 1 : 0;
        if (ok) {
            finish(acc);
            if (st) *st = acc;
            return EXPI_OK;
        }
        if (learned_sub) {
            // the predicted substep count failed: the plain method, from u
            wasted_mv += acc.matvecs;
            wasted_newton += acc.newton_steps;
            wasted_fin += acc.finalized;
            fallbacks += 1;
            learned_sub = false;
            C.selector = nullptr;
            sub = s_plain;
            --attempt;
            continue;
        }
        sub *= 2;
    }
    finish(acc);
    if (st) *st = acc;
    return fail(EXPI_ENOTCONV, "no convergence within m_max products after all substep doublings");
}

// ---- complex operators: phi_k(-i tau H) v ------------------------------------------
// Hermitian H in complex CSR; the same Newton recurrence on (H - cI)/gamma
// with the complex divided differences of x -> phi_k(-i delta (c + gamma x))
// (single products; the loop, stop test and status read-backs are those of
// phi_action).  k = 0: y_{l+1} = e^{-i delta H} y_l.  k = 1: y(t) = t phi_1(-i t H) v
// solves y' = -i H y + v; y' = y/tau is kept in y and r = -i tau H y' + v.
static int run_skew(Op& op, int k, double tau, const double* v, double* y, double tol,
                    const Params& P, char* ws, expi_stats* st, hipStream_t s) {
    double ia, ib;
    int rc = common_setup(op, tau, tol, EXPI_F64, P, ws, s, &ia, &ib);
    if (rc) return rc;
    const double c = 0.5 * (ia + ib), gamma = 0.25 * (ib - ia);
    const int count = P.m_max + 1;
    const double* xi = leja_points(count);
    const WsLayout L = layout(op, EXPI_F64);
    const int64_t nd = op.size * 2;   // doubles per vector
    int sub = substep_count(tau, ia, ib, P.l_max);
    Ctx C{&op, 0, ws, L, reinterpret_cast<NewtonState*>(ws + L.state),
          reinterpret_cast<double*>(ws + L.partials), s, xi, {}, c, gamma, tol, P.m_max, {},
          P.profile, nullptr, 0, ia, ib, tau, false};
    expi_stats acc{};
    for (int attempt = 0; attempt <= P.max_retries; ++attempt) {
        const double delta = tau / sub;
        // the key's k is offset so the real and complex coefficients never share a cache slot
        C.key = DdKey(1000 + k, delta, c, gamma, count);
        get_dd_skew(op, k, C.key, &C.d, &C.di);
        const int rerun = acc.rerun_products;
        acc = expi_stats{};
        acc.rerun_products = rerun;
        acc.substeps = sub;
        acc.retries = attempt;
        acc.interval_a = ia;
        acc.interval_b = ib;
        HIP_TRY(launch_reset(C.st, s));
        bool ok = true;
        LoopOut stop;   // a loop to be run again
        C.spare = ws + L.y;   // not used otherwise
        C.spare_bytes = (size_t)nd * 8;
        for (int l = 0; l < sub && ok; ++l) {
            const bool p_in_y = (sub == 1);
            void* p = p_in_y ? (void*)y : (void*)(ws + L.p);
            const void* src = v;
            if (k == 1 && l > 0) {
                SweepArgs a{};
                a.x = y;
                a.out = ws + L.w1;
                a.g = v;
                a.gmode = G_VEC;
                a.sigma = 0.0;
                a.sigmai = -tau;
                HIP_TRY(launch_sweep(op, EPI_START, 0, 0, a, s));
                acc.matvecs += 1;
                src = ws + L.w1;
            } else if (k == 0 && l > 0) {
                src = y;
            }
            LoopOut lo;
            C.defer = true;
            C.substep = l;
            C.known = stop.redo ? &stop : nullptr;
            rc = newton_loop(C, src, 0, p, &lo);
            if (rc) return rc;
            if (lo.redo) {
                // the same substep up to the degree found
                const int start = k == 1 && l > 0 ? 1 : 0;   // (its start vector is formed again)
                acc.matvecs -= start;
                acc.rerun_products += lo.abandoned + start;
                stop = lo;
                --l;
                continue;
            }
            stop.redo = false;
            stats_add(&acc, lo);
            if (lo.done == 2) return fail(EXPI_ENONFINITE, "a norm became inf/NaN (non-finite input?)");
            if (lo.done != 1) {
                ok = false;
                break;
            }
            if (!p_in_y) {
                // k = 1: y' <- y' + p/s; k = 0: y <- p (complex vectors as pairs of doubles)
                const double* yin = (k == 1 && l > 0) ? y : nullptr;
                HIP_TRY(launch_update(nd, y, yin, p, 0, k == 1 ? 1.0 / sub : 1.0, C.st, 1, s));
            }
        }
        acc.converged = ok ? 1 : 0;
        if (ok) {
            if (st) *st = acc;
            return EXPI_OK;
        }
        sub *= 2;
    }
    if (st) *st = acc;
    return fail(EXPI_ENOTCONV, "no convergence within m_max products after all substep doublings");
}

// ---- second-order exponential Runge-Kutta step ---------------------------------
// U = u + tau phi_1(tau A)(A u + g(u)); u <- U + tau phi_2(tau A)(g(U) - g(u)).
// Workspace: phi_action's layout, then u_n (float64).  g(U) - g(u_n) goes to
// the layout's y slot (unused by run_phi), phi_2 of it into the u_n slot.
size_t exprk2_bytes(const Op& op, int dtype) {
    return layout(op, dtype).total + align256((size_t)op.size * 8);
}

static int run_exprk2(Op& op, int nonlin, double tau, double* u, double tol, int dtype,
                      const Params& P, char* ws, expi_stats* st, hipStream_t s) {
    const WsLayout L = layout(op, dtype);
    const int64_t n = op.size;
    double* un = reinterpret_cast<double*>(ws + L.total);
    double* dg = reinterpret_cast<double*>(ws + L.y);
    HIP_TRY(hipMemcpyAsync(un, u, (size_t)n * 8, hipMemcpyDeviceToDevice, s));
    expi_stats s1{}, s2{};
    int rc = run_expeuler(op, nonlin, tau, u, tol, dtype, P, ws, &s1, s);
    if (rc) {
        if (st) *st = s1;
        return rc;
    }
    HIP_TRY(launch_gdiff(nonlin, n, u, un, dg, s));
    rc = run_phi(op, 2, tau, dg, un, tol, dtype, P, ws, &s2, s, false);
    expi_stats acc = s1;
    acc.substeps = std::max(s1.substeps, s2.substeps);
    acc.newton_steps += s2.newton_steps;
    acc.matvecs += s2.matvecs;
    acc.retries += s2.retries;
    acc.converged = s1.converged && s2.converged;
    acc.degree_max = std::max(s1.degree_max, s2.degree_max);
    acc.degree_last = s2.degree_last;
    acc.err_est = std::max(s1.err_est, s2.err_est);
    acc.timed_products += s2.timed_products;
    acc.newton_ms += s2.newton_ms;
    acc.finalized += s2.finalized;
    acc.timed_pairs += s2.timed_pairs;
    acc.pair_ms += s2.pair_ms;
    acc.pair_launches += s2.pair_launches;
    acc.single_launches += s2.single_launches;
    acc.rerun_products += s2.rerun_products;
    if (st) *st = acc;
    if (rc) return rc;
    // u <- U + tau phi_2(tau A)(g(U) - g(u_n))
    HIP_TRY(launch_update(n, u, u, un, 0, tau, nullptr, 0, s));
    return EXPI_OK;
}

// ---- allocation-free phi_action ---------------------------------------------
// The scratch array lives in the library's code object, one copy per GPU.
// Host code never passes `scratch` itself to a kernel (its host-side name is
// not a device address): expi_noalloc_init looks up each device's address
// with hipGetSymbolAddress and every later use goes through that pointer.
static __device__ __align__(256) unsigned char scratch[EXPI_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch[kMaxDevices] = {};

int noalloc_init() {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(EXPI_EINVAL, "device index out of range");
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch[dev]) {
            void* ptr = nullptr;
            HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
            if (!ptr || ((uintptr_t)ptr & 255) != 0)
                return fail(EXPI_EHIP, "scratch array has no 256-byte aligned device address");
            g_scratch[dev] = static_cast<char*>(ptr);
        }
    }
    // the calling thread's pinned status slots and timing events
    int rc = ctx_init();
    if (rc) return rc;
    return timing_events();
}

// This thread's set-up for the current device, or an error (no allocation).
int noalloc_scratch(char** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    char* ptr = nullptr;
    if (dev >= 0 && dev < kMaxDevices) {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        ptr = g_scratch[dev];
    }
    if (!ptr || tl_ctx.device != dev || !tl_ctx.pinned || !tl_ctx.have_tev)
        return fail(EXPI_EINVAL, "expi_noalloc_init has not run on this thread for the current device");
    *out = ptr;
    return EXPI_OK;
}

}  // namespace expi

using namespace expi;

extern "C" {

const char* expi_last_error(void) { return tl_error.c_str(); }

int expi_op_create_stencil(expi_op** op, int dim, const int64_t* n, const double* h, int bc,
                           int coef_kind, double c0, double c1, const double* tab_x,
                           const double* tab_y, const double* tab_z, const double* field) {
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    *op = nullptr;
    if (dim != 2 && dim != 3) return fail(EXPI_EINVAL, "dim must be 2 or 3");
    if (!n || !h) return fail(EXPI_EINVAL, "n and h must be non-NULL");
    int64_t total = 1;
    for (int d = 0; d < dim; ++d) {
        if (n[d] < 1) return fail(EXPI_EINVAL, "grid sizes must be >= 1");
        if (!(h[d] > 0) || !std::isfinite(h[d])) return fail(EXPI_EINVAL, "grid spacings must be finite and > 0");
        total *= n[d];
        // marched indices run one plane past the grid, so stay well inside int32
        if (total >= ((int64_t)1 << 30)) return fail(EXPI_EINVAL, "grid has 2^30 points or more");
    }
    if (bc != EXPI_DIRICHLET0 && bc != EXPI_NEUMANN0 && bc != EXPI_INTERIOR_ONLY)
        return fail(EXPI_EINVAL, "unknown boundary condition");
    if (!std::isfinite(c0) || !std::isfinite(c1)) return fail(EXPI_EINVAL, "c0, c1 must be finite");
    if (coef_kind == EXPI_COEF_SEPARABLE) {
        if (!tab_x || !tab_y || (dim == 3 && !tab_z))
            return fail(EXPI_EINVAL, "separable coefficient needs tab_x, tab_y (and tab_z in 3D)");
    } else if (coef_kind == EXPI_COEF_FIELD) {
        if (!field) return fail(EXPI_EINVAL, "field coefficient needs a field pointer");
    } else if (coef_kind != EXPI_COEF_CONST && coef_kind != EXPI_COEF_DLAP) {
        return fail(EXPI_EINVAL, "unknown coefficient kind");
    }
    Op* o = new Op();
    o->kind = 0;
    o->dim = dim;
    for (int d = 0; d < 3; ++d) {
        o->n[d] = d < dim ? (int)n[d] : 1;
        o->h[d] = d < dim ? h[d] : 1.0;
    }
    o->bc = bc;
    o->coef = coef_kind;
    o->c0 = c0;
    o->c1 = (coef_kind == EXPI_COEF_SEPARABLE) ? c1 : 0.0;
    o->tx = tab_x;
    o->ty = tab_y;
    o->tz = tab_z;
    o->field = field;
    o->nrows = o->nnz = 0;
    o->rowptr = o->colind = nullptr;
    o->val = nullptr;
    o->size = total;
    o->tiles = default_tiles(*o);
    *op = reinterpret_cast<expi_op*>(o);
    return EXPI_OK;
}

int expi_op_set_boundary_data(expi_op* op, int kind, int mode) {
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    if (kind < EXPI_BDATA_NONE || kind > EXPI_BDATA_SINPIZ_EXPMXY) return fail(EXPI_EINVAL, "unknown boundary data");
    if (mode != EXPI_BDATA_IN_KERNEL && mode != EXPI_BDATA_SEPARATE)
        return fail(EXPI_EINVAL, "mode must be EXPI_BDATA_IN_KERNEL or EXPI_BDATA_SEPARATE");
    if (kind != EXPI_BDATA_NONE) {
        if (o.kind != 0 || o.dim != 3) return fail(EXPI_EINVAL, "boundary data need a 3D stencil");
        if (o.bc != EXPI_DIRICHLET0) return fail(EXPI_EINVAL, "boundary data need EXPI_DIRICHLET0");
        if (o.coef == EXPI_COEF_DLAP) return fail(EXPI_EINVAL, "boundary data are not defined for EXPI_COEF_DLAP");
    }
    std::lock_guard<std::mutex> lock(o.mu);
    o.bdata = kind;
    o.bdata_mode = mode;
    return EXPI_OK;
}

int expi_op_create_csr(expi_op** op, int64_t n, int64_t nnz, const int32_t* rowptr,
                       const int32_t* colind, const double* val) {
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    *op = nullptr;
    if (n < 1 || n >= ((int64_t)1 << 31) - 1) return fail(EXPI_EINVAL, "n must be in [1, 2^31-2]");
    if (nnz < 0 || nnz >= ((int64_t)1 << 31)) return fail(EXPI_EINVAL, "nnz must be in [0, 2^31)");
    if (!rowptr || (nnz > 0 && (!colind || !val))) return fail(EXPI_EINVAL, "CSR arrays must be non-NULL");
    Op* o = new Op();
    o->kind = 1;
    o->dim = 0;
    for (int d = 0; d < 3; ++d) {
        o->n[d] = 1;
        o->h[d] = 1.0;
    }
    o->bc = 0;
    o->coef = 0;
    o->c0 = o->c1 = 0;
    o->tx = o->ty = o->tz = o->field = nullptr;
    o->nrows = n;
    o->nnz = nnz;
    o->rowptr = rowptr;
    o->colind = colind;
    o->val = val;
    o->size = n;
    o->tiles = default_tiles(*o);
    *op = reinterpret_cast<expi_op*>(o);
    return EXPI_OK;
}

int expi_op_create_csr_complex(expi_op** op, int64_t n, int64_t nnz, const int32_t* rowptr,
                               const int32_t* colind, const double* val) {
    int rc = expi_op_create_csr(op, n, nnz, rowptr, colind, val);
    if (rc) return rc;
    Op* o = reinterpret_cast<Op*>(*op);
    o->kind = 2;
    o->tiles = default_tiles(*o);
    return EXPI_OK;
}

int expi_op_destroy(expi_op* op) {
    delete reinterpret_cast<Op*>(op);
    return EXPI_OK;
}

int64_t expi_op_size(const expi_op* op) {
    return op ? reinterpret_cast<const Op*>(op)->size : -1;
}

int expi_op_set_tiles(expi_op* op, int vec, int waves, int march) {
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    Tiles t;
    t.vec = vec;
    t.waves = waves;
    t.march = march;
    if (!tiles_valid(o, t)) return fail(EXPI_EINVAL, "tile setting out of range for this operator");
    std::lock_guard<std::mutex> lock(o.mu);
    o.tiles = t;
    o.tiles_set = true;
    return EXPI_OK;
}

int expi_op_set_pairs(expi_op* op, int use) {
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    if (use != 0 && use != 1 && !(pair2d_supported(o, 0) && pair2d_rows_valid(use)))
        return fail(EXPI_EINVAL, "use must be 0 or 1 (or, on a 2D operator with pair sweeps, a row count "
                                 "4..64, a multiple of 4)");
    std::lock_guard<std::mutex> lock(o.mu);
    o.use_pairs = use;
    return EXPI_OK;
}

int expi_op_get_pairs(const expi_op* op, int* use) {
    if (!op || !use) return fail(EXPI_EINVAL, "op and use must be non-NULL");
    *use = reinterpret_cast<const Op*>(op)->use_pairs;
    return EXPI_OK;
}

int expi_op_get_tiles(const expi_op* op, int* vec, int* waves, int* march) {
    if (!op || !vec || !waves || !march) return fail(EXPI_EINVAL, "NULL argument");
    const Op& o = *reinterpret_cast<const Op*>(op);
    *vec = o.tiles.vec;
    *waves = o.tiles.waves;
    *march = o.tiles.march;
    return EXPI_OK;
}

int expi_op_autotune(expi_op* op, int dtype, int reps, void* ws, size_t ws_bytes, void* stream,
                     int* cand, float* us, int max_cand, int* n_cand) {
    if (!op || !ws || !n_cand) return fail(EXPI_EINVAL, "op, ws, n_cand must be non-NULL");
    if (dtype != EXPI_F64 && dtype != EXPI_F32) return fail(EXPI_EINVAL, "dtype must be EXPI_F64 or EXPI_F32");
    if (reps < 1 || reps > 1000) return fail(EXPI_EINVAL, "reps must be in [1, 1000]");
    if (((uintptr_t)ws & 255) != 0) return fail(EXPI_EWORKSPACE, "workspace must be 256-byte aligned");
    Op& o = *reinterpret_cast<Op*>(op);
    const WsLayout L = layout(o, dtype);
    if (ws_bytes < L.total) return fail(EXPI_EWORKSPACE, "workspace too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int tw = dtype == EXPI_F32 ? 1 : 0;
    char* w = static_cast<char*>(ws);
    // candidate tile settings
    std::vector<Tiles> C;
    if (o.kind == 2) {
        for (int v : {1, 2, 4, 8, 16})
            for (int wv : {1, 2, 4, 8}) C.push_back(Tiles{v, wv, 1});
    } else if (o.kind != 0) {
        for (int v : {4, 8, 16})
            for (int wv : {1, 2, 4, 8}) C.push_back(Tiles{v, wv, 1});
    } else {
        const int marches3[] = {8, 16, 32, 64};
        const int marches2[] = {4, 8, 16, 32};
        for (int v : {2, 1})
            for (int wv : {1, 2, 4, 8})
                for (int q = 0; q < 4; ++q) C.push_back(Tiles{v, wv, o.dim == 3 ? marches3[q] : marches2[q]});
    }
    // deterministic data in w0 and p; w1 is written by the sweep
    if (o.kind == 2 && tw != 0) return fail(EXPI_EINVAL, "complex operators run in FP64 only");
    const int64_t nfill = o.size * (o.kind == 2 ? 2 : 1);
    HIP_TRY(launch_fill(w + L.w0, nfill, tw, 1.0, s));
    HIP_TRY(launch_fill(w + L.p, nfill, tw, 0.5, s));
    hipEvent_t e0, e1;   // timing only (no system-scope fence)
    HIP_TRY(hipEventCreateWithFlags(&e0, hipEventDisableSystemFence));
    HIP_TRY(hipEventCreateWithFlags(&e1, hipEventDisableSystemFence));
    SweepArgs a{};
    a.x = w + L.w0;
    a.out = w + L.w1;
    a.p = w + L.p;
    a.st = reinterpret_cast<NewtonState*>(w + L.state);
    a.partials = reinterpret_cast<double*>(w + L.partials);
    a.alpha = 1e-6;
    a.beta = -0.5;
    a.d1 = 1e-3;
    a.tol = 1e-300;   // never met: every timed product does its work
    a.j = 1;
    a.guard = 0;
    const Tiles keep = o.tiles;
    const bool keep_set = o.tiles_set;
    o.tiles_set = true;
    Tiles best = keep;
    float best_us = 1e30f;
    int nc = 0;
    hipError_t err = hipSuccess;
    for (const Tiles& t : C) {
        if (!tiles_valid(o, t)) continue;
        o.tiles = t;
        err = launch_sweep(o, EPI_NEWTON, tw, tw, a, s);   // warm up
        if (err == hipSuccess) err = hipEventRecord(e0, s);
        for (int r = 0; r < reps && err == hipSuccess; ++r) err = launch_sweep(o, EPI_NEWTON, tw, tw, a, s);
        if (err == hipSuccess) err = hipEventRecord(e1, s);
        if (err == hipSuccess) err = hipEventSynchronize(e1);
        float ms = 0.f;
        if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
        if (err != hipSuccess) break;
        const float per = 1e3f * ms / reps;
        if (nc < max_cand && cand && us) {
            cand[3 * nc] = t.vec;
            cand[3 * nc + 1] = t.waves;
            cand[3 * nc + 2] = t.march;
            us[nc] = per;
        }
        ++nc;
        if (per < best_us) {
            best_us = per;
            best = t;
        }
    }
    // the dominant kernel's form: where a pair sweep can run, it is timed
    // against two single products at the best tiles (the same data, every
    // product doing full work) and kept if it takes less per product.  It is
    // listed as the candidate (0, 0, 2), its time per launch (two products).
    // A 2D pair sweep is timed at several tile heights (candidates
    // (0, rows, 2)) and kept with the fastest: use_pairs then holds its rows.
    int use_pairs = o.use_pairs;
    if (err == hipSuccess && pair_any_supported(o, tw) && best_us < 1e30f) {
        PairArgs b{};
        b.x = w + L.w0;
        b.out = w + L.w1;
        b.p = w + L.p;
        b.partials = reinterpret_cast<double*>(w + L.partials);
        b.st = reinterpret_cast<NewtonState*>(w + L.state);
        b.alpha = 1e-6;
        b.beta1 = -0.5;
        b.beta2 = -0.5;
        b.d1 = 1e-3;
        b.d2 = 1e-3;
        b.tol = 1e-300;
        b.j = 1;
        b.guard = 0;
        std::vector<int> heights{0};
        if (o.dim == 2) {
            heights.clear();
            for (int r = 4; r <= 64; r *= 2)
                if (r <= 16 || r / 2 < o.n[1]) heights.push_back(r);
        }
        // microseconds per launch (after one to warm up), 1e30 if it failed
        auto time_us = [&](const std::function<hipError_t()>& launch) -> float {
            err = launch();
            if (err == hipSuccess) err = hipEventRecord(e0, s);
            for (int r = 0; r < reps && err == hipSuccess; ++r) err = launch();
            if (err == hipSuccess) err = hipEventRecord(e1, s);
            if (err == hipSuccess) err = hipEventSynchronize(e1);
            float ms = 0.f;
            if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
            return err == hipSuccess ? 1e3f * ms / reps : 1e30f;
        };
        float best_pair = 1e30f;
        int best_rows = 1;
        for (int rows : heights) {
            const float per = time_us([&] { return launch_pair_op(o, tw, b, s, nullptr, false, PAIR_NEWTON, rows); });
            if (err != hipSuccess) break;
            if (nc < max_cand && cand && us) {
                cand[3 * nc] = 0;
                cand[3 * nc + 1] = rows;
                cand[3 * nc + 2] = 2;
                us[nc] = per;
            }
            ++nc;
            if (per < best_pair) {
                best_pair = per;
                best_rows = rows ? rows : 1;
            }
        }
        // single products only if nothing that the setting also turns off
        // takes less: the longest chain, or the loop in one workgroup
        float passes = 0.5f * best_pair;
        if (err == hipSuccess && chain2d_supported(o, tw)) {
            // |alpha A| <= 1, so that a loop of many products stays finite
            double norm = 0.0;
            for (int q = 0; q < 2; ++q) norm += 4.0 * std::fabs(o.c0) / (o.h[q] * o.h[q]);
            const double alpha = norm > 0.0 ? 1.0 / norm : 0.0;
            const int m = 32;
            if (resident2d_supported(o, tw, m)) {
                ResidentArgs r{};
                r.x = static_cast<const double*>(b.x);
                r.p = static_cast<double*>(b.p);
                r.st = r.mirror = b.st;
                r.tol = 1e-300;
                r.m_max = m;
                for (int q = 0; q <= m; ++q) r.d[q] = 1e-3;
                for (int q = 0; q < m; ++q) r.beta[q] = -0.5;
                passes = std::min(passes, time_us([&] { return launch_resident2d(o, r, alpha, s); }) / m);
            } else {
                const int n = chain2d_length(o, 6) ? 6 : 4;
                ChainArgs c{};
                c.x = b.x;
                c.out = b.out;
                c.p = b.p;
                c.partials = b.partials;
                c.st = b.st;
                c.alpha = alpha;
                for (int q = 0; q < n; ++q) {
                    c.beta[q] = -0.5;
                    c.d[q] = 1e-3;
                }
                int np = 0;
                const size_t room = partials_bytes(o);
                passes = std::min(passes, time_us([&] {
                           return launch_chain2d(o, tw, n, c, device_cus(), room, &np, s);
                       }) / n);
            }
        }
        if (err == hipSuccess) use_pairs = (passes < best_us) ? best_rows : 0;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    {
        std::lock_guard<std::mutex> lock(o.mu);
        o.tiles = (err == hipSuccess) ? best : keep;
        o.tiles_set = (err == hipSuccess) || keep_set;
        if (err == hipSuccess) o.use_pairs = use_pairs;
    }
    *n_cand = nc;
    if (err != hipSuccess) {
        set_error(std::string("autotune: ") + hipGetErrorString(err));
        return EXPI_EHIP;
    }
    return EXPI_OK;
}

size_t expi_workspace_bytes(const expi_op* op, int dtype) {
    if (!op || (dtype != EXPI_F64 && dtype != EXPI_F32)) return 0;
    return layout(*reinterpret_cast<const Op*>(op), dtype).total;
}

int expi_op_interval(expi_op* op, double* a, double* b, void* ws, size_t ws_bytes, void* stream) {
    if (!op || !a || !b) return fail(EXPI_EINVAL, "op, a, b must be non-NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    {
        std::lock_guard<std::mutex> lock(o.mu);
        if (o.have_interval) {
            *a = o.ia;
            *b = o.ib;
            return EXPI_OK;
        }
    }
    if (!ws) return fail(EXPI_EWORKSPACE, "workspace is NULL");
    if (((uintptr_t)ws & 255) != 0) return fail(EXPI_EWORKSPACE, "workspace must be 256-byte aligned");
    const WsLayout L = layout(o, EXPI_F64);
    if (ws_bytes < L.partials + partials_bytes(o)) return fail(EXPI_EWORKSPACE, "workspace too small");
    return op_interval(o, a, b, static_cast<char*>(ws), static_cast<hipStream_t>(stream));
}

int apply_op(const expi_op* op, double alpha, double beta, const void* x, void* y, int dtype,
             void* stream) {
    if (!op || !x || !y) return fail(EXPI_EINVAL, "op, x, y must be non-NULL");
    if (dtype != EXPI_F64 && dtype != EXPI_F32) return fail(EXPI_EINVAL, "dtype must be EXPI_F64 or EXPI_F32");
    if (!std::isfinite(alpha) || !std::isfinite(beta)) return fail(EXPI_EINVAL, "alpha, beta must be finite");
    const Op& o = *reinterpret_cast<const Op*>(op);
    if (o.kind == 2 && dtype != EXPI_F64) return fail(EXPI_EINVAL, "complex operators run in FP64 only");
    const size_t bytes = (size_t)o.size * (dtype == EXPI_F32 ? 4 : 8) * (o.kind == 2 ? 2 : 1);
    if (overlap(x, bytes, y, bytes)) return fail(EXPI_EALIAS, "y overlaps x");
    SweepArgs a{};
    a.x = x;
    a.out = y;
    a.alpha = alpha;
    a.beta = beta;
    a.bdata = o.bdata;
    const int t = dtype == EXPI_F32 ? 1 : 0;
    HIP_TRY(launch_sweep(o, EPI_APPLY, t, t, a, static_cast<hipStream_t>(stream)));
    return EXPI_OK;
}

int phi_action(expi_op* op, int k, double tau, const double* v, double* y, double tol, int dtype,
               const expi_params* params, void* ws, size_t ws_bytes, expi_stats* st, void* stream) {
    if (st) std::memset(st, 0, sizeof(*st));
    int rc = validate_call(op, tau, tol, dtype, ws, ws_bytes);
    if (rc) return rc;
    if (k < 0 || k > 20) return fail(EXPI_EINVAL, "k must be in [0, 20]");
    if (!v || !y) return fail(EXPI_EINVAL, "v, y must be non-NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    if (o.kind == 2) return fail(EXPI_EINVAL, "complex operator: use expi_skew_phi_action");
    const size_t bytes = (size_t)o.size * 8;
    if (overlap(v, bytes, y, bytes)) return fail(EXPI_EALIAS, "y overlaps v");
    if (overlap(ws, ws_bytes, v, bytes) || overlap(ws, ws_bytes, y, bytes))
        return fail(EXPI_EALIAS, "workspace overlaps v or y");
    Params P;
    rc = read_params(params, &P);
    if (rc) return rc;
    return run_phi(o, k, tau, v, y, tol, dtype, P, static_cast<char*>(ws), st,
                   static_cast<hipStream_t>(stream));
}

int expeuler_step(expi_op* op, int nonlin, double tau, double* u, double tol, int dtype,
                  const expi_params* params, void* ws, size_t ws_bytes, expi_stats* st,
                  void* stream) {
    if (st) std::memset(st, 0, sizeof(*st));
    int rc = validate_call(op, tau, tol, dtype, ws, ws_bytes);
    if (rc) return rc;
    if (nonlin < EXPI_G_CUBIC || nonlin > EXPI_G_COMBUSTION_FAST)
        return fail(EXPI_EINVAL, "nonlin must be EXPI_G_CUBIC, EXPI_G_COMBUSTION or EXPI_G_COMBUSTION_FAST");
    if (!u) return fail(EXPI_EINVAL, "u must be non-NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    if (o.kind == 2) return fail(EXPI_EINVAL, "complex operators have no exponential Euler step here");
    if (overlap(ws, ws_bytes, u, (size_t)o.size * 8)) return fail(EXPI_EALIAS, "workspace overlaps u");
    Params P;
    rc = read_params(params, &P);
    if (rc) return rc;
    return run_expeuler(o, nonlin, tau, u, tol, dtype, P, static_cast<char*>(ws), st,
                        static_cast<hipStream_t>(stream));
}

size_t expi_exprk2_workspace_bytes(const expi_op* op, int dtype) {
    if (!op || (dtype != EXPI_F64 && dtype != EXPI_F32)) return 0;
    return exprk2_bytes(*reinterpret_cast<const Op*>(op), dtype);
}

int exprk2_step(expi_op* op, int nonlin, double tau, double* u, double tol, int dtype,
                const expi_params* params, void* ws, size_t ws_bytes, expi_stats* st, void* stream) {
    if (st) std::memset(st, 0, sizeof(*st));
    int rc = validate_call(op, tau, tol, dtype, ws, ws_bytes);
    if (rc) return rc;
    if (nonlin < EXPI_G_CUBIC || nonlin > EXPI_G_COMBUSTION_FAST)
        return fail(EXPI_EINVAL, "nonlin must be EXPI_G_CUBIC, EXPI_G_COMBUSTION or EXPI_G_COMBUSTION_FAST");
    if (!u) return fail(EXPI_EINVAL, "u must be non-NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    if (o.kind == 2) return fail(EXPI_EINVAL, "complex operators have no Runge-Kutta step here");
    const size_t need = exprk2_bytes(o, dtype);
    if (ws_bytes < need)
        return fail(EXPI_EWORKSPACE, "workspace too small: need " + std::to_string(need) + " bytes");
    if (overlap(ws, ws_bytes, u, (size_t)o.size * 8)) return fail(EXPI_EALIAS, "workspace overlaps u");
    Params P;
    rc = read_params(params, &P);
    if (rc) return rc;
    return run_exprk2(o, nonlin, tau, u, tol, dtype, P, static_cast<char*>(ws), st,
                      static_cast<hipStream_t>(stream));
}

int expi_skew_phi_action(expi_op* op, int k, double tau, const double* v, double* y, double tol,
                         const expi_params* params, void* ws, size_t ws_bytes, expi_stats* st,
                         void* stream) {
    if (st) std::memset(st, 0, sizeof(*st));
    if (op && reinterpret_cast<Op*>(op)->kind != 2)
        return fail(EXPI_EINVAL, "expi_skew_phi_action needs a complex CSR operator");
    int rc = validate_call(op, tau, tol, EXPI_F64, ws, ws_bytes);
    if (rc) return rc;
    if (k != 0 && k != 1) return fail(EXPI_EINVAL, "k must be 0 or 1");
    if (!v || !y) return fail(EXPI_EINVAL, "v, y must be non-NULL");
    Op& o = *reinterpret_cast<Op*>(op);
    const size_t bytes = (size_t)o.size * 16;
    if (overlap(v, bytes, y, bytes)) return fail(EXPI_EALIAS, "y overlaps v");
    if (overlap(ws, ws_bytes, v, bytes) || overlap(ws, ws_bytes, y, bytes))
        return fail(EXPI_EALIAS, "workspace overlaps v or y");
    Params P;
    rc = read_params(params, &P);
    if (rc) return rc;
    if (P.selector) return fail(EXPI_EINVAL, "no step selector for complex operators");
    return run_skew(o, k, tau, v, y, tol, P, static_cast<char*>(ws), st, static_cast<hipStream_t>(stream));
}

int expi_divided_differences_skew(int k, double delta, double c, double gamma, int count, double* re,
                                  double* im) {
    if (!re || !im || count < 1 || count > kMaxLeja) return fail(EXPI_EINVAL, "count must be in [1, 256]");
    if (k < 0 || k > 20) return fail(EXPI_EINVAL, "k must be in [0, 20]");
    if (!std::isfinite(delta) || !std::isfinite(c) || !std::isfinite(gamma))
        return fail(EXPI_EINVAL, "delta, c, gamma must be finite");
    divided_differences_skew(k, delta, c, gamma, count, re, im);
    return EXPI_OK;
}

int expi_nonlinearity(int nonlin, int64_t n, const void* u, void* g, int dtype, void* stream) {
    if (nonlin < EXPI_G_CUBIC || nonlin > EXPI_G_COMBUSTION_FAST)
        return fail(EXPI_EINVAL, "nonlin must be EXPI_G_CUBIC, EXPI_G_COMBUSTION or EXPI_G_COMBUSTION_FAST");
    if (dtype != EXPI_F64 && dtype != EXPI_F32) return fail(EXPI_EINVAL, "dtype must be EXPI_F64 or EXPI_F32");
    if (n < 0) return fail(EXPI_EINVAL, "n must be >= 0");
    if (n == 0) return EXPI_OK;
    if (!u || !g) return fail(EXPI_EINVAL, "u, g must be non-NULL");
    const size_t bytes = (size_t)n * (dtype == EXPI_F32 ? 4 : 8);
    if (u != g && overlap(u, bytes, g, bytes)) return fail(EXPI_EALIAS, "g overlaps u (other than in place)");
    if ((((uintptr_t)u | (uintptr_t)g) & 15) != 0)
        return fail(EXPI_EINVAL, "u and g must be 16-byte aligned");
    HIP_TRY(launch_nonlin(nonlin, n, u, g, dtype, static_cast<hipStream_t>(stream)));
    return EXPI_OK;
}

int expi_noalloc_init(void) { return noalloc_init(); }

int phi_action_noalloc(expi_op* op, int k, double tau, const double* v, double* y, double tol,
                       int dtype, const expi_params* params, expi_stats* st, void* stream) {
    if (st) std::memset(st, 0, sizeof(*st));
    if (!op) return fail(EXPI_EINVAL, "op is NULL");
    if (dtype != EXPI_F64 && dtype != EXPI_F32) return fail(EXPI_EINVAL, "dtype must be EXPI_F64 or EXPI_F32");
    const size_t need = layout(*reinterpret_cast<const Op*>(op), dtype).total;
    if (need > EXPI_NOALLOC_SCRATCH_BYTES)
        return fail(EXPI_EWORKSPACE, "operator needs " + std::to_string(need) +
                                         " bytes of workspace, more than the allocation-free scratch array (" +
                                         std::to_string((size_t)EXPI_NOALLOC_SCRATCH_BYTES) + " bytes)");
    char* ws = nullptr;
    int rc = noalloc_scratch(&ws);
    if (rc) return rc;
    return phi_action(op, k, tau, v, y, tol, dtype, params, ws, EXPI_NOALLOC_SCRATCH_BYTES, st, stream);
}

int expi_leja_points(double* out, int count) {
    if (!out || count < 1 || count > kMaxLeja) return fail(EXPI_EINVAL, "count must be in [1, 256]");
    const double* xi = leja_points(count);
    std::memcpy(out, xi, sizeof(double) * count);
    return EXPI_OK;
}

int expi_divided_differences(int k, double delta, double c, double gamma, int count, double* out) {
    if (!out || count < 1 || count > kMaxLeja) return fail(EXPI_EINVAL, "count must be in [1, 256]");
    if (k < 0 || k > 20) return fail(EXPI_EINVAL, "k must be in [0, 20]");
    if (!std::isfinite(delta) || !std::isfinite(c) || !std::isfinite(gamma))
        return fail(EXPI_EINVAL, "delta, c, gamma must be finite");
    divided_differences(k, delta, c, gamma, count, out);
    return EXPI_OK;
}

}  // extern "C"
