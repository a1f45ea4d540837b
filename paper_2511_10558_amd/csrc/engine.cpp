// Host orchestration: slot pool, admission, the integration launches and harvest.
//
// Cells are admitted into slots and queued on the device; a launch of the
// persistent integration kernel lets every workgroup carry one queued cell
// after another to its end (integrate.hip).  The launch returns when the queue
// is empty, when its time is up (work of other streams gets in then), when a
// workgroup runs idle while cells still wait on the host for a slot, or, in the
// server, for a new or a completed request; the host then reads the counts,
// copies finished results out, and refills freed slots with pending cells.
#include "engine.hpp"

#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "../../include/astrobdf.h"

namespace abdf {

namespace {
size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// A named host range for rocprofv3 --marker-trace (one library call each way
// when no tool is attached).
struct TraceRange {
    explicit TraceRange(const char *name) { roctxRangePush(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};

#define HIP_TRY(expr)                                                           \
    do {                                                                        \
        hipError_t e__ = (expr);                                                \
        if (e__ != hipSuccess) {                                                \
            err = std::string(#expr ": ") + hipGetErrorString(e__);            \
            return ABDF_E_DEVICE;                                               \
        }                                                                       \
    } while (0)
}  // namespace

namespace {
std::atomic<bool> g_prof_on{false};
std::mutex g_prof_mu;
int64_t g_prof_launches[ABDF_PROF_KINDS];
double g_prof_ms[ABDF_PROF_KINDS];
}  // namespace

bool Profiler::on() { return g_prof_on.load(std::memory_order_relaxed); }
void Profiler::enable(bool v) { g_prof_on.store(v); }
void Profiler::add(int kind, double ms) {
    std::lock_guard<std::mutex> l(g_prof_mu);
    g_prof_launches[kind] += 1;
    g_prof_ms[kind] += ms;
}
void Profiler::read(int64_t *launches, double *ms, bool reset) {
    std::lock_guard<std::mutex> l(g_prof_mu);
    for (int i = 0; i < ABDF_PROF_KINDS; ++i) {
        launches[i] = g_prof_launches[i];
        ms[i] = g_prof_ms[i];
        if (reset) { g_prof_launches[i] = 0; g_prof_ms[i] = 0.0; }
    }
}

hipEvent_t Engine::timer_begin(hipStream_t st) {
    if (ext_ || !Profiler::on()) return nullptr;
    hipEvent_t e = nullptr;
    if (!event_pool_.empty()) {
        e = event_pool_.back();
        event_pool_.pop_back();
    } else if (hipEventCreate(&e) != hipSuccess) {
        return nullptr;
    }
    if (hipEventRecord(e, st) != hipSuccess) {
        event_pool_.push_back(e);
        return nullptr;
    }
    return e;
}

void Engine::timer_end(int kind, hipEvent_t a, hipStream_t st) {
    if (!a) return;
    hipEvent_t b = nullptr;
    if (!event_pool_.empty()) {
        b = event_pool_.back();
        event_pool_.pop_back();
    } else if (hipEventCreate(&b) != hipSuccess) {
        event_pool_.push_back(a);
        return;
    }
    (void)hipEventRecord(b, st);
    pending_.push_back({kind, a, b});
}

// Called after the stream has been synchronised.
void Engine::flush_timers() {
    for (auto &p : pending_) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) Profiler::add(p.kind, double(ms));
        event_pool_.push_back(p.a);
        event_pool_.push_back(p.b);
    }
    pending_.clear();
}

Engine::Engine(const HostNetwork &net, const DeviceNet &dn, int prec, int max_steps)
    : net_(net), dn_(dn), prec_(prec), max_steps_(max_steps) {}

Engine::~Engine() {
    for (auto &p : pending_) {
        event_pool_.push_back(p.a);
        event_pool_.push_back(p.b);
    }
    for (hipEvent_t e : event_pool_) (void)hipEventDestroy(e);
    if (ext_) return;   // nothing below was allocated
    if (cached_ && block_.ptr && block_.host)
        net_.keep_workspace(dn_.device, block_);
    else
        block_.free();
}

// Factor storage per slot: FP64-sized in both forms, since an FP32-LU cell can
// fall back to FP64 factors.
static size_t lu_bytes(const DeviceNet &dn, bool padded) {
    return size_t(dn.NP) * size_t(padded ? lu_leading_dim(dn.NP) : dn.NP) * sizeof(double);
}

size_t Engine::bytes_per_slot(const DeviceNet &dn, bool padded) {
    const size_t S = dn.S, R = dn.R, NP = dn.NP;
    return sizeof(SlotCtl) + 5 * sizeof(double) + R * sizeof(double) + kDRows * S * sizeof(double) +
           5 * S * sizeof(double) + size_t(std::max(dn.nnzJ, 1)) * sizeof(double) + lu_bytes(dn, padded) +
           dinv_bytes(int(NP), ABDF_PREC_FP64) +
           NP * sizeof(int32_t) + 4 * sizeof(int32_t) + sizeof(long long);
}

int Engine::set_options(const abdf_options &o, std::string &err, double *atol_host) {
    set_lu_reuse(o.lu_reuse);
    set_max_order(o.max_order);
    set_step_bounds(o.h0, o.h_max);
    method_ = o.method;
    s_.method = method_;
    s_.newton_maxiter = method_ == ABDF_METHOD_ESDIRK5 ? kRkNewtonMaxIter : kNewtonMaxIter;
    tvar_ = o.phi_tc != nullptr;
    for (int j = 0; j < 5; ++j) phi_exp_[j] = o.phi_exp[j];
    s_.tvar = tvar_;
    for (int j = 0; j < 5; ++j) s_.phi_exp[j] = phi_exp_[j];
    atol_sp_ = nullptr;
    if (o.atol_species) {
        if (dn_.S > kMaxSpecies) {
            err = "network too large";
            return ABDF_E_ARG;
        }
        double *h = atol_host;
        if (!h) {
            atol_store_.resize(size_t(dn_.S));
            h = atol_store_.data();
        }
        HIP_TRY(hipMemcpy(h, o.atol_species, size_t(dn_.S) * sizeof(double), hipMemcpyDeviceToHost));
        for (int i = 0; i < dn_.S; ++i)
            if (!(h[i] >= 0.0) || !std::isfinite(h[i])) {
                err = "atol_species entries must be finite and >= 0";
                return ABDF_E_ARG;
            }
        atol_sp_ = h;
    }
    return ABDF_OK;
}

namespace {
// The slot arrays of n slots in the order init lays them out (each part
// 256-byte aligned).
struct Layout {
    static constexpr int kParts = 20;
    size_t bytes[kParts];
    Layout(const DeviceNet &dn, size_t n, bool padded) {
        const size_t S = dn.S, R = dn.R, NP = dn.NP;
        const size_t lu_stride = lu_bytes(dn, padded), dinv_stride = dinv_bytes(int(NP), ABDF_PREC_FP64);
        const size_t b[kParts] = {
            n * sizeof(SlotCtl), n * 5 * sizeof(double), n * R * sizeof(double), n * kDRows * S * sizeof(double),
            n * S * sizeof(double), n * S * sizeof(double), n * S * sizeof(double), n * S * sizeof(double),
            n * S * sizeof(double), n * size_t(std::max(dn.nnzJ, 1)) * sizeof(double),
            n * lu_stride, n * dinv_stride, n * NP * sizeof(int32_t), n * sizeof(int32_t), n * sizeof(int32_t),
            n * sizeof(int32_t), sizeof(SlotQueue), n * sizeof(int32_t), n * sizeof(long long), S * sizeof(double)};
        for (int i = 0; i < kParts; ++i) bytes[i] = b[i];
    }
    size_t total() const {
        size_t t = 0;
        for (size_t b : bytes) t += align256(b);
        return t;
    }
};
}  // namespace

size_t Engine::workspace_bytes(const DeviceNet &dn, long long n, bool padded) {
    return Layout(dn, size_t(n), padded).total();
}

// Points the slot arrays into base (workspace_bytes(nslots) bytes) and sets
// the launch shapes.
int Engine::layout(int nslots, void *base, std::string &err) {
    const size_t n = size_t(nslots), S = dn_.S, NP = dn_.NP;
    const Layout lay(dn_, n, padded_);
    void *part[Layout::kParts];
    size_t off = 0;
    for (int i = 0; i < Layout::kParts; ++i) {
        part[i] = static_cast<char *>(base) + off;
        off += align256(lay.bytes[i]);
    }
    s_.nslots = nslots;
    s_.S = dn_.S;
    s_.R = dn_.R;
    s_.NP = dn_.NP;
    s_.prec = prec_;
    s_.max_steps = max_steps_;
    s_.ctl = static_cast<SlotCtl *>(part[0]);
    s_.phi = static_cast<double *>(part[1]);
    s_.k = static_cast<double *>(part[2]);
    s_.D = static_cast<double *>(part[3]);
    s_.xJ = static_cast<double *>(part[4]);
    s_.x = static_cast<double *>(part[5]);
    s_.d = static_cast<double *>(part[6]);
    s_.psi = static_cast<double *>(part[7]);
    s_.rb = static_cast<double *>(part[8]);
    s_.jval = static_cast<double *>(part[9]);
    s_.lu = part[10];
    s_.dinv = part[11];
    s_.lu_stride = lu_bytes(dn_, padded_);
    s_.lda = padded_ ? lu_leading_dim(int(NP)) : int(NP);
    s_.dinv_stride = dinv_bytes(int(NP), ABDF_PREC_FP64);
    s_.perm = static_cast<int32_t *>(part[12]);
    s_.fifo = static_cast<int32_t *>(part[13]);
    s_.held = static_cast<int32_t *>(part[14]);
    s_.fin = static_cast<int32_t *>(part[15]);
    s_.q = static_cast<SlotQueue *>(part[16]);
    d_admit_slots_ = static_cast<int32_t *>(part[17]);
    d_admit_cells_ = static_cast<long long *>(part[18]);
    s_.lu_reuse = lu_reuse_;
    s_.max_order = max_order_;
    s_.h0 = h0_;
    s_.h_max = h_max_;
    s_.method = method_;
    s_.newton_maxiter = method_ == ABDF_METHOD_ESDIRK5 ? kRkNewtonMaxIter : kNewtonMaxIter;
    s_.tvar = tvar_;
    for (int j = 0; j < 5; ++j) s_.phi_exp[j] = phi_exp_[j];
    s_.atol_sp = nullptr;
    if (atol_sp_) {
        HIP_TRY(hipMemcpy(part[19], atol_sp_, S * sizeof(double), hipMemcpyHostToDevice));
        s_.atol_sp = static_cast<const double *>(part[19]);
    }
    lds_admit_ = admit_lds(dn_);
    if (dn_.NP > 512 || lds_admit_ + kAdmitFixedLds > kMaxLds || integrate_lds(dn_, prec_, true) > kMaxLds) {
        err = "network too large for one workgroup's LDS";
        return ABDF_E_ARG;
    }
    int dev = 0, cus = 256;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
        cus = prop.multiProcessorCount;
    grid_max_ = cus * integrate_resident_per_cu(dn_, prec_, false);
    grid_fp64_max_ = cus * integrate_resident_per_cu(dn_, prec_, true);
    grid_reverse_max_ = cus * reverse_resident_per_cu(dn_);
    if (grid_max_ == 0 || grid_fp64_max_ == 0) {
        err = "network too large for one compute unit";
        return ABDF_E_ARG;
    }
    n_free_ = 0;
    for (int i = nslots - 1; i >= 0; --i) free_[n_free_++] = i;
    (void)n;
    return ABDF_OK;
}

int Engine::init(int nslots, std::string &err, bool cache_workspace) {
    const size_t n = size_t(nslots);
    const size_t total = workspace_bytes(dn_, nslots, padded_);
    cached_ = cache_workspace;
    // pinned: the queue's counts, cells to admit, slots to admit, finished slots
    // (copies to and from ordinary memory hold up other threads' calls)
    const size_t host_total = sizeof(SlotQueue) + n * (sizeof(long long) + 2 * sizeof(int32_t));
    if (cached_) block_ = net_.take_workspace(dn_.device, total, host_total);
    if (!block_.ptr) {
        hipError_t e = hipMalloc(&block_.ptr, total);
        if (e != hipSuccess) {
            block_.ptr = nullptr;
            err = "device workspace of " + std::to_string(total) + " bytes: " + hipGetErrorString(e);
            return ABDF_E_NOMEM;
        }
        block_.bytes = total;
        HIP_TRY(hipHostMalloc(&block_.host, host_total, hipHostMallocDefault));
        block_.host_bytes = host_total;
    }
    h_q_ = static_cast<SlotQueue *>(block_.host);
    h_admit_cells_ = reinterpret_cast<long long *>(h_q_ + 1);
    h_admit_slots_ = reinterpret_cast<int32_t *>(h_admit_cells_ + n);
    h_fin_ = h_admit_slots_ + n;
    free_store_.resize(n);
    free_ = free_store_.data();
    return layout(nslots, block_.ptr, err);
}

int Engine::init_external(int nslots, void *base, size_t bytes, const HostBuffers &hb, std::string &err) {
    ext_ = true;
    if (nslots < 1 || nslots > hb.max_slots || workspace_bytes(dn_, nslots, padded_) > bytes) {
        err = "slot count beyond the external workspace";
        return ABDF_E_ARG;
    }
    free_ = hb.free_list;
    h_q_ = hb.queue;
    h_fin_ = hb.fin;
    h_admit_slots_ = hb.admit_slots;
    h_admit_cells_ = hb.admit_cells;
    return layout(nslots, base, err);
}

int Engine::reset_counts(hipStream_t st, std::string &err) {
    HIP_TRY(launch_fill_i32(reinterpret_cast<int32_t *>(s_.q), 0, kQueueInts, st));
    held_seen_ = 0;
    n64_seen_ = 0;
    fp64_too_ = false;
    for (unsigned long long &t : ticks_seen_) t = 0;
    launch_ = 0;
    bound_ = 0;
    return ABDF_OK;
}

double Engine::newton_tolerance(const abdf_options &opt) {
    return opt.newton_tol > 0 ? opt.newton_tol
                              : std::max(10.0 * kURound / opt.rtol, std::min(0.03, std::sqrt(opt.rtol)));
}

int Engine::admit_cells(const AdmitArgs &a, hipStream_t st, std::string &err) {
    if (a.count <= 0) return ABDF_OK;
    TraceRange tr("abdf admit");
    hipEvent_t t0 = timer_begin(st);
    HIP_TRY(launch_admit(s_, dn_, a, lds_admit_, st));
    timer_end(ABDF_PROF_ADMIT, t0, st);
    bound_ += a.count;
    return ABDF_OK;
}

int Engine::admit(const BatchIO &io, const abdf_options &opt, long long &next, hipStream_t st, std::string &err) {
    const long long want = std::min<long long>(static_cast<long long>(n_free_), io.n_cells - next);
    if (want <= 0) return ABDF_OK;
    for (long long i = 0; i < want; ++i) {
        h_admit_slots_[i] = take_slot();
        h_admit_cells_[i] = next + i;
    }
    HIP_TRY(hipMemcpyAsync(d_admit_slots_, h_admit_slots_, want * sizeof(int32_t), hipMemcpyHostToDevice, st));
    HIP_TRY(hipMemcpyAsync(d_admit_cells_, h_admit_cells_, want * sizeof(long long), hipMemcpyHostToDevice, st));
    AdmitArgs a{};
    a.count = int(want);
    a.slots = d_admit_slots_;
    a.cells = d_admit_cells_;
    a.T = io.T;
    a.nH = io.nH;
    a.Av = io.Av;
    a.zeta = io.zeta;
    a.G0 = io.G0;
    a.x0 = io.x0;
    a.t_end = io.t_end;
    a.rtol = opt.rtol;
    a.atol = opt.atol;
    a.newton_tol = newton_tolerance(opt);
    a.tc = opt.phi_tc;
    // the admission buffers are rewritten only after the next poll's synchronisation
    next += want;
    return admit_cells(a, st, err);
}

// One launch of a persistent kernel over the occupied slots.
IntegrateArgs Engine::next_launch(bool stop_on_idle) {
    IntegrateArgs a{};
    a.held_limit = held_seen_;
    a.ticks = (unsigned long long)(kLaunchMs * 1e5);   // the device's constant clock: 100 MHz
    a.launch = ++launch_;
    if (stop_on_idle) a.flags |= kStopOnIdle;
    if (!ext_ && Profiler::on()) a.flags |= kProf;
    if (serve_) a.flags |= kServe;
    return a;
}

// A server's launch does not look at its call before this, so that requests in quick
// succession do not end one launch after another at its first attempt.
constexpr double kCallMs = 0.5;

int Engine::serve(const int32_t *call, int32_t *fin_host, hipStream_t st, std::string &err) {
    int rc = reset_counts(st, err);
    if (rc != ABDF_OK) return rc;
    SlotQueue q{};
    q.call = call;
    q.ticks_call = (unsigned long long)(kCallMs * 1e5);
    q.fin_host = fin_host;
    *h_q_ = q;
    HIP_TRY(hipMemcpyAsync(s_.q, h_q_, sizeof(SlotQueue), hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    serve_ = true;
    return ABDF_OK;
}

int Engine::integrate(bool stop_on_idle, hipStream_t st, std::string &err) {
    if (bound_ <= 0) return ABDF_OK;
    TraceRange tr("abdf integrate");
    // while cells of the one-wave FP32-LU kernel are on FP64 factors, its form that
    // holds those runs in every other launch (all cells advance in it, fewer at once)
    fp64_too_ = n64_seen_ > 0 && !fp64_too_;
    grid_ = std::min(bound_, fp64_too_ ? grid_fp64_max_ : grid_max_);
    HIP_TRY(launch_integrate(s_, dn_, next_launch(stop_on_idle), fp64_too_, grid_, st));
    return ABDF_OK;
}

int Engine::sync_counts(hipStream_t st, int &nfin, std::string &err) {
    TraceRange tr("abdf poll");
    HIP_TRY(hipMemcpyAsync(h_q_, s_.q, sizeof(SlotQueue), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    flush_timers();
    nfin = h_q_->nfin;
    held_seen_ = h_q_->held_tail;
    n64_seen_ = h_q_->n64;
    // a phase's time: the mean over the launch's workgroups
    static const int kind[kPhases] = {ABDF_PROF_CONTROL, ABDF_PROF_FACTOR,    ABDF_PROF_RHS,
                                      ABDF_PROF_NEWTON,  ABDF_PROF_ADJ_SOLVE, ABDF_PROF_ADJ_STEP};
    for (int p = 0; p < kPhases; ++p) {
        const unsigned long long d = h_q_->ticks[p] - ticks_seen_[p];
        ticks_seen_[p] = h_q_->ticks[p];
        if (d > 0 && grid_ > 0) Profiler::add(kind[p], double(d) * 1e-5 / grid_);
    }
    return ABDF_OK;
}

int Engine::harvest(HarvestArgs h, hipStream_t st, std::string &err) {
    const int nfin = h.count;
    if (nfin <= 0) return ABDF_OK;
    TraceRange tr("abdf harvest");
    HIP_TRY(hipMemcpyAsync(h_fin_, s_.fin, nfin * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    h.slots = s_.fin;
    hipEvent_t t0 = timer_begin(st);
    HIP_TRY(launch_harvest(s_, h, st));
    timer_end(ABDF_PROF_HARVEST, t0, st);
    HIP_TRY(hipStreamSynchronize(st));
    for (int i = 0; i < nfin; ++i) free_[n_free_++] = h_fin_[i];
    bound_ -= nfin;
    return ABDF_OK;
}

int Engine::solve(const BatchIO &io, const abdf_options &opt, hipStream_t st, std::string &err) {
    TraceRange tr("abdf solve");
    long long next = 0;
    {
        // the queue starts empty: an external workspace keeps the previous
        // call's contents, and an engine's earlier sweep leaves its counts
        int rc0 = reset_counts(st, err);
        if (rc0 != ABDF_OK) return rc0;
    }
    int rc = admit(io, opt, next, st, err);
    if (rc != ABDF_OK) return rc;
    while (bound_ > 0) {
        rc = integrate(next < io.n_cells, st, err);
        if (rc != ABDF_OK) return rc;
        int nfin = 0;
        rc = sync_counts(st, nfin, err);
        if (rc != ABDF_OK) return rc;
        HarvestArgs h{};
        h.count = nfin;
        h.x_out = io.x_out;
        h.status = io.status;
        h.stats = io.stats;
        rc = harvest(h, st, err);
        if (rc != ABDF_OK) return rc;
        rc = admit(io, opt, next, st, err);
        if (rc != ABDF_OK) return rc;
    }
    flush_timers();
    return ABDF_OK;
}

int Engine::reverse(const AdjIO &io, hipStream_t st, std::string &err) {
    TraceRange tr("abdf reverse sweep");
    {
        int rc0 = reset_counts(st, err);
        if (rc0 != ABDF_OK) return rc0;
    }
    const size_t lds_adj = adj_lds(dn_);
    if (lds_adj > kMaxLds || reverse_lds(dn_) > kMaxLds || grid_reverse_max_ == 0) {
        err = "network too large for one workgroup's LDS";
        return ABDF_E_ARG;
    }
    long long next = 0;
    auto admit_rev = [&]() -> int {
        const long long want = std::min<long long>(static_cast<long long>(n_free_), io.n_cells - next);
        if (want <= 0) return ABDF_OK;
        for (long long i = 0; i < want; ++i) {
            h_admit_slots_[i] = take_slot();
            h_admit_cells_[i] = next + i;
        }
        HIP_TRY(hipMemcpyAsync(d_admit_slots_, h_admit_slots_, want * sizeof(int32_t), hipMemcpyHostToDevice, st));
        HIP_TRY(hipMemcpyAsync(d_admit_cells_, h_admit_cells_, want * sizeof(long long), hipMemcpyHostToDevice, st));
        AdjArgs a{int(want), d_admit_slots_, d_admit_cells_, io.phi, io.dLdx, io.status};
        hipEvent_t t0 = timer_begin(st);
        HIP_TRY(launch_adj_admit(s_, dn_, a, lds_adj, st));
        timer_end(ABDF_PROF_ADMIT, t0, st);
        next += want;
        bound_ += int(want);
        return ABDF_OK;
    };
    int rc = admit_rev();
    if (rc != ABDF_OK) return rc;
    while (bound_ > 0) {
        grid_ = std::min(bound_, grid_reverse_max_);
        HIP_TRY(launch_reverse(s_, dn_, next_launch(next < io.n_cells), grid_, st));
        int nfin = 0;
        rc = sync_counts(st, nfin, err);
        if (rc != ABDF_OK) return rc;
        if (nfin > 0) {
            HIP_TRY(hipMemcpyAsync(h_fin_, s_.fin, nfin * sizeof(int32_t), hipMemcpyDeviceToHost, st));
            AdjHarvestArgs h{nfin, s_.fin, io.g_cell, io.dx0, io.dphi};
            hipEvent_t t0 = timer_begin(st);
            HIP_TRY(launch_adj_harvest(s_, dn_, h, st));
            timer_end(ABDF_PROF_HARVEST, t0, st);
            HIP_TRY(hipStreamSynchronize(st));
            for (int i = 0; i < nfin; ++i) free_[n_free_++] = h_fin_[i];
            bound_ -= nfin;
        }
        rc = admit_rev();
        if (rc != ABDF_OK) return rc;
    }
    flush_timers();
    return ABDF_OK;
}

}  // namespace abdf
