// libpmx C ABI: context, workspace plan, argument checks and the orchestration
// of the PM forward run and its reverse-time adjoint (see include/pm.h).
//
// Forward (kick-drift-kick with growth-factor coefficients, merged kicks):
//   ICs -> F(x_0) -> for n = 0..N: gather F(x_n),
//   p += (kick_b_{n-1} + kick_a_n) F_n   (kick_b_{-1} = kick_a_N = 0),
//   x += drift_n p (n < N), F(x_{n+1}) ...
// Adjoint (pmwd paper, Statement of Need: dual equations integrated backward in
// time with the forward states recovered by reverse time integration; the
// discrete transpose of the forward steps).  Cotangents xi (positions) and pi
// (momenta); at each x_m the force's transpose J_F^T[(kick_b_{m-1}+kick_a_m) pi]
// has three parts: (i) the gather's position derivative, (ii) a CIC scatter of
// the cotangent through the transposed spectral operator and (iii) the
// scatter's position derivative.  Walking back from x_{n+1}:
//   (ii)+(iii) at x_{n+1};  xi complete -> dL/ddrift_n = Sum xi.p_{n+1/2},
//   pi += drift_n xi, x_n = x_{n+1} - drift_n p_{n+1/2};  recompute F(x_n);
//   p_{n-1/2} = p_{n+1/2} - (kick_b_{n-1} + kick_a_n) F_n together with (i) at x_n
//   and Sum pi.F_n (= dL/dkick_a_n = dL/dkick_b_{n-1}).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <utility>
#include <string>
#include <vector>

#include "fft_plan.h"
#include "host_cosmo.h"
#include "kernels.h"
#include "pm.h"

using namespace pmx;

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kNParam = 4417;
constexpr int kExtraSlots = 16 + 2 * PM_MAX_CHECKPOINTS;

thread_local std::string g_err;

// Pinned host memory for the scalar results of the process's contexts.  Freeing it
// waits for the whole device and invalidates captures on other streams, so a block
// that pm_destroy gives back is kept for a later pm_init, up to kKept blocks and
// kKeptBytes; only what is beyond that is freed.  No kernel writes to a block that is
// given back: every call that has one do so waits for it.
class ResultBlocks {
  public:
    static constexpr int kKept = 32;
    static constexpr size_t kKeptBytes = 1u << 20;

    // a block of at least `need` bytes (sizes are powers of two, so that contexts of
    // one configuration find each other's), on any device; null when that fails
    void* take(size_t need, size_t* bytes) {
        *bytes = 4096;
        while (*bytes < need) *bytes *= 2;
        {
            std::lock_guard<std::mutex> lock(mu_);
            for (int i = 0; i < n_; ++i)
                if (kept_[i].bytes == *bytes) {
                    void* p = kept_[i].p;
                    kept_[i] = kept_[--n_];
                    total_ -= *bytes;
                    return p;
                }
        }
        void* p = nullptr;
        return hipHostMalloc(&p, *bytes, hipHostMallocMapped | hipHostMallocPortable) == hipSuccess
                   ? p
                   : nullptr;
    }
    void give(void* p, size_t bytes) {
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (n_ < kKept && total_ + bytes <= kKeptBytes) {
                kept_[n_++] = {p, bytes};
                total_ += bytes;
                return;
            }
        }
        (void)hipHostFree(p);
    }

  private:
    struct Block {
        void* p;
        size_t bytes;
    };
    std::mutex mu_;
    Block kept_[kKept];
    int n_ = 0;
    size_t total_ = 0;
};
ResultBlocks g_results;

bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

int check_config(const pm_config* c, std::string* why) {
    if (!c) { *why = "config is null"; return PM_EINVAL; }
    if (!is_pow2(c->ptcl_grid) || c->ptcl_grid < 8 || c->ptcl_grid > 1024) {
        *why = "ptcl_grid must be a power of two in [8, 1024]"; return PM_EINVAL;
    }
    if (!is_pow2(c->mesh) || c->mesh < 8 || c->mesh > 1024) {
        *why = "mesh must be a power of two in [8, 1024]"; return PM_EINVAL;
    }
    if (c->mesh % c->ptcl_grid != 0) { *why = "mesh must be a multiple of ptcl_grid"; return PM_EINVAL; }
    if (!(c->box > 0.0) || !std::isfinite(c->box)) { *why = "box must be positive"; return PM_EINVAL; }
    if (!(c->a_start > 0.0 && c->a_stop > c->a_start) || !std::isfinite(c->a_stop)) {
        *why = "need 0 < a_start < a_stop"; return PM_EINVAL;
    }
    if (c->n_steps < 1 || c->n_steps > 100000) { *why = "n_steps must be >= 1"; return PM_EINVAL; }
    if (c->checkpoint_every < 0) { *why = "checkpoint_every must be >= 0"; return PM_EINVAL; }
    if (c->checkpoint_every > 0 && (c->n_steps - 1) / c->checkpoint_every > PM_MAX_CHECKPOINTS) {
        *why = "too many checkpoints"; return PM_EINVAL;
    }
    if (c->filter != 0 && c->filter != 1) { *why = "filter must be 0 or 1"; return PM_EINVAL; }
    if ((c->flags & ~(uint64_t)(PM_F_TIMING | PM_F_2LPT)) != 0) {
        *why = "unknown flags"; return PM_EINVAL;
    }
    return PM_OK;
}

int check_cosmo(const pm_cosmology* c, std::string* why) {
    if (!c) { *why = "cosmology is null"; return PM_EINVAL; }
    if (!(c->omega_m > 0.0 && c->omega_m <= 1.0)) { *why = "omega_m must be in (0, 1]"; return PM_EINVAL; }
    if (!(c->omega_b >= 0.0 && c->omega_b < c->omega_m)) { *why = "need 0 <= omega_b < omega_m"; return PM_EINVAL; }
    if (!(c->h > 0.0) || !(c->sigma8 > 0.0) || !std::isfinite(c->n_s)) {
        *why = "h and sigma8 must be positive, n_s finite"; return PM_EINVAL;
    }
    return PM_OK;
}

Cosmo to_cosmo(const pm_cosmology* c) {
    return Cosmo{c->omega_m, c->omega_b, c->h, c->sigma8, c->n_s, c->T_cmb > 0 ? c->T_cmb : 2.7255};
}

// Fixed-point units of the particle state: positions in box / 2^32 (periodic wrap
// is integer overflow); momenta in cell * 2^-22, doubled while the int32 range
// 2^31 units falls short of kMomBound, so that |p| <= kMomBound Mpc/h per unit
// time (10^4 km/s of peculiar velocity at a = 1, far above cluster velocities)
// is representable at any cell size.
constexpr double kMomBound = 100.0;

void state_units(const pm_config& c, double* pos, double* mom) {
    *pos = c.box / 4294967296.0;
    double u = c.box / c.mesh * std::ldexp(1.0, -22);
    while (u * 2147483648.0 < kMomBound) u *= 2.0;
    *mom = u;
}

int n_checkpoints(const pm_config& c) {
    return c.checkpoint_every > 0 ? (c.n_steps - 1) / c.checkpoint_every : 0;
}

// Workspace plan: byte offsets of every buffer, 256-byte aligned.
struct Plan {
    size_t total = 0;
    size_t cplx, disp, mom, xi, pi, disp2, mom2, xi2, pi2, id, id2, fin_disp, fin_mom, tmpv,
        noise, ckpt;
    size_t counts, offsets, keys, ranks, ord, scan_tmp;
    size_t radial_f, radial_ic, radial_ic_dom, radial_lpt, losstab, tw, tw_stages, partials, sums, maxbits,
        pkbins;
    size_t theta, gtheta, fbar, mlp_scratch, ovf;
    size_t step_parts, parts_a, parts_b, pmax;
    long cplx_elems, P, nkeys, ntab_f, ntab_p, tab_stride;
    int cs, cs_p, tile, nt, nckpt, ntables;

    size_t take(size_t bytes) {
        size_t off = total;
        total += (bytes + 255) / 256 * 256;
        return off;
    }
    explicit Plan(const pm_config& c) {
        const int ng = c.mesh, np = c.ptcl_grid;
        cs = complex_row_stride(ng);
        cs_p = complex_row_stride(np);
        cplx_elems = (long)ng * ng * cs;
        P = (long)np * np * np;
        tile = choose_tile(ng);
        nt = ng / tile;
        nkeys = (long)nt * nt * nt * 8;
        ntab_f = 3L * (ng / 2) * (ng / 2) + 1;
        ntab_p = 3L * (np / 2) * (np / 2) + 1;
        // learned runs: as many force evaluations' filter tables are formed in one
        // launch as fit in 2^17 entries, and their cotangents go through the network
        // in one.  A table of a 128^3 mesh (12289 entries, 193 work-groups) takes
        // 16 us alone and nine of them 34 us, the backward pass 25 us for one and
        // 69 us for eight; from 256^3 on a table fills the GPU by itself.  A batch and
        // its cotangents stay within 1 MB; a single table may be larger (with its
        // cotangent 1.6 MB at 512^3, 6.3 MB at 1024^3).
        tab_stride = (ntab_f + 63) / 64 * 64;
        ntables = c.filter ? (int)std::min<long>({std::max<long>(1, (1L << 17) / tab_stride),
                                                  (long)c.n_steps + 1, kMaxTables})
                           : 1;
        nckpt = n_checkpoints(c);
        const size_t vec = (size_t)P * 3 * sizeof(float);
        // a fifth buffer where the plane kernels read G while they write the
        // second and third force mesh
        cplx = take((ng <= kMaxPlane ? 5 : 4) * (size_t)cplx_elems * sizeof(float2));
        disp = take(vec);
        mom = take(vec);
        xi = take(vec);
        pi = take(vec);
        disp2 = take(vec);
        mom2 = take(vec);
        xi2 = take(vec);
        pi2 = take(vec);
        id = take((size_t)P * sizeof(uint32_t));
        id2 = take((size_t)P * sizeof(uint32_t));
        fin_disp = take(vec);
        fin_mom = take(vec);
        tmpv = take(vec);
        noise = take((size_t)P * sizeof(float));
        ckpt = take((size_t)nckpt * 2 * vec);
        counts = take((nkeys + 1) * sizeof(uint32_t));
        offsets = take((nkeys + 1) * sizeof(uint32_t));
        keys = take((size_t)P * sizeof(uint32_t));
        ranks = take((size_t)P * sizeof(uint32_t));
        ord = take((size_t)P * sizeof(uint32_t));
        scan_tmp = take(scan_tmp_elems(nkeys) * sizeof(uint32_t));
        radial_f = take((size_t)ntables * tab_stride * sizeof(float));
        radial_ic = take(ntab_p * sizeof(float));
        radial_ic_dom = take(ntab_p * sizeof(float));
        radial_lpt = take(ntab_p * sizeof(float));
        losstab = take(std::max(ntab_f * sizeof(float),
                                ng * (sizeof(double) + sizeof(float)) + sizeof(int)));
        tw = take((size_t)ng * sizeof(float2));
        tw_stages = take(kStageTableSize * sizeof(float2));
        // FP64 block partials: sets of at most 4096 grid-stride blocks (nine of
        // 1024 at the adjoint's end, checks, losses), and one set for each of the
        // two gathers of a reverse step (one value per tile, or per block of the
        // un-drift), whose sums and maximum |pi| one launch forms
        step_parts = std::max((size_t)gather_partials(np, ng), (size_t)4096);
        partials = take((3 * (size_t)((P + 255) / 256) + 3 * 4096) * sizeof(double));
        parts_a = take(step_parts * sizeof(double));
        parts_b = take(step_parts * sizeof(double));
        pmax = take(step_parts * sizeof(float));
        sums = take((2 * (size_t)c.n_steps + 2 + kExtraSlots) * sizeof(double));
        maxbits = take(kExtraSlots * sizeof(unsigned));
        pkbins = take(3 * (size_t)ng * sizeof(double));
        theta = take(kNParam * sizeof(float));
        gtheta = take(kNParam * sizeof(float));
        fbar = take(c.filter ? (size_t)ntables * tab_stride * sizeof(float) : 0);
        mlp_scratch = take(c.filter ? mlp_backward_scratch(ng) * sizeof(float) : 0);
        ovf = take(sizeof(unsigned));
    }
};

}  // namespace

namespace pmx {
void set_context_free_error(const char* msg) { g_err = msg; }
}  // namespace pmx

struct pm_ctx {
    pm_config cfg;
    pm_cosmology cosmo;
    hipStream_t stream;
    char* ws;
    size_t ws_bytes;
    Plan plan;
    Lattice lat;
    Bins bins;
    int np, ng, cs, cs_p;
    long P;
    float2* C[5];   // C[4] on meshes up to kMaxPlane only
    // Working particle records, kept in bin order and double-buffered: each
    // sort moves them from the current arrays to the *_alt arrays, which then
    // become current.  id is the lattice index of each record.
    uint32_t *xq, *xq_alt, *id, *id_alt;
    int32_t *pq, *pq_alt;
    float *xi, *xi_alt, *pi, *pi_alt;
    uint32_t *fin_x, *ckpt;        // final state and checkpoints, lattice order
    int32_t* fin_p;
    float *tmpv, *noise;
    float *radial_f, *radial_ic, *radial_ic_dom, *radial_lpt, *theta, *gtheta, *fbar, *mlp_scratch;
    float* losstab;                    // targets, loss and shell factors of pm_loss_pk
    std::vector<double> loss_target;   // the targets, kept alive across their async upload
    // Pinned host memory that kernels write the scalar results to (res_host as the
    // device sees it: res_dev): after the synchronisation they are there.  Copying
    // them to ordinary memory took 23 us from the last kernel's launch to the end of
    // the wait, this takes 12.5.
    double* res_host = nullptr;
    double* res_dev = nullptr;
    size_t res_bytes = 0;
    bool hip_failed = false;   // a call ended without its wait: writes may be under way
    float2* tw;
    float2* tw_stages;
    Twiddles twd;
    double *partials, *sums, *pkbins;
    double *parts_a, *parts_b;      // partials of a reverse step's two gathers
    float* pmax;                    // and max |pi| beside the first's
    unsigned* maxbits;
    unsigned* ovf;                  // set by the forward kicks on a momentum overflow
    Schedule sched, dsched;         // KDK factors in use (scaled) and their d/dOmega_m
    Schedule sched0, dsched0;       // the unscaled growth-factor schedule and derivative
    std::vector<double> step_scale; // [3N] multipliers of kick_a | drift | kick_b
    std::vector<double> g_step;     // [3N] dL/d(step_scale) of the last adjoint
    bool have_step_grads = false;
    bool have_forward = false;
    // sorts since the records were last moved into bin order; kLatticeOrder
    // after the records were (re)written in lattice order
    int sorts_since_compact = 0;
    // the gather that last moved the particles also counted them into the bins
    bool counts_ready = false;
    bool have_filter = false;
    std::string err;
    pm_stats stats;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    // PM_F_TIMING: event pairs around launches, flushed into the stats
    static constexpr int kPool = 2048;
    bool timing = false;
    std::vector<hipEvent_t> pool;
    struct Pending { int cls; double bytes; int slot; };
    std::vector<Pending> pending;

    pm_ctx(const pm_config& c) : cfg(c), plan(c) {}
    void flush_timing() {
        if (pending.empty()) return;
        (void)hipEventSynchronize(pool[2 * pending.back().slot + 1]);
        for (const Pending& q : pending) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, pool[2 * q.slot], pool[2 * q.slot + 1]) == hipSuccess) {
                stats.kernel_ms[q.cls] += ms;
                stats.kernel_launches[q.cls] += 1;
                stats.kernel_bytes[q.cls] += q.bytes;
            }
        }
        pending.clear();
    }
    int acquire_slot() {
        if ((int)pending.size() == kPool) flush_timing();
        return (int)pending.size();
    }
    template <class Tp>
    Tp* at(size_t off) { return reinterpret_cast<Tp*>(ws + off); }
    int fail(int code, const std::string& msg) {
        if (code == PM_EHIP) {
            bins.dirty = true;   // a sort may have been left half done
            hip_failed = true;
        }
        err = msg;
        return code;
    }
    int hip_check(const char* where) {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(PM_EHIP, std::string(where) + ": " + hipGetErrorString(e));
        return PM_OK;
    }
    int wait(const char* what) {
        if (hipStreamSynchronize(stream) != hipSuccess)
            return fail(PM_EHIP, std::string("reading ") + what + " failed");
        return PM_OK;
    }
    float* creal(int k) { return reinterpret_cast<float*>(C[k]); }
    bool lpt2() const { return (cfg.flags & PM_F_2LPT) != 0; }
    long creal_stride() const { return 2 * plan.cplx_elems; }
    float mass() const { return (float)(lat.ratio * lat.ratio * lat.ratio); }
};

namespace {

// Times the launches enqueued during its lifetime (PM_F_TIMING), attributing
// `bytes` of algorithmic HBM traffic to kernel family `cls`.
struct KTimer {
    pm_ctx* c;
    int cls;
    double bytes;
    int slot = -1;
    KTimer(pm_ctx* ctx, int k, double b) : c(ctx), cls(k), bytes(b) {
        if (c->timing) {
            slot = c->acquire_slot();
            (void)hipEventRecord(c->pool[2 * slot], c->stream);
        }
    }
    ~KTimer() {
        if (slot >= 0) {
            (void)hipEventRecord(c->pool[2 * slot + 1], c->stream);
            c->pending.push_back({cls, bytes, slot});
        }
    }
};

// Algorithmic bytes: real mesh, half spectrum and one particle of FP32.
double mesh_r(int n) { return 4.0 * n * (double)n * n; }
double mesh_c(int n) { return 8.0 * n * (double)n * (n / 2 + 1); }

#define PM_TRY(expr)                 \
    do {                             \
        int _rc = (expr);            \
        if (_rc != PM_OK) return _rc; \
    } while (0)

// The schedule in use: sched0 and dsched0 (the cosmology's growth-factor schedule
// and its Omega_m derivative, integrals that take the host about 20 us per step)
// with the kick/drift factors multiplied by the per-step scales.
void apply_step_scales(pm_ctx* ctx) {
    const int N = ctx->cfg.n_steps;
    if (ctx->step_scale.empty()) ctx->step_scale.assign(3 * (size_t)N, 1.0);
    ctx->sched = ctx->sched0;
    ctx->dsched = ctx->dsched0;
    const double* f = ctx->step_scale.data();
    for (Schedule* t : {&ctx->sched, &ctx->dsched})
        for (int n = 0; n < N; ++n) {
            t->kick_a[n] *= f[n];
            t->drift[n] *= f[N + n];
            t->kick_b[n] *= f[2 * N + n];
        }
}

// Upload the cosmology-dependent tables (schedule on host; P(k) tables to the GPU).
int upload_tables(pm_ctx* ctx) {
    const pm_config& c = ctx->cfg;
    Cosmo co = to_cosmo(&ctx->cosmo);
    ctx->sched0 = schedule(co.omega_m, c.a_start, c.a_stop, c.n_steps);
    ctx->dsched0 = schedule_domega(co.omega_m, c.a_start, c.a_stop, c.n_steps);
    apply_step_scales(ctx);
    const int np = ctx->np, ng = ctx->ng;
    const long ntp = ctx->plan.ntab_p, ntf = ctx->plan.ntab_f;
    std::vector<double> pk = pk_table(co, c.box, (int)(ntp - 1));
    std::vector<double> dpk = pk_table_domega(co, c.box, (int)(ntp - 1));
    const double vcell = std::pow(c.box / np, 3.0);
    const double norm_p = c.box / (2.0 * kPi) / ((double)np * np * np);
    std::vector<float> ric(ntp), ricd(ntp), rlpt(ntp), rf(ntf);
    for (long n2 = 0; n2 < ntp; ++n2) {
        // second-order displacement s2_k = -i k S_k / k^2 (with the 1/Np^3 of the inverse)
        rlpt[n2] = n2 == 0 ? 0.f : (float)(-norm_p / n2);
        if (n2 == 0 || pk[n2] <= 0.0) {
            ric[n2] = 0.f;
            ricd[n2] = 0.f;
            continue;
        }
        const double sq = std::sqrt(pk[n2] / vcell);
        ric[n2] = (float)(sq * norm_p / n2);
        // d sqrt(P/V)/dOm = dP/dOm / (2 sqrt(P V))
        ricd[n2] = (float)(dpk[n2] / (2.0 * std::sqrt(pk[n2] * vcell)) * norm_p / n2);
    }
    // same FP32 expression as the filter path (f * fscale / n2 with f = 1), so a
    // zero filter reproduces the plain force bit for bit
    const float fscale = (float)(c.box / (2.0 * kPi) / std::pow((double)ng, 3.0));
    for (long n2 = 0; n2 < ntf; ++n2) rf[n2] = n2 == 0 ? 0.f : (1.0f * fscale) / (float)n2;
    std::vector<float2> tw(ng), stages(kStageTableSize);
    fill_stage_twiddles(stages.data());
    for (int m = 0; m < ng; ++m) {
        const double ang = -2.0 * kPi * m / ng;
        tw[m] = make_float2((float)std::cos(ang), (float)std::sin(ang));
    }
    hipStream_t s = ctx->stream;
    if (hipMemcpyAsync(ctx->radial_ic, ric.data(), ntp * sizeof(float), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ctx->radial_ic_dom, ricd.data(), ntp * sizeof(float), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ctx->radial_lpt, rlpt.data(), ntp * sizeof(float), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ctx->radial_f, rf.data(), ntf * sizeof(float), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ctx->tw, tw.data(), ng * sizeof(float2), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(ctx->tw_stages, stages.data(), kStageTableSize * sizeof(float2),
                       hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return ctx->fail(PM_EHIP, "uploading tables failed");
    return PM_OK;
}

// Radial tables of the force at sf's scale factors (plain: the precomputed one;
// learned: from the filter network, table t at t tab_stride).
void force_radials(pm_ctx* ctx, const ScaleFactors& sf) {
    if (!ctx->cfg.filter) return;
    KTimer t(ctx, PM_K_MLP, 0);
    const float fscale = (float)(ctx->cfg.box / (2.0 * kPi) / std::pow((double)ctx->ng, 3.0));
    launch_mlp_table(ctx->theta, ctx->ng, sf, fscale, ctx->plan.tab_stride, ctx->radial_f, nullptr,
                     ctx->stream);
}
const float* force_radial(pm_ctx* ctx, double a) {
    ScaleFactors sf;
    sf.add(a);
    force_radials(ctx, sf);
    return ctx->radial_f;
}

// A run's n evaluations 0, 1, ... of the force, at scale factors a[i stride]: the table of
// evaluation i, formed with those of the next ones (their number is bounded by
// the plan) when it is the first of a batch, and of the transposed pass's cotangent.
struct RunTables {
    pm_ctx* ctx;
    const double* a;   // outlives this
    int n, stride;
    int first_bar = -1;   // evaluations first_bar .. last_bar: cotangents not yet
    int last_bar = -1;    // taken through the network

    const float* radial(int i) {
        const int K = ctx->plan.ntables;
        if (ctx->cfg.filter && i % K == 0) {
            ScaleFactors sf;
            for (int k = i; k < std::min(i + K, n); ++k) sf.add(a[k * stride]);
            force_radials(ctx, sf);
        }
        return ctx->radial_f + offset(i);
    }
    // where evaluation i's dL/df goes (null for plain runs)
    float* bar(int i) {
        if (!ctx->cfg.filter) return nullptr;
        if (first_bar < 0) first_bar = i;
        last_bar = i;
        return ctx->fbar + offset(i);
    }
    // after evaluation i's transposed pass: a full batch, or the last one, is taken on
    void done(int i) {
        if (!ctx->cfg.filter || first_bar < 0) return;
        if ((i + 1) % ctx->plan.ntables != 0 && i + 1 < n) return;
        ScaleFactors sf;
        for (int k = first_bar; k <= last_bar; ++k) sf.add(a[k * stride]);
        KTimer t(ctx, PM_K_MLP, 0);
        launch_mlp_backward(ctx->theta, ctx->ng, sf, ctx->plan.tab_stride,
                            ctx->fbar + offset(first_bar), ctx->gtheta, ctx->mlp_scratch,
                            ctx->stream);
        first_bar = -1;
    }

  private:
    long offset(int i) const {
        return ctx->cfg.filter ? (i % ctx->plan.ntables) * ctx->plan.tab_stride : 0;
    }
};

// Records are moved into bin order on every kCompactEvery-th sort, and on the
// first sort after they were written in lattice order; in between, the sort
// only rebuilds the bin order (8 bytes written per particle instead of the 28
// or 52 bytes of its records, read and written).  The particle kernels then
// read the records through the order, a little less coalesced as particles
// change bins: measured at 512^3 particles, every 4th sort (bin family 524 ->
// 290 ms per 1024^3-mesh run, particle kernels +155 ms) beats every 2nd or
// 8th, and compacting on every sort of the adjoint gains nothing.
constexpr int kCompactEvery = 4;
constexpr int kLatticeOrder = 1 << 20;   // forces a compaction

// The working records are (re)written in lattice order.  Particles already counted
// for the next sort were counted where they no longer are (a checkpoint reset after
// the un-drift): those counts are to be cleared.
void records_in_lattice_order(pm_ctx* ctx) {
    ctx->sorts_since_compact = kLatticeOrder;
    if (ctx->counts_ready) ctx->bins.dirty = true;
    ctx->counts_ready = false;
}

// Where the records of a reverse run come from at x_N, in lattice order: the stored
// final state and the caller's cotangents (null: zero).
struct ReverseStart {
    const uint32_t* x;
    const int32_t* p;
    const float *xi, *pi;
};

// Bin the working particles (bin offsets and order in ctx->bins); compact the
// records (positions, momenta, ids, and with `cotangents` also xi and pi) when
// due.  With `start` (with cotangents) the compaction takes the records from there,
// so that they are never copied in lattice order first (512^3 particles: 2.7 ms of
// copies, clears and their reading back).  Returns the bytes moved, for the timing
// statistics.
double sort_particles(pm_ctx* ctx, bool cotangents, const ReverseStart* start = nullptr) {
    const double P = (double)ctx->P;
    cotangents = cotangents || start;
    if (start) records_in_lattice_order(ctx);
    launch_bin(start ? start->x : ctx->xq, ctx->lat, ctx->bins,
               ctx->counts_ready ? kCounted : kNotCounted, ctx->stream);
    // positions read, keys and ranks written and read, order written (the
    // gather that counted accounts for its own key and rank writes)
    double bytes = ctx->counts_ready ? 12.0 * P : 32.0 * P;
    ctx->counts_ready = false;
    if (++ctx->sorts_since_compact <= kCompactEvery) return bytes;
    ctx->sorts_since_compact = 1;
    Records rec;
    rec.state(start ? start->x : ctx->xq, ctx->xq_alt, start ? start->p : ctx->pq, ctx->pq_alt,
              ctx->id, ctx->id_alt);
    // without a momentum cotangent nothing reads pi before the un-drift writes it
    // (512^3 particles on 1024^3: compaction 3.93 -> 2.64 ms, un-kick at x_N,
    // which then leaves xi alone, 6.18 -> 5.15)
    if (start)
        rec.add_cotangents(start->xi, ctx->xi_alt, start->pi, start->pi ? ctx->pi_alt : nullptr, true);
    else if (cotangents)
        rec.add_cotangents(ctx->xi, ctx->xi_alt, ctx->pi, ctx->pi_alt, false);
    launch_compact(ctx->bins, rec, ctx->P, ctx->stream);
    std::swap(ctx->xq, ctx->xq_alt);
    std::swap(ctx->pq, ctx->pq_alt);
    std::swap(ctx->id, ctx->id_alt);
    if (cotangents) {
        std::swap(ctx->xi, ctx->xi_alt);
        std::swap(ctx->pi, ctx->pi_alt);
    }
    if (start) return bytes + (72.0 + (start->xi ? 12 : 0) + (start->pi ? 24 : 0)) * P;
    return bytes + (cotangents ? 112.0 : 64.0) * P;
}

// Fixed-point positions of a caller's displacements in the working positions,
// in lattice order and counted into the bins; the running state is gone.
void load_once(pm_ctx* ctx, const float* disp) {
    records_in_lattice_order(ctx);
    launch_to_fixed_count(disp, ctx->xq, ctx->lat, ctx->bins, ctx->stream);
}

// Bins the positions of load_once; the records stay in lattice order.
double order_once(pm_ctx* ctx) {
    launch_bin(ctx->xq, ctx->lat, ctx->bins, kCountedOnce, ctx->stream);
    return 12.0 * ctx->P;
}

// Zero bin counts for a gather that counts the particles it moves into the next
// sort's bins.
void count_next_bins(pm_ctx* ctx) { launch_bin_zero(ctx->bins, ctx->stream); }

// What compute_force and the building blocks bin: the running state (with or
// without its cotangents), whose records compact every few sorts, or one set of
// positions used once (counted by launch_to_fixed_count), which stays in
// lattice order: compacting its records costs more than the one or two kernels
// that read them through the order save (512^3 particles: 2.24 ms for the
// compaction alone; force on a 512^3 mesh 9.88 -> 7.52 ms without it, with the
// count in the pass that loads the positions and with slot-ordered
// output; density and P(k) at 256^3 0.948 -> 0.607 ms; sparse sets, 128^3 on
// 512^3, gain nothing and lose nothing).
enum Particles { kState, kStateCotangents, kOnce };

// PM force meshes of the working particles: sort into bins, delta -> C0
// (x,y-transformed spectrum left in C0) and, when given, to the caller's plain
// array `dens` in the same write-out, F~_j real meshes in C1..C3.
void compute_force(pm_ctx* ctx, const float* radial, Particles which, float* dens = nullptr,
                   const ReverseStart* start = nullptr) {
    hipStream_t s = ctx->stream;
    const int ng = ctx->ng, cs = ctx->cs;
    const long cst = ctx->plan.cplx_elems;
    const double r = mesh_r(ng), c = mesh_c(ng), P = (double)ctx->P;
    { KTimer t(ctx, PM_K_BIN, 0);
      t.bytes = which == kOnce ? order_once(ctx)
                               : sort_particles(ctx, which == kStateCotangents, start); }
    { KTimer t(ctx, PM_K_SCATTER, 12 * P + (dens ? 2 : 1) * r);
      launch_scatter_density(ctx->xq, ctx->lat, ctx->bins, ctx->creal(0), dens, s); }
    if (ng <= kMaxPlane) {   // planes: one launch for axes 2 and 1, timed with the last axis
        { KTimer t(ctx, PM_K_FFT_X, r + c);
          launch_fft_xy_r2c(nullptr, ctx->C[0], ng, cs, 1, cst, ctx->twd, s); }
        { KTimer t(ctx, PM_K_GRAD_Z, 3 * c);
          launch_grad_z(ctx->C[0], ctx->C[1], ctx->C[4], ng, cs, radial, ctx->twd, s); }
        { KTimer t(ctx, PM_K_FFT_X, 3 * r + 2 * c);
          launch_plane_c2r_force(ctx->C[1], ctx->C[4], ng, cs, cst, ctx->twd, s); }
        return;
    }
    { KTimer t(ctx, PM_K_FFT_X, r + c); launch_fft_x_r2c(ctx->C[0], ng, cs, 1, cst, ctx->twd, s); }
    { KTimer t(ctx, PM_K_FFT_STRIDED, 2 * c);
      launch_fft_y(ctx->C[0], ng, cs, -1, 1, cst, ctx->twd, s); }
    // F~_0 -> C1 and G -> C2; axis 1: F~_0 in place, G -> F~_1 (C2) and IFFT_1(G)
    // (C3); last axis: C2R of the three, C3 times i k2 first (= F~_2)
    { KTimer t(ctx, PM_K_GRAD_Z, 3 * c);
      launch_grad_z(ctx->C[0], ctx->C[1], ctx->C[2], ng, cs, radial, ctx->twd, s); }
    { KTimer t(ctx, PM_K_FFT_STRIDED, 5 * c);
      launch_fft_y(ctx->C[1], ng, cs, 1, 1, cst, ctx->twd, s);
      launch_fft_y_split(ctx->C[2], ctx->C[3], ng, cs, ctx->twd, s); }
    { KTimer t(ctx, PM_K_FFT_X, 3 * (r + c));
      launch_fft_x_c2r_dk2(ctx->C[1], ng, cs, 3, cst, 2, ctx->twd, s); }
}

// delta_bar (real, in C0) = transposed spectral operator applied to the CIC
// scatter of coeff * v at the current bins; the cotangent of the filter table to fbar
// (learned).  The word vmax_word(ctx) holds max |v| as float bits.
unsigned* vmax_word(pm_ctx* ctx) { return ctx->maxbits + kExtraSlots - 1; }
void vjp_mesh(pm_ctx* ctx, const uint32_t* xq, const float* v, float coeff, const float* radial,
              float* fbar) {
    hipStream_t s = ctx->stream;
    const int ng = ctx->ng, cs = ctx->cs;
    const long cst = ctx->plan.cplx_elems;
    const double r = mesh_r(ng), c = mesh_c(ng), P = (double)ctx->P;
    { KTimer t(ctx, PM_K_SCATTER_VEC, 24 * P + 3 * r);
      launch_scatter_vec(xq, v, coeff, vmax_word(ctx), ctx->lat, ctx->bins, ctx->creal(1),
                         ctx->creal_stride(), s); }
    // G_0 into C1 and n1 G_1 + n2 G_2 into C2, the transposed axis-0 pass's inputs
    const bool planes = ng <= kMaxPlane;
    if (planes) {
        KTimer t(ctx, PM_K_FFT_X, 3 * r + 2 * c);
        launch_plane_r2c_merge(ctx->C[1], ng, cs, cst, ctx->twd, s);
    } else {
        { KTimer t(ctx, PM_K_FFT_X, 3 * (r + c));
          launch_fft_x_r2c(ctx->C[1], ng, cs, 3, cst, ctx->twd, s); }
        { KTimer t(ctx, PM_K_FFT_STRIDED, 2 * c);
          launch_fft_y(ctx->C[1], ng, cs, -1, 1, cst, ctx->twd, s); }
        { KTimer t(ctx, PM_K_FFT_STRIDED, 3 * c);
          launch_fft_y_merge(ctx->C[2], ctx->C[3], ng, cs, ctx->twd, s); }
    }
    const float fscale = (float)(ctx->cfg.box / (2.0 * kPi) / std::pow((double)ng, 3.0));
    // (C3 is free: its spectrum went into C2's)
    // filter: delta_k read again, and the terms of +-n0 written and read (4 bytes each)
    const double terms = 4.0 * ng * (ng / 2 + 1.0) * (ng / 2 + 1.0);
    { KTimer t(ctx, PM_K_GRAD_ADJ_Z, fbar ? 4 * c + 2 * terms : 3 * c);
      launch_grad_adj_z(ctx->C[1], cst, ctx->C[0], ctx->C[0], ng, cs, radial, fbar,
                        ctx->creal(3), fscale, ctx->twd, s); }
    if (planes) {
        KTimer t(ctx, PM_K_FFT_X, r + c);
        launch_fft_yx_c2r(ctx->C[0], nullptr, ng, cs, 1, cst, ctx->twd, s);
    } else {
        { KTimer t(ctx, PM_K_FFT_STRIDED, 2 * c);
          launch_fft_y(ctx->C[0], ng, cs, 1, 1, cst, ctx->twd, s); }
        { KTimer t(ctx, PM_K_FFT_X, r + c);
          launch_fft_x_c2r(ctx->C[0], ng, cs, 1, cst, ctx->twd, s); }
    }
}

// Gradient synthesis on the particle lattice: the real mesh in C0 (or `field`,
// a dense [Np]^3 array, when given) becomes s_j = IDFT(i n_j radial(|n|^2) DFT(C0))
// in C1..C3 (the force chain; radial carries the 1/k^2, the k units and the
// 1/Np^3 of the inverse).
void grad_synthesis(pm_ctx* ctx, const float* radial, const float* field = nullptr) {
    hipStream_t s = ctx->stream;
    const int np = ctx->np, cs = ctx->cs_p;
    const long cst = ctx->plan.cplx_elems;
    launch_fft_xy_r2c(field, ctx->C[0], np, cs, 1, cst, ctx->twd, s);
    if (np <= kMaxPlane) {
        // G needs a buffer of its own: on a finer mesh the second half of C0, whose
        // size is 4 or more of the particle grid's, is free
        float2* g = np < ctx->ng ? ctx->C[0] + ctx->plan.cplx_elems / 2 : ctx->C[4];
        launch_grad_z(ctx->C[0], ctx->C[1], g, np, cs, radial, ctx->twd, s);
        launch_plane_c2r_force(ctx->C[1], g, np, cs, cst, ctx->twd, s);
        return;
    }
    launch_grad_z(ctx->C[0], ctx->C[1], ctx->C[2], np, cs, radial, ctx->twd, s);
    launch_fft_y(ctx->C[1], np, cs, 1, 1, cst, ctx->twd, s);
    launch_fft_y_split(ctx->C[2], ctx->C[3], np, cs, ctx->twd, s);
    launch_fft_x_c2r_dk2(ctx->C[1], np, cs, 3, cst, 2, ctx->twd, s);
}

// Transpose of grad_synthesis: the real mesh Sum_j IDFT(conj(i n_j radial)
// DFT(v_j)) of v [P][3] (lattice order; nullptr: of the real meshes in C1..C3) in
// C0, or in the dense array `out`.  With radial2 the same transpose with that
// table, from the same forward transforms, in C3.
void grad_transpose(pm_ctx* ctx, const float* v, const float* radial, float* out = nullptr,
                    const float* radial2 = nullptr) {
    hipStream_t s = ctx->stream;
    const int np = ctx->np, cs = ctx->cs_p;
    const long cst = ctx->plan.cplx_elems;
    const long rp = 2L * cs;
    if (v) launch_deinterleave(v, ctx->creal(1), ctx->creal_stride(), np, rp, s);
    if (np <= kMaxPlane) {
        launch_plane_r2c_merge(ctx->C[1], np, cs, cst, ctx->twd, s);
    } else {
        launch_fft_x_r2c(ctx->C[1], np, cs, 3, cst, ctx->twd, s);
        launch_fft_y(ctx->C[1], np, cs, -1, 1, cst, ctx->twd, s);
        launch_fft_y_merge(ctx->C[2], ctx->C[3], np, cs, ctx->twd, s);
    }
    for (const float* r : {radial, radial2}) {
        if (!r) continue;
        float2* dst = r == radial ? ctx->C[0] : ctx->C[3];
        launch_grad_adj_z(ctx->C[1], cst, dst, dst, np, cs, r, nullptr, nullptr, 0.f, ctx->twd, s);
        launch_fft_yx_c2r(dst, r == radial ? out : nullptr, np, cs, 1, cst, ctx->twd, s);
    }
}

// Zel'dovich displacement (a = 1) of white noise `noise` [Np^3] with the radial
// table: s_j as real meshes in C1..C3 (particle-grid geometry).
void ic_synthesis(pm_ctx* ctx, const float* noise) {
    KTimer t(ctx, PM_K_OTHER, 0);
    grad_synthesis(ctx, ctx->radial_ic, noise);
}

// The six Hessian entries (a, b), a <= b, of the potential of the linear density.
constexpr int kPairs[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {0, 2}, {1, 2}};

// Second-order (2LPT) displacement at a = 1 of white noise `noise` [Np^3]:
// Hessian entries phi_ab = IDFT(k_a k_b sqrt(P/V_c) noise_k / k^2) (the
// off-diagonal ones zero on the Nyquist planes of a and b), source
// S = Sum_{a<b} (phi_aa phi_bb - phi_ab^2), s2_k = -i k S_k / k^2 (the gradient's
// own Nyquist rule).  Writes s2_out [P][3] in lattice order; uses C0..C3.
void lpt_second_order(pm_ctx* ctx, const float* noise, float* s2_out) {
    hipStream_t s = ctx->stream;
    const int np = ctx->np, cs = ctx->cs_p;
    const long cst = ctx->plan.cplx_elems, rp = 2L * cs;
    // radial_ic holds sqrt(P/V_c) (L/2pi) / (Np^3 |n|^2): times 2pi/L and n_a n_b
    // it is the Hessian multiplier including the 1/Np^3 of the inverse
    const float kf = (float)(2.0 * kPi / ctx->cfg.box);
    float *r0 = ctx->creal(0), *r1 = ctx->creal(1), *r2 = ctx->creal(2), *r3 = ctx->creal(3);
    KTimer t(ctx, PM_K_OTHER, 0);
    launch_fft3_r2c_dense(noise, ctx->C[0], nullptr, np, cs, ctx->twd, s);
    // phi_ab's spectrum transformed back along axis 0, to buffer k
    auto hessian = [&](int k, int a, int b) {
        launch_fft_z_mul(ctx->C[0], ctx->C[k], np, cs, 1, a, b, 0, ctx->radial_ic, kf, false,
                         ctx->twd, s);
    };
    for (int a = 0; a < 3; ++a) hessian(1 + a, a, a);
    launch_fft_yx_c2r(ctx->C[1], nullptr, np, cs, 3, cst, ctx->twd, s);
    launch_lpt_pointwise(r1, r2, r3, r1, np, rp, 0, 1.f, s);
    hessian(2, 0, 1);
    hessian(3, 0, 2);
    launch_fft_yx_c2r(ctx->C[2], nullptr, np, cs, 2, cst, ctx->twd, s);
    launch_lpt_pointwise(r1, r2, r3, r1, np, rp, 1, 1.f, s);
    hessian(2, 1, 2);
    launch_fft_yx_c2r(ctx->C[2], nullptr, np, cs, 1, cst, ctx->twd, s);
    launch_lpt_pointwise(r1, r2, nullptr, r0, np, rp, 1, 1.f, s);   // S in C0
    grad_synthesis(ctx, ctx->radial_lpt);
    launch_ic_field(r1, ctx->creal_stride(), rp, ctx->lat, s2_out, s);
}

// Transpose of lpt_second_order at `noise`: g_noise [Np^3] += its transpose
// applied to s2_bar [P][3] (lattice order), and sums[slot] = the Omega_m
// derivative of <s2_bar, s2> through sqrt(P/V_c).  Reverse mode through the
// source: S_bar = transpose of the s2 gradient, phi_aa_bar = S_bar (phi_bb +
// phi_cc) over the two other axes, phi_ab_bar = -2 S_bar phi_ab; each Hessian
// entry is a real even multiplier of the noise, so its transpose is itself.
int lpt_second_order_transpose(pm_ctx* ctx, const float* noise, const float* s2_bar,
                               float* g_noise, int slot, int nb) {
    hipStream_t s = ctx->stream;
    const int np = ctx->np, cs = ctx->cs_p;
    const long cst = ctx->plan.cplx_elems, rp = 2L * cs;
    const float kf = (float)(2.0 * kPi / ctx->cfg.box);
    float *r0 = ctx->creal(0), *r2 = ctx->creal(2), *r3 = ctx->creal(3);
    KTimer t(ctx, PM_K_OTHER, 0);
    grad_transpose(ctx, s2_bar, ctx->radial_lpt);
    if (hipMemcpyAsync(r3, r0, (size_t)np * np * rp * sizeof(float), hipMemcpyDeviceToDevice, s) !=
        hipSuccess)
        return ctx->fail(PM_EHIP, "device copy failed");
    launch_fft3_r2c_dense(noise, ctx->C[0], nullptr, np, cs, ctx->twd, s);
    // C1 = Sum_ab (n_a n_b / |n|^2) DFT(phi_ab_bar)
    for (int k = 0; k < 6; ++k) {
        const int a = kPairs[k][0], b = kPairs[k][1];
        launch_fft_z_mul(ctx->C[0], ctx->C[2], np, cs, 1, a, b, a == b ? 1 : 0, ctx->radial_ic, kf,
                         false, ctx->twd, s);
        launch_fft_yx_c2r(ctx->C[2], nullptr, np, cs, 1, cst, ctx->twd, s);
        launch_lpt_pointwise(r2, r3, nullptr, r2, np, rp, 2, a == b ? 1.f : -2.f, s);
        launch_fft_xy_r2c(nullptr, ctx->C[2], np, cs, 1, cst, ctx->twd, s);
        launch_fft_z_mul(ctx->C[2], ctx->C[1], np, cs, -1, a, b, 0, nullptr, 1.f, k > 0, ctx->twd,
                         s);
    }
    // Omega_m: < IDFT(d sqrt(P/V_c)/dOmega_m C1), noise >
    launch_fft_z_mul(ctx->C[1], ctx->C[2], np, cs, 1, 0, 0, 2, ctx->radial_ic_dom, kf, false,
                     ctx->twd, s);
    launch_fft_yx_c2r(ctx->C[2], nullptr, np, cs, 1, cst, ctx->twd, s);
    launch_dot_pitched(r2, noise, np, rp, ctx->partials, nb, s);
    launch_reduce(ctx->partials, nb, ctx->sums, slot, s);
    // noise: IDFT(sqrt(P/V_c) C1)
    launch_fft_z_mul(ctx->C[1], ctx->C[2], np, cs, 1, 0, 0, 2, ctx->radial_ic, kf, false, ctx->twd,
                     s);
    launch_fft_yx_c2r(ctx->C[2], nullptr, np, cs, 1, cst, ctx->twd, s);
    launch_add_from_pitched(r2, g_noise, np, rp, 1.f, s);
    return PM_OK;
}

int copy_d2d(pm_ctx* ctx, void* dst, const void* src, size_t bytes) {
    if (hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, ctx->stream) != hipSuccess)
        return ctx->fail(PM_EHIP, "device copy failed");
    return PM_OK;
}

int ctx_check(pm_ctx* ctx) {
    if (!ctx) {
        g_err = "context is null";
        return PM_EINVAL;
    }
    return PM_OK;
}

}  // namespace

extern "C" {

size_t pm_workspace_bytes(const pm_config* cfg, int* status) {
    std::string why;
    int rc = check_config(cfg, &why);
    if (status) *status = rc;
    if (rc != PM_OK) {
        g_err = why;
        return 0;
    }
    return Plan(*cfg).total;
}

int pm_host_tables(const pm_config* cfg, const pm_cosmology* cosmo, double* coeffs,
                   double* dcoeffs, double* growth_out, double* pk_out) {
    std::string why;
    int rc = check_config(cfg, &why);
    if (rc == PM_OK) rc = check_cosmo(cosmo, &why);
    if (rc != PM_OK) {
        g_err = why;
        return rc;
    }
    Cosmo co = to_cosmo(cosmo);
    const int N = cfg->n_steps;
    auto fill = [N](const Schedule& s, double* out) {
        for (int n = 0; n < N; ++n) {
            out[n] = s.kick_a[n];
            out[N + n] = s.drift[n];
            out[2 * N + n] = s.kick_b[n];
        }
        out[3 * N] = s.D0;
        out[3 * N + 1] = s.G0;
    };
    Schedule s = schedule(co.omega_m, cfg->a_start, cfg->a_stop, N);
    if (coeffs) fill(s, coeffs);
    if (dcoeffs) fill(schedule_domega(co.omega_m, cfg->a_start, cfg->a_stop, N), dcoeffs);
    if (growth_out)
        for (int n = 0; n <= N; ++n) {
            growth_out[n] = s.D[n];
            growth_out[N + 1 + n] = s.dD[n];
            growth_out[2 * (N + 1) + n] = s.G[n];
        }
    if (pk_out) {
        const int n2max = 3 * (cfg->ptcl_grid / 2) * (cfg->ptcl_grid / 2);
        std::vector<double> t = pk_table(co, cfg->box, n2max);
        std::memcpy(pk_out, t.data(), t.size() * sizeof(double));
    }
    return PM_OK;
}

int pm_state_units(const pm_config* cfg, double* out) {
    std::string why;
    int rc = check_config(cfg, &why);
    if (rc == PM_OK && !out) {
        why = "out is required";
        rc = PM_EINVAL;
    }
    if (rc != PM_OK) {
        g_err = why;
        return rc;
    }
    state_units(*cfg, &out[0], &out[1]);
    out[2] = out[1] * 2147483648.0;
    return PM_OK;
}

int pm_lpt2_growth(const pm_config* cfg, const pm_cosmology* cosmo, double* out) {
    std::string why;
    int rc = check_config(cfg, &why);
    if (rc == PM_OK) rc = check_cosmo(cosmo, &why);
    if (rc == PM_OK && !out) {
        why = "out is required";
        rc = PM_EINVAL;
    }
    if (rc != PM_OK) {
        g_err = why;
        return rc;
    }
    const double om = to_cosmo(cosmo).omega_m;
    Schedule s = schedule(om, cfg->a_start, cfg->a_stop, cfg->n_steps);
    Schedule d = schedule_domega(om, cfg->a_start, cfg->a_stop, cfg->n_steps);
    out[0] = s.D20;
    out[1] = s.G20;
    out[2] = d.D20;
    out[3] = d.G20;
    return PM_OK;
}

int pm_init(const pm_config* cfg, const pm_cosmology* cosmo, void* workspace, size_t ws_bytes,
            void* hip_stream, pm_ctx** out) {
    std::string why;
    int rc = check_config(cfg, &why);
    if (rc == PM_OK) rc = check_cosmo(cosmo, &why);
    if (rc == PM_OK && (!workspace || !out)) {
        why = "workspace and out must be non-null";
        rc = PM_EINVAL;
    }
    if (rc == PM_OK && (reinterpret_cast<uintptr_t>(workspace) & 255u)) {
        why = "workspace must be 256-byte aligned";
        rc = PM_EINVAL;
    }
    if (rc == PM_OK && ws_bytes < Plan(*cfg).total) {
        why = "workspace too small";
        rc = PM_ENOMEM;
    }
    if (rc != PM_OK) {
        g_err = why;
        return rc;
    }
    pm_ctx* ctx = new pm_ctx(*cfg);
    ctx->cosmo = *cosmo;
    ctx->stream = reinterpret_cast<hipStream_t>(hip_stream);
    ctx->ws = static_cast<char*>(workspace);
    ctx->ws_bytes = ws_bytes;
    const Plan& p = ctx->plan;
    ctx->np = cfg->ptcl_grid;
    ctx->ng = cfg->mesh;
    ctx->cs = p.cs;
    ctx->cs_p = p.cs_p;
    ctx->P = p.P;
    for (int k = 0; k < 4; ++k) ctx->C[k] = ctx->at<float2>(p.cplx) + k * p.cplx_elems;
    ctx->C[4] = ctx->ng <= kMaxPlane ? ctx->C[3] + p.cplx_elems : nullptr;
    ctx->xq = ctx->at<uint32_t>(p.disp);
    ctx->pq = ctx->at<int32_t>(p.mom);
    ctx->xi = ctx->at<float>(p.xi);
    ctx->pi = ctx->at<float>(p.pi);
    ctx->xq_alt = ctx->at<uint32_t>(p.disp2);
    ctx->pq_alt = ctx->at<int32_t>(p.mom2);
    ctx->xi_alt = ctx->at<float>(p.xi2);
    ctx->pi_alt = ctx->at<float>(p.pi2);
    ctx->id = ctx->at<uint32_t>(p.id);
    ctx->id_alt = ctx->at<uint32_t>(p.id2);
    ctx->fin_x = ctx->at<uint32_t>(p.fin_disp);
    ctx->fin_p = ctx->at<int32_t>(p.fin_mom);
    ctx->tmpv = ctx->at<float>(p.tmpv);
    ctx->noise = ctx->at<float>(p.noise);
    ctx->ckpt = ctx->at<uint32_t>(p.ckpt);
    ctx->radial_f = ctx->at<float>(p.radial_f);
    ctx->radial_ic = ctx->at<float>(p.radial_ic);
    ctx->radial_ic_dom = ctx->at<float>(p.radial_ic_dom);
    ctx->radial_lpt = ctx->at<float>(p.radial_lpt);
    ctx->losstab = ctx->at<float>(p.losstab);
    ctx->tw = ctx->at<float2>(p.tw);
    ctx->tw_stages = ctx->at<float2>(p.tw_stages);
    ctx->twd = Twiddles{ctx->tw, ctx->ng, ctx->tw_stages};
    ctx->partials = ctx->at<double>(p.partials);
    ctx->parts_a = ctx->at<double>(p.parts_a);
    ctx->parts_b = ctx->at<double>(p.parts_b);
    ctx->pmax = ctx->at<float>(p.pmax);
    ctx->sums = ctx->at<double>(p.sums);
    ctx->maxbits = ctx->at<unsigned>(p.maxbits);
    ctx->pkbins = ctx->at<double>(p.pkbins);
    ctx->theta = ctx->at<float>(p.theta);
    ctx->gtheta = ctx->at<float>(p.gtheta);
    ctx->fbar = ctx->at<float>(p.fbar);
    ctx->mlp_scratch = ctx->at<float>(p.mlp_scratch);
    ctx->ovf = ctx->at<unsigned>(p.ovf);
    {
        Lattice& L = ctx->lat;
        int lg = 0;
        while ((1 << lg) < ctx->ng) ++lg;
        L.np = ctx->np;
        L.ng = ctx->ng;
        L.ratio = ctx->ng / ctx->np;
        L.inv_cell = (float)(ctx->ng / cfg->box);
        L.rp = 2L * p.cs;
        L.shift = 32 - lg;
        L.half = 1u << (L.shift - 1);
        L.qstep = (uint32_t)(4294967296.0 / ctx->np);
        L.frac = (float)std::ldexp(1.0, -L.shift);
        L.len_to_pos = (float)(4294967296.0 / cfg->box);
        L.pos_to_len = (float)(cfg->box / 4294967296.0);
        double pos_unit, mom_unit;
        state_units(*cfg, &pos_unit, &mom_unit);
        L.mom_unit = (float)mom_unit;
        L.inv_mom_unit = (float)(1.0 / mom_unit);
    }
    ctx->bins.tile = p.tile;
    ctx->bins.nt = p.nt;
    ctx->bins.counts = ctx->at<uint32_t>(p.counts);
    ctx->bins.offsets = ctx->at<uint32_t>(p.offsets);
    ctx->bins.keys = ctx->at<uint32_t>(p.keys);
    ctx->bins.ranks = ctx->at<uint32_t>(p.ranks);
    ctx->bins.ord = ctx->at<uint32_t>(p.ord);
    ctx->bins.scan_tmp = ctx->at<uint32_t>(p.scan_tmp);
    std::memset(&ctx->stats, 0, sizeof(ctx->stats));
    ctx->stats.workspace_bytes = p.total;
    for (int k = 0; k < 4; ++k)
        if (hipEventCreate(&ctx->ev[k]) != hipSuccess) {
            g_err = "hipEventCreate failed";
            delete ctx;
            return PM_EHIP;
        }
    {
        const size_t n = std::max<size_t>(3 * (size_t)ctx->ng,
                                          2 * (size_t)cfg->n_steps + 2 + 2 * kExtraSlots);
        void* dev = nullptr;
        ctx->res_host = static_cast<double*>(g_results.take(n * sizeof(double), &ctx->res_bytes));
        if (!ctx->res_host ||
            hipHostGetDevicePointer(&dev, ctx->res_host, 0) != hipSuccess) {
            g_err = "hipHostMalloc failed";
            pm_destroy(ctx);
            return PM_EHIP;
        }
        ctx->res_dev = static_cast<double*>(dev);
    }
    if (cfg->flags & PM_F_TIMING) {
        ctx->timing = true;
        ctx->pool.assign(2 * pm_ctx::kPool, nullptr);
        for (hipEvent_t& e : ctx->pool)
            if (hipEventCreate(&e) != hipSuccess) {
                g_err = "hipEventCreate failed";
                pm_destroy(ctx);
                return PM_EHIP;
            }
    }
    // what later calls take for granted, on whatever stream a captured one is
    // replayed: done when pm_init returns (upload_tables waits for the stream)
    launch_zero(ctx->theta, kNParam * sizeof(float), ctx->stream);
    launch_zero(ctx->ovf, sizeof(unsigned), ctx->stream);
    launch_zero(ctx->bins.counts, (ctx->bins.nkeys() + 1) * sizeof(uint32_t), ctx->stream);
    rc = ctx->hip_check("pm_init");
    if (rc == PM_OK) rc = upload_tables(ctx);
    if (rc != PM_OK) {
        g_err = ctx->err;
        pm_destroy(ctx);
        return rc;
    }
    *out = ctx;
    return PM_OK;
}

int pm_set_cosmology(pm_ctx* ctx, const pm_cosmology* cosmo) {
    PM_TRY(ctx_check(ctx));
    std::string why;
    if (check_cosmo(cosmo, &why) != PM_OK) return ctx->fail(PM_EINVAL, why);
    ctx->cosmo = *cosmo;
    ctx->have_forward = false;
    return upload_tables(ctx);
}

int pm_set_step_scales(pm_ctx* ctx, const double* scales) {
    PM_TRY(ctx_check(ctx));
    if (!scales) return ctx->fail(PM_EINVAL, "scales are null");
    const int N = ctx->cfg.n_steps;
    for (int i = 0; i < 3 * N; ++i)
        if (!std::isfinite(scales[i])) return ctx->fail(PM_EINVAL, "step scales must be finite");
    ctx->step_scale.assign(scales, scales + 3 * (size_t)N);
    apply_step_scales(ctx);
    ctx->have_forward = false;
    ctx->have_step_grads = false;
    return PM_OK;
}

int pm_step_gradients(pm_ctx* ctx, double* out) {
    PM_TRY(ctx_check(ctx));
    if (!out) return ctx->fail(PM_EINVAL, "out is null");
    if (!ctx->have_step_grads) return ctx->fail(PM_ESTATE, "no pm_adjoint since the last pm_forward");
    std::memcpy(out, ctx->g_step.data(), ctx->g_step.size() * sizeof(double));
    return PM_OK;
}

int pm_set_filter(pm_ctx* ctx, const float* weights_dev) {
    PM_TRY(ctx_check(ctx));
    if (!ctx->cfg.filter) return ctx->fail(PM_ESTATE, "context was created with filter = 0");
    if (!weights_dev) return ctx->fail(PM_EINVAL, "weights are null");
    PM_TRY(copy_d2d(ctx, ctx->theta, weights_dev, kNParam * sizeof(float)));
    ctx->have_forward = false;
    ctx->have_filter = true;
    return ctx->hip_check("pm_set_filter");
}

int pm_forward(pm_ctx* ctx, const float* noise, float* disp_out, float* mom_out, float* dens) {
    PM_TRY(ctx_check(ctx));
    if (!noise || !disp_out || !mom_out) return ctx->fail(PM_EINVAL, "noise, disp and mom are required");
    if (ctx->cfg.filter && !ctx->have_filter) return ctx->fail(PM_ESTATE, "pm_set_filter not called");
    // the stored run is overwritten from here on: valid again only once the whole
    // new run has been enqueued without error
    ctx->have_forward = false;
    ctx->have_step_grads = false;
    hipStream_t s = ctx->stream;
    const pm_config& c = ctx->cfg;
    const Schedule& sc = ctx->sched;
    const int N = c.n_steps;
    (void)hipEventRecord(ctx->ev[0], s);
    PM_TRY(copy_d2d(ctx, ctx->noise, noise, (size_t)ctx->P * sizeof(float)));
    launch_zero(ctx->ovf, sizeof(unsigned), s);
    if (ctx->lpt2()) lpt_second_order(ctx, ctx->noise, ctx->tmpv);
    ic_synthesis(ctx, ctx->noise);
    {
        KTimer t(ctx, PM_K_OTHER, 0);
        launch_ic_state(ctx->creal(1), ctx->creal_stride(), 2L * ctx->cs_p, (float)sc.D0,
                        (float)sc.G0, ctx->lat, ctx->xq, ctx->pq, ctx->id, s,
                        ctx->lpt2() ? ctx->tmpv : nullptr, (float)sc.D20, (float)sc.G20);
    }
    records_in_lattice_order(ctx);
    RunTables tables{ctx, sc.a.data(), N + 1, 1};
    for (int n = 0; n <= N; ++n) {
        // the last force is taken at the final positions: its density is the run's
        // (a sort and a scatter of their own took 3.6 ms at 512^3/1024^3)
        compute_force(ctx, tables.radial(n), kState, n == N ? dens : nullptr);
        const double kick = (n > 0 ? sc.kick_b[n - 1] : 0.0) + (n < N ? sc.kick_a[n] : 0.0);
        uint32_t* ckx = nullptr;
        int32_t* ckp = nullptr;
        if (c.checkpoint_every > 0 && n > 0 && n < N && n % c.checkpoint_every == 0) {
            const int slot = n / c.checkpoint_every - 1;
            ckx = ctx->ckpt + (size_t)slot * 6 * ctx->P;
            ckp = reinterpret_cast<int32_t*>(ckx + 3 * ctx->P);
        }
        const bool count = n < N;   // the drifted particles are binned for the next force
        if (count) count_next_bins(ctx);
        KTimer t(ctx, PM_K_GATHER,
                 ((ckx ? 72.0 : 48.0) + (count ? 8.0 : 0.0)) * ctx->P + 3 * mesh_r(ctx->ng));
        launch_gather_kick_drift(ctx->xq, ctx->pq, ctx->id, ctx->creal(1), ctx->creal_stride(),
                                 ctx->lat, ctx->bins, (float)kick,
                                 n < N ? (float)sc.drift[n] : 0.f, n < N, ckx, ckp, ctx->ovf,
                                 count, s);
        ctx->counts_ready = count;
    }
    {
        KTimer t(ctx, PM_K_OTHER, 0);
        // final state in lattice order (private copy for the adjoint) and outputs
        launch_final_state(ctx->xq, ctx->pq, ctx->id, ctx->lat, ctx->fin_x, ctx->fin_p, disp_out,
                           mom_out, s);
    }
    (void)hipEventRecord(ctx->ev[1], s);
    PM_TRY(ctx->hip_check("pm_forward"));
    ctx->have_forward = true;
    return PM_OK;
}

int pm_adjoint(pm_ctx* ctx, const float* g_dens, const float* g_disp, const float* g_mom,
               float* g_noise, double* g_cosmo, float* g_filter) {
    PM_TRY(ctx_check(ctx));
    if (!g_noise) return ctx->fail(PM_EINVAL, "g_noise is required");
    if (g_filter && !ctx->cfg.filter) return ctx->fail(PM_EINVAL, "g_filter needs filter = 1");
    if (!ctx->have_forward) return ctx->fail(PM_ESTATE, "pm_adjoint needs a preceding pm_forward");
    hipStream_t s = ctx->stream;
    const pm_config& c = ctx->cfg;
    const Schedule& sc = ctx->sched;
    const int N = c.n_steps;
    const long P = ctx->P;
    const size_t vec = (size_t)P * 3 * sizeof(float);
    // grid-stride reductions over the particles: block partials + one max per block
    const int nb = std::min(particle_blocks(P), 4096);
    const int nb_ic = std::min(nb, 1024);   // nine sets of partials
    const int slotS = 0, slotD = N + 1, slotX = 2 * N + 1;   // S_m, D_n, extras
    const int xD0 = slotX, xG0 = slotX + 1, xSig = slotX + 2, xOm = slotX + 3,
              xIc = slotX + 4, xIcMom = slotX + 5, xIcMomRef = slotX + 6, xCk = slotX + 8,
              xD20 = xCk + PM_MAX_CHECKPOINTS, xG20 = xD20 + 1, xSig2 = xD20 + 2,
              xOm2 = xD20 + 3;
    const bool lpt2 = ctx->lpt2();
    const float mass = ctx->mass();
    const double bytes_unkick = 72.0 * P + 3 * mesh_r(ctx->ng);
    const double bytes_wgrad = 84.0 * P + mesh_r(ctx->ng);
    (void)hipEventRecord(ctx->ev[2], s);
    launch_zero(ctx->sums, (2 * (size_t)N + 2 + kExtraSlots) * sizeof(double), s);
    launch_zero(ctx->maxbits, kExtraSlots * sizeof(unsigned), s);
    if (c.filter) launch_zero(ctx->gtheta, kNParam * sizeof(float), s);

    // seed at x_N: xi = dL/dx_N (lattice order), sorted with the state by the
    // force evaluation, then + m grad w . dL/ddelta.  The vector scatters need max
    // |pi|: of a caller's cotangent here, later from the kernels that write pi (a
    // pass of its own read pi once more per step, 16 us at 128^3 particles, 0.3 ms
    // at 512^3, and cleared the word before it)
    if (g_mom) launch_absmax(g_mom, 3 * P, vmax_word(ctx), s);
    const ReverseStart start{ctx->fin_x, ctx->fin_p, g_disp, g_mom};
    RunTables tables{ctx, sc.a.data() + N, N + 1, -1};   // evaluation N - n is at x_n
    const float* radial = tables.radial(0);
    compute_force(ctx, radial, kStateCotangents, nullptr, &start);
    const int ngather = (int)gather_partials(ctx->np, ctx->ng);
    if (g_dens) {
        KTimer t(ctx, PM_K_WGRAD, 36.0 * P + mesh_r(ctx->ng));
        launch_wgrad(g_dens, ctx->ng, mass, ctx->xq, ctx->pq, ctx->xi, ctx->pi, ctx->lat,
                     ctx->bins, 0.f, 2, nullptr, s, true);
    }
    {
        KTimer t(ctx, PM_K_UNKICK_VJP, g_mom ? bytes_unkick : 36.0 * P + 3 * mesh_r(ctx->ng));
        launch_unkick_vjp(ctx->xq, ctx->pq, ctx->creal(1), ctx->creal_stride(), ctx->lat,
                          ctx->bins, (float)sc.kick_b[N - 1], g_mom ? ctx->pi : nullptr, ctx->xi,
                          false, ctx->parts_b, s);
    }
    launch_reduce(ctx->parts_b, ngather, ctx->sums, slotS + N, s);

    int nck = 0;
    for (int n = N - 1; n >= 0; --n) {
        // (ii) + (iii) at x_{n+1}; then un-drift to x_n.  Without a momentum
        // cotangent pi is zero at x_N, and (ii) and (iii), linear in pi, add zero:
        // the first step is then the un-drift alone (one VJP less per run: 28 ms
        // of 312 ms on 512^3 particles, 1024^3 mesh, two steps)
        const double c1 = sc.kick_b[n] + (n + 1 < N ? sc.kick_a[n + 1] : 0.0);
        const bool pi_zero = n == N - 1 && !g_mom;
        if (!pi_zero)
            vjp_mesh(ctx, ctx->xq, ctx->pi, (float)c1, radial, tables.bar(N - n - 1));
        tables.done(N - n - 1);
        count_next_bins(ctx);   // the un-drifted particles are binned for F(x_n)
        if (pi_zero) {
            KTimer t(ctx, PM_K_WGRAD, 68.0 * P);
            launch_undrift(ctx->xq, ctx->pq, ctx->xi, ctx->pi, ctx->lat, ctx->bins,
                           (float)sc.drift[n], ctx->parts_a, ctx->pmax, nb, s);
        } else {
            KTimer t(ctx, PM_K_WGRAD, bytes_wgrad + 8.0 * P);
            launch_wgrad(ctx->creal(0), ctx->lat.rp, mass, ctx->xq, ctx->pq, ctx->xi, ctx->pi,
                         ctx->lat, ctx->bins, (float)sc.drift[n], 1, ctx->parts_a, s, false,
                         true, ctx->pmax);
        }
        ctx->counts_ready = true;
        // checkpoint: compare the reconstructed (x_n, p_{n+1/2}) and reset to it
        if (c.checkpoint_every > 0 && n > 0 && n % c.checkpoint_every == 0) {
            const int slot = n / c.checkpoint_every - 1;
            const uint32_t* ckx = ctx->ckpt + (size_t)slot * 6 * P;
            launch_recon_err(ctx->xq, ctx->id, ckx, ctx->lat, ctx->partials, nb,
                             ctx->maxbits + 2 + nck, s);
            launch_reduce(ctx->partials, nb, ctx->sums, xCk + nck, s);
            // reset to the stored (lattice-order) state; cotangents to lattice order
            PM_TRY(copy_d2d(ctx, ctx->xq, ckx, vec));
            PM_TRY(copy_d2d(ctx, ctx->pq, ckx + 3 * P, vec));
            launch_permute_by_id(ctx->xi, ctx->id, ctx->xi_alt, P, s);
            launch_permute_by_id(ctx->pi, ctx->id, ctx->pi_alt, P, s);
            std::swap(ctx->xi, ctx->xi_alt);
            std::swap(ctx->pi, ctx->pi_alt);
            launch_iota(ctx->id, P, s);
            records_in_lattice_order(ctx);
            ++nck;
        }
        // recompute F(x_n); un-kick and (i) at x_n
        radial = tables.radial(N - n);
        compute_force(ctx, radial, kStateCotangents);
        const double c0 = (n > 0 ? sc.kick_b[n - 1] : 0.0) + sc.kick_a[n];
        {
            KTimer t(ctx, PM_K_UNKICK_VJP, bytes_unkick);
            launch_unkick_vjp(ctx->xq, ctx->pq, ctx->creal(1), ctx->creal_stride(), ctx->lat,
                              ctx->bins, (float)c0, ctx->pi, ctx->xi, false, ctx->parts_b, s);
        }
        ReduceSets step;
        step.add(ctx->parts_a, pi_zero ? nb : ngather, slotD + n);
        step.add(ctx->parts_b, ngather, slotS + n);
        step.maxs = ctx->pmax;
        step.nmax = step.n[0];
        step.vmax = vmax_word(ctx);
        launch_reduce_sets(step, ctx->sums, s);
    }
    // (ii) + (iii) at x_0
    vjp_mesh(ctx, ctx->xq, ctx->pi, (float)sc.kick_a[0], radial, tables.bar(N));
    tables.done(N);
    {
        KTimer t(ctx, PM_K_WGRAD, 36.0 * P + mesh_r(ctx->ng));
        launch_wgrad(ctx->creal(0), ctx->lat.rp, mass, ctx->xq, ctx->pq, ctx->xi, ctx->pi,
                     ctx->lat, ctx->bins, 0.f, 2, nullptr, s);
    }

    // ICs: x_0 = q + D0 s (+ D20 s2), p_0 = G0 s (+ G20 s2).  Reconstruction
    // check against the ICs.  2LPT: s2 in pi_alt (lattice order; free here).
    if (lpt2) lpt_second_order(ctx, ctx->noise, ctx->pi_alt);
    ic_synthesis(ctx, ctx->noise);
    {
        KTimer t(ctx, PM_K_OTHER, 0);
        // checks and scalar sums; s_bar = D0 xi + G0 pi over s in C1..C3, and s2_bar =
        // D20 xi + G20 pi in xi_alt (lattice order)
        const int slots[9] = {xIc, xIcMom, xIcMomRef, xD0, xG0, xSig, xD20, xG20, xSig2};
        ReduceSets end;
        for (int k = 0; k < (lpt2 ? 9 : 6); ++k)
            end.add(ctx->partials + (long)k * nb_ic, nb_ic, slots[k]);
        launch_ic_adjoint(ctx->creal(1), ctx->creal_stride(), 2L * ctx->cs_p, (float)sc.D0,
                          (float)sc.G0, ctx->lat, ctx->xq, ctx->pq, ctx->id, ctx->xi, ctx->pi,
                          ctx->partials, nb_ic, ctx->maxbits, s, lpt2 ? ctx->pi_alt : nullptr,
                          lpt2 ? ctx->xi_alt : nullptr, (float)sc.D20, (float)sc.G20);
        launch_reduce_sets(end, ctx->sums, s);
        // dL/dnoise = transpose of the synthesis applied to s_bar; and, with the
        // Omega_m derivative of its table, the field whose product with the noise is
        // <s_bar, ds/dOmega_m> (the synthesis is linear in the noise)
        grad_transpose(ctx, nullptr, ctx->radial_ic, g_noise, ctx->radial_ic_dom);
        launch_dot_pitched(ctx->creal(3), ctx->noise, ctx->np, 2L * ctx->cs_p, ctx->partials, nb, s);
        launch_reduce(ctx->partials, nb, ctx->sums, xOm, s);
    }
    if (lpt2) PM_TRY(lpt_second_order_transpose(ctx, ctx->noise, ctx->xi_alt, g_noise, xOm2, nb));
    if (g_filter) PM_TRY(copy_d2d(ctx, g_filter, ctx->gtheta, kNParam * sizeof(float)));
    (void)hipEventRecord(ctx->ev[3], s);
    PM_TRY(ctx->hip_check("pm_adjoint"));

    // scalar results (synchronises)
    const int nsum = 2 * N + 1 + kExtraSlots;
    launch_collect(ctx->sums, nsum, ctx->maxbits, kExtraSlots, ctx->ovf, ctx->res_dev, s);
    PM_TRY(ctx->hip_check("pm_adjoint"));
    PM_TRY(ctx->wait("adjoint sums"));
    const double* h = ctx->res_host;
    const unsigned* mb = reinterpret_cast<const unsigned*>(h + nsum);
    const unsigned ovf = mb[kExtraSlots];
    if (ovf)
        return ctx->fail(PM_ENUMERIC, "a momentum of the forward run left the fixed-point range "
                                      "(see pm_state_units)");
    const Schedule& d = ctx->dsched;
    double g_om = 0.0;
    for (int n = 0; n < N; ++n)
        g_om += h[slotS + n] * d.kick_a[n] + h[slotS + n + 1] * d.kick_b[n] + h[slotD + n] * d.drift[n];
    g_om += h[xD0] * d.D0 + h[xG0] * d.G0 + h[xOm];
    // 2LPT: s2 ~ sigma_8^2, hence the factor 2 (the slots stay 0 otherwise)
    g_om += h[xD20] * d.D20 + h[xG20] * d.G20 + h[xOm2];
    const double g_s8 = (h[xSig] + 2.0 * h[xSig2]) / ctx->cosmo.sigma8;
    for (int i = 0; i < nsum; ++i)
        if (!std::isfinite(h[i])) return ctx->fail(PM_ENUMERIC, "non-finite adjoint sum");
    // dL/d(scale) = unscaled factor * dL/d(factor) per step
    ctx->g_step.assign(3 * (size_t)N, 0.0);
    for (int n = 0; n < N; ++n) {
        ctx->g_step[n] = h[slotS + n] * ctx->sched0.kick_a[n];
        ctx->g_step[N + n] = h[slotD + n] * ctx->sched0.drift[n];
        ctx->g_step[2 * N + n] = h[slotS + n + 1] * ctx->sched0.kick_b[n];
    }
    ctx->have_step_grads = true;
    if (g_cosmo) {
        g_cosmo[0] = g_om;
        g_cosmo[1] = g_s8;
    }
    auto as_float = [](unsigned b) {
        float f;
        std::memcpy(&f, &b, sizeof(f));
        return (double)f;
    };
    ctx->stats.n_checkpoints = nck;
    for (int k = 0; k < nck; ++k) {
        ctx->stats.ckpt_rms_cells[k] = std::sqrt(h[xCk + k] / P);
        ctx->stats.ckpt_max_cells[k] = as_float(mb[2 + k]);
    }
    ctx->stats.ic_rms_cells = std::sqrt(h[xIc] / P);
    ctx->stats.ic_max_cells = as_float(mb[0]);
    ctx->stats.ic_mom_rel_rms = h[xIcMomRef] > 0 ? std::sqrt(h[xIcMom] / h[xIcMomRef]) : 0.0;
    return PM_OK;
}

int pm_initial_conditions(pm_ctx* ctx, const float* noise, float* disp_out, float* mom_out) {
    PM_TRY(ctx_check(ctx));
    if (!noise || !disp_out || !mom_out) return ctx->fail(PM_EINVAL, "noise, disp and mom are required");
    if (ctx->lpt2()) lpt_second_order(ctx, noise, ctx->tmpv);
    ic_synthesis(ctx, noise);
    {
        KTimer t(ctx, PM_K_OTHER, 0);
        const Schedule& sc = ctx->sched;
        launch_ic_float(ctx->creal(1), ctx->creal_stride(), 2L * ctx->cs_p, (float)sc.D0,
                        (float)sc.G0, ctx->lat, disp_out, mom_out, ctx->stream,
                        ctx->lpt2() ? ctx->tmpv : nullptr, (float)sc.D20, (float)sc.G20);
    }
    return ctx->hip_check("pm_initial_conditions");
}

int pm_loss_mse(pm_ctx* ctx, const float* dens, const float* target, float* g_dens,
                double* loss) {
    PM_TRY(ctx_check(ctx));
    if (!dens || !target) return ctx->fail(PM_EINVAL, "dens and target are required");
    const long n3 = (long)ctx->ng * ctx->ng * ctx->ng;
    const int nb = std::min(particle_blocks(n3), 4096);
    launch_mse(dens, target, g_dens, n3, ctx->partials, nb, ctx->stream);
    PM_TRY(ctx->hip_check("pm_loss_mse"));
    if (loss) {
        launch_reduce(ctx->partials, nb, ctx->res_dev, 0, ctx->stream);
        PM_TRY(ctx->hip_check("pm_loss_mse"));
        PM_TRY(ctx->wait("the loss"));
        *loss = ctx->res_host[0] / n3;
    }
    return PM_OK;
}

int pm_loss_pk(pm_ctx* ctx, const float* dens, int32_t n_bins, const double* pk_target,
               double weight, double* loss, float* g_dens) {
    PM_TRY(ctx_check(ctx));
    if (!dens || !pk_target) return ctx->fail(PM_EINVAL, "dens and pk_target are required");
    if (n_bins < 1 || n_bins > ctx->ng) return ctx->fail(PM_EINVAL, "n_bins must be in [1, mesh]");
    if (!std::isfinite(weight)) return ctx->fail(PM_EINVAL, "weight must be finite");
    // shells b <= round(sqrt(3) ng / 2) hold modes; further ones are empty
    const int b_max = (int)std::floor(std::sqrt(0.75) * ctx->ng + 0.5);
    bool usable = false;
    for (int b = 1; b <= n_bins && b <= b_max; ++b)
        usable = usable || (pk_target[b - 1] != 0.0 && std::isfinite(pk_target[b - 1]));
    if (!usable) return ctx->fail(PM_EINVAL, "no shell has both modes and a nonzero target");
    hipStream_t s = ctx->stream;
    const int ng = ctx->ng;
    // P_b = L^3 / Ng^6 <|delta_k|^2>_b; dL/d delta(x) = 2 Sum_k t_k delta_k e^{ik.x}
    // (unnormalised inverse DFT) with t_k = dL/dP_b L^3 / (Ng^6 N_b), one value per
    // shell.  Targets, shell factors and whether the loss is finite (only then is
    // g_dens written) live in losstab: [n_bins] | [n_bins] | 1
    const double L = ctx->cfg.box, norm = L * L * L / std::pow((double)ng, 6.0);
    double* target_dev = reinterpret_cast<double*>(ctx->losstab);
    float* table_dev = reinterpret_cast<float*>(target_dev + n_bins);
    int* finite_dev = reinterpret_cast<int*>(table_dev + n_bins);
    ctx->loss_target.assign(pk_target, pk_target + n_bins);
    if (hipMemcpyAsync(target_dev, ctx->loss_target.data(), n_bins * sizeof(double),
                       hipMemcpyHostToDevice, s) != hipSuccess)
        return ctx->fail(PM_EHIP, "upload of the loss targets failed");
    launch_fft_shells(dens, ctx->C[0], ctx->C[1], ng, ctx->cs, n_bins, ctx->pkbins, ctx->twd, s);
    launch_pk_loss(ctx->pkbins, target_dev, n_bins, norm, weight, ctx->res_dev, table_dev,
                   finite_dev, s);
    if (g_dens)
        launch_fft_shell_scale(ctx->C[0], g_dens, ng, ctx->cs, n_bins, table_dev, finite_dev,
                               ctx->twd, s);
    PM_TRY(ctx->hip_check("pm_loss_pk"));
    PM_TRY(ctx->wait("the P(k) loss"));
    if (loss) *loss = ctx->res_host[0];
    if (!std::isfinite(ctx->res_host[1])) return ctx->fail(PM_ENUMERIC, "non-finite P(k) loss");
    return PM_OK;
}

int pm_loss_disp(pm_ctx* ctx, const float* disp, const float* disp_target, double weight,
                 double* loss, float* g_disp) {
    PM_TRY(ctx_check(ctx));
    if (!disp || !disp_target) return ctx->fail(PM_EINVAL, "disp and disp_target are required");
    if (!std::isfinite(weight)) return ctx->fail(PM_EINVAL, "weight must be finite");
    const long n = 3 * ctx->P;
    const double cell = ctx->cfg.box / ctx->ng;
    const double norm = weight / ((double)ctx->P * cell * cell);
    const int nb = std::min(particle_blocks(n), 4096);
    launch_mse_periodic(disp, disp_target, g_disp, n, (float)ctx->cfg.box, (float)(2.0 * norm),
                        ctx->partials, nb, ctx->stream);
    PM_TRY(ctx->hip_check("pm_loss_disp"));
    if (loss) {
        launch_reduce(ctx->partials, nb, ctx->res_dev, 0, ctx->stream);
        PM_TRY(ctx->hip_check("pm_loss_disp"));
        PM_TRY(ctx->wait("the loss"));
        *loss = norm * ctx->res_host[0];
    }
    return PM_OK;
}

int pm_power_spectrum(pm_ctx* ctx, const float* dens, int32_t n_bins, double* k_out,
                      double* pk_out, double* nmodes_out) {
    PM_TRY(ctx_check(ctx));
    if (!dens) return ctx->fail(PM_EINVAL, "dens is required");
    if (n_bins < 1 || n_bins > ctx->ng) return ctx->fail(PM_EINVAL, "n_bins must be in [1, mesh]");
    hipStream_t s = ctx->stream;
    const int ng = ctx->ng;
    launch_fft_shells(dens, ctx->C[0], ctx->C[0], ng, ctx->cs, n_bins, ctx->res_dev, ctx->twd, s);
    PM_TRY(ctx->hip_check("pm_power_spectrum"));
    PM_TRY(ctx->wait("P(k)"));
    const double* h = ctx->res_host;
    const double L = ctx->cfg.box, n6 = std::pow((double)ng, 6.0);
    for (int b = 0; b < n_bins; ++b) {
        const double cnt = h[3 * b + 2];
        if (k_out) k_out[b] = cnt > 0 ? h[3 * b + 1] / cnt * 2.0 * kPi / L : NAN;
        if (pk_out) pk_out[b] = cnt > 0 ? h[3 * b] / cnt * L * L * L / n6 : NAN;
        if (nmodes_out) nmodes_out[b] = cnt;
    }
    return PM_OK;
}

int pm_density(pm_ctx* ctx, const float* disp, float* dens) {
    PM_TRY(ctx_check(ctx));
    if (!disp || !dens) return ctx->fail(PM_EINVAL, "disp and dens are required");
    load_once(ctx, disp);
    order_once(ctx);
    launch_scatter_density(ctx->xq, ctx->lat, ctx->bins, nullptr, dens, ctx->stream);
    return ctx->hip_check("pm_density");
}

int pm_force(pm_ctx* ctx, const float* disp, double a, float* force) {
    PM_TRY(ctx_check(ctx));
    if (!disp || !force) return ctx->fail(PM_EINVAL, "disp and force are required");
    if (ctx->cfg.filter && !ctx->have_filter) return ctx->fail(PM_ESTATE, "pm_set_filter not called");
    load_once(ctx, disp);
    compute_force(ctx, force_radial(ctx, a), kOnce);
    launch_gather_force(ctx->xq, ctx->creal(1), ctx->creal_stride(), ctx->lat, ctx->bins, force,
                        ctx->stream);
    return ctx->hip_check("pm_force");
}

int pm_force_vjp(pm_ctx* ctx, const float* disp, double a, const float* v, float* xi) {
    PM_TRY(ctx_check(ctx));
    if (!disp || !v || !xi) return ctx->fail(PM_EINVAL, "disp, v and xi are required");
    if (ctx->cfg.filter && !ctx->have_filter) return ctx->fail(PM_ESTATE, "pm_set_filter not called");
    hipStream_t s = ctx->stream;
    load_once(ctx, disp);
    RunTables tables{ctx, &a, 1, 1};
    const float* radial = tables.radial(0);
    compute_force(ctx, radial, kOnce);
    launch_unkick_vjp(ctx->xq, nullptr, ctx->creal(1), ctx->creal_stride(), ctx->lat, ctx->bins,
                      1.f, v, xi, true, nullptr, s);
    if (ctx->cfg.filter) launch_zero(ctx->gtheta, kNParam * sizeof(float), s);
    launch_zero(vmax_word(ctx), sizeof(unsigned), s);
    launch_absmax(v, 3 * ctx->P, vmax_word(ctx), s);
    vjp_mesh(ctx, ctx->xq, v, 1.f, radial, tables.bar(0));
    tables.done(0);
    launch_wgrad(ctx->creal(0), ctx->lat.rp, ctx->mass(), ctx->xq, nullptr, xi, nullptr, ctx->lat,
                 ctx->bins, 0.f, 2, nullptr, s);
    return ctx->hip_check("pm_force_vjp");
}

int pm_fft_r2c(pm_ctx* ctx, const float* real, float* spec) {
    PM_TRY(ctx_check(ctx));
    if (!real || !spec) return ctx->fail(PM_EINVAL, "real and spec are required");
    hipStream_t s = ctx->stream;
    const int ng = ctx->ng;
    launch_fft3_r2c_dense(real, ctx->C[0], reinterpret_cast<float2*>(spec), ng, ctx->cs, ctx->twd, s);
    return ctx->hip_check("pm_fft_r2c");
}

int pm_fft_c2r(pm_ctx* ctx, const float* spec, float* real) {
    PM_TRY(ctx_check(ctx));
    if (!real || !spec) return ctx->fail(PM_EINVAL, "real and spec are required");
    hipStream_t s = ctx->stream;
    const int ng = ctx->ng;
    launch_fft3_c2r_dense(reinterpret_cast<const float2*>(spec), ctx->C[0], real, ng, ctx->cs,
                          ctx->twd, s);
    return ctx->hip_check("pm_fft_c2r");
}

int pm_filter_table(pm_ctx* ctx, double a, float* table) {
    PM_TRY(ctx_check(ctx));
    if (!table) return ctx->fail(PM_EINVAL, "table is required");
    if (!ctx->cfg.filter || !ctx->have_filter) return ctx->fail(PM_ESTATE, "no filter weights set");
    ScaleFactors sf;
    sf.add(a);
    launch_mlp_table(ctx->theta, ctx->ng, sf, 0.f, 0, nullptr, table, ctx->stream);
    return ctx->hip_check("pm_filter_table");
}

int pm_adam(pm_ctx* ctx, float* param, const float* grad, int32_t n_grads, float* m, float* v,
            int32_t n, double lr, double beta1, double beta2, double eps, int32_t t) {
    PM_TRY(ctx_check(ctx));
    if (!param || !grad || !m || !v || n < 1 || t < 1 || n_grads < 1)
        return ctx->fail(PM_EINVAL, "bad Adam arguments");
    const double bc1 = 1.0 - std::pow(beta1, t), bc2 = 1.0 - std::pow(beta2, t);
    launch_adam(param, grad, n_grads, m, v, n, (float)lr, (float)beta1, (float)beta2, (float)eps,
                (float)bc1, (float)bc2, ctx->stream);
    return ctx->hip_check("pm_adam");
}

int pm_stats_get(pm_ctx* ctx, pm_stats* out) {
    PM_TRY(ctx_check(ctx));
    if (!out) return ctx->fail(PM_EINVAL, "out is null");
    float ms = 0.f;
    if (hipEventSynchronize(ctx->ev[3]) == hipSuccess &&
        hipEventElapsedTime(&ms, ctx->ev[2], ctx->ev[3]) == hipSuccess)
        ctx->stats.adjoint_ms = ms;
    if (hipEventSynchronize(ctx->ev[1]) == hipSuccess &&
        hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]) == hipSuccess)
        ctx->stats.forward_ms = ms;
    ctx->flush_timing();
    (void)hipGetLastError();
    unsigned ovf = 0;
    if (hipMemcpyAsync(&ovf, ctx->ovf, sizeof(unsigned), hipMemcpyDeviceToHost, ctx->stream) !=
            hipSuccess ||
        hipStreamSynchronize(ctx->stream) != hipSuccess)
        return ctx->fail(PM_EHIP, "reading the overflow flag failed");
    ctx->stats.momentum_overflow = ovf ? 1 : 0;
    *out = ctx->stats;
    return PM_OK;
}

int pm_stats_reset(pm_ctx* ctx) {
    PM_TRY(ctx_check(ctx));
    ctx->flush_timing();
    for (int k = 0; k < PM_NKERNELS; ++k) {
        ctx->stats.kernel_ms[k] = 0.0;
        ctx->stats.kernel_launches[k] = 0;
        ctx->stats.kernel_bytes[k] = 0.0;
    }
    return PM_OK;
}

void pm_destroy(pm_ctx* ctx) {
    if (!ctx) return;
    for (int k = 0; k < 4; ++k)
        if (ctx->ev[k]) (void)hipEventDestroy(ctx->ev[k]);
    for (hipEvent_t e : ctx->pool)
        if (e) (void)hipEventDestroy(e);
    if (ctx->res_host && ctx->hip_failed) (void)hipHostFree(ctx->res_host);   // waits
    else if (ctx->res_host) g_results.give(ctx->res_host, ctx->res_bytes);
    delete ctx;
}

const char* pm_last_error(const pm_ctx* ctx) {
    return ctx ? ctx->err.c_str() : g_err.c_str();
}

}  // extern "C"
