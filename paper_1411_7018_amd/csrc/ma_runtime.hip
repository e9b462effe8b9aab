// Host runtime behind the C ABI of include/ma.h: parameter checks, hierarchy
// allocation, the component entry points (single-grid kernels) and the
// solve driver.  Full solves run through the batched engine (a single solve
// is a batch of one), following Algorithm 1 repeated under the stopping rule
// of Section 4 after the Poisson initial guess.
#include "ma.h"
#include "ma_engine.h"
#include "ma_internal.h"
#include "ma_runtime.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <functional>
#include <string>
#include <utility>
#include <vector>

using namespace mafas;

namespace {

thread_local std::string g_create_error;

bool valid_params(const ma_params *p, std::string &why)
{
    if (!p) {
        why = "params is NULL";
        return false;
    }
    if (p->n < 2 || p->n > 2048) {
        why = "n must satisfy 2 <= n <= 2048";
        return false;
    }
    if (p->nu1 < 0 || p->nu2 < 0 || p->nu0 < 1 || p->nu1 > 16 || p->nu2 > 16 || p->nu0 > 16) {
        why = "smoothing counts must satisfy 0 <= nu1, nu2 <= 16 and 1 <= nu0 <= 16";
        return false;
    }
    if (p->order != MA_COLOR4 && p->order != MA_COLOR8) {
        why = "order must be MA_COLOR4 or MA_COLOR8";
        return false;
    }
    if (p->restriction != MA_RESTRICT_FULL && p->restriction != MA_RESTRICT_HALF) {
        why = "restriction must be MA_RESTRICT_FULL or MA_RESTRICT_HALF";
        return false;
    }
    if (p->precision != MA_FP64 && p->precision != MA_MIXED) {
        why = "precision must be MA_FP64 or MA_MIXED";
        return false;
    }
    if (p->smoother < MA_SMOOTHER_AUTO || p->smoother > MA_SMOOTHER_FUSED) {
        why = "unknown smoother";
        return false;
    }
    if (p->tile_config < 0 || p->tile_config > bsweep_num_configs() || p->block_n < -1 ||
        p->block_n > 2048) {
        why = "tile_config must be in 0..12 and block_n in -1..2048";
        return false;
    }
    if (p->max_cycles < 0 || p->init_max_cycles < 0 || p->inner_cycles < 1 ||
        p->inner_cycles > 16) {
        why = "cycle counts must be >= 0 and 1 <= inner_cycles <= 16";
        return false;
    }
    if (p->coarse_n < 0 || p->coarse_n > kCoarseMax) {
        why = "coarse_n must be in 0..32";
        return false;
    }
    if (p->max_blocks < 0 || p->max_blocks % 8 != 0 || p->max_blocks > (1 << 20)) {
        why = "max_blocks must be 0 or a multiple of 8 up to 2^20";
        return false;
    }
    if (p->strip_rows < 0 || p->strip_rows > 4096) {
        why = "strip_rows must be in 0..4096";
        return false;
    }
    if (p->zsweep_n < -1 || p->zsweep_n > 2048) {
        why = "zsweep_n must be in -1..2048";
        return false;
    }
    if (p->fuse_prolong != 0 && p->fuse_prolong != -1) {
        why = "fuse_prolong must be 0 or -1";
        return false;
    }
    if (p->graphs != 0 && p->graphs != 1) {
        why = "graphs must be 0 or 1";
        return false;
    }
    if (!std::isfinite(p->tol) || !std::isfinite(p->init_tol)) {
        why = "tolerances must be finite";
        return false;
    }
    return true;
}

// Workspace of gs_steps (none: gs_solve sweeps and tests one by one).  A
// sweep with its test, gs_steps against one by one, in us: 4 colours, n = 32:
// 12 / 33, 64: 17 / 37, 96: 38 / 49, 128: 67 / 68; 8 colours, n = 32: 12 / 53,
// 64: 19 / 53, 96: 71 / 58.
size_t gs_doubles(const ma_params *p)
{
    if (p->n > (p->order == MA_COLOR4 ? 96 : 80) || p->smoother == MA_SMOOTHER_COLOR)
        return 0;
    return 2 * size_t(gs_blocks(p->order, p->n)) + 2 * kGsBatch + 3;
}

} // namespace

// the message ma_last_error(NULL) returns, for calls that have no solver
void mafas::set_global_error(const std::string &why) { g_create_error = why; }

double mafas::now_seconds()
{
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

// ---------------------------------------------------------------------------
// Hierarchy layout (FP64, (n_l+1)^3 each):
//   level 0: r (residual), R (Poisson right-hand side), t (block-sweep target),
//            fs (colour-ordered right-hand side, FP64 4-colour solvers);
//   level l >= 1: u, b, w, r, t.
// Plus the single-grid norm partials, the batch-of-one engine's partials and
// lists, and the MA_MIXED FP32 hierarchy.
// ---------------------------------------------------------------------------
size_t mafas::hierarchy_bytes(const ma_params *p)
{
    int ns[32];
    const int L = ma_levels(p->n, ns, 32);
    size_t b = 0;
    for (int l = 0; l < L; ++l) {
        const size_t c = npts(ns[l]) * sizeof(double);
        b += (l == 0) ? 3 * c : 5 * c;
    }
    if (p->order == MA_COLOR4 && p->precision == MA_FP64 && p->n >= 2)
        b += size_t(4 * fs_colour_count(p->n)) * sizeof(double);
    b += (residual_partials(p->n) + gs_doubles(p)) * sizeof(double);
    const size_t rows = size_t((p->n - 1 + 63) / 64) * size_t(p->n - 1) * size_t(p->n - 1);
    b += rows * sizeof(double) + (64 << 10) + 4096;
    if (p->precision == MA_MIXED)
        b += mixed_bytes(p);
    return b;
}

extern "C" {

void ma_params_default(ma_params *p, int n)
{
    std::memset(p, 0, sizeof(*p));
    p->n = n;
    p->nu1 = 2;
    p->nu2 = 2;
    p->nu0 = 1;
    p->order = MA_COLOR4;
    p->restriction = MA_RESTRICT_FULL;
    p->precision = MA_FP64;
    p->smoother = MA_SMOOTHER_AUTO;
    p->max_cycles = 100;
    p->tol = 1e-8;
    p->init_tol = 1e-6;
    p->init_max_cycles = 30;
    p->inner_cycles = 2;
    p->graphs = 1;
    p->coarse_n = 16;
    p->max_blocks = 0;
}

int ma_levels(int n, int *ns, int cap)
{
    int L = 0;
    if (n < 2 || cap < 1 || !ns)
        return 0;
    ns[L++] = n;
    while (n % 2 == 0 && n >= 4 && L < cap) {
        n /= 2;
        ns[L++] = n;
    }
    return L;
}

size_t ma_footprint_bytes(const ma_params *p)
{
    std::string why;
    if (!valid_params(p, why))
        return 0;
    return hierarchy_bytes(p);
}

ma_status ma_create(const ma_params *p, void *hip_stream, ma_solver **out)
{
    std::string why;
    if (!out) {
        g_create_error = "out is NULL";
        return MA_ERR_ARG;
    }
    *out = nullptr;
    if (!valid_params(p, why)) {
        g_create_error = why;
        return MA_ERR_ARG;
    }
    ma_solver *s = new ma_solver();
    s->p = *p;
    s->stream = static_cast<hipStream_t>(hip_stream);
    const ma_status st = s->allocate();
    if (st != MA_OK) {
        g_create_error = s->err;
        delete s;
        return st;
    }
    *out = s;
    return MA_OK;
}

void ma_destroy(ma_solver *s) { delete s; }

const char *ma_last_error(const ma_solver *s)
{
    return s ? s->err.c_str() : g_create_error.c_str();
}

ma_status ma_set_stream(ma_solver *s, void *hip_stream)
{
    if (!s)
        return MA_ERR_ARG;
    s->stream = static_cast<hipStream_t>(hip_stream);
    return MA_OK;
}

ma_status ma_retune(ma_solver *s, int coarse_n, int max_blocks, int strip_rows, int block_n)
{
    if (!s)
        return MA_ERR_ARG;
    ma_params q = s->p;
    q.coarse_n = coarse_n;
    q.max_blocks = max_blocks;
    q.strip_rows = strip_rows;
    q.block_n = block_n;
    std::string why;
    if (!valid_params(&q, why))
        return s->fail(MA_ERR_ARG, why);
    s->p = q;
    return MA_OK;
}

ma_status ma_retune_smoother(ma_solver *s, int block_n, int zsweep_n, int tile_config)
{
    if (!s)
        return MA_ERR_ARG;
    ma_params q = s->p;
    q.block_n = block_n;
    q.zsweep_n = zsweep_n;
    q.tile_config = tile_config;
    std::string why;
    if (!valid_params(&q, why))
        return s->fail(MA_ERR_ARG, why);
    s->p = q;
    return MA_OK;
}

ma_status ma_solve(ma_solver *s, double *u, const double *f, double tol, unsigned flags,
                   ma_report *rep)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    if ((flags & MA_INIT_POISSON) && (flags & MA_INIT_FMG))
        return s->fail(MA_ERR_ARG, "MA_INIT_POISSON and MA_INIT_FMG exclude each other");
    SolveState st;
    st.tol = tol > 0.0 ? tol : s->p.tol;
    st.phase = (flags & MA_INIT_POISSON) ? SolveState::INIT0 : SolveState::MAIN0;
    st.t0 = now_seconds();
    std::memset(&st.rep, 0, sizeof(st.rep));
    if (flags & MA_INIT_FMG)
        MA_TRY(fmg_start(s, u, f, st));
    Engine *E = nullptr;
    MA_TRY(s->own_engine(&E, u, f));
    if (E->reset_counters(0) != MA_OK)
        return s->fail(MA_ERR_DEVICE, E->error());
    std::vector<SolveState *> states{&st};
    while (st.phase != SolveState::DONE) {
        if (drive_step(*E, states, false, true) != MA_OK)
            return s->fail(MA_ERR_DEVICE, E->error());
    }
    std::vector<unsigned long long> nc, fb;
    if (E->read_counters(nc, fb) == MA_OK) {
        st.rep.nonconvex = (long long)nc[0] + st.fmg_nonconvex;
        st.rep.fp64_fallbacks = (long long)fb[0];
    }
    if (s->p.profile) {
        int launches = 0;
        E->take_profile(&st.rep.smooth_seconds, &launches, &st.rep.smooth_bytes);
        st.rep.smooth_launches = launches;
    }
    st.rep.seconds = now_seconds() - st.t0;
    if (rep)
        *rep = st.rep;
    if (st.status != MA_OK)
        return s->fail(st.status, st.err);
    return MA_OK;
}

ma_status ma_vcycle(ma_solver *s, double *u, const double *f)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    if (s->p.precision == MA_MIXED)
        return s->fail(MA_ERR_ARG, "ma_vcycle runs FP64 cycles; MA_MIXED solvers use ma_solve");
    Engine *E = nullptr;
    MA_TRY(s->own_engine(&E, u, f));
    std::vector<double> norms;
    if (E->tick(Engine::MODE_MA, std::vector<char>{1}, norms) != MA_OK)
        return s->fail(MA_ERR_DEVICE, E->error());
    return MA_OK;
}

ma_status ma_residual(ma_solver *s, const double *u, const double *f, double *r_or_null,
                      double *l2_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    MA_HIP(s, launch_residual(s->stream, OP_MA, s->p.n, u, f, r_or_null, s->partials));
    if (l2_host) {
        double l2;
        MA_TRY(s->finish_norm(s->p.n, &l2));
        *l2_host = l2;
    }
    return MA_OK;
}

ma_status ma_sweep(ma_solver *s, double *u, const double *f, int count, long long *nonconvex_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f || count < 0)
        return s->fail(MA_ERR_ARG, "u, f must be device pointers and count >= 0");
    MA_HIP(s, launch_fill_u64(s->stream, 1, 0ull, s->dcount));
    MA_TRY(s->smooth(0, u, f, count, OP_MA));
    if (nonconvex_host) {
        MA_HIP(s, hipMemcpyAsync(s->hpin_u64, s->dcount, sizeof(unsigned long long),
                                 hipMemcpyDeviceToHost, s->stream));
        MA_HIP(s, hipStreamSynchronize(s->stream));
        *nonconvex_host = (long long)s->hpin_u64[0];
    }
    return MA_OK;
}

ma_status ma_restrict(ma_solver *s, const double *u, const double *f, double *w_c, double *b_c)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f || !w_c || !b_c)
        return s->fail(MA_ERR_ARG, "null device pointer");
    if (s->lv.size() < 2)
        return s->fail(MA_ERR_ARG, "n must be even and >= 4 for a coarser level");
    const int n = s->p.n;
    // One launch reads f and writes the coarse arrays, in no order between
    // its blocks: outputs laid over f get it from a copy.
    const double *f_end = f + npts(n);
    auto over_f = [&](const double *o) { return o < f_end && f < o + npts(n / 2); };
    if (over_f(w_c) || over_f(b_c)) {
        s->tick_state = 0;
        MA_HIP(s, launch_copy(s->stream, npts(n), f, s->lv[0].r));
        f = s->lv[0].r;
    }
    MA_HIP(s, launch_restrict(s->stream, s->rmode(), n, u, f, w_c, s->lv[1].u, b_c));
    return MA_OK;
}

ma_status ma_prolong_correct(ma_solver *s, double *u, const double *u_c, const double *w_c)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !u_c || !w_c)
        return s->fail(MA_ERR_ARG, "null device pointer");
    if (s->p.n % 2 || s->p.n < 4)
        return s->fail(MA_ERR_ARG, "n must be even and >= 4");
    MA_HIP(s, launch_prolong(s->stream, s->p.n, u, u_c, w_c));
    return MA_OK;
}

ma_status ma_gs_solve(ma_solver *s, double *u, const double *f, double tol, int max_sweeps,
                      ma_report *rep)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f || max_sweeps < 0)
        return s->fail(MA_ERR_ARG, "u, f must be device pointers and max_sweeps >= 0");
    const double t0 = now_seconds();
    const int n = s->p.n;
    const double target = tol > 0.0 ? tol : s->p.tol;
    ma_report r;
    std::memset(&r, 0, sizeof(r));
    auto norm = [&](double *l2) -> ma_status {
        MA_HIP(s, launch_residual(s->stream, OP_MA, n, u, f, nullptr, s->partials));
        return s->finish_norm(n, l2);
    };
    MA_TRY(norm(&r.res0));
    r.res = r.res0;
    ma_status st = MA_ERR_NOT_CONVERGED;
    // the stopping test after sweep q of residual res; true: stop
    auto test = [&](int q, double res) {
        r.cycles = q;
        r.res = res;
        if (q <= 64)
            r.history[q - 1] = res;
        if (!std::isfinite(res))
            st = MA_ERR_NONFINITE;
        else if (res <= target * r.res0)
            st = MA_OK;
        return st != MA_ERR_NOT_CONVERGED;
    };
    if (!std::isfinite(r.res0)) {
        st = MA_ERR_NONFINITE;
    } else if (r.res0 == 0.0) {
        st = MA_OK;
    } else if (s->gs_work) {
        MA_TRY(s->gs_steps(u, f, max_sweeps, sum_threshold(target * r.res0, n), test, &r.nonconvex));
    } else {
        MA_HIP(s, launch_fill_u64(s->stream, 1, 0ull, s->dcount));
        for (int q = 1; q <= max_sweeps; ++q) {
            MA_TRY(s->smooth(0, u, f, 1, OP_MA));
            double res;
            MA_TRY(norm(&res));
            if (test(q, res))
                break;
        }
        MA_HIP(s, hipMemcpyAsync(s->hpin_u64, s->dcount, sizeof(unsigned long long),
                                 hipMemcpyDeviceToHost, s->stream));
        MA_HIP(s, hipStreamSynchronize(s->stream));
        r.nonconvex = (long long)s->hpin_u64[0];
    }
    r.point_updates = double(r.cycles) * interior(n);
    r.alg_bytes = 40.0 * r.point_updates;   // sweep 24, residual check 16
    r.rel_res = r.res0 > 0.0 ? r.res / r.res0 : 0.0;
    r.converged = st == MA_OK;
    r.seconds = now_seconds() - t0;
    if (rep)
        *rep = r;
    if (st == MA_ERR_NOT_CONVERGED)
        return s->fail(st, "max_sweeps reached before the tolerance");
    if (st == MA_ERR_NONFINITE)
        return s->fail(st, "residual is not finite");
    return MA_OK;
}

ma_status ma_fmg(ma_solver *s, double *u, const double *f, long long *nonconvex_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    long long nc = 0;
    MA_TRY(s->fmg(u, f, &nc, nullptr, nullptr));
    if (nonconvex_host)
        *nonconvex_host = nc;
    return MA_OK;
}

ma_status ma_poisson_init(ma_solver *s, double *u, const double *f, int *cycles_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    Engine *E = nullptr;
    MA_TRY(s->own_engine(&E, u, f));
    SolveState st;
    st.phase = SolveState::INIT0;
    std::memset(&st.rep, 0, sizeof(st.rep));
    std::vector<SolveState *> states{&st};
    // drive the Poisson phases only: stop once the solve would start its
    // main phase (the residual of the guess is not needed here)
    while (st.phase == SolveState::INIT0 || st.phase == SolveState::INIT) {
        if (drive_step(*E, states, true) != MA_OK)
            return s->fail(MA_ERR_DEVICE, E->error());
    }
    if (st.status != MA_OK)
        return s->fail(st.status, st.err);
    if (cycles_host)
        *cycles_host = st.rep.init_cycles;
    return MA_OK;
}

} // extern "C"

// ---------------------------------------------------------------------------
// ma_solver methods
// ---------------------------------------------------------------------------
ma_solver::~ma_solver()
{
    delete eng;
    for (double *q : owned)
        (void)hipFree(q);
    if (hpin)
        (void)hipHostFree(hpin);
    if (hpin_u64)
        (void)hipHostFree(hpin_u64);
    mixed_release();
}

ma_status ma_solver::fail(ma_status st, const std::string &msg)
{
    err = msg;
    return st;
}

ma_status ma_solver::alloc(double **q, size_t count)
{
    *q = nullptr;
    if (count == 0)
        return MA_OK;
    const hipError_t e = hipMalloc(reinterpret_cast<void **>(q), count * sizeof(double));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *q = nullptr;
        return fail(e == hipErrorOutOfMemory ? MA_ERR_OOM : MA_ERR_DEVICE,
                    std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    owned.push_back(*q);
    const hipError_t z = launch_fill(stream, count, 0.0, *q);
    if (z != hipSuccess)
        return fail(MA_ERR_DEVICE, std::string("fill: ") + hipGetErrorString(z));
    return MA_OK;
}

ma_status ma_solver::allocate()
{
    int ns[32];
    const int L = ma_levels(p.n, ns, 32);
    lv.resize(L);
    for (int l = 0; l < L; ++l) {
        Level &v = lv[l];
        v.n = ns[l];
        const size_t c = npts(v.n);
        if (l == 0) {
            MA_TRY(alloc(&v.r, c));
            MA_TRY(alloc(&R, c));
            MA_TRY(alloc(&v.t, c));
            if (p.order == MA_COLOR4 && p.precision == MA_FP64 && v.n >= 2) {
                fs_cs = fs_colour_count(v.n);
                MA_TRY(alloc(&fs, size_t(4 * fs_cs)));
            }
        } else {
            MA_TRY(alloc(&v.u, c));
            MA_TRY(alloc(&v.b, c));
            MA_TRY(alloc(&v.w, c));
            MA_TRY(alloc(&v.r, c));
            MA_TRY(alloc(&v.t, c));
        }
    }
    MA_TRY(alloc(&partials, residual_partials(p.n)));
    MA_TRY(alloc(&dsum, 4));
    MA_TRY(alloc(&gs_work, gs_doubles(&p)));
    {
        const hipError_t e = hipMalloc(reinterpret_cast<void **>(&dcount), 64);
        if (e != hipSuccess)
            return fail(MA_ERR_OOM, std::string("hipMalloc: ") + hipGetErrorString(e));
        owned.push_back(reinterpret_cast<double *>(dcount));
    }
    if (hipHostMalloc(reinterpret_cast<void **>(&hpin), (2 * kGsBatch + 2) * sizeof(double)) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void **>(&hpin_u64), 4 * sizeof(unsigned long long)) !=
            hipSuccess ||
        hipHostGetDevicePointer(reinterpret_cast<void **>(&hpin_dev), hpin, 0) != hipSuccess)
        return fail(MA_ERR_OOM, "hipHostMalloc failed");
    if (p.precision == MA_MIXED)
        MA_TRY(mixed_allocate());
    const hipError_t e = hipStreamSynchronize(stream);
    if (e != hipSuccess)
        return fail(MA_ERR_DEVICE, std::string("allocate: ") + hipGetErrorString(e));
    return MA_OK;
}

int ma_solver::rmode() const { return p.restriction == MA_RESTRICT_HALF ? 1 : 0; }

// Shape (launch_bsweep_one) of single-grid sweeps of an n grid, -1 for the
// automatic block shape; false: one launch per colour phase.  One launch per
// sweep where the engine's levels take it: block sweeps up to block_limit
// and, with 4 colours, z-stream sweeps from zsweep_n on; in between the colour
// phases are faster.
bool ma_solver::sweep_shape(int n, int *cfg) const
{
    *cfg = -1;
    if (p.smoother == MA_SMOOTHER_COLOR)
        return false;
    if (p.smoother == MA_SMOOTHER_FUSED && n <= kBlockMaxN) {
        *cfg = p.order == MA_COLOR4 ? p.tile_config - 1 : n >= kGroupN ? kGroupConfig8 : -1;
        return true;
    }
    const int zn = p.zsweep_n != 0 ? p.zsweep_n : kZsweepAuto;
    if (p.order == MA_COLOR4 && zn > 0 && n >= zn) {
        *cfg = p.tile_config > kZsFirstConfig ? p.tile_config - 1 : bsweep_zs_pick(n);
        return true;
    }
    if (p.order == MA_COLOR4 && p.tile_config > 0 && p.tile_config <= kZsFirstConfig)
        *cfg = p.tile_config - 1;
    const bool block = n <= block_limit(p.order, p.block_n);
    if (p.order != MA_COLOR4 && n >= kGroupN && (block || group_level(p.order, p.block_n, n, kGroupSweepN))) {
        *cfg = kGroupConfig8;
        return true;
    }
    return block;
}

// Whether a lone one-launch sweep of shape cfg, which ends in t and is copied
// back to u, takes less than its colour launches (8-colour halves go u -> t ->
// u).  us, 4 colours n = 48: 13.0 / 14.9, 56 (more blocks of 8^3 than compute
// units): 16.2 / 15.5, 64: 17.5 / 16.5; 8 colours n = 80: 25 / 27, 88: 34 / 29.
bool ma_solver::alone_pays(int n, int cfg) const
{
    if (p.order != MA_COLOR4)
        return cfg == kGroupConfig8 || n <= 80;
    return bsweep_is_zstream(0, cfg) ? bsweep_zs_alone(n) : n <= 49;
}

// count single-grid sweeps of op on level l; the result ends in u: one-launch
// sweeps go u -> t -> u, and an odd last one is copied back or runs per colour.
ma_status ma_solver::smooth(int l, double *u, const double *F, int count, int op)
{
    const int n = lv[l].n;
    int cfg, whole = 0;   // sweeps in one launch
    if (sweep_shape(n, &cfg))
        whole = alone_pays(n, cfg) ? count : count / 2 * 2;
    if (whole > 0)
        tick_state = 0;
    double *a = u, *b = lv[l].t;
    for (int k = 0; k < whole; ++k) {
        MA_HIP(this, launch_bsweep_one(stream, op, p.order, cfg, n, a, b, F, dcount));
        if (p.order != MA_COLOR4 && cfg == kGroupConfig8)
            MA_HIP(this, launch_bsweep_one(stream, op, p.order, cfg + 1, n, b, a, F, dcount));
        else
            std::swap(a, b);
    }
    if (a != u)
        MA_HIP(this, launch_copy(stream, npts(n), a, u));
    for (int k = whole; k < count; ++k)
        MA_HIP(this, launch_sweep_color(stream, op, p.order, n, u, F, dcount));
    return MA_OK;
}

// The standalone Gauss-Seidel iteration on u by launches of k_gs_step (one
// sweep each, GsStep in ma_fsweep.h), in batches with a look at the sums behind
// each.  Launches chain from iterate base, in x[0]: launch e takes iterate base + e,
// in x[e & 1], to the next and tests iterate base + e - 1, so a look knows all but
// the chain's last two iterates.  A batch that closes the chain takes their sums
// too, and a new one starts from its last iterate.  test(q, residual) is the host's
// test of iterate q, the same on the same sum (thr: sum_threshold), so both stop at
// the same iterate; *nonconvex counts the sweeps up to it.
//
// Where the batches end: a look costs 20 to 25 us, a launch queued behind the
// iterate a solve stops at still loads its block (3.5 us at n = 32, 11 at 96), and
// a sweep looked at by itself 30 to 50.  So the first batch is what costs about
// as much as one such look (from n = 77, 8 colours 73, on eight lone sweeps, as colour
// launches: k_gs_step takes a residual that a lone sweep has no use for), the next
// ones double, and from 32 sweeps on the waste is bounded by a batch of 32.  us a
// solve, every sweep looked at / batches of 32 throughout / so: 4 colours n = 32, 1
// sweep 87 / 183 / 97, 5: 208 / 203 / 185, 20: 661 / 271 / 302, 888: 26130 / 7990 /
// 7855; n = 64, 2: 116 / 251 / 130, 8: 328 / 317 / 287, 60: 2090 / 1016 / 1067; n =
// 84 (lone sweeps by k_gs_step in batches of 1, 2, 5 ..: 3: 263, 8: 499), 3: 195 /
// 495 / 161, 8: 430 / 586 / 364; n = 96, 3: 215 / 567 / 182, 40: 2081 / 1788 / 1840.
ma_status ma_solver::gs_steps(double *u, const double *F, int max_sweeps, double thr,
                              const std::function<bool(int, double)> &test, long long *nonconvex)
{
    const int n = p.n, blocks = gs_blocks(p.order, n);
    const bool colours = n > (p.order == MA_COLOR4 ? 76 : 72);
    const double h = 1.0 / double(n);
    // block sums of two iterates; a batch's counts and, behind them, its sums
    double *part[2] = {gs_work, gs_work + blocks}, *res = gs_work + 2 * blocks;
    unsigned long long *counts = reinterpret_cast<unsigned long long *>(res);
    int *stop = reinterpret_cast<int *>(res + 2 * kGsBatch + 2);
    double *x[2] = {u, lv[0].t};
    tick_state = 0;
    MA_HIP(this, launch_fill(stream, 2 * kGsBatch + 3, 0.0, res));
    *nonconvex = 0;
    static constexpr int kEnds[4][5] = {{4, 16, 32}, {2, 8, 16, 32}, {1, 3, 8, 16, 32}, {8, 12, 20, 32}};
    const auto &ends = kEnds[colours ? 3 : n > 56 ? 2 : n > 40 ? 1 : 0];
    auto batch_end = [&](int q) {   // of the batch that starts after q sweeps
        if (colours && q < 8)
            return q + 1;
        for (int e : ends)
            if (e > q)
                return e;
        return q + kGsBatch;
    };
    int base = 0, done = 0, tested = 0;   // launches since base; iterates tested
    std::vector<unsigned long long> pending;   // counts of the sweeps not tested
    bool stopped = false;
    while (!stopped && base + done < max_sweeps) {
        const int q0 = base + done;
        const int m = std::min(batch_end(q0), max_sweeps) - q0;
        const bool close = q0 == 0 || m < 3 || q0 + m == max_sweeps;
        const bool here = m == 1 && done == 0 && colours;   // a lone sweep, in x[0]
        double *sums = res + m;
        if (here)
            MA_HIP(this, launch_sweep_color(stream, OP_MA, p.order, n, x[0], F, counts));
        for (int b = 0; b < m && !here; ++b) {
            const int e = done + b;
            MA_HIP(this, launch_gs_step(stream, p.order, n, x[e & 1], x[1 - (e & 1)], F,
                                        e >= 2 ? part[1 - (e & 1)] : nullptr, part[e & 1],
                                        sums + b, counts + b, stop, base + e + 1, thr));
        }
        const int before = done;
        done += m;
        if (close) {
            if (done >= 2)   // the block sums of iterate base + done - 1 are there
                MA_HIP(this, launch_reduce(stream, part[1 - (done & 1)], blocks, sums + m));
            MA_HIP(this, launch_residual(stream, OP_MA, n, x[here ? 0 : done & 1], F, nullptr,
                                         partials));
            MA_HIP(this, launch_reduce(stream, partials, residual_partials(n), sums + m + 1));
        }
        MA_HIP(this, launch_take(stream, 2 * m + 2, res, hpin_dev));
        MA_HIP(this, hipStreamSynchronize(stream));
        for (int b = 0; b < m; ++b) {
            unsigned long long c;
            std::memcpy(&c, hpin + b, sizeof(c));
            pending.push_back(c);
        }
        const int last = base + (close ? done : done - 2);   // iterates whose sums are there
        size_t k = 0;
        while (!stopped && tested < last) {
            ++tested;
            *nonconvex += (long long)pending[k++];
            stopped = test(tested, std::sqrt(hpin[m + tested - base + 1 - before] * h * h * h));
        }
        pending.erase(pending.begin(), pending.begin() + k);
        if (close || stopped) {
            if (!here && ((tested - base) & 1))
                std::swap(x[0], x[1]);
            base = tested;
            done = 0;
        }
    }
    if (x[0] != u)
        MA_HIP(this, launch_copy(stream, npts(n), x[0], u));
    return MA_OK;
}

// partials of an n grid -> host l2 = sqrt(h^3 sum r^2) (synchronises).
ma_status ma_solver::finish_norm(int n, double *l2)
{
    MA_HIP(this, launch_reduce(stream, partials, residual_partials(n), dsum));
    return read_norm(n, l2);
}

// the same of a sum in dsum
ma_status ma_solver::read_norm(int n, double *l2)
{
    MA_HIP(this, hipMemcpyAsync(hpin, dsum, sizeof(double), hipMemcpyDeviceToHost, stream));
    MA_HIP(this, hipStreamSynchronize(stream));
    const double h = 1.0 / double(n);
    *l2 = std::sqrt(hpin[0] * h * h * h);
    return MA_OK;
}

ma_status ma_solver::own_engine(Engine **out, double *u, const double *f)
{
    if (!eng)
        eng = new Engine();
    tick_state = 0;
    std::vector<SolveRef> refs(1);
    refs[0].s = this;
    refs[0].u = u;
    refs[0].f = f;
    if (eng->set(refs, stream, p.graphs != 0, p.profile != 0) != MA_OK)
        return fail(MA_ERR_DEVICE, eng->error());
    *out = eng;
    return MA_OK;
}

// Algorithm 2 unrolled: inject f (b_H := injection of b_h) and the
// Dirichlet data of u down the hierarchy; on the coarsest grid start from
// zero and sweep nu0 times; then on the way up interpolate (cubic FMG
// interpolation) and run one FAS V-cycle per level.  All of it is queued on the
// engine's stream, which the host waits for once: with a norm and the counters
// of every level fetched on the way, the seven levels of 129^3 spent 300 of
// their 1370 us on what nobody used.
ma_status ma_solver::fmg(double *u, const double *f, long long *nonconvex, double *updates,
                         double *bytes)
{
    Engine *E = nullptr;
    MA_TRY(own_engine(&E, u, f));
    const hipStream_t user = stream;
    hipStream_t st = nullptr;
    if (E->begin_cycles(&st) != MA_OK)
        return fail(MA_ERR_DEVICE, E->error());
    long long nc = 0;
    double up = 0.0, by = 0.0;
    stream = st;
    const ma_status r = fmg_queued(*E, u, f, &nc, &up, &by);
    stream = user;
    // also after a failure: what was queued is done before the arrays go on
    const hipError_t e = hipStreamSynchronize(st);
    MA_TRY(r);
    MA_HIP(this, e);
    if (nonconvex)
        *nonconvex += nc + (long long)hpin_u64[0];
    if (updates)
        *updates += up;
    if (bytes)
        *bytes += by;
    return MA_OK;
}

// The same on this->stream, the engine's; leaves the count of the levels that
// no profiled tick counted (nc) in hpin_u64[0] once the stream has run.
ma_status ma_solver::fmg_queued(Engine &E, double *u, const double *f, long long *nc, double *up,
                                double *by)
{
    const int L = int(lv.size());
    auto U = [&](int l) { return l == 0 ? u : lv[l].u; };
    InjectLevels in;
    in.u0 = u;
    in.f0 = f;
    in.n0 = p.n;
    in.levels = L - 1;
    if (L - 1 > int(sizeof(in.u) / sizeof(in.u[0])))
        return fail(MA_ERR_ARG, "too many levels");
    for (int l = 1; l < L; ++l) {
        in.u[l - 1] = lv[l].u;
        in.f[l - 1] = lv[l].b;
    }
    MA_HIP(this, launch_inject_levels(stream, in));
    // coarsest grid: zero inside, then an approximate solve -- nu0 sweeps
    // solve a one-unknown grid exactly; a 3-interval grid (8 unknowns)
    // takes 8 sweeps
    const int c = L - 1;
    const int csweeps = (lv[c].n == 3 && p.nu0 < 8) ? 8 : p.nu0;
    MA_HIP(this, launch_zero_interior(stream, lv[c].n, U(c)));
    MA_HIP(this, launch_fill_u64(stream, 1, 0ull, dcount));
    MA_TRY(smooth(c, U(c), c == 0 ? f : lv[c].b, csweeps, OP_MA));
    *up = double(csweeps) * interior(lv[c].n);
    *by = 24.0 * *up;
    for (int l = L - 2; l >= 0; --l) {
        MA_HIP(this, launch_fmg_interp(stream, lv[l + 1].n, U(l + 1), U(l)));
        if (l == 0 && p.profile) {   // the profiled tick of the finest level
            std::vector<double> nrm;
            std::vector<unsigned long long> cnt, fb;
            if (E.reset_counters(0) != MA_OK || E.tick(Engine::MODE_MA, {1}, nrm) != MA_OK ||
                E.read_counters(cnt, fb) != MA_OK)
                return fail(MA_ERR_DEVICE, E.error());
            *nc += (long long)cnt[0];
        } else if (E.cycle_from(l, dcount) != MA_OK) {
            return fail(MA_ERR_DEVICE, E.error());
        }
        double tu, tb;
        E.tick_cost(Engine::MODE_MA, 0, &tu, &tb, l);
        *up += tu;
        *by += tb;
    }
    MA_HIP(this, hipMemcpyAsync(hpin_u64, dcount, sizeof(unsigned long long),
                                hipMemcpyDeviceToHost, stream));
    return MA_OK;
}

ma_status mafas::fmg_start(ma_solver *s, double *u, const double *f, SolveState &st)
{
    MA_HIP(s, launch_zero_interior(s->stream, s->p.n, u));
    Engine *E = nullptr;
    MA_TRY(s->own_engine(&E, u, f));
    std::vector<double> nrm;
    if (E->norms_only(Engine::MODE_MA, {1}, nrm) != MA_OK)
        return s->fail(MA_ERR_DEVICE, E->error());
    st.rep.res0 = st.rep.res = nrm[0];
    MA_TRY(s->fmg(u, f, &st.fmg_nonconvex, &st.rep.point_updates, &st.rep.alg_bytes));
    st.fmg = true;
    st.phase = SolveState::MAIN0;
    return MA_OK;
}

// ---------------------------------------------------------------------------
// Per-solve phase machine shared by ma_solve, ma_solve_batch and ma_batch.
// ---------------------------------------------------------------------------
ma_status mafas::drive_step(Engine &eng, std::vector<SolveState *> &states, bool init_only,
                            bool ahead)
{
    const int S = int(states.size());
    std::vector<char> act(S, 0);
    std::vector<double> nrm;
    auto finish = [&](SolveState *st, ma_status s, const char *why) {
        st->status = s;
        if (s != MA_OK)
            st->err = why;
        st->phase = SolveState::DONE;
    };
    auto select = [&](SolveState::Phase ph) {
        bool any = false;
        for (int i = 0; i < S; ++i) {
            act[i] = states[i] && states[i]->phase == ph;
            any |= act[i] != 0;
        }
        return any;
    };
    const Engine::Mode main_mode = eng.mixed() ? Engine::MODE_MIXED : Engine::MODE_MA;

    // 1. Poisson right-hand sides and the linear residuals of the start
    if (select(SolveState::INIT0)) {
        for (int i = 0; i < S; ++i)
            if (act[i])
                eng.ref(i).s->tick_state = 0;   // R is formed ahead of the norm
        MA_TRY(eng.norms_only(Engine::MODE_LAP, act, nrm));
        for (int i = 0; i < S; ++i)
            if (act[i]) {
                SolveState *st = states[i];
                st->lin0 = st->last = nrm[i];
                st->prev = 0.0;
                if (!std::isfinite(nrm[i]))
                    finish(st, MA_ERR_NONFINITE, "Poisson initial residual is not finite");
                else if (nrm[i] == 0.0 || eng.ref(i).s->p.init_max_cycles == 0)
                    st->phase = SolveState::MAIN0;
                else
                    st->phase = SolveState::INIT;
            }
    }
    // A tick is queued ahead of the host's stopping test only while every
    // live solve is in the phase being ticked and none can reach its cycle
    // limit at the tick being read: every other reason to stop is one the
    // device sees (the tolerance test and a non-finite norm, on the same sum
    // through sum_threshold), so a solve that stops skips the tick queued
    // after it.
    auto only = [&](SolveState::Phase ph) {
        for (int i = 0; i < S; ++i)
            if (states[i] && states[i]->phase != SolveState::DONE && states[i]->phase != ph)
                return false;
        return true;
    };
    // the host's and the device's stopping decisions on the tick just read
    auto agree = [&](int i, bool host_stop) {
        return eng.halted(i) == host_stop;
    };
    // Whether the tick about to be read will leave solve st above its
    // threshold c, guessed from its contraction so far (a factor of 10 per
    // cycle before two norms are known) with a margin of 8: a tick queued
    // ahead of a solve that then stops is skipped on the device but still
    // costs its launches, while one not queued costs only a host round trip.
    auto goes_on = [](const SolveState *st, double c) {
        const double rho = st->prev > 0.0 ? st->last / st->prev : 0.1;
        return st->last * rho > 8.0 * c;
    };
    // The same guess one tick further: what is queued ahead may be two ticks
    // in one graph (one graph boundary fewer) when the solve is guessed to
    // go on after the tick following the one being read as well.
    auto goes_on2 = [](const SolveState *st, double c) {
        const double rho = st->prev > 0.0 ? st->last / st->prev : 0.1;
        return st->last * rho * rho > 8.0 * c;
    };
    // 2. one linear V-cycle of the Poisson guess
    bool init_ahead = false;
    if (select(SolveState::INIT)) {
        std::vector<double> thr(S, -1.0);
        bool spec = ahead && only(SolveState::INIT);
        bool pair = spec;
        for (int i = 0; i < S; ++i)
            if (act[i]) {
                const ma_params &p = eng.ref(i).s->p;
                const double c = p.init_tol * states[i]->lin0;
                thr[i] = sum_threshold(c, p.n);
                spec &= states[i]->rep.init_cycles + 2 <= p.init_max_cycles &&
                        goes_on(states[i], c);
                pair &= states[i]->rep.init_cycles + 3 <= p.init_max_cycles &&
                        goes_on2(states[i], c);
            }
        MA_TRY(eng.tick_ahead(Engine::MODE_LAP, act, thr, spec, nrm, spec && pair));
        init_ahead = eng.pending() > 0;
        for (int i = 0; i < S; ++i)
            if (act[i]) {
                SolveState *st = states[i];
                const ma_params &p = eng.ref(i).s->p;
                if (!agree(i, !std::isfinite(nrm[i]) || nrm[i] <= p.init_tol * st->lin0))
                    return eng.fail(MA_ERR_DEVICE, "internal: device stopping flag disagrees "
                                                   "with the Poisson stopping test");
                double up, by;
                eng.tick_cost(Engine::MODE_LAP, i, &up, &by);
                st->rep.alg_bytes += by;
                st->rep.init_cycles += 1;
                st->prev = st->last;
                st->last = nrm[i];
                if (!std::isfinite(nrm[i]))
                    finish(st, MA_ERR_NONFINITE, "Poisson residual is not finite");
                else if (nrm[i] <= p.init_tol * st->lin0 ||
                         st->rep.init_cycles >= p.init_max_cycles)
                    st->phase = SolveState::MAIN0;
            }
    }
    // When this step's Poisson tick left one queued ahead, the solves that
    // left the phase start the next one in the next step: a launch for them
    // now would queue behind a tick that other solves have yet to read.  (A
    // queued tick that no solve reads any more is one they all skip; the
    // next launch waits for it.)
    if (init_only || init_ahead)
        return MA_OK;
    // 3. residual of the initial guess (res0 of the stopping rule)
    if (select(SolveState::MAIN0)) {
        MA_TRY(eng.norms_only(main_mode, act, nrm));
        for (int i = 0; i < S; ++i)
            if (act[i]) {
                SolveState *st = states[i];
                const int maxc = eng.ref(i).s->p.max_cycles;
                if (st->fmg) {
                    // the FMG-FAS iteration is the first cycle; res0 is the
                    // residual of the zero-interior start
                    ma_report &r = st->rep;
                    r.cycles = 1;
                    r.outer = eng.mixed() ? 1 : 0;
                    r.res = r.history[0] = nrm[i];
                    st->last = nrm[i];
                    st->prev = 0.0;
                    st->best = r.res0;
                    st->stall = 0;
                    r.rel_res = r.res0 > 0.0 ? r.res / r.res0 : 0.0;
                    if (!std::isfinite(nrm[i]))
                        finish(st, MA_ERR_NONFINITE, "residual after FMG is not finite");
                    else if (r.res <= st->tol * r.res0) {
                        r.converged = 1;
                        finish(st, MA_OK, "");
                    } else if (maxc <= 1) {
                        finish(st, MA_ERR_NOT_CONVERGED, "max_cycles reached before the tolerance");
                    } else {
                        st->phase = SolveState::MAIN;
                    }
                    continue;
                }
                st->rep.res0 = st->rep.res = st->last = nrm[i];
                st->prev = 0.0;
                st->best = nrm[i];
                st->stall = 0;
                if (!std::isfinite(nrm[i]))
                    finish(st, MA_ERR_NONFINITE, "initial residual is not finite");
                else if (nrm[i] == 0.0) {
                    st->rep.converged = 1;
                    finish(st, MA_OK, "");
                } else if (maxc == 0) {
                    finish(st, MA_ERR_NOT_CONVERGED, "max_cycles is 0");
                } else {
                    st->phase = SolveState::MAIN;
                }
            }
    }
    // 4. one V-cycle (FP64) or one outer correction (mixed)
    if (select(SolveState::MAIN)) {
        std::vector<double> thr(S, -1.0);
        bool spec = ahead && only(SolveState::MAIN);
        bool pair = spec;
        for (int i = 0; i < S; ++i)
            if (act[i]) {
                const ma_params &p = eng.ref(i).s->p;
                const ma_report &r = states[i]->rep;
                const double c = states[i]->tol * r.res0;
                thr[i] = sum_threshold(c, p.n);
                const int done = main_mode == Engine::MODE_MIXED ? r.outer : r.cycles;
                // a stall stop is the host's own decision too: no tick ahead
                // of one that could make it
                spec &= done + 2 <= p.max_cycles && goes_on(states[i], c) &&
                        states[i]->stall + 1 < 3;
                pair &= done + 3 <= p.max_cycles && goes_on2(states[i], c) &&
                        states[i]->stall + 2 < 3;
            }
        MA_TRY(eng.tick_ahead(main_mode, act, thr, spec, nrm, spec && pair));
        for (int i = 0; i < S; ++i)
            if (act[i]) {
                SolveState *st = states[i];
                const ma_params &p = eng.ref(i).s->p;
                ma_report &r = st->rep;
                if (!agree(i, !std::isfinite(nrm[i]) || nrm[i] <= st->tol * r.res0))
                    return eng.fail(MA_ERR_DEVICE, "internal: device stopping flag disagrees "
                                                   "with the stopping test");
                double up, by;
                eng.tick_cost(main_mode, i, &up, &by);
                r.point_updates += up;
                r.alg_bytes += by;
                int steps;
                if (main_mode == Engine::MODE_MIXED) {
                    r.cycles += p.inner_cycles;
                    r.outer += 1;
                    steps = r.outer;
                } else {
                    r.cycles += 1;
                    steps = r.cycles;
                }
                if (steps - 1 < 64)
                    r.history[steps - 1] = nrm[i];
                r.res = nrm[i];
                st->prev = st->last;
                st->last = nrm[i];
                r.rel_res = r.res / r.res0;
                const int stalled = r.res < 0.9 * st->best ? 0 : st->stall + 1;
                if (stalled == 0)
                    st->best = r.res;
                st->stall = stalled;
                if (!std::isfinite(r.res)) {
                    finish(st, MA_ERR_NONFINITE, "residual is not finite");
                } else if (r.res <= st->tol * r.res0) {
                    r.converged = 1;
                    finish(st, MA_OK, "");
                } else if (st->stall >= 3) {
                    finish(st, MA_ERR_NOT_CONVERGED,
                           "the residual stagnated above the tolerance (round-off floor)");
                } else if (steps >= p.max_cycles) {
                    finish(st, MA_ERR_NOT_CONVERGED, "max_cycles reached before the tolerance");
                }
            }
    }
    return MA_OK;
}
