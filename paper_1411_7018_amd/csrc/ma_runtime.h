// Solver object behind the opaque ma_solver handle of include/ma.h.
#pragma once

#include "ma.h"
#include "ma_internal.h"

#include <functional>
#include <string>
#include <vector>

#define MA_TRY(expr)                                                                             \
    do {                                                                                         \
        const ma_status st_ = (expr);                                                            \
        if (st_ != MA_OK)                                                                        \
            return st_;                                                                          \
    } while (0)

#define MA_HIP(obj, expr)                                                                        \
    do {                                                                                         \
        const hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                                    \
            return (obj)->fail(MA_ERR_DEVICE,                                                    \
                               std::string(#expr) + ": " + hipGetErrorString(e_));             \
    } while (0)

namespace mafas {

class Engine;

constexpr int kCoarseMax = 32;   // largest coarse_n

struct Level {
    int n = 0;
    double *u = nullptr;   // iterate (coarse levels; level 0 is the caller's array)
    double *b = nullptr;   // right-hand side (coarse levels)
    double *w = nullptr;   // injected fine approximation (coarse levels)
    double *r = nullptr;   // residual
    double *t = nullptr;   // out-of-place target of the block sweep
};

// FP32 inner hierarchy of the mixed-precision form (one per level).
struct MixedLevel {
    int n = 0;
    float *d = nullptr;    // correction delta
    float *b = nullptr;    // right-hand side of T(delta) = b
    float *w = nullptr;    // injected delta
    float *r = nullptr;    // residual of the inner problem (n <= kCoarseMax: k_tail)
    double *U = nullptr;   // injected FP64 approximation (coarse levels)
};

size_t hierarchy_bytes(const ma_params *p);
// Doubles per colour of the colour-ordered right-hand side of an n grid
// (rows of the 4-colour sweep x 64 lanes).
inline long fs_colour_count(int n)
{
    return 64L * colour_items(n, n - 1) * (n / 2);
}
// largest n of a block sweep (its element offsets are 32-bit)
constexpr int kBlockMaxN = 1289;
// Largest n whose sweeps MA_SMOOTHER_AUTO runs as block sweeps (-1: none).
// A sweep of Monge-Ampere, one launch against the colour launches, in us: 4
// colours, n = 64: 11 / 14, 96: 26 / 20, 128: 47 / 31; 8 colours (a block
// recomputes 2.2-2.7 x its updates, with 4 colours 2.9 x, and replaces eight
// launches), n = 32: 9 / 24, 64: 13 / 24, 80: 16 / 27, 88: 22 / 28, 96: 33 / 28, 128:
// 60 / 39.
inline int block_limit(int order, int block_n)
{
    return block_n == 0 ? (order == MA_COLOR4 ? 64 : 88) : block_n < kBlockMaxN ? block_n : kBlockMaxN;
}
// With 8 colours the grids of a depth of up to 64 intervals take colour launches
// when they have more 8^3 tiles together: many small grids fill the chip as one
// large one does, and their 8-wide blocks recompute most.  Six cycles of a batch,
// colour launches / blocks, ms: 2 grids of n = 64 (1024 tiles) 2.48 / 2.11, 3: 2.22
// / 2.46, 16: 4.8 / 7.5; 64 of n = 24 2.7 / 3.6; wider blocks pay: 2 of n = 80
// (2000) 2.58 / 2.18, 2 of n = 88 2.67 / 2.50.
constexpr long kBlockTiles8 = 1200;
// 8-colour sweeps above that limit as two launches of four phases each, from n
// = least on.  In the engine from kGroupN; a V-cycle with them against colour
// launches on those levels, in us: n = 136: 426 / 438, 144: 487 / 493, 160: 552 /
// 602, 192: 804 / 893, 256: 1606 / 1831.  Repeated on one grid, as ma_sweep runs
// them, colour launches find u in the last-level cache and are faster, so there
// from kGroupSweepN; a sweep in us: n = 144: 64 / 51, 160: 73 / 73, 190: 122 / 113,
// 256: 310 / 267, 304: 529 / 470, 320: 584 / 588 (u and F no longer fit that cache,
// and eight launches read u eight times), 384: 853 / 1133.
constexpr int kGroupSweepN = 320;
inline bool group_level(int order, int block_n, int n, int least)
{
    return order != MA_COLOR4 && block_n >= 0 && n >= least && n <= kBlockMaxN;
}
size_t mixed_bytes(const ma_params *p);
// most launches of the Gauss-Seidel iteration between looks at its sums
constexpr int kGsBatch = 32;

hipError_t launch_fill(hipStream_t st, size_t count, double v, double *dst);
hipError_t launch_fill_u64(hipStream_t st, size_t count, unsigned long long v,
                           unsigned long long *dst);

double now_seconds();

// Sets the message ma_last_error(NULL) returns (calls without a solver).
void set_global_error(const std::string &why);

} // namespace mafas

struct ma_solver {
    ma_params p{};
    hipStream_t stream = nullptr;
    std::vector<mafas::Level> lv;
    double *R = nullptr;                  // Poisson right-hand side, finest level
    // The finest right-hand side in the order the 4-colour sweep visits it:
    // colour c, work item q, lane t at fs[c * fs_cs + 64 q + t]
    // (FP64 4-colour solvers; filled by the engine when stale).
    double *fs = nullptr;
    long fs_cs = 0;
    double *partials = nullptr;           // norm partials of the single-grid kernels
    double *dsum = nullptr;
    double *gs_work = nullptr;            // sums and counts of gs_steps (small grids)
    unsigned long long *dcount = nullptr; // counter of the single-grid kernels
    double *hpin = nullptr;               // pinned host scalars
    double *hpin_dev = nullptr;           // the same as kernels see them
    unsigned long long *hpin_u64 = nullptr;
    std::vector<double *> owned;
    std::vector<void *> mixed_owned;
    std::vector<mafas::MixedLevel> mx;
    std::string err;
    mafas::Engine *eng = nullptr;         // batch-of-one engine of ma_solve / ma_vcycle
    // What the scratch arrays carry from one tick of a resident batch to the
    // next is the state of engine tick_state's last tick; 0 once another call
    // has written them (calls on a resident solve's solver may come between its
    // ticks), and the engine forms that state again ahead of its next tick
    // (Engine::restore_state).
    unsigned long long tick_state = 0;
    bool tick_rows = false;   // mixed: the finest level had row kernels then (H formed, b in split rows)

    ~ma_solver();
    ma_status fail(ma_status st, const std::string &msg);
    ma_status alloc(double **q, size_t count);
    ma_status allocate();
    bool sweep_shape(int n, int *cfg) const;
    bool alone_pays(int n, int cfg) const;
    int rmode() const;
    // single-grid kernels behind the component entry points
    ma_status smooth(int l, double *u, const double *F, int count, int op);
    ma_status finish_norm(int n, double *l2);
    ma_status read_norm(int n, double *l2);
    ma_status gs_steps(double *u, const double *F, int max_sweeps, double thr,
                       const std::function<bool(int, double)> &test, long long *nonconvex);
    ma_status own_engine(mafas::Engine **out, double *u, const double *f);
    ma_status fmg_queued(mafas::Engine &E, double *u, const double *f, long long *nc, double *up,
                         double *by);
    // One FMG-FAS iteration (Algorithm 2) on u, whose interior is not read;
    // adds its non-certified updates, point updates and algorithmic bytes.
    ma_status fmg(double *u, const double *f, long long *nonconvex, double *updates,
                  double *bytes);
    // H of a mixed solve's level l, two floats a node each (xx yy, zz xy, xz yz),
    // in FP64 arrays that its inner cycles leave alone.  Level 0's outlives the
    // tick that forms it: a call that writes one of these arrays clears
    // tick_state.
    void *mixed_h(int l, int q) const
    {
        return q == 0 ? lv[l].r : q == 1 ? lv[l].t : l == 0 ? R : lv[l].u;
    }
    ma_status mixed_allocate();
    void mixed_release();
};

namespace mafas {

// Progress of one solve driven tick by tick inside an Engine.
struct SolveState {
    enum Phase { INIT0, INIT, MAIN0, MAIN, DONE };
    Phase phase = MAIN0;
    double tol = 1e-8;
    double lin0 = 0.0;      // linear residual of the Poisson guess's start
    ma_status status = MA_OK;
    std::string err;
    ma_report rep{};
    double t0 = 0.0;        // start time (seconds)
    bool fmg = false;       // started by one FMG-FAS iteration: res0 is the
                            // residual of the zero-interior start, and the
                            // FMG iteration is the first cycle
    long long fmg_nonconvex = 0;
    // the phase's last two norms read (prev 0: only the phase's start is
    // known), for the guess whether the tick being read will stop the solve
    double last = 0.0, prev = 0.0;
    // the main phase's best residual so far and the cycles since it last
    // dropped below 0.9 x that best (three in a row: stagnation)
    double best = 0.0;
    int stall = 0;
};

// The FMG start of a solve (Section 4 protocol): zero the interior of u, take
// r^0 there, run one FMG-FAS iteration; st then continues at MAIN0.
ma_status fmg_start(ma_solver *s, double *u, const double *f, SolveState &st);

// One scheduling step over the engine's slots: the entry residuals of solves
// starting a phase, then one tick of every solve that is cycling (Poisson
// guess, FAS V-cycle or mixed correction).  states[i] may be null (empty
// slot).  Per-solve outcomes land in the states; the return value reports
// engine failures only.
// init_only: stop after the Poisson phases.
// ahead: let the engine queue a tick ahead of the stopping test (a closed
// set of solves: the caller adds or removes none between steps).
ma_status drive_step(Engine &eng, std::vector<SolveState *> &states, bool init_only = false,
                     bool ahead = false);

} // namespace mafas
