// Internal declarations shared by the host runtime and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace mafas {

enum Op { OP_MA = 0, OP_LAP = 1 };

inline size_t npts(int n) { return size_t(n + 1) * size_t(n + 1) * size_t(n + 1); }
// Wavefronts of `rows` rows of one colour, packed (n / 2 nodes a row).
inline int colour_items(int n, int rows) { return int((long(rows) * (n / 2) + 63) / 64); }
// Factor of colour_node's divisions by n / 2.
inline unsigned colour_div(int n) { return unsigned(((1ull << 31) + n / 2 - 1) / (n / 2)); }
// Wavefronts per block of a launch of row items, each on items of its own.  A
// large launch takes four a block, four times fewer blocks to dispatch (4 colours
// n = 160, two sweeps, us: 114 with one, 110 with four; 8 colours n = 272: 636 /
// 620).  A small one takes one: its few blocks spread over more compute units (8
// colours n = 104: 63 with one, 68 with four; 4 colours n = 104: 46.5 / 48.7).
// (The number is a kernel argument: reading it as blockDim.x costs each
// wavefront a load before its first item, 3-5% of those times.)
constexpr int kRowWaves = 4, kManyWaves = 6144;
inline int row_waves(int waves) { return waves > kManyWaves ? kRowWaves : 1; }
inline double interior(int n) { return double(n - 1) * double(n - 1) * double(n - 1); }

// Number of blocks (and partial sums) the residual-norm kernel produces for
// an n grid; the partial buffer must hold at least this many doubles.
size_t residual_partials(int n);

// --- smoother -------------------------------------------------------------
// One sweep of the operator op (MA: nonlinear GS, LAP: linear 7-point GS) on
// u in place, one launch per colour phase.  order 0: 4 colours, 1: 8 colours.
// nonconvex: device counter (may be null) incremented per non-certified update.
hipError_t launch_sweep_color(hipStream_t st, int op, int order, int n, double *u,
                              const double *F, unsigned long long *nonconvex);

// The block sweep (ma_fsweep.h): one sweep, all colour phases in a single
// launch reading u_in and writing u_out; u_out receives the Dirichlet layer
// too.  cfg: shape index of that ordering (< 0: automatic for n; the z-stream
// shapes of the 4-colour ordering among them).  Bitwise equal to
// launch_sweep_color.
hipError_t launch_bsweep_one(hipStream_t st, int op, int order, int cfg, int n,
                             const double *u_in, double *u_out, const double *F,
                             unsigned long long *nonconvex);
// The first of two 8-colour shapes that run half of a sweep's phases each, and
// the least n of a block sweep that takes them (128: 62 us as whole sweeps; 144:
// 64 as halves).
constexpr int kGroupConfig8 = 3;
constexpr int kGroupN = 136;
int bsweep_num_configs();
// Automatic block shape for grids of up to n intervals whose 8^3 tiles number
// tiles8 in all.
int bsweep_pick(int order, int n, long tiles8);
// One step of the standalone Gauss-Seidel iteration (GsStep in ma_fsweep.h);
// part_in / part_out hold gs_blocks doubles.
int gs_blocks(int order, int n);
hipError_t launch_gs_step(hipStream_t st, int order, int n, const double *u_in, double *u_out,
                          const double *F, const double *part_in, double *part_out, double *sum,
                          unsigned long long *count, int *stop, int q, double thr);
// Whether one z-stream sweep of an n grid and the copy back to u take less than
// its colour launches.  The sweep by the chunk model, its steps 1.42 us / 100;
// the copy 3.0 ns a node and the launches 11.5, until u and F no longer fit the
// last-level cache.  us, sweep and copy / launches: n = 192: 90 / 86, 208: 112 /
// 108, 224: 125 / 131, 240: 168 / 161, 256: 200 / 203, 272: 266 / 300.
bool bsweep_zs_alone(int n);
// automatic z-stream shape (config index) of an n grid
int bsweep_zs_pick(int n);

// --- residual and norm ----------------------------------------------------
// r = F - S(u) (0 on the boundary, written; r may be null) and per-block sums
// of r^2 into partials[0..residual_partials(n)).
hipError_t launch_residual(hipStream_t st, int op, int n, const double *u, const double *F,
                           double *r, double *partials);
// out[0] = sum of partials[0..count) in a fixed order (one block).
hipError_t launch_reduce(hipStream_t st, const double *partials, size_t count, double *out);

// --- transfers --------------------------------------------------------------
// Residual and FAS restriction nf -> nf/2 in one launch: wc = uc = injection
// of uf; bc = S_H(wc) + I (F - S(uf)).  rmode 0: full weighting, 1:
// half-weighting.
hipError_t launch_restrict(hipStream_t st, int rmode, int nf, const double *uf, const double *F,
                           double *wc, double *uc, double *bc);
// uf += trilinear(uc - wc) at fine interior nodes.
hipError_t launch_prolong(hipStream_t st, int nf, double *uf, const double *uc,
                          const double *wc);
// R = 3 cbrt(f) at every node.
hipError_t launch_poisson_rhs(hipStream_t st, int n, const double *f, double *R);
// dst = src (count doubles).
hipError_t launch_copy(hipStream_t st, size_t count, const double *src, double *dst);
// src copied to dst (pinned host memory) and cleared
hipError_t launch_take(hipStream_t st, size_t count, double *src, double *dst);
// u0 and f0 of an n0 grid injected onto levels n0 / 2, n0 / 4, ... (levels of
// them; block is set by the launch).
struct InjectLevels {
    const double *u0, *f0;
    double *u[12], *f[12];
    int block[12];
    int levels, n0;
};
hipError_t launch_inject_levels(hipStream_t st, InjectLevels &A);
// Interior of uf (2 nc intervals) = FMG cubic interpolation of uc.
hipError_t launch_fmg_interp(hipStream_t st, int nc, const double *uc, double *uf);
// Interior of u = 0.
hipError_t launch_zero_interior(hipStream_t st, int n, double *u);

} // namespace mafas
