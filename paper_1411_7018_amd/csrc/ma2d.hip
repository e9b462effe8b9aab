// Two-dimensional variant (include/ma2d.h): 9-point nonlinear Gauss-Seidel
// smoother, FAS V-cycle and FMG for u_xx u_yy - u_xy^2 = f.  A V-cycle is two
// launches per level (k2_leg: the sweeps of one leg with the transfer beside
// them) driven from the host, and one for all the levels n <= 64 (k2_tail): a
// 2D grid of the sizes this variant targets (up to 8193^2) fills the chip on
// its own, so no batching is needed.  A lone sweep of a middle grid is a launch
// per phase (k2_phase).
#include "ma2d.h"
#include "ma_device.h"
#include "ma_fsweep.h"
#include "ma_runtime.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

namespace {

constexpr int BX = 64, BY = 4;

// Two nodes side by side.  The compiler takes an elementwise operation as two
// neighbouring instructions, so two updates run as one interleaved sequence;
// written one after the other they stay so, and a phase on a small grid waits
// out two dependent chains of ~45 64-bit operations (1200 against 700 clocks).
using Two = double __attribute__((ext_vector_type(2)));

// Discrete Hessian at a node: second differences as differences of first
// differences, the mixed one over the four diagonal neighbours.
template <typename T>
struct Hes2 {
    T xx, yy, xy;
};
using H2 = Hes2<double>;

template <typename T>
__device__ __forceinline__ Hes2<T> hess2(T c, T w, T e, T s, T n, T sw, T se, T nw, T ne, double k)
{
    Hes2<T> g;
    g.xx = ((e - c) - (c - w)) * k;
    g.yy = ((n - c) - (c - s)) * k;
    g.xy = ((ne - nw) - (se - sw)) * (0.25 * k);
    return g;
}

template <typename T>
__device__ __forceinline__ T det2(const Hes2<T> &g)
{
    return g.xx * g.yy - g.xy * g.xy;
}

// Smaller root of (xx - sigma)(yy - sigma) - xy^2 = F.  With t = tr G and
// D = (xx - yy)^2 + 4 xy^2 + 4 F the roots are (t -+ sqrt D) / 2; for t > 0
// the smaller one is evaluated as 2 (det G - F) / (t + sqrt D), free of
// cancellation.  D < 0 (no real root, F far below zero): the vertex t / 2.
// unconvex: F <= 0 or D < 0.
//
// One node: branches that almost no wavefront takes.  A large grid is bound
// by the instructions it issues (selecting between both forms instead takes
// 15% longer at 8193^2).
__device__ __forceinline__ double root2(const H2 &g, double F, int &unconvex)
{
    const double t = g.xx + g.yy;
    const double a = g.xx - g.yy;
    const double D = a * a + 4.0 * g.xy * g.xy + 4.0 * F;
    unconvex = int(!(F > 0.0) | (D < 0.0));
    if (D < 0.0)
        return 0.5 * t;
    const double r = sqrt(D);
    if (t > 0.0)
        return 2.0 * (det2(g) - F) / (t + r);
    return 0.5 * (t - r);
}

// Two nodes: both forms evaluated and selected, since a branch would split
// the interleaved sequence.
__device__ __forceinline__ Two root2(const Hes2<Two> &g, Two F, int &ua, int &ub)
{
    const Two t = g.xx + g.yy;
    const Two a = g.xx - g.yy;
    const Two D = a * a + 4.0 * g.xy * g.xy + 4.0 * F;
    const Two r = __builtin_elementwise_sqrt(D);
    const Two pos = 2.0 * (det2(g) - F) / (t + r);
    ua = int(!(F.x > 0.0) | (D.x < 0.0));
    ub = int(!(F.y > 0.0) | (D.y < 0.0));
    auto select = [](double t1, double D1, double r1, double pos1) {
        asm("" : "+v"(pos1));   // keeps the selects from becoming branches around it
        const double v = t1 > 0.0 ? pos1 : 0.5 * (t1 - r1);
        return D1 < 0.0 ? 0.5 * t1 : v;
    };
    return Two{select(t.x, D.x, r.x, pos.x), select(t.y, D.y, r.y, pos.y)};
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_down(v, off, 64);
    return v;
}

// Updates a wavefront found not convex, added to the counter once.
__device__ __forceinline__ void count_nonconvex(int mine, unsigned long long *cnt)
{
    if (__builtin_amdgcn_ballot_w64(mine > 0) == 0)
        return;
    for (int off = 32; off > 0; off >>= 1)
        mine += __shfl_down(mine, off, 64);
    if ((threadIdx.x & 63) == 0)
        atomicAdd(cnt, (unsigned long long)mine);
}

// Restricted residual at a coarse interior node from r(dx, dy) around it.
template <typename R>
__device__ __forceinline__ double restricted(R r, bool half)
{
    if (half)
        return (4.0 * r(0, 0) + (r(-1, 0) + r(1, 0)) + (r(0, -1) + r(0, 1))) / 8.0;
    const double w[3] = {0.25, 0.5, 0.25};
    double rh = 0.0;
#pragma unroll
    for (int b = -1; b <= 1; ++b)
#pragma unroll
        for (int a = -1; a <= 1; ++a)
            rh += (w[b + 1] * w[a + 1]) * r(a, b);
    return rh;
}

// 1D rule of the FMG interpolation as four taps at coarse nodes first ..
// first + 3 (a coarse node is copied; a midpoint takes the cubic Lagrange
// value through the 4 nearest coarse nodes, one-sided at the boundary; the
// quadratic value on a 3-node grid, whose fourth tap has weight 0 and is
// never read past the grid).
__device__ __forceinline__ int rule2(int nc, int i, double w[4])
{
    const int m = i >> 1;
    if (nc < 3) {
        w[0] = (i & 1) ? (m == 0 ? 0.375 : -0.125) : (m == 0 ? 1.0 : 0.0);
        w[1] = (i & 1) ? 0.75 : (m == 1 ? 1.0 : 0.0);
        w[2] = (i & 1) ? (m == 0 ? -0.125 : 0.375) : (m == 2 ? 1.0 : 0.0);
        w[3] = 0.0;
        return 0;
    }
    const int first = min(max(m - 1, 0), nc - 3);
    if ((i & 1) == 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
            w[a] = first + a == m ? 1.0 : 0.0;
        return first;
    }
    const bool lo = m == 0, hi = m == nc - 1;
    w[0] = lo ? 0.3125 : hi ? 0.0625 : -0.0625;
    w[1] = lo ? 0.9375 : hi ? -0.3125 : 0.5625;
    w[2] = lo ? -0.3125 : hi ? 0.9375 : 0.5625;
    w[3] = lo ? 0.0625 : hi ? 0.3125 : -0.0625;
    return first;
}

// FMG value at fine node (i, j); uc(I, J) reads the coarse grid.
template <typename U>
__device__ __forceinline__ double fmg_value(U uc, int nc, int i, int j)
{
    double wi[4], wj[4];
    const int fi = rule2(nc, i, wi), fj = rule2(nc, j, wj);
    double v = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int a = 0; a < 4; ++a)
            v += wj[b] * wi[a] * uc(min(fi + a, nc), min(fj + b, nc));
    return v;
}

// ---------------------------------------------------------------------------
// One leg of a V-cycle on one level in one launch: up to two sweeps with the
// work before and after them.  A workgroup owns a TX x TY tile of nodes; it
// loads the tile and a halo into LDS, applies every colour phase there (one
// barrier each, halo nodes recomputed from the values their own tiles start
// from), and writes its tile out of place (neighbouring tiles read the same
// input at the same time).  A leg reads u and F and writes u once for all of
// its phases; a launch per colour phase, with a second one to commit it, moved
// about 150 B a node and sweep and cost 2-4 us each on the coarse levels.
// Section 4 solves, phase launches against legs and the coarse-level kernel:
// 8193^2 red-black 16.9 -> 4.7 ms, 1537^2 4-colour 2.9 -> 0.77 ms, 129^2
// 1.45 -> 0.23 ms.  At 8193^2 a leg takes 0.99-1.11 ms: the ~65 vector
// instructions (55 of them 64-bit) of an update on 1.9 x the nodes keep the
// vector units busy 60% of it, its memory traffic alone would take 0.4 ms, and
// a tile's load and phases overlap only with other tiles', so the wavefronts
// count: within 64 registers (launch bound) 6-8% faster than with 70 (the 32 x 32
// 4-colour legs, which no large grid takes, stay at 70).  From 512^2 down a leg
// takes 7-11 us, mostly the latency of its load, phases and store.
//   IN   LEG_U    the values of uin
//        LEG_PRO  uin plus the bilinear interpolation of uc - wc (the
//                 coarse-grid correction; interior nodes)
//        LEG_FMG  the FMG interpolation of uc inside, uin on the boundary
//   OUT  LEG_RESTRICT  also the FAS restriction of the result: cw = the
//                 injection, cb = det(D^2_H w) + restricted residual (the
//                 coarse u starts from cw: an array of its own, since tiles
//                 of a LEG_FMG launch still read the coarse u)
//        LEG_NORM also the squared residuals of the result, one sum per tile
//
// Halo.  Red-black phases read one node further each in x and y, so after
// two sweeps (4 phases) values 4 nodes inside the loaded tile are right; the
// residual reads one more and the restriction (residuals next to the coarse
// node, u two nodes away) another: 6.  The 4-colour phases come in pairs on
// the same rows: phases 0, 1 update even rows and 2, 3 odd rows, so a sweep
// reads two rows further (two sweeps and the transfer: 4 + 2 = 6) but four
// columns (8 + 2 = 10).
//
// A thread owns a 2 x 2 quad, so it updates two nodes per red-black phase
// and one per 4-colour phase, and keeps their values and F in registers.
// LDS rows hold the even columns, then the odd ones: the nodes of a phase
// are contiguous.
// ---------------------------------------------------------------------------
enum { LEG_U, LEG_PRO, LEG_FMG };
enum { LEG_PLAIN, LEG_RESTRICT, LEG_NORM };

// BIG: the tile of 4-colour legs from n = kLegBigN on, whose wider halo makes
// 32 x 32 tiles update 2.2 x their nodes (52 x 44: 1.8 x).  A leg of two sweeps
// and the restriction, 32 x 32 / 52 x 44, us: n = 384: 8.7 / 11.0, 768: 18.5 /
// 18.2, 1536: 64 / 43.  Red-black legs (1.9 x) gain nothing by 56 x 44 tiles:
// 4096: 239 / 250, 8192: 993 / 980.
constexpr int kLegBigN = 768;
template <int ORDER, bool BIG>
struct LegShape {
    static constexpr int TX = BIG ? 52 : 32, TY = BIG ? 44 : 32;
    static constexpr int HX = ORDER == MA2D_RED_BLACK ? 6 : 10, HY = 6;
    static constexpr int LX = TX + 2 * HX, LY = TY + 2 * HY;   // loaded tile
    static constexpr int QX = LX / 2, QY = LY / 2;             // quads
    static constexpr int NT = (QX * QY + 63) / 64 * 64;
};

struct LegArgs {
    const double *uin;
    double *uout;
    const double *F;
    const double *uc, *wc;
    double *cw, *cb;
    double *part;
    unsigned long long *cnt;
    int n, sweeps, half, tiles_x;
};

// The neighbours of the node of column parity q at LDS offset base (its row
// start + its quad column).  Those along the axes come from oth and the
// diagonal ones from same (a red-black phase keeps the two colours in
// different buffers).
struct Nine {
    double w, e, s, n, sw, se, nw, ne;
};
template <int QX>
__device__ __forceinline__ Nine around(const double *same, const double *oth, int base, int q)
{
    constexpr int LX = 2 * QX;
    const int o = base + q * QX, l = q ? base : base + QX - 1, r = q ? base + 1 : base + QX;
    Nine v;
    v.w = oth[l];
    v.e = oth[r];
    v.s = oth[o - LX];
    v.n = oth[o + LX];
    v.sw = same[l - LX];
    v.se = same[r - LX];
    v.nw = same[l + LX];
    v.ne = same[r + LX];
    return v;
}
__device__ __forceinline__ H2 hess_of(double c, const Nine &v, double k)
{
    return hess2<double>(c, v.w, v.e, v.s, v.n, v.sw, v.se, v.nw, v.ne, k);
}
__device__ __forceinline__ Hes2<Two> hess_of(Two c, const Nine &a, const Nine &b, double k)
{
    return hess2<Two>(c, Two{a.w, b.w}, Two{a.e, b.e}, Two{a.s, b.s}, Two{a.n, b.n},
                      Two{a.sw, b.sw}, Two{a.se, b.se}, Two{a.nw, b.nw}, Two{a.ne, b.ne}, k);
}

// New values of two nodes, and of one; bad counts the uncertified ones of
// those whose flag is set.
__device__ __forceinline__ Two update2(Two c, const Nine &a, const Nine &b, Two F, double k,
                                       double hh, bool ca, bool cb, int &bad)
{
    int ua, ub;
    const Two x = root2(hess_of(c, a, b, k), F, ua, ub);
    bad += (ca ? ua : 0) + (cb ? ub : 0);
    return c + x * hh;
}
__device__ __forceinline__ double update1(double c, const Nine &a, double F, double k, double hh,
                                          bool ca, int &bad)
{
    int ua;
    const double x = root2(hess_of(c, a, k), F, ua);
    bad += ca ? ua : 0;
    return c + x * hh;
}

template <int ORDER, int IN, int OUT, bool BIG>
__global__ __launch_bounds__((LegShape<ORDER, BIG>::NT), 8) void k2_leg(LegArgs A)
{
    using Sh = LegShape<ORDER, BIG>;
    constexpr int QX = Sh::QX, QY = Sh::QY, LX = Sh::LX, LY = Sh::LY, HX = Sh::HX, HY = Sh::HY;
    constexpr bool RB = ORDER == MA2D_RED_BLACK;
    // red-black: the two buffers a colour's values alternate between; the
    // restriction's residuals take the buffer the result is not in
    __shared__ double S[RB || OUT == LEG_RESTRICT ? 2 : 1][LX * LY];
    const int n = A.n, tid = int(threadIdx.x);
    const int tile = mafas::tile_of_block(int(blockIdx.x), int(gridDim.x));
    const int tx = tile % A.tiles_x, ty = tile / A.tiles_x;
    const int qx = tid % QX, qy = tid / QX;
    const bool quad = qy < QY;
    const int x0 = 2 * qx, y0 = 2 * qy;                        // in the loaded tile
    const int gi = tx * Sh::TX - HX + x0, gj = ty * Sh::TY - HY + y0;
    const long sy = n + 1;
    const double s = double(n) * double(n);
    const bool own = quad && x0 >= HX && x0 < HX + Sh::TX && y0 >= HY && y0 < HY + Sh::TY;

    // ---- load
    double u[2][2], f[2][2];
    bool in[2][2];
    {
        bool ok[2][2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int i = gi + q, j = gj + r;
                ok[r][q] = quad && i >= 0 && i <= n && j >= 0 && j <= n;
                in[r][q] = quad && i >= 1 && i <= n - 1 && j >= 1 && j <= n - 1;
                const long p = i + sy * j;
                const bool rd = IN == LEG_FMG ? ok[r][q] && !in[r][q] : ok[r][q];
                u[r][q] = A.uin[rd ? p : 0];
                f[r][q] = A.F[in[r][q] ? p : 0];
            }
        if (IN == LEG_PRO && quad) {
            // coarse corners of the quad, clamped where no interior node of
            // the quad uses them
            const int nc = n / 2;
            const long cy = nc + 1;
            const int I0 = min(max(gi >> 1, 0), nc), J0 = min(max(gj >> 1, 0), nc);
            const int I1 = min(I0 + 1, nc), J1 = min(J0 + 1, nc);
            const double e00 = A.uc[I0 + cy * J0] - A.wc[I0 + cy * J0];
            const double e10 = A.uc[I1 + cy * J0] - A.wc[I1 + cy * J0];
            const double e01 = A.uc[I0 + cy * J1] - A.wc[I0 + cy * J1];
            const double e11 = A.uc[I1 + cy * J1] - A.wc[I1 + cy * J1];
            if (in[0][0])
                u[0][0] += e00;
            if (in[0][1])
                u[0][1] += 0.5 * e00 + 0.5 * e10;
            if (in[1][0])
                u[1][0] += 0.5 * e00 + 0.5 * e01;
            if (in[1][1])
                u[1][1] += ((0.25 * e00 + 0.25 * e10) + 0.25 * e01) + 0.25 * e11;
        }
        if (IN == LEG_FMG) {
            // The coarse nodes under the tile and three more on each side go
            // through LDS (in the tile's own buffer, ahead of its values):
            // 25 reads a quad, 16 of them the patch of its odd-odd node.
            constexpr int CX = QX + 6, CY = QY + 6;
            static_assert(CX * CY <= LX * LY, "the coarse patch fits the tile's buffer");
            const int nc = n / 2;
            const long cy = nc + 1;
            const int cx0 = (tx * Sh::TX - HX) / 2 - 3, cy0 = (ty * Sh::TY - HY) / 2 - 3;
            for (int e = tid; e < CX * CY; e += Sh::NT) {
                const int I = cx0 + e % CX, J = cy0 + e / CX;
                const bool ok = I >= 0 && I <= nc && J >= 0 && J <= nc;
                S[0][e] = ok ? A.uc[I + cy * J] : 0.0;
            }
            mafas::lds_barrier();
            if (quad) {
                // the four taps of the odd column and row; the first coarse
                // node lies at most three from the quad's own
                double wi[4], wj[4];
                const int I = gi >> 1, J = gj >> 1;
                const int fi = rule2(nc, gi + 1, wi), fj = rule2(nc, gj + 1, wj);
                auto uc = [&](int X, int Y) {
                    return S[0][(min(X, nc) - cx0) + CX * (min(Y, nc) - cy0)];
                };
                if (in[0][0])
                    u[0][0] = uc(I, J);
                if (in[0][1]) {
                    double v = 0.0;
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        v += wi[a] * uc(fi + a, J);
                    u[0][1] = v;
                }
                if (in[1][0]) {
                    double v = 0.0;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        v += wj[b] * uc(I, fj + b);
                    u[1][0] = v;
                }
                if (in[1][1]) {
                    double v = 0.0;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int a = 0; a < 4; ++a)
                            v += wj[b] * wi[a] * uc(fi + a, fj + b);
                    u[1][1] = v;
                }
            }
            mafas::lds_barrier();
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (!ok[r][q])
                    u[r][q] = 0.0;
                if (quad)
                    S[0][(y0 + r) * LX + q * QX + qx] = u[r][q];
            }
    }
    mafas::lds_barrier();

    // ---- sweeps
    // LDS offsets of this quad's nodes by row and column parity, moved inside
    // for nodes on the rim of the loaded tile: they compute from the wrong
    // neighbours and keep their values
    const int yc = min(qy, QY - 1) * 2;
    const int row[2] = {max(yc, 1) * LX, min(yc + 1, LY - 2) * LX};
    const int col[2] = {max(qx, 1), min(qx, QX - 2)};
    const double hh = 0.5 / s;
    // quads all of whose neighbours are loaded: the others' nodes are never
    // read by a node that counts (the halo leaves room for a whole quad)
    const bool rim = quad && qx >= 1 && qx < QX - 1 && qy >= 1 && qy < QY - 1;
    int bad = 0;
    if (RB) {
        for (int w = 0; w < A.sweeps; ++w) {
            // at the start of a sweep both colours are in buffer w & 1
            const double *cur = S[w & 1];
            double *nxt = S[1 - (w & 1)];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double *oth = c == 0 ? cur : nxt;
                const int lo = 2 * w + c + 1;   // first right row and column
                // one node after the other: side by side they take 92-124
                // registers, and a large grid needs the wavefronts
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int q = c ^ r;
                    const int x = x0 + q, y = y0 + r;
                    if (in[r][q] && x >= lo && x < LX - lo && y >= lo && y < LY - lo)
                        u[r][q] = update1(u[r][q], around<QX>(cur, oth, row[r] + col[q], q),
                                          f[r][q], s, hh, own, bad);
                }
                if (quad) {
#pragma unroll
                    for (int r = 0; r < 2; ++r)
                        nxt[(y0 + r) * LX + (c ^ r) * QX + qx] = u[r][c ^ r];
                }
                mafas::lds_barrier();
            }
        }
    } else {
        for (int w = 0; w < A.sweeps; ++w) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int q = c & 1, r = c >> 1;
                if (in[r][q] && rim) {
                    u[r][q] = update1(u[r][q], around<QX>(S[0], S[0], row[r] + col[q], q),
                                      f[r][q], s, hh, own, bad);
                    S[0][row[r] + col[q] + q * QX] = u[r][q];
                }
                mafas::lds_barrier();
            }
        }
    }
    if (A.sweeps > 0)
        count_nonconvex(bad, A.cnt);

    // ---- results
    if (own) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (gi + q <= n && gj + r <= n)
                    A.uout[gi + q + sy * (gj + r)] = u[r][q];
    }
    if (OUT == LEG_PLAIN)
        return;
    const double *U = S[RB ? A.sweeps & 1 : 0];
    // residuals of the tile's own nodes and, for the restriction, of the ones
    // around them
    constexpr int m = OUT == LEG_RESTRICT ? 1 : 0;
    double res[2][2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int x = x0 + q, y = y0 + r;
            res[r][q] = 0.0;
            if (in[r][q] && x >= HX - m && x < HX + Sh::TX + m && y >= HY - m &&
                y < HY + Sh::TY + m)
                res[r][q] = f[r][q] - det2(hess_of(u[r][q], around<QX>(U, U, y * LX + qx, q), s));
        }
    if (OUT == LEG_RESTRICT) {
        double *R = S[RB ? 1 - (A.sweeps & 1) : 1];
        if (quad) {
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    R[(y0 + r) * LX + q * QX + qx] = res[r][q];
        }
        mafas::lds_barrier();
        const int nc = n / 2, I = gi >> 1, J = gj >> 1;
        if (own && I <= nc && J <= nc) {
            const long c = I + long(nc + 1) * J;
            A.cw[c] = u[0][0];
            double b = 0.0;
            if (I >= 1 && I <= nc - 1 && J >= 1 && J <= nc - 1) {
                const int o = y0 * LX + qx;   // this node in U and R (even column)
                auto r = [&](int dx, int dy) {
                    return R[o + dy * LX + (dx == 0 ? 0 : dx < 0 ? QX - 1 : QX)];
                };
                const double rh = restricted(r, A.half != 0);
                // D^2_H of the injected values: even columns two rows apart
                const double sc = double(nc) * double(nc), v = u[0][0];
                const double *a = U + o - 2 * LX, *m = U + o, *t = U + o + 2 * LX;
                b = det2(hess2<double>(v, m[-1], m[1], a[0], t[0], a[-1], a[1], t[-1], t[1], sc)) +
                    rh;
            }
            A.cb[c] = b;
        }
    }
    if (OUT == LEG_NORM) {
        double v = 0.0;
        if (own)
            v = (res[0][0] * res[0][0] + res[0][1] * res[0][1]) +
                (res[1][0] * res[1][0] + res[1][1] * res[1][1]);
        v = wave_sum(v);
        mafas::lds_barrier();   // every read of the tile is done
        if ((tid & 63) == 0)
            S[0][tid >> 6] = v;
        mafas::lds_barrier();
        if (tid == 0) {
            double t = 0.0;
            for (int w = 0; w < Sh::NT / 64; ++w)
                t += S[0][w];
            A.part[tile] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// The levels n <= kTail2N of a V-cycle (or of the whole FMG iteration) in one
// workgroup with every array in LDS.  A thread owns a 2 x 2 quad of interior
// nodes; levels of at most 64 quads (n <= 16) run on the first wavefront
// alone, which needs no barrier between phases.  A V-cycle from n = 64 takes
// 42 us and the FMG iteration 113 us on one compute unit (one launch per phase
// cost 2-4 us for each of ~100 and ~350 phases): n = 64 is bound by the 64-bit
// instruction rate, the levels below by the dependent chain of each phase
// (~700 clocks: sqrt 110, division 70, LDS write to read 110).
// ---------------------------------------------------------------------------
constexpr int kTail2N = 64;
constexpr int kTail2Levels = 6;         // 64, 32, 16, 8, 4, 2
constexpr int kTail2Threads = 1024;     // quads of the largest level
constexpr int kTail2Doubles = 19200;    // LDS: 153.6 kB
constexpr int kTail2Wave = 16;          // levels the first wavefront runs alone
static_assert((kTail2N / 2 + 1) * (kTail2N / 2 + 1) * (kTail2N / 2) < 65536 &&
                  kTail2Threads * (kTail2N / 2) < 65536, "range of div16");

struct Tail2Args {
    const double *uin;          // top level
    double *u;                  // its result
    const double *F;
    unsigned long long *cnt;
    int levels, nu1, nu2, nu0, half, fmg, coarsest;   // coarsest: FMG sweeps there
    int n[kTail2Levels];
    unsigned mq[kTail2Levels], mc[kTail2Levels];   // div16 by n / 2 and by n / 2 + 1
    int ou[kTail2Levels], ob[kTail2Levels], ow[kTail2Levels], orr[kTail2Levels];
};

// q / d for q (d - 1) < 65536 with m = ceil(65536 / d): the integer division
// by a variable takes ~35 instructions, on the critical path of each phase.
__device__ __forceinline__ int div16(int q, unsigned m) { return int((unsigned(q) * m) >> 16); }

// One level: rows of P doubles hold the even columns, then (from H on) the
// odd ones.
struct Lev2 {
    int n, H, P;
    unsigned mq, mc;
    double *u, *b, *w, *r;
    __device__ __forceinline__ int at(int i, int j) const
    {
        return j * P + (i & 1) * H + (i >> 1);
    }
    // neighbours of the node at offset o whose row neighbours are at l and r
    __device__ __forceinline__ Nine around(int o, int l, int r) const
    {
        return Nine{u[l], u[r], u[o - P], u[o + P], u[l - P], u[r - P], u[l + P], u[r + P]};
    }
};

template <int ORDER>
__global__ __launch_bounds__(kTail2Threads) void k2_tail(Tail2Args A)
{
    __shared__ double S[kTail2Doubles];
    const int tid = int(threadIdx.x), L = A.levels;
    int bad = 0;
    auto lev = [&](int l) {
        Lev2 V;
        V.n = A.n[l];
        V.H = V.n / 2 + 1;
        V.P = 2 * V.H;
        V.mq = A.mq[l];
        V.mc = A.mc[l];
        V.u = S + A.ou[l];
        V.b = S + A.ob[l];
        V.w = S + A.ow[l];
        V.r = S + A.orr[l];
        return V;
    };
    auto sync = [](bool one) {
        if (one)
            mafas::lds_wave_order();
        else
            mafas::lds_barrier();
    };
    // The calls below take ONE = std::true_type when the caller is the first
    // wavefront alone, and the thread's quad: nodes m = 0..3 at (2a + 1 + (m &
    // 1), 2b + 1 + (m >> 1)), of which on[m] are interior.  p is the offset of
    // the quad's first row and column pair: its odd column is at p + H, the
    // next even one at p + 1.
    struct Quad {
        int a, b, p;
        bool any, on[4];
    };
    auto quad_of = [&](const Lev2 &V) {
        Quad q;
        q.b = div16(tid, V.mq);
        q.a = tid - q.b * (V.n / 2);
        q.p = (2 * q.b + 1) * V.P + q.a;
        q.any = q.b < V.n / 2;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            q.on[m] = bool(q.any & (2 * q.a + 1 + (m & 1) <= V.n - 1) &
                           (2 * q.b + 1 + (m >> 1) <= V.n - 1));
        return q;
    };
    auto offset = [](const Lev2 &V, const Quad &q, int m) {
        return q.p + (m >> 1) * V.P + ((m & 1) ? 1 : V.H);
    };
    auto nine = [](const Lev2 &V, const Quad &q, int m) {
        const int r = q.p + (m >> 1) * V.P;
        return V.around(r + ((m & 1) ? 1 : V.H), (m & 1) ? r + V.H : r,
                        (m & 1) ? r + V.H + 1 : r + 1);
    };
    auto sweep = [&](auto ONE, const Lev2 &V, const Quad &Q, int count) {
        const double s = double(V.n) * double(V.n), hh = 0.5 / s;
        double f[4];
        if (Q.any) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                f[m] = V.b[offset(V, Q, m)];
        }
        for (int k = 0; k < count; ++k) {
            if (ORDER == MA2D_RED_BLACK) {
                // colour 0: nodes 0 and 3 of the quad (i + j even), then 1, 2
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int m0 = c, m1 = 3 - c;
                    const int o0 = offset(V, Q, m0), o1 = offset(V, Q, m1);
                    Two v{0.0, 0.0};
                    if (Q.any)
                        v = update2(Two{V.u[o0], V.u[o1]}, nine(V, Q, m0), nine(V, Q, m1),
                                    Two{f[m0], f[m1]}, s, hh, Q.on[m0], Q.on[m1], bad);
                    sync(ONE);
                    if (Q.on[m0])
                        V.u[o0] = v.x;
                    if (Q.on[m1])
                        V.u[o1] = v.y;
                    sync(ONE);
                }
            } else {
                // colour (i mod 2) + 2 (j mod 2); node 0 is odd in both
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int m = 3 - c, o = offset(V, Q, m);
                    if (Q.on[m])
                        V.u[o] = update1(V.u[o], nine(V, Q, m), f[m], s, hh, true, bad);
                    sync(ONE);
                }
            }
        }
    };
    // residual of V, then the restriction to the interior of C (the boundary
    // of C's u and w is injected once, at the start); the quad's last node is
    // the coarse node (a + 1, b + 1)
    auto restrict_to = [&](auto ONE, const Lev2 &V, const Quad &Q, const Lev2 &C) {
        const double s = double(V.n) * double(V.n), sc = 0.25 * s;
        if (Q.any) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {   // nodes 0, 3 and 1, 2 together
                const int o0 = offset(V, Q, m), o1 = offset(V, Q, 3 - m);
                const Two c{V.u[o0], V.u[o1]}, F{V.b[o0], V.b[o1]};
                const Two r = F - det2(hess_of(c, nine(V, Q, m), nine(V, Q, 3 - m), s));
                if (Q.on[m])
                    V.r[o0] = r.x;
                if (Q.on[3 - m])
                    V.r[o1] = r.y;
            }
        }
        sync(ONE);
        if (Q.on[3]) {
            const int o = offset(V, Q, 3), P = V.P, c = C.at(Q.a + 1, Q.b + 1);
            const double v = V.u[o];
            C.w[c] = v;
            C.u[c] = v;
            auto r = [&](int dx, int dy) {
                return V.r[o + dy * P + (dx == 0 ? 0 : dx < 0 ? V.H - 1 : V.H)];
            };
            const double rh = restricted(r, A.half != 0);
            const double *a = V.u + o - 2 * P, *m = V.u + o, *t = V.u + o + 2 * P;
            C.b[c] = det2(hess2<double>(v, m[-1], m[1], a[0], t[0], a[-1], a[1], t[-1], t[1], sc)) + rh;
        }
        sync(ONE);
    };
    // correction of V from the next level C
    auto correct = [&](auto ONE, const Lev2 &V, const Quad &Q, const Lev2 &C) {
        if (Q.any) {
            auto e = [&](int da, int db) {
                const int c = C.at(Q.a + da, Q.b + db);
                return C.u[c] - C.w[c];
            };
            const double e00 = e(0, 0), e10 = e(1, 0), e01 = e(0, 1), e11 = e(1, 1);
            const double d[4] = {((0.25 * e00 + 0.25 * e10) + 0.25 * e01) + 0.25 * e11,
                                 0.5 * e10 + 0.5 * e11, 0.5 * e01 + 0.5 * e11, e11};
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (Q.on[m])
                    V.u[offset(V, Q, m)] += d[m];
        }
        sync(ONE);
    };
    // one visit of level l on the way down (or on the coarsest, with nu0
    // sweeps) or up
    auto visit = [&](auto ONE, int l, bool dn, int nu0) {
        const Lev2 V = lev(l), C = lev(min(l + 1, L - 1));
        const Quad Q = quad_of(V);
        if (!dn)
            correct(ONE, V, Q, C);
        sweep(ONE, V, Q, !dn ? A.nu2 : l < L - 1 ? A.nu1 : nu0);
        if (dn && l < L - 1)
            restrict_to(ONE, V, Q, C);
    };
    // V-cycle from level top: the larger levels on the whole workgroup, the
    // others, down and up again, on the first wavefront.  Each loop has one
    // call of visit, which keeps the kernel within the instruction cache.
    auto vcycle = [&](int top, int nu0) {
        int few = top;   // first level of the wavefront
        while (few < L && A.n[few] > kTail2Wave)
            ++few;
        const int many = few - top;
        for (int k = 0; k <= 2 * many; ++k) {
            if (k == many) {
                const int m = L - few;
                if (tid < 64)
                    for (int q = 0; q < 2 * m - 1; ++q)
                        visit(std::true_type{}, few + (q < m ? q : 2 * m - 2 - q), q < m, nu0);
                mafas::lds_barrier();
                continue;
            }
            const int l = k < many ? top + k : top + 2 * many - k;
            if (k < many || l < L - 1)   // the coarsest has no way up
                visit(std::false_type{}, l, k < many, nu0);
        }
    };

    // ---- load, every value of a thread in flight together; the residuals'
    // boundary is zero and never written
    const int n = A.n[0];
    {
        constexpr int KQ = ((kTail2N + 1) * (kTail2N + 1) + kTail2Threads - 1) / kTail2Threads;
        const Lev2 V = lev(0);
        double u[KQ], f[KQ];
        int at[KQ];
#pragma unroll
        for (int m = 0; m < KQ; ++m) {
            const int q = tid + m * kTail2Threads;
            const int i = q % (n + 1), j = q / (n + 1);
            const bool in = i >= 1 && i <= n - 1 && j >= 1 && j <= n - 1;
            at[m] = j <= n ? V.at(i, j) : -1;
            u[m] = A.uin[j <= n ? q : 0];
            f[m] = A.F[in ? q : 0];
        }
        for (int q = tid; q < kTail2Doubles; q += kTail2Threads)
            S[q] = 0.0;
        mafas::lds_barrier();
#pragma unroll
        for (int m = 0; m < KQ; ++m)
            if (at[m] >= 0) {
                V.u[at[m]] = u[m];
                V.b[at[m]] = f[m];   // boundary values are never used
            }
    }
    mafas::lds_barrier();
    // the Dirichlet data of every level (u - w is 0 there); F too, which the
    // FMG starts from (a V-cycle overwrites it)
    for (int l = 1; l < L; ++l) {
        const Lev2 V = lev(l - 1), C = lev(l);
        const int m = C.n + 1;
        for (int q = tid; q < m * m; q += kTail2Threads) {
            const int J = div16(q, V.mc), I = q - J * m;
            const int c = C.at(I, J), o = V.at(2 * I, 2 * J);
            C.u[c] = C.w[c] = V.u[o];
            C.b[c] = V.b[o];
        }
        mafas::lds_barrier();
    }
    // FMG (Algorithm 2): each level starts from the interpolation of the next
    // (the coarsest from zero) and takes a V-cycle
    for (int l = A.fmg ? L - 1 : 0; l >= 0; --l) {
        if (A.fmg) {
            const Lev2 V = lev(l), C = lev(min(l + 1, L - 1));
            const int m = V.n - 1;
            auto uc = [&](int I, int J) { return C.u[C.at(I, J)]; };
            for (int q = tid; q < m * m; q += kTail2Threads) {
                const int i = 1 + q % m, j = 1 + q / m;
                V.u[V.at(i, j)] = l == L - 1 ? 0.0 : fmg_value(uc, C.n, i, j);
            }
            mafas::lds_barrier();
        }
        vcycle(l, A.fmg && l == L - 1 ? A.coarsest : A.nu0);
    }
    count_nonconvex(bad, A.cnt);
    {
        // the boundary too: the prolongation reads u - w there
        const Lev2 V = lev(0);
        for (int q = tid; q < (n + 1) * (n + 1); q += kTail2Threads)
            A.u[q] = V.u[V.at(q % (n + 1), q / (n + 1))];
    }
}

// r = F - det(D^2 u) (r may be null; 0 on the boundary) and one sum of r^2
// per block.  A lane walks kResRows rows of one column with the three columns
// around it of three rows in registers, the next row's loads issued before
// the current row's residual.  ZERO: u is taken as zero inside (the start of
// the Section 4 protocol), so u is read on the boundary alone.
constexpr int kResRows = 16, kResWaves = 4;

template <bool ZERO>
__global__ __launch_bounds__(64 * kResWaves) void k2_residual(const double *__restrict__ u,
                                                              const double *__restrict__ F,
                                                              double *__restrict__ r,
                                                              double *__restrict__ part, int n)
{
    __shared__ double ws[kResWaves];
    const int lane = int(threadIdx.x) & 63, w = int(threadIdx.x) >> 6;
    const int i = int(blockIdx.x) * 64 + lane;
    const int j0 = (int(blockIdx.y) * kResWaves + w) * kResRows, j1 = min(j0 + kResRows, n + 1);
    const long sy = n + 1;
    const double s = double(n) * double(n);
    const bool col = i >= 1 && i <= n - 1;
    const int ic = min(max(i, 1), n - 1);   // a lane outside computes a copy
    double acc = 0.0;
    auto val = [&](int x, int y) {
        y = min(max(y, 0), n);
        if (ZERO && x >= 1 && x <= n - 1 && y >= 1 && y <= n - 1)
            return 0.0;
        return u[x + sy * y];
    };
    double R[4][3], fn = 0.0;
    auto load = [&](double *v, int y) {
        v[0] = val(ic - 1, y);
        v[1] = val(ic, y);
        v[2] = val(ic + 1, y);
    };
    auto rhs = [&](int y) { return F[ic + sy * min(max(y, 1), n - 1)]; };
    if (j0 < j1) {
        load(R[0], j0 - 1);
        load(R[1], j0);
        load(R[2], j0 + 1);
        fn = rhs(j0);
    }
    for (int j = j0; j < j1; ++j) {
        const double f = fn;
        load(R[3], j + 2);
        fn = rhs(j + 1);
        const double c = R[1][1];
        H2 g;
        g.xx = ((R[1][2] - c) - (c - R[1][0])) * s;
        g.yy = ((R[2][1] - c) - (c - R[0][1])) * s;
        g.xy = ((R[2][2] - R[2][0]) - (R[0][2] - R[0][0])) * (0.25 * s);
        const bool in = col && j >= 1 && j <= n - 1;
        const double rv = in ? f - det2(g) : 0.0;
        acc += rv * rv;
        if (r && i <= n)
            r[i + sy * j] = rv;
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                R[m][k] = R[m + 1][k];
    }
    acc = wave_sum(acc);
    if (lane == 0)
        ws[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0)
        part[blockIdx.x + gridDim.x * blockIdx.y] = ((ws[0] + ws[1]) + ws[2]) + ws[3];
}

// Injection of F and of u's Dirichlet data from the finest grid (n
// intervals) to every level of the list at once; level q's blocks start at
// start[q].  The interior of a coarser u is not written: the FMG fills it.
constexpr int kInjLevels = 16;
struct InjectArgs {
    const double *u, *F;
    double *lu[kInjLevels], *lb[kInjLevels];
    int start[kInjLevels];
    int levels, n;
};

__global__ __launch_bounds__(256) void k2_inject(InjectArgs A)
{
    int q = 0;
    while (q + 1 < A.levels && int(blockIdx.x) >= A.start[q + 1])
        ++q;
    const int nc = A.n >> (q + 1), m = nc + 1;
    const long p = (long(blockIdx.x) - A.start[q]) * 256 + threadIdx.x;
    if (p >= long(m) * m)
        return;
    const int I = int(p % m), J = int(p / m);
    const long f = (long(I) << (q + 1)) + long(A.n + 1) * (long(J) << (q + 1));
    if (I >= 1 && I <= nc - 1 && J >= 1 && J <= nc - 1)
        A.lb[q][p] = A.F[f];
    else
        A.lu[q][p] = A.u[f];
}

__global__ __launch_bounds__(BX *BY) void k2_zero_interior(double *__restrict__ u, int n)
{
    const int i = 1 + int(blockIdx.x * BX + threadIdx.x);
    const int j = 1 + int(blockIdx.y * BY + threadIdx.y);
    if (i > n - 1 || j > n - 1)
        return;
    u[i + long(n + 1) * j] = 0.0;
}

// A phase of a lone sweep as a launch of its own.  4 colours: in place.
// Red-black: the colour's new values into t (out = t), then back (commit).
template <int ORDER>
__global__ __launch_bounds__(BX *BY) void k2_phase(double *u, const double *__restrict__ F,
                                                   double *out, int n, int color,
                                                   unsigned long long *cnt, bool commit)
{
    const int y = int(blockIdx.y * BY + threadIdx.y);
    const int j = ORDER == MA2D_COLOR4 ? ((color & 2) ? 1 : 2) + 2 * y : 1 + y;
    const bool odd = ORDER == MA2D_COLOR4 ? (color & 1) != 0 : ((color + j) & 1) != 0;
    const int i = (odd ? 1 : 2) + 2 * int(blockIdx.x * BX + threadIdx.x);
    const bool in = i <= n - 1 && j <= n - 1;
    int bad = 0;
    if (in) {
        const long sy = n + 1, p = i + sy * j;
        if (commit) {
            u[p] = out[p];
        } else {
            const double s = double(n) * double(n);
            const Nine v{u[p - 1],      u[p + 1],      u[p - sy],     u[p + sy],
                         u[p - sy - 1], u[p - sy + 1], u[p + sy - 1], u[p + sy + 1]};
            out[p] = update1(u[p], v, F[p], s, 0.5 / s, true, bad);
        }
    }
    count_nonconvex(bad, cnt);
}

inline dim3 grid2(int cx, int cy) { return dim3((cx + BX - 1) / BX, (cy + BY - 1) / BY); }

double now_s()
{
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

thread_local std::string g_err2;

bool valid2(const ma2d_params *p, std::string &why)
{
    if (!p) {
        why = "params is NULL";
        return false;
    }
    if (p->n < 2 || p->n > 65536) {
        why = "n must satisfy 2 <= n <= 65536";
        return false;
    }
    if (p->nu1 < 0 || p->nu2 < 0 || p->nu0 < 1 || p->nu1 > 16 || p->nu2 > 16 || p->nu0 > 16) {
        why = "smoothing counts must satisfy 0 <= nu1, nu2 <= 16 and 1 <= nu0 <= 16";
        return false;
    }
    if (p->order != MA2D_COLOR4 && p->order != MA2D_RED_BLACK) {
        why = "order must be MA2D_COLOR4 or MA2D_RED_BLACK";
        return false;
    }
    if (p->restriction != MA_RESTRICT_FULL && p->restriction != MA_RESTRICT_HALF) {
        why = "restriction must be MA_RESTRICT_FULL or MA_RESTRICT_HALF";
        return false;
    }
    if (p->max_cycles < 0 || !std::isfinite(p->tol)) {
        why = "max_cycles must be >= 0 and tol finite";
        return false;
    }
    return true;
}

int levels2(int n, int *ns, int cap)
{
    int L = 0;
    ns[L++] = n;
    while (n % 2 == 0 && n >= 4 && L < cap) {
        n /= 2;
        ns[L++] = n;
    }
    return L;
}

size_t pts2(int n) { return size_t(n + 1) * size_t(n + 1); }

// First level the coarse-level kernel takes over from (the level count when
// none is small enough).
int tail_level(const int *ns, int L)
{
    int l = 0;
    while (l < L && ns[l] > kTail2N)
        ++l;
    return l;
}

// Tiles of a leg in x and y.
bool leg_big(int order, int n) { return order == MA2D_COLOR4 && n >= kLegBigN; }
dim3 leg_grid(int order, int n)
{
    using Small = LegShape<MA2D_COLOR4, false>;
    using Big = LegShape<MA2D_COLOR4, true>;
    static_assert(LegShape<MA2D_RED_BLACK, false>::TX == Small::TX &&
                      LegShape<MA2D_RED_BLACK, false>::TY == Small::TY,
                  "the small tile serves both orderings");
    const int tx = leg_big(order, n) ? Big::TX : Small::TX;
    const int ty = leg_big(order, n) ? Big::TY : Small::TY;
    return dim3((n + tx) / tx, (n + ty) / ty);
}

dim3 residual_grid(int n)
{
    return dim3((n + 64) / 64, (n + kResRows * kResWaves) / (kResRows * kResWaves));
}

// sums of squares of the finest level: one per tile of a leg or per block of
// the residual kernel
size_t partials2(int order, int n)
{
    const dim3 g = residual_grid(n), t = leg_grid(order, n);
    return std::max(size_t(g.x) * g.y, size_t(t.x) * t.y);
}

} // namespace

struct ma2d_solver {
    ma2d_params p{};
    hipStream_t st = nullptr;
    std::vector<int> ns;
    int tail = 0;                          // first level of the coarse-level kernel
    std::vector<double *> u, b, w, t;      // per level up to tail (u, b, w unused on level 0)
    double *part = nullptr, *dsum = nullptr, *hpin = nullptr;
    unsigned long long *cnt = nullptr, *hcnt = nullptr;
    std::vector<void *> owned;
    std::string err;

    ~ma2d_solver()
    {
        if (st)
            (void)hipStreamSynchronize(st);
        for (void *q : owned)
            (void)hipFree(q);
        if (hpin)
            (void)hipHostFree(hpin);
        if (hcnt)
            (void)hipHostFree(hcnt);
    }
    ma_status fail(ma_status s, const std::string &m)
    {
        err = m;
        return s;
    }
    ma_status alloc(double **q, size_t count)
    {
        const hipError_t e = hipMalloc(reinterpret_cast<void **>(q), count * sizeof(double));
        if (e != hipSuccess) {
            (void)hipGetLastError();
            *q = nullptr;
            return fail(MA_ERR_OOM, std::string("hipMalloc: ") + hipGetErrorString(e));
        }
        owned.push_back(*q);
        return MA_OK;
    }
};

#define H2_HIP(s, expr)                                                                          \
    do {                                                                                         \
        const hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                                    \
            return (s)->fail(MA_ERR_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)
#define H2_TRY(expr)                                                                             \
    do {                                                                                         \
        const ma_status s_ = (expr);                                                             \
        if (s_ != MA_OK)                                                                         \
            return s_;                                                                           \
    } while (0)

namespace {

struct Leg {
    int in = LEG_U, out = LEG_PLAIN;
    int sweeps = 0;
};

template <int ORDER, bool BIG>
void launch_leg_t(hipStream_t st, const Leg &g, const LegArgs &A, int tiles)
{
    const dim3 grid(tiles), block(LegShape<ORDER, BIG>::NT);
#define MA2D_LEG(IN, OUT)                                                                        \
    if (g.in == IN && g.out == OUT)                                                              \
        hipLaunchKernelGGL((k2_leg<ORDER, IN, OUT, BIG>), grid, block, 0, st, A);
    MA2D_LEG(LEG_U, LEG_PLAIN)
    MA2D_LEG(LEG_U, LEG_RESTRICT)
    MA2D_LEG(LEG_FMG, LEG_PLAIN)
    MA2D_LEG(LEG_FMG, LEG_RESTRICT)
    MA2D_LEG(LEG_PRO, LEG_PLAIN)
    MA2D_LEG(LEG_PRO, LEG_NORM)
    MA2D_LEG(LEG_U, LEG_NORM)
#undef MA2D_LEG
}

// One leg on level l: uin -> uout (different arrays).
ma_status leg2(ma2d_solver *s, int l, const Leg &g, const double *uin, double *uout,
               const double *F)
{
    LegArgs A{};
    A.uin = uin;
    A.uout = uout;
    A.F = F;
    A.cnt = s->cnt;
    A.part = s->part;
    A.n = s->ns[l];
    A.sweeps = g.sweeps;
    A.half = s->p.restriction == MA_RESTRICT_HALF ? 1 : 0;
    const dim3 t = leg_grid(s->p.order, A.n);
    A.tiles_x = int(t.x);
    if (g.in != LEG_U) {
        A.uc = s->u[l + 1];
        A.wc = s->w[l + 1];
    }
    if (g.out == LEG_RESTRICT) {
        A.cw = s->w[l + 1];
        A.cb = s->b[l + 1];
    }
    const int tiles = int(t.x * t.y);
    if (s->p.order == MA2D_RED_BLACK)
        launch_leg_t<MA2D_RED_BLACK, false>(s->st, g, A, tiles);
    else if (leg_big(s->p.order, A.n))
        launch_leg_t<MA2D_COLOR4, true>(s->st, g, A, tiles);
    else
        launch_leg_t<MA2D_COLOR4, false>(s->st, g, A, tiles);
    H2_HIP(s, hipGetLastError());
    return MA_OK;
}

// Legs of at most two sweeps that run count sweeps (at least one leg).
std::vector<Leg> legs_of(int count)
{
    std::vector<Leg> v;
    do {
        Leg g;
        g.sweeps = std::min(count, 2);
        count -= g.sweeps;
        v.push_back(g);
    } while (count > 0);
    return v;
}

// Runs the legs on level l from x to u; they alternate between u and t, the
// last one ending in u.  x may be u when their number is even.
ma_status run_legs(ma2d_solver *s, int l, const std::vector<Leg> &v, const double *x, double *u,
                   const double *F)
{
    for (size_t k = 0; k < v.size(); ++k) {
        double *y = (v.size() - 1 - k) % 2 ? s->t[l] : u;
        if (x == y)
            return s->fail(MA_ERR_DEVICE, "internal: a leg in place");
        H2_TRY(leg2(s, l, v[k], x, y, F));
        x = y;
    }
    return MA_OK;
}

// Whether a lone sweep in place takes less as a launch per phase than as a leg,
// which needs a copy beside it.  In between, u and F are in the L2 caches and
// the copy takes half the time; above, the phases read them again from farther
// away, and below, the launches count.  us, phases / leg: 4 colours n = 640: 15.5
// / 14.6, 768: 16.4 / 18.7, 1024: 19.1 / 23.4, 1536: 29.8 / 34.9, 1700: 38.9 / 38.4;
// red-black n = 900: 21.2 / 20.1, 1024: 22.4 / 24.5, 1100: 26.0 / 24.6.
bool lone_phases(int order, int n)
{
    return order == MA2D_COLOR4 ? n >= 704 && n <= 1664 : n >= 992 && n <= 1056;
}

ma_status sweep_phases(ma2d_solver *s, int l, double *u, const double *F)
{
    const int n = s->ns[l];
    for (int c = 0; c < (s->p.order == MA2D_COLOR4 ? 4 : 2); ++c) {
        if (s->p.order == MA2D_COLOR4) {
            hipLaunchKernelGGL((k2_phase<MA2D_COLOR4>), grid2(n / 2, n / 2), dim3(BX, BY), 0, s->st,
                               u, F, u, n, c, s->cnt, false);
        } else {
            for (int commit = 0; commit < 2; ++commit)
                hipLaunchKernelGGL((k2_phase<MA2D_RED_BLACK>), grid2(n / 2, n - 1), dim3(BX, BY),
                                   0, s->st, u, F, s->t[l], n, c, s->cnt, commit != 0);
        }
        H2_HIP(s, hipGetLastError());
    }
    return MA_OK;
}

// count sweeps of level l from x to u (x may be u)
ma_status sweep2(ma2d_solver *s, int l, const double *x, double *u, const double *F, int count)
{
    if (count <= 0 && x == u)
        return MA_OK;
    if (count == 1 && x == u && lone_phases(s->p.order, s->ns[l]))
        return sweep_phases(s, l, u, F);
    const std::vector<Leg> v = legs_of(count);
    if (x == u && v.size() % 2) {
        H2_HIP(s, mafas::launch_copy(s->st, pts2(s->ns[l]), u, s->t[l]));
        x = s->t[l];
    }
    return run_legs(s, l, v, x, u, F);
}

// sum of the count partials -> host l2 = sqrt(h^2 sum) on the finest grid
ma_status finish_norm2(ma2d_solver *s, size_t count, double *l2)
{
    H2_HIP(s, mafas::launch_reduce(s->st, s->part, count, s->dsum));
    H2_HIP(s, hipMemcpyAsync(s->hpin, s->dsum, sizeof(double), hipMemcpyDeviceToHost, s->st));
    H2_HIP(s, hipStreamSynchronize(s->st));
    *l2 = std::sqrt(s->hpin[0]) / double(s->p.n);
    return MA_OK;
}

// finest residual into r (may be null) and, with l2 set, its norm; zero: of
// u with a zero interior (u's own interior is not read)
ma_status residual2(ma2d_solver *s, const double *u, const double *F, double *r, double *l2,
                    bool zero = false)
{
    const int n = s->p.n;
    const dim3 g = residual_grid(n), block(64 * kResWaves);
    if (zero)
        hipLaunchKernelGGL(k2_residual<true>, g, block, 0, s->st, u, F, r, s->part, n);
    else
        hipLaunchKernelGGL(k2_residual<false>, g, block, 0, s->st, u, F, r, s->part, n);
    H2_HIP(s, hipGetLastError());
    return l2 ? finish_norm2(s, size_t(g.x) * g.y, l2) : MA_OK;
}

// The coarse-level kernel from level l down: a V-cycle from x to u (x may be
// u), or the FMG iteration (which needs x on the boundary alone).
ma_status tail2(ma2d_solver *s, int l, const double *x, double *u, const double *F, bool fmg)
{
    const int L = int(s->ns.size());
    Tail2Args A{};
    A.uin = x;
    A.u = u;
    A.F = F;
    A.cnt = s->cnt;
    A.levels = L - l;
    A.nu1 = s->p.nu1;
    A.nu2 = s->p.nu2;
    A.nu0 = s->p.nu0;
    A.half = s->p.restriction == MA_RESTRICT_HALF ? 1 : 0;
    A.fmg = fmg ? 1 : 0;
    A.coarsest = (s->ns[L - 1] == 3 && s->p.nu0 < 8) ? 8 : s->p.nu0;
    int off = 0;
    for (int q = 0; q < A.levels; ++q) {
        const int n = s->ns[l + q], size = (n + 1) * 2 * (n / 2 + 1);
        A.n[q] = n;
        A.mq[q] = (65536u + n / 2 - 1) / (n / 2);
        A.mc[q] = (65536u + n / 2) / (n / 2 + 1);
        A.ou[q] = off;
        A.ob[q] = off += size;
        A.orr[q] = off += size;
        off += size;
        A.ow[q] = off;
        off += q > 0 ? size : 0;
    }
    if (off > kTail2Doubles || A.levels > kTail2Levels)
        return s->fail(MA_ERR_ARG, "internal: coarse levels exceed the coarse-level kernel");
    if (s->p.order == MA2D_RED_BLACK)
        hipLaunchKernelGGL(k2_tail<MA2D_RED_BLACK>, dim3(1), dim3(kTail2Threads), 0, s->st, A);
    else
        hipLaunchKernelGGL(k2_tail<MA2D_COLOR4>, dim3(1), dim3(kTail2Threads), 0, s->st, A);
    H2_HIP(s, hipGetLastError());
    return MA_OK;
}

// FAS V-cycle on level l from x to u (x may be u).  fmg: the interior starts
// as the FMG interpolation of the next level's u, and x holds the boundary.
// norm: the last leg leaves the sums of squared residuals of the result in
// part (one per tile; levels above the coarse-level kernel with a
// coarser level).
ma_status vcycle2(ma2d_solver *s, int l, const double *x, double *u, const double *b,
                  bool fmg = false, bool norm = false)
{
    const int L = int(s->ns.size());
    if (l >= s->tail)
        return tail2(s, l, x, u, b, false);
    if (l == L - 1)
        return sweep2(s, l, x, u, b, s->p.nu0);
    std::vector<Leg> dn = legs_of(s->p.nu1), up = legs_of(s->p.nu2);
    if (x == u && (dn.size() + up.size()) % 2) {
        // one leg more: split a leg of two sweeps, or add one without sweeps
        Leg g;
        if (up.front().sweeps == 2)
            up.front().sweeps = g.sweeps = 1;
        up.push_back(g);
    }
    if (fmg)
        dn.front().in = LEG_FMG;
    dn.back().out = LEG_RESTRICT;
    up.front().in = LEG_PRO;
    if (norm)
        up.back().out = LEG_NORM;
    // the legs of the whole cycle alternate between u and t as one sequence
    double *mid = up.size() % 2 ? s->t[l] : u;
    for (size_t k = 0; k < dn.size(); ++k) {
        double *y = (dn.size() - 1 - k) % 2 ? (mid == u ? s->t[l] : u) : mid;
        H2_TRY(leg2(s, l, dn[k], x, y, b));
        x = y;
    }
    H2_TRY(vcycle2(s, l + 1, s->w[l + 1], s->u[l + 1], s->b[l + 1]));
    return run_legs(s, l, up, x, u, b);
}

// One V-cycle of the whole hierarchy (fmg: one FMG iteration) and, with l2
// set, the norm of the residual after it.
ma_status cycle2(ma2d_solver *s, double *u, const double *f, bool fmg, double *l2)
{
    const int L = int(s->ns.size());
    const bool fused = s->tail > 0 && L > 1;   // the finest leg can take the norm
    if (!fmg) {
        H2_TRY(vcycle2(s, 0, u, u, f, false, fused && l2));
    } else if (s->tail == 0) {
        H2_TRY(tail2(s, 0, u, u, f, true));
    } else {
        // F and the Dirichlet data on every level the legs or the
        // coarse-level kernel read from memory
        const int last = std::min(s->tail, L - 1);
        if (last > 0) {
            InjectArgs A{};
            A.u = u;
            A.F = f;
            A.n = s->p.n;
            A.levels = last;
            int blocks = 0;
            for (int l = 1; l <= last; ++l) {
                A.lu[l - 1] = s->u[l];
                A.lb[l - 1] = s->b[l];
                A.start[l - 1] = blocks;
                blocks += int((pts2(s->ns[l]) + 255) / 256);
            }
            hipLaunchKernelGGL(k2_inject, dim3(blocks), dim3(256), 0, s->st, A);
            H2_HIP(s, hipGetLastError());
        }
        auto U = [&](int l) { return l == 0 ? u : s->u[l]; };
        auto B = [&](int l) -> const double * { return l == 0 ? f : s->b[l]; };
        int l = last;
        if (s->tail < L) {
            H2_TRY(tail2(s, l, U(l), U(l), B(l), true));
        } else {
            // coarsest: zero inside, then an approximate solve (nu0 sweeps)
            const int n0 = s->ns[l];
            hipLaunchKernelGGL(k2_zero_interior, grid2(n0 - 1, n0 - 1), dim3(BX, BY), 0, s->st,
                               U(l), n0);
            H2_HIP(s, hipGetLastError());
            H2_TRY(sweep2(s, l, U(l), U(l), B(l), s->p.nu0));
        }
        for (--l; l >= 0; --l)
            H2_TRY(vcycle2(s, l, U(l), U(l), B(l), true, l == 0 && fused && l2));
    }
    if (!l2)
        return MA_OK;
    if (!fused)
        return residual2(s, u, f, nullptr, l2);
    const dim3 t = leg_grid(s->p.order, s->p.n);
    return finish_norm2(s, size_t(t.x) * t.y, l2);
}

ma_status read_count(ma2d_solver *s, long long *out)
{
    H2_HIP(s, hipMemcpyAsync(s->hcnt, s->cnt, sizeof(unsigned long long), hipMemcpyDeviceToHost,
                             s->st));
    H2_HIP(s, hipStreamSynchronize(s->st));
    *out = (long long)s->hcnt[0];
    return MA_OK;
}

// point updates of one V-cycle and of the FMG start (sweeps on every level)
double vcycle_updates(const ma2d_solver *s)
{
    double up = 0.0;
    const int L = int(s->ns.size());
    for (int l = 0; l < L; ++l) {
        const double in = double(s->ns[l] - 1) * double(s->ns[l] - 1);
        up += (l < L - 1 ? s->p.nu1 + s->p.nu2 : s->p.nu0) * in;
    }
    return up;
}

} // namespace

extern "C" {

void ma2d_params_default(ma2d_params *p, int n)
{
    std::memset(p, 0, sizeof(*p));
    p->n = n;
    p->nu1 = 2;
    p->nu2 = 2;
    p->nu0 = 1;
    p->order = MA2D_RED_BLACK;
    p->restriction = MA_RESTRICT_HALF;
    p->max_cycles = 100;
    p->tol = 1e-6;
}

size_t ma2d_footprint_bytes(const ma2d_params *p)
{
    std::string why;
    if (!valid2(p, why))
        return 0;
    int ns[40];
    const int L = levels2(p->n, ns, 40);
    size_t b = 0;
    for (int l = 0; l < L && l <= tail_level(ns, L); ++l)
        b += (l == 0 ? 1 : 4) * pts2(ns[l]) * sizeof(double);
    return b + partials2(p->order, p->n) * sizeof(double) + 4096;
}

ma_status ma2d_create(const ma2d_params *p, void *hip_stream, ma2d_solver **out)
{
    std::string why;
    if (!out) {
        g_err2 = "out is NULL";
        return MA_ERR_ARG;
    }
    *out = nullptr;
    if (!valid2(p, why)) {
        g_err2 = why;
        return MA_ERR_ARG;
    }
    ma2d_solver *s = new ma2d_solver();
    s->p = *p;
    s->st = static_cast<hipStream_t>(hip_stream);
    int ns[40];
    const int L = levels2(p->n, ns, 40);
    s->ns.assign(ns, ns + L);
    s->u.assign(L, nullptr);
    s->b.assign(L, nullptr);
    s->w.assign(L, nullptr);
    s->tail = tail_level(ns, L);
    s->t.assign(L, nullptr);
    ma_status st = MA_OK;
    for (int l = 0; l < L && l <= s->tail && st == MA_OK; ++l) {
        const size_t c = pts2(ns[l]);
        if (l > 0) {
            st = s->alloc(&s->u[l], c);
            if (st == MA_OK)
                st = s->alloc(&s->b[l], c);
            if (st == MA_OK)
                st = s->alloc(&s->w[l], c);
        }
        if (st == MA_OK)
            st = s->alloc(&s->t[l], c);
    }
    if (st == MA_OK)
        st = s->alloc(&s->part, partials2(p->order, p->n));
    if (st == MA_OK)
        st = s->alloc(&s->dsum, 4);
    if (st == MA_OK) {
        void *q = nullptr;
        if (hipMalloc(&q, 64) != hipSuccess)
            st = s->fail(MA_ERR_OOM, "hipMalloc of the counter");
        else {
            s->owned.push_back(q);
            s->cnt = static_cast<unsigned long long *>(q);
        }
    }
    if (st == MA_OK && (hipHostMalloc(reinterpret_cast<void **>(&s->hpin), 4 * sizeof(double)) !=
                            hipSuccess ||
                        hipHostMalloc(reinterpret_cast<void **>(&s->hcnt),
                                      4 * sizeof(unsigned long long)) != hipSuccess))
        st = s->fail(MA_ERR_OOM, "hipHostMalloc failed");
    if (st == MA_OK && hipStreamSynchronize(s->st) != hipSuccess)
        st = s->fail(MA_ERR_DEVICE, "allocation");
    if (st != MA_OK) {
        g_err2 = s->err;
        delete s;
        return st;
    }
    *out = s;
    return MA_OK;
}

void ma2d_destroy(ma2d_solver *s) { delete s; }

const char *ma2d_last_error(const ma2d_solver *s) { return s ? s->err.c_str() : g_err2.c_str(); }

ma_status ma2d_sweep(ma2d_solver *s, double *u, const double *f, int count,
                     long long *nonconvex_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f || count < 0)
        return s->fail(MA_ERR_ARG, "u, f must be device pointers and count >= 0");
    H2_HIP(s, mafas::launch_fill_u64(s->st, 1, 0ull, s->cnt));
    H2_TRY(sweep2(s, 0, u, u, f, count));
    if (nonconvex_host)
        H2_TRY(read_count(s, nonconvex_host));
    return MA_OK;
}

ma_status ma2d_residual(ma2d_solver *s, const double *u, const double *f, double *r_or_null,
                        double *l2_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    double l2 = 0.0;
    H2_TRY(residual2(s, u, f, r_or_null, l2_host ? &l2 : nullptr));
    if (l2_host)
        *l2_host = l2;
    return MA_OK;
}

ma_status ma2d_vcycle(ma2d_solver *s, double *u, const double *f)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    return cycle2(s, u, f, false, nullptr);
}

ma_status ma2d_fmg(ma2d_solver *s, double *u, const double *f, long long *nonconvex_host)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    H2_HIP(s, mafas::launch_fill_u64(s->st, 1, 0ull, s->cnt));
    H2_TRY(cycle2(s, u, f, true, nullptr));
    long long nc = 0;
    H2_TRY(read_count(s, &nc));
    if (nonconvex_host)
        *nonconvex_host = nc;
    return MA_OK;
}

ma_status ma2d_solve(ma2d_solver *s, double *u, const double *f, double tol, unsigned flags,
                     ma_report *rep)
{
    if (!s)
        return MA_ERR_ARG;
    if (!u || !f)
        return s->fail(MA_ERR_ARG, "u and f must be device pointers");
    if (flags & MA_INIT_POISSON)
        return s->fail(MA_ERR_ARG, "the 2D solver starts from u or from MA_INIT_FMG");
    const double t0 = now_s();
    const double target = tol > 0.0 ? tol : s->p.tol;
    const int n = s->p.n;
    ma_report r;
    std::memset(&r, 0, sizeof(r));
    H2_HIP(s, mafas::launch_fill_u64(s->st, 1, 0ull, s->cnt));
    const bool fmg = (flags & MA_INIT_FMG) != 0;
    H2_TRY(residual2(s, u, f, nullptr, &r.res0, fmg));
    r.res = r.res0;
    const double vc_up = vcycle_updates(s);
    const double in0 = double(n - 1) * double(n - 1);
    ma_status st = MA_ERR_NOT_CONVERGED;
    if (!std::isfinite(r.res0)) {
        st = MA_ERR_NONFINITE;
        if (fmg) {   // u is the start whose residual this is
            hipLaunchKernelGGL(k2_zero_interior, grid2(n - 1, n - 1), dim3(BX, BY), 0, s->st, u,
                               n);
            H2_HIP(s, hipGetLastError());
        }
    } else {
        if (fmg) {
            H2_TRY(cycle2(s, u, f, true, &r.res));
            r.cycles = 1;
            r.point_updates += vc_up * (4.0 / 3.0);
            r.history[0] = r.res;
        }
        if (!std::isfinite(r.res))
            st = MA_ERR_NONFINITE;
        else if (r.res <= target * r.res0)
            st = MA_OK;
        while (st == MA_ERR_NOT_CONVERGED && r.cycles < s->p.max_cycles) {
            H2_TRY(cycle2(s, u, f, false, &r.res));
            r.cycles += 1;
            r.point_updates += vc_up;
            if (r.cycles <= 64)
                r.history[r.cycles - 1] = r.res;
            if (!std::isfinite(r.res))
                st = MA_ERR_NONFINITE;
            else if (r.res <= target * r.res0)
                st = MA_OK;
        }
    }
    r.rel_res = r.res0 > 0.0 ? r.res / r.res0 : 0.0;
    r.converged = st == MA_OK;
    r.alg_bytes = r.point_updates * 24.0 + double(r.cycles + 1) * 16.0 * in0;
    long long nc = 0;
    H2_TRY(read_count(s, &nc));
    r.nonconvex = nc;
    r.seconds = now_s() - t0;
    if (rep)
        *rep = r;
    if (st == MA_ERR_NOT_CONVERGED)
        return s->fail(st, "max_cycles reached before the tolerance");
    if (st == MA_ERR_NONFINITE)
        return s->fail(st, "residual is not finite");
    return MA_OK;
}

} // extern "C"
