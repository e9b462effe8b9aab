// One complete nonlinear Gauss-Seidel sweep per launch (Section 2: the
// pointwise update of eqs. 2.7-2.9 applied colour by colour), for many
// grids at once: the block sweep.
//
// A node reads only nodes of other colours, so a sweep is one phase per colour
// (4: c = ((i+j) mod 2) + 2 ((i+k) mod 2); 8: the parities of i, j, k), each
// updating all nodes of one colour at once.  Launched phase by phase, a
// sweep costs four or eight kernel launches, which on the smaller grids of the
// V-cycle take longer than the work itself.  The block sweep runs all
// phases in one launch:
//
// * A workgroup owns a TX x TY x TZ block of output nodes.  It loads the
//   block with a halo into LDS (rows de-interleaved by x parity,
//   so the nodes of one colour in a row are contiguous), and prefetches the
//   right-hand side of every node it will update into registers.
// * It applies phase c to the colour-c nodes of the block grown by ext(c) in
//   every direction, with a workgroup barrier after each phase: the nodes
//   whose values the later phases read, directly or through one another.  With
//   4 colours each pair of colours meets along every axis, so the grown blocks
//   shrink by one node per phase (3, 2, 1, 0).  With 8 colours two nodes of
//   colours c < c' are neighbours only along the axes in whose parity bits c
//   and c' differ (one or two of them), so ext(c) is per axis the largest
//   ext(c') + 1 over those c'.  The nodes outside the owned block are
//   recomputed from the same values by the neighbouring workgroups.
// * It writes the owned block (and the Dirichlet layer next to it) to
//   u_out.  The sweep reads u_in and writes u_out (out of place), so halos
//   read from a neighbouring block are never modified during the launch.
//
// The update of a node evaluates the same expressions (hessian3 and the root
// rule of ma_device.h) on the same values as the colour-phase kernels, so
// the results are bitwise identical to the colour phases.
//
// Algorithmic bytes per interior node and sweep: read u 8, read F 8,
// write u 8.  The recomputation costs ALU work, which on the grids this
// kernel is used for is cheaper than three extra launches.
#pragma once

#include "ma_device.h"
#include "ma_internal.h"

#include <type_traits>

namespace mafas {

// One grid of a block-sweep launch.
struct FsGrid {
    const double *uin;
    double *uout;
    const double *F;
    int n;          // intervals per side
    int tiles_x, tiles_y, tiles_z;
    int start;      // first block of this grid in the launch
    int slot;       // counter slot of the solve
    double s, s4;   // 1/h^2, 1/(4h^2)
    double hk;      // h^2/2 (nonlinear update) or 1/(6s) (linear update)
    // z-stream sweeps that also prolong (the first sweep after the coarse
    // correction): the coarse level's u and w, whose difference is
    // interpolated onto u_in as it is read; null otherwise
    const double *cu, *cw;
};

constexpr int kFsMaxGrids = 64;

struct FsList {
    int ngrids;
    int total;      // blocks over all grids
    unsigned long long stopped;  // bit s: solve s has stopped, skip it
    FsGrid g[kFsMaxGrids];
};
constexpr size_t fs_list_bytes(int ngrids) { return 16 + sizeof(FsGrid) * size_t(ngrids); }
static_assert(offsetof(FsList, g) == 16, "list header is 16 bytes");

// A launch runs PH consecutive phases of a sweep: all of them, or a group whose
// other phases are launches of their own.
//
// Growth of phase c's block along an axis (0: x, 1: y, 2: z): what the later
// phases of its launch read.
__host__ __device__ constexpr int fs_ext(int order, int ph, int c, int axis)
{
    const int p = c % ph;
    if (order == 0)
        return ph - 1 - p;
    // colours 0-3 (4-7) lie in planes of one parity, and each two of them in
    // columns beside one another
    constexpr int e8[8][3] = {{5, 3, 1}, {4, 3, 1}, {3, 2, 1}, {2, 2, 1},
                              {3, 1, 0}, {2, 1, 0}, {1, 0, 0}, {0, 0, 0}};
    return e8[8 - ph + p][axis];
}

template <int ORDER, int PH, int TX, int TY, int TZ, int NT>
struct FsShape {
    // halo loaded around the block: the first phase's growth and one node
    static constexpr int HX = fs_ext(ORDER, PH, 0, 0) + 1, HY = fs_ext(ORDER, PH, 0, 1) + 1,
                         HZ = fs_ext(ORDER, PH, 0, 2) + 1;
    static constexpr int LX = TX + 2 * HX;   // LDS row length
    static constexpr int LY = TY + 2 * HY;   // LDS rows per plane
    static constexpr int LZ = TZ + 2 * HZ;   // LDS planes
    static constexpr int HW = LX / 2;        // one parity half of a row
    static constexpr int PE = LX * LY;       // elements of a plane
    // Doubles per plane.  The items of a wavefront lie in several rows and
    // planes whose starts would all be in one bank; with 4 colours this pad
    // brings the reads of 8-wide blocks from 2.9 cycles a pass to 1.8, and a
    // sweep of n = 64 from 12.2 to 11.0 us (wider blocks and 8 colours do not
    // gain).
    static constexpr int PL = PE + (ORDER == 0 && LX == 16 ? 3 : 0);
    static constexpr int NL = PL * LZ;       // doubles in LDS
    // phase c covers columns and planes of one parity and (4 colours) all
    // rows or (8 colours) those of one parity of its grown block
    static constexpr int ncol(int c) { return TX / 2 + fs_ext(ORDER, PH, c, 0); }
    static constexpr int nrow(int c)
    {
        return ORDER == 0 ? TY + 2 * fs_ext(ORDER, PH, c, 1) : TY / 2 + fs_ext(ORDER, PH, c, 1);
    }
    static constexpr int npl(int c) { return TZ / 2 + fs_ext(ORDER, PH, c, 2); }
    static constexpr int count(int c) { return ncol(c) * nrow(c) * npl(c); }
    // rounds of a workgroup over phase c, and those of the phases before it
    static constexpr int rounds(int c) { return (count(c) + NT - 1) / NT; }
    static constexpr int before(int c) { return c % PH == 0 ? 0 : before(c - 1) + rounds(c - 1); }
    static constexpr int total = before(PH - 1) + rounds(PH - 1);
    static constexpr int SX = TX + 2, SY = TY + 2, SZ = TZ + 2;   // store bound
    static_assert(TX % 2 == 0 && TY % 2 == 0 && TZ % 2 == 0, "block sides must be even");
    static_assert(LX % 2 == 0, "LDS rows hold two parity halves");
};

// Workgroup barrier that orders LDS accesses only: global loads issued
// before it (the right-hand side prefetch) stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The same for accesses of one wavefront alone: its LDS accesses run in order,
// so this only keeps the compiler from moving them across.
__device__ __forceinline__ void lds_wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Phase C and those after it, the item counts of each a constant.
template <int C, int NC, typename F>
__device__ __forceinline__ void fs_phases(F f)
{
    if constexpr (C < NC) {
        f(std::integral_constant<int, C>{});
        fs_phases<C + 1, NC>(f);
    }
}

// One step of the standalone Gauss-Seidel iteration: sweep q, u_{q-1} (in) to
// u_q (out), with the residual norm of u_{q-1} taken from the block in LDS
// before its first phase, and the stopping test of u_{q-2}.
//
// The test of an iterate comes a launch after its sums, and the iterate is
// still whole then: launch q leaves the sums of squares of u_{q-1}, one per
// block, in part_out; launch q + 1, which would overwrite u_{q-1}, first adds
// them up -- every block the same sum in the same order -- and when the sum
// meets the test (<= thr, or not finite) sets *stop to its number q and
// stores nothing, like every launch after it (q > *stop).  So a sweep is one
// launch, and the host looks at the sums once per batch of launches.  Bound by the latency of one block's chain
// (launch, loads, residual, phases): the sums are loaded with the block and
// added up with its residual, and the test is taken just before the phases.
// n = 32, a sweep and its test: 29 us as colour launches, a residual, a
// reduction and a host round trip, 9.3 us so (9.7 with the sums added up
// before the block was loaded).
struct GsStep {
    const double *part_in;      // sums of squares of u_{q-2} (null: none yet)
    double *part_out;           // of u_{q-1}
    double *sum;                // total of part_in (written by block 0)
    unsigned long long *count;  // uncertified updates of this sweep
    int *stop;                  // 0, or the launch that stopped
    int q;                      // this launch, from 1
    double thr;
};

// Block `tile` of grid G by a workgroup of NT threads; su: LDS.  Global
// offsets are 32-bit: grids up to n = 1289.  GS: a step of the Gauss-Seidel
// iteration A, with sums over `blocks` blocks (waves: NT / 32 doubles of LDS).
template <int OP, int ORDER, int PH, int GRP, int TX, int TY, int TZ, int NT, bool GS>
__device__ __forceinline__ void bsweep_tile(const FsGrid &G, int tile, double *__restrict__ su,
                                            unsigned long long *__restrict__ ncount,
                                            const GsStep *A = nullptr, int blocks = 0,
                                            double *__restrict__ waves = nullptr)
{
    using S = FsShape<ORDER, PH, TX, TY, TZ, NT>;
    constexpr int LX = S::LX, HW = S::HW, PE = S::PE, PL = S::PL, NE = PE * S::LZ;
    constexpr int KL = (NE + NT - 1) / NT;
    constexpr int KS = (S::SX * S::SY * S::SZ + NT - 1) / NT;

    const int n = G.n;
    const int tid = int(threadIdx.x);
    const int tx = tile % G.tiles_x;
    const int rest = tile / G.tiles_x;
    const int ty = rest % G.tiles_y;
    const int tz = rest / G.tiles_y;
    const int x0 = 1 + tx * TX, y0 = 1 + ty * TY, z0 = 1 + tz * TZ;
    const int x1 = min(x0 + TX, n), y1 = min(y0 + TY, n), z1 = min(z0 + TZ, n);
    const int lx0 = x0 - S::HX, ly0 = y0 - S::HY, lz0 = z0 - S::HZ;
    const int sy = n + 1, sz = sy * sy;
    const auto uin = to_global(G.uin);
    const auto uout = to_global(G.uout);
    const auto F = to_global(G.F);

    // Node of item m of phase c over the grown block: planes and columns of
    // the colour's parities (4 colours: k = j + c0 + c1, i = j + c0 mod 2) and
    // rows, all or those of its parity.  Returns false when the item lies
    // outside the grid interior.
    auto node = [&](auto cc, int item, int &i, int &j, int &k) -> bool {
        constexpr int c = decltype(cc)::value;
        constexpr int ex = fs_ext(ORDER, PH, c, 0), ey = fs_ext(ORDER, PH, c, 1), ez = fs_ext(ORDER, PH, c, 2);
        constexpr int nc = S::ncol(c);
        const int q = item % nc;
        const int r2 = item / nc;
        int pi, pk;
        if (ORDER == 0) {
            constexpr int c0 = c & 1, c1 = c >> 1, np = S::npl(c);
            const int kk = r2 % np;
            j = y0 - ey + r2 / np;
            pk = (j + c0 + c1) & 1;
            pi = (j + c0) & 1;
            k = (z0 - ez) + (((z0 - ez) ^ pk) & 1) + 2 * kk;
        } else {
            constexpr int nr = S::nrow(c);
            pi = c & 1;
            pk = c >> 2;
            j = (y0 - ey) + (((y0 - ey) ^ (c >> 1)) & 1) + 2 * (r2 % nr);
            k = (z0 - ez) + (((z0 - ez) ^ pk) & 1) + 2 * (r2 / nr);
        }
        i = (x0 - ex) + (((x0 - ex) ^ pi) & 1) + 2 * q;
        return item < S::count(c) && i >= max(1, x0 - ex) && i <= min(n - 1, x1 - 1 + ex) &&
               j >= max(1, y0 - ey) && j <= min(n - 1, y1 - 1 + ey) && k >= max(1, z0 - ez) &&
               k <= min(n - 1, z1 - 1 + ez);
    };
    auto lds_off = [&](int i, int j, int k) {
        const int lx = i - lx0;
        return (k - lz0) * PL + (j - ly0) * LX + (lx & 1) * HW + (lx >> 1);
    };

    // ---- the sums of the iterate before u_in
    int stop = 0;
    double before = 0.0;
    if (GS) {
        stop = *A->stop;   // this launch's own value is not a stop yet
        stop = stop != 0 && stop < A->q;
        if (A->part_in)
            for (int q = tid; q < blocks; q += NT)
                before += A->part_in[q];
    }

    // ---- right-hand sides of every item of this lane, in flight during
    // the block load (a lane without a node reads node 0 and discards it)
    double f[S::total];
    fs_phases<GRP * PH, GRP * PH + PH>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
#pragma unroll
        for (int m = 0; m < S::rounds(c); ++m) {
            int i, j, k;
            const bool ok = node(cc, tid + m * NT, i, j, k);
            f[S::before(c) + m] = F[ok ? i + sy * j + sz * k : 0];
        }
    });

    // ---- the block and its halo into LDS (0 outside the grid): every load
    // of the lane first, then the LDS writes, so all of them are in flight
    // together
    double lv[KL];
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int el = tid + k * NT;
        const int lz = el / PE, rem = el - (el / PE) * PE;
        const int ly = rem / LX, lx = rem - (rem / LX) * LX;
        const int gx = lx0 + lx, gy = ly0 + ly, gz = lz0 + lz;
        const bool in = el < NE && gx >= 0 && gx <= n && gy >= 0 && gy <= n && gz >= 0 &&
                        gz <= n;
        const double v = uin[in ? gx + sy * gy + sz * gz : 0];
        lv[k] = in ? v : 0.0;
    }
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int el = tid + k * NT;
        const int lz = el / PE, rem = el - (el / PE) * PE;
        const int ly = rem / LX, lx = rem - (rem / LX) * LX;
        if (el < NE)
            su[lz * PL + ly * LX + (lx & 1) * HW + (lx >> 1)] = lv[k];
    }
    lds_barrier();

    auto value = [&](int i, int j, int k, double fv, bool resid, bool &nc) {
        double *C = su + lds_off(i, j, k);
        const double *D = C - PL;
        const double *U = C + PL;
        const int odd = (i - lx0) & 1;
        const int xp = odd ? 1 - HW : HW;
        const int xm = odd ? -HW : HW - 1;
        if (OP == OP_MA) {
            const Hess h = hessian3(D, C, U, xp, xm, LX, G.s, G.s4);
            return resid ? fv - det3(h) : ma_point_update(h, C[0], fv, G.hk, nc);
        }
        const double lap = laplacian3(D, C, U, xp, xm, LX, G.s);
        return resid ? fv - lap : lap_point_update(lap, C[0], fv, G.hk);
    };

    // ---- the residual of u_in on the owned nodes, and the test of the iterate
    // before it
    if (GS) {
        if (stop)
            return;
        constexpr int KN = (TX * TY * TZ + NT - 1) / NT;
        double acc = 0.0;
#pragma unroll
        for (int m = 0; m < KN; ++m) {
            const int el = tid + m * NT;
            const int i = x0 + el % TX, r = el / TX, j = y0 + r % TY, k = z0 + r / TY;
            if (el < TX * TY * TZ && i < x1 && j < y1 && k < z1) {
                bool nc = false;
                const double rv = value(i, j, k, F[i + sy * j + sz * k], true, nc);
                acc += rv * rv;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            acc += __shfl_down(acc, off, 64);
            before += __shfl_down(before, off, 64);
        }
        if ((tid & 63) == 0) {
            waves[tid >> 6] = acc;
            waves[NT / 64 + (tid >> 6)] = before;
        }
        lds_barrier();
        double now = 0.0, prev = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) {
            now += waves[w];
            prev += waves[NT / 64 + w];
        }
        const bool done = A->part_in && (prev <= A->thr || !isfinite(prev));
        if (tid == 0) {
            A->part_out[tile] = now;
            if (A->part_in && blockIdx.x == 0) {
                *A->sum = prev;
                if (done)
                    *A->stop = A->q;
            }
        }
        if (done)
            return;
    }

    // ---- the phases
    fs_phases<GRP * PH, GRP * PH + PH>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
#pragma unroll
        for (int m = 0; m < S::rounds(c); ++m) {
            int i, j, k;
            if (!node(cc, tid + m * NT, i, j, k))
                continue;
            bool nc = false;
            su[lds_off(i, j, k)] = value(i, j, k, f[S::before(c) + m], false, nc);
            // recomputed halo nodes are counted by their own block
            if (nc && ncount && i >= x0 && i < x1 && j >= y0 && j < y1 && k >= z0 && k < z1)
                atomicAdd(ncount + G.slot, 1ull);
        }
        lds_barrier();
    });

    // ---- the owned block and the Dirichlet layer next to it to u_out
    const int xs0 = x0 == 1 ? 0 : x0, xs1 = x1 == n ? n + 1 : x1;
    const int ys0 = y0 == 1 ? 0 : y0, ys1 = y1 == n ? n + 1 : y1;
    const int zs0 = z0 == 1 ? 0 : z0, zs1 = z1 == n ? n + 1 : z1;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        const int el = tid + k * NT;
        const int c2 = el / (S::SX * S::SY), rem = el - c2 * (S::SX * S::SY);
        const int b = rem / S::SX, a = rem - b * S::SX;
        const int gx = xs0 + a, gy = ys0 + b, gz = zs0 + c2;
        if (el < S::SX * S::SY * S::SZ && gx < xs1 && gy < ys1 && gz < zs1)
            uout[gx + sy * gy + sz * gz] = su[lds_off(gx, gy, gz)];
    }
}

// Blocks are dispatched round-robin over the 8 XCDs; tile_of_block gives
// each XCD a contiguous range of tiles, so tiles that share halos share an
// L2.  One tile per workgroup.
template <int OP, int ORDER, int PH, int GRP, int TX, int TY, int TZ, int NT>
__global__ __launch_bounds__(NT) void k_bsweep(const FsList *__restrict__ L,
                                                unsigned long long *__restrict__ ncount)
{
    __shared__ double su[FsShape<ORDER, PH, TX, TY, TZ, NT>::NL];
    const int total = L->total;
    const int t = tile_of_block(int(blockIdx.x), int(gridDim.x));
    if (t >= total)
        return;
    const int ng = L->ngrids;
    int g = 0;
    while (g + 1 < ng && L->g[g + 1].start <= t)
        ++g;
    const FsGrid G = L->g[g];   // the whole descriptor in one set of loads
    if ((L->stopped >> G.slot) & 1ull)
        return;
    bsweep_tile<OP, ORDER, PH, GRP, TX, TY, TZ, NT, false>(G, t - G.start, su, ncount);
}

// The same for one grid passed by value (gridDim.x = its tile count).
template <int OP, int ORDER, int PH, int GRP, int TX, int TY, int TZ, int NT>
__global__ __launch_bounds__(NT) void k_bsweep1(FsGrid G, unsigned long long *__restrict__ ncount)
{
    __shared__ double su[FsShape<ORDER, PH, TX, TY, TZ, NT>::NL];
    const int t = tile_of_block(int(blockIdx.x), int(gridDim.x));
    bsweep_tile<OP, ORDER, PH, GRP, TX, TY, TZ, NT, false>(G, t, su, ncount);
}

template <int ORDER, int TX, int TY, int TZ, int NT>
__global__ __launch_bounds__(NT) void k_gs_step(FsGrid G, GsStep A)
{
    constexpr int PH = ORDER == 0 ? 4 : 8;
    __shared__ double su[FsShape<ORDER, PH, TX, TY, TZ, NT>::NL];
    __shared__ double waves[NT / 32];
    const int blocks = int(gridDim.x);
    bsweep_tile<OP_MA, ORDER, PH, 0, TX, TY, TZ, NT, true>(G, tile_of_block(int(blockIdx.x), blocks), su,
                                                    A.count, &A, blocks, waves);
}

} // namespace mafas
