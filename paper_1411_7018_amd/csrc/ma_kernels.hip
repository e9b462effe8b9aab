// FP64 kernels of the FAS V-cycle (Algorithm 1) for det(D^2 u) = f and of
// the linear 7-point V-cycle used for the initial guess.  All grid functions
// are (n+1)^3 x-fastest arrays; Dirichlet nodes are read, never written.
#include "ma_device.h"
#include "ma_walk.h"
#include "ma_internal.h"
#include "ma_runtime.h"

namespace mafas {

namespace {

constexpr int RES_BX = 64;   // residual / transfer block: 64 x 4 threads
constexpr int RES_BY = 4;

__device__ __forceinline__ double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_down(v, off, 64);
    return v;
}

// Sum over a block of exactly nwaves full wavefronts, fixed order.
template <int NWAVES>
__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double part[NWAVES];
    const int lane = threadIdx.x & 63;
    const int wid = (threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z)) >> 6;
    v = wave_sum(v);
    if (lane == 0)
        part[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (wid == 0 && lane == 0)
        for (int w = 0; w < NWAVES; ++w)
            t += part[w];
    return t;
}

// ---------------------------------------------------------------------------
// Smoother, one launch per colour phase.  Colour of node (i,j,k):
//   4 colours: ((i+j) mod 2) + 2 ((i+k) mod 2)   [i = j + c0, k parity from c1]
//   8 colours: (i mod 2) + 2 (j mod 2) + 4 (k mod 2)
// Nodes of one colour are never stencil neighbours, so the in-place updates
// of a phase do not interact.
// ---------------------------------------------------------------------------
template <int OP, int ORDER>
__global__ __launch_bounds__(64 * kRowWaves) void k_sweep_color(
    double *__restrict__ u, const double *__restrict__ F, int n, unsigned md, int waves, int color,
    int gy, int gz, int nb, double s, double s4, double hk, unsigned long long *__restrict__ ncount)
{
    // One wavefront per colour item (rows packed: with a row in segments of 64 a
    // row of 65-95 nodes left its second wavefront mostly idle; two sweeps, us,
    // segments / packed: 4 colours n = 66: 31.7 / 28.4, 96: 43.4 / 40.0, 128:
    // 62.3 / 62.3, 130: 97.7 / 67.0, 160: 145 / 108, 240: 320 / 305; 8 colours n =
    // 104: 62.4 / 59.4, 127: 76.5 / 77.8); blocks in XCD-contiguous order.
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = tile_of_block(blockIdx.x, nb) * waves + wave;
    const int bz = q / gy, by = q - bz * gy;
    if (bz >= gz)
        return;
    int i, j, k;
    colour_node<ORDER>(color, n, md, by, bz, int(threadIdx.x & 63), i, j, k);
    if (i > n - 1 || j > n - 1 || k > n - 1)
        return;
    const long sy = n + 1, sz = sy * sy;
    const long p = i + sy * j + sz * k;
    if (OP == OP_MA) {
        const Hess g = hessian_at(u, p, 1, sy, sz, s, s4);
        bool nc = false;
        u[p] = ma_point_update(g, u[p], F[p], hk, nc);
        if (nc && ncount)
            atomicAdd(ncount, 1ull);
    } else {
        u[p] = lap_point_update(laplacian_at(u, p, 1, sy, sz, s), u[p], F[p], hk);
    }
}

// ---------------------------------------------------------------------------
// Residual r = F - S(u) (0 on the boundary; r may be null) and per-block sums
// of r^2 over interior nodes.  A wavefront takes 64 columns of one row and
// walks a chunk of planes along z (ma_walk.h).  Bound by HBM; 298^3 with r: 375
// us as a gather and a separate clear of r, 250 us with nine loads a node and a
// plane in flight, 204 us so.  On small grids a launch lasts as long as one
// wavefront's walk, so their chunks are two planes; residual and norm, us, a
// gather / chunks of eight / of two: n = 32: 19.3 / 21.5 / 19.3, 64: 20.6 / 23.1 /
// 20.9, 72: 24.0 / 23.1 / 22.8.
// ---------------------------------------------------------------------------
constexpr int kResPlanes = 8, kResPlanesSmall = 2;
int residual_planes(int n) { return n <= 65 ? kResPlanesSmall : kResPlanes; }
// First column of a row's wavefronts: 1 where that saves the row a wavefront of
// one or two columns (its end columns then write the boundary ones beside them),
// else 0, without the end columns' stores.  Us, from 0 / 1: residual and norm, 64:
// 22.0 / 20.9, 129: 33.2 / 30.4; residual, 96: 11.6 / 12.4, 130: 19.5 / 20.7.
int residual_column(int n) { return n >= 64 && n % RES_BX <= 1 ? 1 : 0; }

template <int OP, int PLANES>
__global__ __launch_bounds__(RES_BX *RES_BY) void k_residual(const double *__restrict__ u,
                                                             const double *__restrict__ F,
                                                             double *__restrict__ r,
                                                             double *__restrict__ partials,
                                                             int n, int x0, double s,
                                                             double s4)
{
    const int i = x0 + blockIdx.x * RES_BX + threadIdx.x;
    const int j = blockIdx.y * RES_BY + threadIdx.y;
    const int k0 = blockIdx.z * PLANES, k1 = min(k0 + PLANES, n + 1);
    const bool col = i >= 1 && i <= n - 1 && j >= 1 && j <= n - 1;
    const int sy = n + 1;
    const long sz = long(sy) * sy;
    double acc = 0.0;
    walk_planes<PLANES>(u, F, n, i, min(max(j, 1), n - 1), k0, k1, int(threadIdx.x),
                            [&](int k, const PlaneTerms &C, const PlaneTerms &D,
                                const PlaneTerms &U, double f) {
        double rv;
        if (OP == OP_MA)
            rv = f - det3(hessian_planes(D, C, U, s, s4));
        else
            rv = f - laplacian_planes(D, C, U, s);
        if (!col || k < 1 || k > n - 1)
            rv = 0.0;
        acc = fma(rv, rv, acc);
        if (r && i <= n && j <= n) {
            double *p = r + (i + long(sy) * j + sz * k);
            *p = rv;
            if (x0 == 1 && i == 1)
                p[-1] = 0.0;
            if (x0 == 1 && i == n - 1)
                p[1] = 0.0;
        }
    });
    const double t = block_sum<RES_BX * RES_BY / 64>(acc);
    if (threadIdx.x == 0 && threadIdx.y == 0)
        partials[blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * size_t(blockIdx.z))] = t;
}

// Fixed-order sum of count partials by one block of 1024 threads: thread t
// adds partials t, t + 1024, ... in order, with the loads of eight steps in
// flight together (one load a step waited out the memory latency each time:
// 101 us for the 266k partials of an 8193^2 grid).
__global__ __launch_bounds__(1024) void k_reduce(const double *__restrict__ partials,
                                                 size_t count, double *__restrict__ out)
{
    double v = 0.0;
    size_t q = threadIdx.x;
    for (; q + 7 * 1024 < count; q += 8 * 1024) {
        double a[8];
#pragma unroll
        for (int m = 0; m < 8; ++m)
            a[m] = partials[q + m * 1024];
#pragma unroll
        for (int m = 0; m < 8; ++m)
            v += a[m];
    }
    for (; q < count; q += 1024)
        v += partials[q];
    const double t = block_sum<16>(v);
    if (threadIdx.x == 0)
        out[0] = t;
}

__global__ void k_poisson_rhs(const double *__restrict__ f, double *__restrict__ R, size_t count)
{
    const size_t q = blockIdx.x * size_t(blockDim.x) + threadIdx.x;
    if (q < count)
        R[q] = 3.0 * cbrt(f[q]);
}

__global__ void k_copy(const double *__restrict__ src, double *__restrict__ dst, size_t count)
{
    const size_t q = blockIdx.x * size_t(blockDim.x) + threadIdx.x;
    if (q < count)
        dst[q] = src[q];
}

// A look at device scalars: copied out (dst: pinned host memory) and cleared.
__global__ void k_take(double *__restrict__ src, double *__restrict__ dst, size_t count)
{
    const size_t q = blockIdx.x * size_t(blockDim.x) + threadIdx.x;
    if (q < count) {
        dst[q] = src[q];
        src[q] = 0.0;
    }
}

// Injection of u and f onto every coarser level at once: each coarse node,
// boundary included, takes the finest value at the same point.
__global__ __launch_bounds__(256) void k_inject_levels(InjectLevels A)
{
    int l = 0;
    while (l + 1 < A.levels && int(blockIdx.x) >= A.block[l + 1])
        ++l;
    const int n = A.n0 >> (l + 1), m = n + 1;
    const long q = (long(blockIdx.x) - A.block[l]) * 256 + threadIdx.x;
    if (q >= long(m) * m * m)
        return;
    const int I = int(q % m), J = int(q / m % m), K = int(q / m / m);
    const long fy = A.n0 + 1L, st = 2L << l;
    const long p = st * (I + fy * (J + fy * K));
    A.u[l][q] = A.u0[p];
    A.f[l][q] = A.f0[p];
}

// 1D rule of the FMG interpolation at fine index i (nf = 2 nc intervals):
// a coarse node is copied; a midpoint takes the cubic Lagrange value through
// the four nearest coarse nodes (one-sided next to the boundary), or the
// quadratic value when the coarse grid has only three nodes.
__device__ __forceinline__ int fmg_rule(int nc, int i, int &first, double w[4])
{
    if ((i & 1) == 0) {
        first = i >> 1;
        w[0] = 1.0;
        return 1;
    }
    const int m = i >> 1;  // midpoint between coarse m and m + 1
    if (nc < 3) {
        first = 0;
        w[0] = m == 0 ? 0.375 : -0.125;
        w[1] = 0.75;
        w[2] = m == 0 ? -0.125 : 0.375;
        return 3;
    }
    if (m == 0) {
        first = 0;
        w[0] = 0.3125; w[1] = 0.9375; w[2] = -0.3125; w[3] = 0.0625;
    } else if (m == nc - 1) {
        first = nc - 3;
        w[0] = 0.0625; w[1] = -0.3125; w[2] = 0.9375; w[3] = 0.3125;
    } else {
        first = m - 1;
        w[0] = -0.0625; w[1] = 0.5625; w[2] = 0.5625; w[3] = -0.0625;
    }
    return 4;
}

// FMG values at the odd fine column 2m + 1 and the even one after it, CK x CJ x
// CI coarse nodes from (fi, fj, fk) on, the even column's at m + 1; summed over
// (k, j, i) offsets in order.
template <int CK, int CJ, int CI>
__device__ __forceinline__ void fmg_pair(const double *__restrict__ uc, long cy, int m, int fi,
                                         int fj, int fk, const double *wi, const double *wj,
                                         const double *wk, double &odd, double &even)
{
    double o = 0.0, e = 0.0;
#pragma unroll
    for (int c = 0; c < CK; ++c)
#pragma unroll
        for (int b = 0; b < CJ; ++b) {
            const double *row = uc + cy * ((fj + b) + cy * (fk + c));
#pragma unroll
            for (int a = 0; a < CI; ++a)
                o += wk[c] * wj[b] * wi[a] * row[fi + a];
            e += wk[c] * wj[b] * row[m + 1];
        }
    odd = o;
    even = e;
}

// FMG interpolation (Algorithm 2, step 4) into the interior of uf: tensor
// product of the 1D rule.  A wavefront takes one row, so the taps in y and z
// are the same for its lanes, and a lane two neighbouring columns, so the odd
// one's four taps in x are nobody else's wait.  128^3: 40 us with a node a lane
// and loops of 1 or 4 turns in each direction, 16 us so.
__global__ __launch_bounds__(RES_BX *RES_BY) void k_fmg_interp(const double *__restrict__ uc,
                                                               double *__restrict__ uf, int nc)
{
    const int nf = 2 * nc;
    const int m0 = blockIdx.x * RES_BX + threadIdx.x, m = min(m0, nc - 1);
    const int j = 1 + blockIdx.y * RES_BY + __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int k = 1 + blockIdx.z;
    if (j > nf - 1)
        return;
    int fi, fj, fk;
    double wi[4], wj[4], wk[4];
    fmg_rule(nc, 2 * m + 1, fi, wi);
    const int cj = fmg_rule(nc, j, fj, wj);
    const int ck = fmg_rule(nc, k, fk, wk);
    const long cy = nc + 1;
    double odd, even;
    if (nc < 3) {
        if (ck == 1 && cj == 1)
            fmg_pair<1, 1, 3>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
        else if (ck == 1)
            fmg_pair<1, 3, 3>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
        else if (cj == 1)
            fmg_pair<3, 1, 3>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
        else
            fmg_pair<3, 3, 3>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
    } else if (ck == 1 && cj == 1) {
        fmg_pair<1, 1, 4>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
    } else if (ck == 1) {
        fmg_pair<1, 4, 4>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
    } else if (cj == 1) {
        fmg_pair<4, 1, 4>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
    } else {
        fmg_pair<4, 4, 4>(uc, cy, m, fi, fj, fk, wi, wj, wk, odd, even);
    }
    double *row = uf + long(nf + 1) * (j + long(nf + 1) * k);
    if (m0 < nc)
        row[2 * m + 1] = odd;
    if (m0 < nc - 1)
        row[2 * m + 2] = even;
}

// Zero the interior nodes of an (n+1)^3 grid.
__global__ void k_zero_interior(double *__restrict__ u, int n)
{
    const int i = 1 + blockIdx.x * RES_BX + threadIdx.x;
    const int j = 1 + blockIdx.y * RES_BY + threadIdx.y;
    const int k = 1 + blockIdx.z;
    if (i > n - 1 || j > n - 1)
        return;
    u[i + long(n + 1) * (j + long(n + 1) * k)] = 0.0;
}

inline dim3 res_grid(int cnt_x, int cnt_y, int cnt_z)
{
    return dim3((cnt_x + RES_BX - 1) / RES_BX, (cnt_y + RES_BY - 1) / RES_BY, cnt_z);
}

} // namespace

namespace {
dim3 residual_grid(int n)
{
    return dim3((n - 2 * residual_column(n) + RES_BX) / RES_BX, (n + RES_BY) / RES_BY,
                (n + residual_planes(n)) / residual_planes(n));
}
} // namespace

size_t residual_partials(int n)
{
    const dim3 g = residual_grid(n);
    return size_t(g.x) * g.y * g.z;
}

hipError_t launch_sweep_color(hipStream_t st, int op, int order, int n, double *u,
                              const double *F, unsigned long long *nonconvex)
{
    const double s = double(n) * double(n), s4 = 0.25 * s;
    const double hk = op == OP_MA ? 0.5 / s : 1.0 / (6.0 * s);
    const int ncol = order == 1 ? 8 : 4;
    const int gy = colour_items(n, order == 0 ? n - 1 : n / 2), gz = n / 2;
    const int w = row_waves(gy * gz), nb = (gy * gz + w - 1) / w;
    const unsigned md = colour_div(n);
    for (int c = 0; c < ncol; ++c) {
#define MA_COLOR_LAUNCH(OPV, ORD)                                                                \
    hipLaunchKernelGGL((k_sweep_color<OPV, ORD>), dim3(nb), dim3(64 * w), 0, st, u, F, n, md, w, \
                       c, gy, gz, nb, s, s4, hk, nonconvex)
        if (op == OP_MA) {
            if (order == 0)
                MA_COLOR_LAUNCH(OP_MA, 0);
            else
                MA_COLOR_LAUNCH(OP_MA, 1);
        } else {
            if (order == 0)
                MA_COLOR_LAUNCH(OP_LAP, 0);
            else
                MA_COLOR_LAUNCH(OP_LAP, 1);
        }
#undef MA_COLOR_LAUNCH
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_residual(hipStream_t st, int op, int n, const double *u, const double *F,
                           double *r, double *partials)
{
    const double s = double(n) * double(n), s4 = 0.25 * s;
    const dim3 grid = residual_grid(n), block(RES_BX, RES_BY);
    const bool small = residual_planes(n) == kResPlanesSmall;
#define MA_RESIDUAL_LAUNCH(OPV, PL)                                                              \
    hipLaunchKernelGGL((k_residual<OPV, PL>), grid, block, 0, st, u, F, r, partials, n,       \
                       residual_column(n), s, s4)
    if (op == OP_MA) {
        if (small)
            MA_RESIDUAL_LAUNCH(OP_MA, kResPlanesSmall);
        else
            MA_RESIDUAL_LAUNCH(OP_MA, kResPlanes);
    } else {
        if (small)
            MA_RESIDUAL_LAUNCH(OP_LAP, kResPlanesSmall);
        else
            MA_RESIDUAL_LAUNCH(OP_LAP, kResPlanes);
    }
#undef MA_RESIDUAL_LAUNCH
    return hipGetLastError();
}

hipError_t launch_reduce(hipStream_t st, const double *partials, size_t count, double *out)
{
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(1024), 0, st, partials, count, out);
    return hipGetLastError();
}

hipError_t launch_poisson_rhs(hipStream_t st, int n, const double *f, double *R)
{
    const size_t cnt = npts(n);
    hipLaunchKernelGGL(k_poisson_rhs, dim3((cnt + 255) / 256), dim3(256), 0, st, f, R, cnt);
    return hipGetLastError();
}

hipError_t launch_copy(hipStream_t st, size_t count, const double *src, double *dst)
{
    if (count == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_copy, dim3((count + 255) / 256), dim3(256), 0, st, src, dst, count);
    return hipGetLastError();
}

hipError_t launch_take(hipStream_t st, size_t count, double *src, double *dst)
{
    hipLaunchKernelGGL(k_take, dim3((count + 255) / 256), dim3(256), 0, st, src, dst, count);
    return hipGetLastError();
}

hipError_t launch_inject_levels(hipStream_t st, InjectLevels &A)
{
    long blocks = 0;
    for (int l = 0; l < A.levels; ++l) {
        const long m = (A.n0 >> (l + 1)) + 1;
        A.block[l] = int(blocks);
        blocks += (m * m * m + 255) / 256;
    }
    if (blocks == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_inject_levels, dim3(unsigned(blocks)), dim3(256), 0, st, A);
    return hipGetLastError();
}

hipError_t launch_fmg_interp(hipStream_t st, int nc, const double *uc, double *uf)
{
    const int nf = 2 * nc;
    hipLaunchKernelGGL(k_fmg_interp, res_grid(nc, nf - 1, nf - 1), dim3(RES_BX, RES_BY), 0, st,
                       uc, uf, nc);
    return hipGetLastError();
}

hipError_t launch_zero_interior(hipStream_t st, int n, double *u)
{
    if (n < 2)
        return hipSuccess;
    hipLaunchKernelGGL(k_zero_interior, res_grid(n - 1, n - 1, n - 1), dim3(RES_BX, RES_BY), 0, st,
                       u, n);
    return hipGetLastError();
}

} // namespace mafas

namespace mafas {
namespace {
template <typename T>
__global__ void k_fill(T *__restrict__ dst, size_t count, T v)
{
    const size_t q = blockIdx.x * size_t(blockDim.x) + threadIdx.x;
    if (q < count)
        dst[q] = v;
}
} // namespace

hipError_t launch_fill(hipStream_t st, size_t count, double v, double *dst)
{
    if (count == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_fill<double>, dim3((count + 255) / 256), dim3(256), 0, st, dst, count, v);
    return hipGetLastError();
}

hipError_t launch_fill_u64(hipStream_t st, size_t count, unsigned long long v,
                           unsigned long long *dst)
{
    if (count == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_fill<unsigned long long>, dim3((count + 255) / 256), dim3(256), 0, st, dst,
                       count, v);
    return hipGetLastError();
}

} // namespace mafas
