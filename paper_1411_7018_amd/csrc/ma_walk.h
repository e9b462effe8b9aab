// The 19-point stencil of a wavefront that walks a row of 64 columns along z.
// A lane loads its own column of three rows; the columns beside it come from
// its neighbours through DPP, and only lanes 0 and 63 load theirs.  Each plane
// is reduced at once to the six differences that its nodes and those of the
// planes beside it need, so the registers hold kAhead planes in flight: a walk
// is bound by the latency of its planes, one after the other, until enough of
// them are.
#pragma once

#include "ma_device.h"

namespace mafas {

// v of the lane before (after) this one; e in lane 0 (63).  Every lane active.
template <int CTRL>
__device__ __forceinline__ double wave_shift(double v, double e)
{
    const long long vb = __builtin_bit_cast(long long, v), eb = __builtin_bit_cast(long long, e);
    const int lo = __builtin_amdgcn_update_dpp(int(eb), int(vb), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(int(eb >> 32), int(vb >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
__device__ __forceinline__ double lane_left(double v, double e)
{
    return wave_shift<0x138>(v, e);   // wave_shr:1
}
__device__ __forceinline__ double lane_right(double v, double e)
{
    return wave_shift<0x130>(v, e);   // wave_shl:1
}

// One plane as loaded: rows j - 1, j, j + 1 at this lane's column, and (lanes 0
// and 63) the column outside the wavefront.
struct PlaneRows {
    double m[3], e[3];
};

// What the stencils take from a plane: the centre, the second differences in x
// and y, the mixed one, and the first differences over two columns and rows.
struct PlaneTerms {
    double c, xx, yy, xy, gx, gy;
};

// The differences are those of hessian3, in its order.
__device__ __forceinline__ PlaneTerms plane_terms(const PlaneRows &R)
{
    const double c = R.m[1];
    const double w = lane_left(c, R.e[1]), e = lane_right(c, R.e[1]);
    const double sw = lane_left(R.m[0], R.e[0]), se = lane_right(R.m[0], R.e[0]);
    const double nw = lane_left(R.m[2], R.e[2]), ne = lane_right(R.m[2], R.e[2]);
    PlaneTerms T;
    T.c = c;
    T.xx = (e - c) - (c - w);
    T.yy = (R.m[2] - c) - (c - R.m[0]);
    T.xy = (ne - nw) - (se - sw);
    T.gx = e - w;
    T.gy = R.m[2] - R.m[0];
    return T;
}

// hessian3 and laplacian3 of the node in plane C between planes D and U.
__device__ __forceinline__ Hess hessian_planes(const PlaneTerms &D, const PlaneTerms &C,
                                               const PlaneTerms &U, double s, double s4)
{
    Hess g;
    g.xx = C.xx * s;
    g.yy = C.yy * s;
    g.zz = ((U.c - C.c) - (C.c - D.c)) * s;
    g.xy = C.xy * s4;
    g.xz = (U.gx - D.gx) * s4;
    g.yz = (U.gy - D.gy) * s4;
    return g;
}
__device__ __forceinline__ double laplacian_planes(const PlaneTerms &D, const PlaneTerms &C,
                                                   const PlaneTerms &U, double s)
{
    return (C.xx + C.yy + ((U.c - C.c) - (C.c - D.c))) * s;
}

// Walk columns i (any; loads are clamped into the grid) of row j (1 <= j <=
// n - 1) over planes k0 .. k0 + PLANES - 1 below k1 (k1 uniform, k0 >= 0):
// node(k, C, D, U, f) takes the terms of plane k and of those below and above it
// and F there (f is F's value at the nearest interior node of lanes and planes
// outside the interior).
template <int PLANES, typename PU, typename PF, typename N>
__device__ __forceinline__ void walk_planes(PU u, PF F, int n, int i, int j, int k0, int k1,
                                            int lane, N node)
{
    constexpr int kAhead = PLANES < 3 ? PLANES : 3;
    const long sy = n + 1, sz = sy * sy;
    const bool outer = lane == 0 || lane == 63;
    const long at = min(max(i, 0), n) + sy * j;
    const long edge = min(max(lane == 0 ? i - 1 : i + 1, 0), n) + sy * j;
    const long fat = min(max(i, 1), n - 1) + sy * j;
    auto load = [&](int k, PlaneRows &R) {
        const long z = sz * min(max(k, 0), n);
#pragma unroll
        for (int y = 0; y < 3; ++y)
            R.m[y] = u[at + z + sy * (y - 1)];
        if (outer)
#pragma unroll
            for (int y = 0; y < 3; ++y)
                R.e[y] = u[edge + z + sy * (y - 1)];
    };
    auto rhs = [&](int k) { return F[fat + sz * min(max(k, 1), n - 1)]; };
    PlaneRows R[kAhead], R0, R1;
    double f[kAhead];
    load(k0 - 1, R0);
    load(k0, R1);
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
        load(k0 + 1 + q, R[q]);
        f[q] = rhs(k0 + q);
    }
    PlaneTerms D = plane_terms(R0), C = plane_terms(R1);
#pragma unroll
    for (int m = 0; m < PLANES; ++m) {
        const int k = k0 + m;
        if (k >= k1)
            break;
        const PlaneTerms U = plane_terms(R[m % kAhead]);
        const double fc = f[m % kAhead];
        if (m + kAhead < PLANES) {
            load(k + 1 + kAhead, R[m % kAhead]);
            f[m % kAhead] = rhs(k + kAhead);
        }
        node(k, C, D, U, fc);
        D = C;
        C = U;
    }
}

} // namespace mafas
