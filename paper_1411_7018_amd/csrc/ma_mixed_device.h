// Device-side pieces of the FP32/FP64 mixed-precision inner problem
// T(delta) = det(H + D^2 delta) - det(H) = r (see ma_mixed.hip).
#pragma once

#include "ma_device.h"

namespace mafas {

struct Sym32 {
    float xx, yy, zz, xy, xz, yz;
};

__device__ __forceinline__ Sym32 to32(const Hess &h)
{
    return Sym32{float(h.xx), float(h.yy), float(h.zz), float(h.xy), float(h.xz), float(h.yz)};
}

// E = D^2 delta at index p (FP32 data, FP32 arithmetic).
template <typename PD>
__device__ __forceinline__ Sym32 hess32(PD d, long p, long sx, long sy, long sz, float s, float s4)
{
#pragma clang fp contract(off)
    const float c = d[p];
    Sym32 e;
    e.xx = ((d[p + sx] - c) - (c - d[p - sx])) * s;
    e.yy = ((d[p + sy] - c) - (c - d[p - sy])) * s;
    e.zz = ((d[p + sz] - c) - (c - d[p - sz])) * s;
    e.xy = ((d[p + sx + sy] - d[p - sx + sy]) - (d[p + sx - sy] - d[p - sx - sy])) * s4;
    e.xz = ((d[p + sx + sz] - d[p - sx + sz]) - (d[p + sx - sz] - d[p - sx - sz])) * s4;
    e.yz = ((d[p + sy + sz] - d[p - sy + sz]) - (d[p + sy - sz] - d[p - sy - sz])) * s4;
    return e;
}

// The same from the 3 x 3 neighbourhoods (x stride 1, y stride 3) of the planes
// below, at and above the node.
__device__ __forceinline__ Sym32 hess32_win(const float *D, const float *C, const float *U,
                                            float s, float s4)
{
#pragma clang fp contract(off)
    const float c = C[0];
    Sym32 e;
    e.xx = ((C[1] - c) - (c - C[-1])) * s;
    e.yy = ((C[3] - c) - (c - C[-3])) * s;
    e.zz = ((U[0] - c) - (c - D[0])) * s;
    e.xy = ((C[4] - C[2]) - (C[-2] - C[-4])) * s4;
    e.xz = ((U[1] - U[-1]) - (D[1] - D[-1])) * s4;
    e.yz = ((U[3] - U[-3]) - (D[3] - D[-3])) * s4;
    return e;
}

// The products below are fused where they are written as fmaf and nowhere else
// (fp contract off), so a node's result does not depend on the kernel that the
// compiler inlined them into.
__device__ __forceinline__ Sym32 adj32(const Sym32 &a)
{
#pragma clang fp contract(off)
    return Sym32{fmaf(a.yy, a.zz, -(a.yz * a.yz)), fmaf(a.xx, a.zz, -(a.xz * a.xz)),
                 fmaf(a.xx, a.yy, -(a.xy * a.xy)), fmaf(a.xz, a.yz, -(a.xy * a.zz)),
                 fmaf(a.xy, a.yz, -(a.xz * a.yy)), fmaf(a.xy, a.xz, -(a.xx * a.yz))};
}

// tr(A B) for symmetric A, B.
__device__ __forceinline__ float trprod(const Sym32 &a, const Sym32 &b)
{
#pragma clang fp contract(off)
    const float o = fmaf(a.yz, b.yz, fmaf(a.xz, b.xz, a.xy * b.xy));
    return fmaf(2.0f, o, fmaf(a.zz, b.zz, fmaf(a.yy, b.yy, a.xx * b.xx)));
}

__device__ __forceinline__ float det32(const Sym32 &a, const Sym32 &adja)
{
#pragma clang fp contract(off)
    return fmaf(a.xz, adja.xz, fmaf(a.xy, adja.xy, a.xx * adja.xx));
}

// T(E) = det(H + E) - det(H) through the identity.
__device__ __forceinline__ float t_of(const Sym32 &H, const Sym32 &adjH, const Sym32 &E)
{
#pragma clang fp contract(off)
    const Sym32 adjE = adj32(E);
    return trprod(adjH, E) + trprod(H, adjE) + det32(E, adjE);
}

struct LevelConst {
    double s, s4;
    float sf, s4f, hkf;
};

__host__ __device__ __forceinline__ LevelConst level_const(int n)
{
    LevelConst c;
    c.s = double(n) * double(n);
    c.s4 = 0.25 * c.s;
    c.sf = float(c.s);
    c.s4f = float(c.s4);
    c.hkf = float(0.5 / c.s);
    return c;
}

// A node of U in memory: its index and the strides of its level's neighbours.
template <typename PU>
struct UNode {
    PU u;
    long p, sx, sy, sz;
};

// FP64 recomputation of one node: sigma of det(H + E - sigma I) = det(H) + r.
// Inlined: as a call its registers and the caller's add up to half the waves.
template <typename PU, typename PD>
__device__ __forceinline__ double mixed_fp64_root(const UNode<PU> &U, PD d, long p, long sy,
                                                  long sz, double s, double s4, float r,
                                                  bool &nonconvex)
{
#pragma clang fp contract(off)
    const Hess H = hessian_at(U.u, U.p, U.sx, U.sy, U.sz, s, s4);
    const Hess E = hessian_at(d, p, 1, sy, sz, s, s4);
    const double F = det3(H) + double(r);
    Hess G;
    G.xx = H.xx + E.xx;
    G.yy = H.yy + E.yy;
    G.zz = H.zz + E.zz;
    G.xy = H.xy + E.xy;
    G.xz = H.xz + E.xz;
    G.yz = H.yz + E.yz;
    return smallest_root(G, F, nonconvex);
}

// New delta at node p of a level with constants lc, H = D^2 U there in FP32:
// returns the updated value and flags.
template <typename PD, typename PU>
__device__ __forceinline__ float mixed_point(const Sym32 &H, PD d, const UNode<PU> &U, float b,
                                             long p, long sy, long sz, const LevelConst &lc, bool &fallback,
                                             bool &nonconvex)
{
#pragma clang fp contract(off)
    const Sym32 adjH = adj32(H);
    const Sym32 E = hess32(d, p, 1, sy, sz, lc.sf, lc.s4f);
    const float T = t_of(H, adjH, E);
    const float detH = det32(H, adjH);
    const Sym32 G{H.xx + E.xx, H.yy + E.yy, H.zz + E.zz, H.xy + E.xy, H.xz + E.xz, H.yz + E.yz};
    const float I1 = G.xx + G.yy + G.zz;
    const Sym32 adjG = adj32(G);
    const float mab = adjG.zz;
    const float I2 = mab + adjG.yy + adjG.xx;
    const float detG = det32(G, adjG);
    const float sc = fabsf(I1) * (1.0f / 3.0f);
    const float m = 1e-3f;
    bool ok = G.xx > m * sc && mab > m * sc * sc && detG > m * sc * sc * sc &&
              detH + b > m * fabsf(detH);
    float sig = 0.0f;
    if (ok) {
        // Stop once the step is below 2e-6 of sigma: the quadratic error
        // left is ~1e-11 of sigma, far below the FP32 noise of q itself,
        // and the outer FP64 residual absorbs what FP32 cannot resolve.
        const float c0 = T - b;
        int it = 0;
#pragma unroll 1
        for (; it < 16; ++it) {
            const float q = fmaf(fmaf(I1 - sig, sig, -I2), sig, c0);
            const float dq = fmaf(fmaf(-3.0f, sig, 2.0f * I1), sig, -I2);
            // a step's own rounding is below the stopping bound squared, so
            // one reciprocal (1 ulp) does
            const float dd = q * __builtin_amdgcn_rcpf(dq);
            sig = sig - dd;
            if (!(fabsf(dd) > 2e-6f * fabsf(sig)))
                break;
        }
        ok = it < 16 && isfinite(sig);
    }
    if (!ok) {
        fallback = true;
        const double sg = mixed_fp64_root(U, d, p, sy, sz, lc.s, lc.s4, b, nonconvex);
        return float(fma(sg, 0.5 / lc.s, double(d[p])));
    }
    return fmaf(sig, lc.hkf, d[p]);
}

} // namespace mafas
