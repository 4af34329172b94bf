// Device helpers shared by the D2Q9 kernels (both fused variants and the
// field-form step): address space views, DPP lane shifts, the
// pairwise-difference stencils, the cubic EOS per site and per component,
// helper wave placement, the factored D2Q9 collision, the LDS block and the
// population row type.
//
// Every D2Q9 kernel gives bitwise the same state, whichever of them takes a
// step, so each rounding is written out here: no contraction by the
// compiler (which would depend on the caller), explicit fma where one is
// meant, and one function per term for all of them.
#pragma once

#include "kernels.h"

#pragma clang fp contract(off)

namespace fused {

// Address-space-qualified views: constant (scalar loads) and global.
template <class T> using cptr = const __attribute__((address_space(4))) T *;
template <class T> using gptr = const __attribute__((address_space(1))) T *;
template <class T> using gmptr = __attribute__((address_space(1))) T *;

// DPP wavefront shifts (GFX9 family): lane l receives lane l-1 (wave_shr:1)
// or lane l+1 (wave_shl:1).  Lanes 0 / 63 receive 0; only lanes 1..62 use
// shifted values.
__device__ __forceinline__ double from_left(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x138, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_right(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x130, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// One row of a field at a lane: own column and its west / east neighbours.
// A ring of these needs each lane shift once per row instead of once per
// stencil that reads it.
struct Row3 {
    double w, c, e;
};
__device__ __forceinline__ Row3 row3(double v) { return {from_left(v), v, from_right(v)}; }

// Pairwise-difference D2Q9 gradient from a 3x3 neighbourhood (S = row
// below, C = own row, N = row above).
__device__ __forceinline__ void grad3(const Row3 &S, const Row3 &C, const Row3 &N, double &gx,
                                      double &gy) {
    const double d1 = C.e - C.w, d2 = N.c - S.c, d5 = N.e - S.w, d6 = N.w - S.e;
    const double m5 = (1.0 / 36.0) * d5;
    gx = 3.0 * fma(-1.0 / 36.0, d6, fma(1.0 / 9.0, d1, m5));
    gy = 3.0 * fma(1.0 / 36.0, d6, fma(1.0 / 9.0, d2, m5));
}
__device__ __forceinline__ void grad3(double S, double C, double N, double &gx, double &gy) {
    grad3(row3(S), row3(C), row3(N), gx, gy);
}

__device__ __forceinline__ double lap3(const Row3 &S, const Row3 &C, const Row3 &N) {
    const double ax = (C.e - C.c) + (N.c - C.c) + (C.w - C.c) + (S.c - C.c);
    const double dg = (N.e - C.c) + (N.w - C.c) + (S.w - C.c) + (S.e - C.c);
    return 6.0 * fma(1.0 / 9.0, ax, (1.0 / 36.0) * dg);
}
__device__ __forceinline__ double lap3(double S, double C, double N) {
    return lap3(row3(S), row3(C), row3(N));
}

// Wave that computes part p (0..3) of the per-site sums.  Waves of a
// workgroup are dealt to the 4 SIMDs of a CU in turn, so with NC % 4 != 0
// the SIMDs s >= NC % 4 hold one wave fewer; the parts go to their waves.
template <int NC>
__device__ constexpr int helper_wave(int p) {
    int light[16] = {0};
    int n = 0;
    for (int w = 0; w < NC; ++w)
        if (NC % 4 == 0 || w % 4 >= NC % 4) light[n++] = w;
    if (n == 0)
        for (int w = 0; w < NC; ++w) light[n++] = w;
    return light[p % n];
}

// D2Q9 collision of one component at one site, Eq. (1a)-(1c) with
// rho^c = 0 and cs^2 = 1/3, factored per opposite pair of directions:
//   g*_a = (1 - omega) g_a + w_a T_a,
//   T_a  = omega geq_a / w_a + c F_a / w_a
//        = eu (A + B eu + 3c eH) + 3c eF + K(|e_a|^2),
//   A = 3 omega rho, B = 4.5 omega rho, c = 1 - 1/(2 tau), H = 3 F + G,
//   K(e2) = -1.5 omega rho u.u - 3c F.u + c (1.5 e2 - 2) G.u,
// and g*_0 = (1 - omega) g_0 + omega rho + w_0 K(0).  A pair +e / -e shares
// its even part E = w (eu (B eu + 3c eH) + K) and odd part
// O = w (A eu + 3c eF): w T+ = E + O, w T- = E - O.
struct SiteTerms {
    double base, Gu, K1, K2;   // K of |e|^2 = 0 is fma(-2c, Gu, base)
};
__device__ __forceinline__ SiteTerms site_terms(double orho, double fcoef, double ux, double uy,
                                                double Fx, double Fy, double Gx, double Gy) {
    const double uu = fma(ux, ux, uy * uy);
    const double Fu = fma(Fx, ux, Fy * uy);
    SiteTerms s;
    s.Gu = fma(Gx, ux, Gy * uy);
    s.base = fma(-1.5 * orho, uu, -((3.0 * fcoef) * Fu));
    s.K1 = fma(-0.5 * fcoef, s.Gu, s.base);
    s.K2 = fma(fcoef, s.Gu, s.base);
    return s;
}

// w T of the eight moving directions (m: direction a = m + 1 of the D2Q9
// order); rest: omega rho + w_0 K(0).
__device__ __forceinline__ void collide_d2q9(double orho, double fcoef, double ux, double uy,
                                             double Fx, double Fy, double Gx, double Gy,
                                             double (&t)[8], double &rest) {
    const SiteTerms s = site_terms(orho, fcoef, ux, uy, Fx, Fy, Gx, Gy);
    const double Hx = fma(3.0, Fx, Gx), Hy = fma(3.0, Fy, Gy);
    auto pair = [](double A, double B, double C, double K, double eu, double eF, double eH,
                   double &tp, double &tm) {
        const double E = fma(eu, fma(C, eH, B * eu), K);
        const double O = fma(eu, A, C * eF);
        tp = E + O;
        tm = E - O;
    };
    {
        const double A = (1.0 / 3.0) * orho, B = 0.5 * orho, C = (1.0 / 3.0) * fcoef;
        const double K = (1.0 / 9.0) * s.K1;
        pair(A, B, C, K, ux, Fx, Hx, t[0], t[2]);
        pair(A, B, C, K, uy, Fy, Hy, t[1], t[3]);
    }
    {
        const double A = (1.0 / 12.0) * orho, B = 0.125 * orho, C = (1.0 / 12.0) * fcoef;
        const double K = (1.0 / 36.0) * s.K2;
        pair(A, B, C, K, ux + uy, Fx + Fy, Hx + Hy, t[4], t[6]);
        pair(A, B, C, K, uy - ux, Fy - Fx, Hy - Hx, t[5], t[7]);
    }
    rest = fma(4.0 / 9.0, fma(-2.0 * fcoef, s.Gu, s.base), orho);
}

// The same collision for FP32 storage: the eight moving populations in
// FP32 arithmetic (they are stored in FP32; the per-site terms A, B, K, u,
// F, G are formed in FP64 and rounded once):
//   P = B eu + 9c eF + 3c eG,  T+- = +-eu (A +- P) +- 3c eF + K.  The caller stores the rest
// population as rho - (the FP64 sum of the eight stored values, in
// direction order), so that Eq. (1a)-(1c), which conserve each
// component's mass, conserve it to FP64 rounding here too; the EOS, psi
// and the gradients stay FP64.  m: direction a = m + 1 of the D2Q9 order.
// KEEP: add (1 - omega) g, which is zero at omega = 1.
template <bool KEEP>
__device__ __forceinline__ double collide_moving_f32(double orho, double fcoef, double omc,
                                                     double ux, double uy, double Fx, double Fy,
                                                     double Gx, double Gy, const float (&g)[8],
                                                     float (&t)[8]) {
    const SiteTerms s = site_terms(orho, fcoef, ux, uy, Fx, Fy, Gx, Gy);
    const float fA = (float)(3.0 * orho), fB = (float)(4.5 * orho);
    const float f9 = (float)(9.0 * fcoef), f3 = (float)(3.0 * fcoef);
    const float fomc = (float)omc;
    const float fux = (float)ux, fuy = (float)uy, fFx = (float)Fx, fFy = (float)Fy;
    const float fGx = (float)Gx, fGy = (float)Gy;
    auto pair = [&](float K, float eu, float eF, float eG, float w, int mp, int mm) {
        const float P = fmaf(f3, eG, fmaf(f9, eF, fB * eu));
        const float tp = fmaf(eu, fA + P, fmaf(f3, eF, K));
        const float tm = fmaf(eu, P - fA, fmaf(-f3, eF, K));
        t[mp] = KEEP ? fmaf(fomc, g[mp], w * tp) : w * tp;
        t[mm] = KEEP ? fmaf(fomc, g[mm], w * tm) : w * tm;
    };
    pair((float)s.K1, fux, fFx, fGx, 1.0f / 9.0f, 0, 2);
    pair((float)s.K1, fuy, fFy, fGy, 1.0f / 9.0f, 1, 3);
    pair((float)s.K2, fux + fuy, fFx + fFy, fGx + fGy, 1.0f / 36.0f, 4, 6);
    pair((float)s.K2, fuy - fux, fFy - fFx, fGy - fGx, 1.0f / 36.0f, 5, 7);
    double msum = 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) msum += (double)t[m];
    return msum;
}

template <int NC>
struct FusedLds {
    double rt[NC][64];      // molar densities of row r
    double jx[NC][64];      // per-component momentum of row r
    double jy[NC][64];
    double xs[NC][64];      // rt_i Sraw_i of row r
    double fx[NC][64];      // per-component force of row y
    double fy[NC][64];
    double tot[4][3][64];   // ring over rows (slot = row & 3): 1/rho, jx, jy
    double mx[2][2][64];    // ring over rows (slot = row & 1): rt, b_m rt
    double eos[5][64];      // row r-1: c1, c2a, c2b, c3b (helper A), lambda (helper B)
};

// Moments of one component's populations at a site (direction order).
template <class V>
__device__ __forceinline__ void moments_d2q9(const V &v, double &rho, double &jx, double &jy) {
    rho = 0.0;
#pragma unroll
    for (int a = 0; a < 9; ++a) rho += v[a];
    jx = (v[1] - v[3]) + (v[5] - v[7]) + (v[8] - v[6]);
    jy = (v[2] - v[4]) + (v[5] - v[7]) + (v[6] - v[8]);
}

// 1/x to ~1 ulp: hardware reciprocal estimate and two Newton steps.
__device__ __forceinline__ double frcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// Eq. (9)-(12) in combined-log form (any of the cubics,
// p = RT/(v - b) - a/((v + d1 b)(v + d2 b))),
//   RT ln f_i = RT ln(rt_i c1) + b_i (c2a + lambda c2b) - lambda c3b Sraw_i,
//   lambda = ln[(1 + d1 eta)/(1 + d2 eta)] / (d1 - d2), or eta for vdW,
// with the mixture's coefficients from rt = sum_j rt_j, eta = b_m rt and
// xsum = sum_j rt_j Sraw_j, Sraw_i = sum_j (a alpha)_ij rt_j.
struct MixCoef {
    double c1, c2a, c2b, c3b;
};
template <class CP>
__device__ __forceinline__ MixCoef mix_coef(CP C, double RT, double invRT, double rt, double eta,
                                            double xsum, uint32_t &bad) {
    const double inv_rt = frcp(rt);
    const double am = (xsum * inv_rt) * inv_rt;
    const double ome = 1.0 - eta;
    if (!(ome > 0.0)) bad |= FUG_ST_COVOLUME;
    const double inv_ome = frcp(ome);
    const double inv_bm = rt * frcp(eta);
    const double den = fma(C->ew * eta, eta, fma(C->eu, eta, 1.0));
    const double zm1 = fma(eta, inv_ome, -(((am * rt) * invRT) * frcp(den)));
    return {RT * inv_ome, (RT * zm1) * inv_bm, (am * inv_bm) * inv_bm, (2.0 * inv_bm) * inv_rt};
}
template <class CP>
__device__ __forceinline__ double mix_lambda(CP C, double eta) {
    if (C->eos == 2) return eta;
    return log(fma(C->d1, eta, 1.0) * frcp(fma(C->d2, eta, 1.0))) * C->dk;
}
__device__ __forceinline__ double rt_lnf(const MixCoef &m, double lam, double RT, double rti,
                                         double bi, double Si) {
    const double t = fma(bi, fma(lam, m.c2b, m.c2a), RT * log(rti * m.c1));
    return fma(-(lam * m.c3b), Si, t);
}

// Populations of one component at one site: the rest one in FP64, the
// moving ones (directions 1..8) in the storage type.
template <typename ST>
struct PopRow {
    double r;
    ST m[8];
};

}  // namespace fused
