// Fused one-pass D2Q9 step for work items of one or two rows (gfx950): the
// register-ring variant's form for small grids.
//
// On a grid of some thousand sites a step is a chain of latencies, not of
// work: a marching item of one row still takes five lead rows one after
// another, each with two workgroup barriers.  Here an item's rows are taken
// together: every row is loaded at once, every phase runs over all rows of
// the item (independent chains of one wavefront, so its latencies overlap),
// and an item has four barriers in all:
//
//      (components)  moments of the rows y0 - 2 .. y0 + R + 1
//   -- 1 --
//      (components)  Sraw_i, rt_i Sraw_i of the rows y0 - 1 .. y0 + R
//      (helpers)     s, rt, b_m rt; 1/rho and j of the output rows
//   -- 2 --
//      (components)  lap s, G_i        (helpers)  mixture coefficients
//   -- 3 --
//      (components)  psi_i, F_i
//   -- 4 --
//      (components)  u, collision, push
//
// (Two rows of nine and ten components in FP64 spill 2 and 4 of 128 registers.)
//
// One wavefront per component, lane = column of a 60-column strip, and one
// helper wavefront per row that needs the EOS.  Terms, orders of summation
// and work-item tables are those of the marching kernels: bitwise the same
// state.
#pragma once

#include "fused_common.h"

namespace block {

using namespace fused;

template <int NC, int R>
struct BlockLds {
    double rt[R + 4][NC][64];
    double jx[R][NC][64];
    double jy[R][NC][64];
    double xs[R + 2][NC][64];
    double s[R + 4][64];
    double eos[R + 2][5][64];
    double tot[R][3][64];        // 1/rho, jx, jy
    double2 F[R][NC][64];
};

template <int NC, typename ST, int R>
__global__ __launch_bounds__(64 * (NC + R + 2)) void k_fused_block(FusedTable T, int flip) {
    __shared__ BlockLds<NC, R> L;
    cptr<FusedItem> itp = (cptr<FusedItem>)T.items + blockIdx.x;
    const FusedItem it = {itp->sim, itp->x0, itp->y0, itp->rows};
    if (it.sim < 0) return;
    // a single simulation's entry does not wait for the item's
    cptr<FusedSim> sm = (cptr<FusedSim>)T.sims + (T.nsims == 1 ? 0 : it.sim);
    const int par = (sm->parity ^ flip) & 1;
    cptr<SimConst> C = (cptr<SimConst>)sm->c;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const double RT = C->RT;
    uint32_t bad = 0;

    if (wave >= NC) {
        // helper k: row y0 - 1 + k (rows of L.rt count from y0 - 2)
        const int k = wave - NC;
        __syncthreads();
        double rtt = 0.0, eta = 0.0;
        auto s_row = [&](int q) {
            double sv = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j) sv = fma(C->sqk[j], L.rt[q][j][lane], sv);
            L.s[q][lane] = sv;
        };
        s_row(k + 1);
        if (k == 0) s_row(0);
        if (k == R + 1) s_row(R + 3);
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const double t = L.rt[k + 1][j][lane];
            rtt += t;
            eta = fma(C->b[j], t, eta);
        }
        if (k >= 1 && k <= R) {
            double rtot = 0.0, jxt = 0.0, jyt = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                rtot = fma(C->M[j], L.rt[k + 1][j][lane], rtot);
                jxt += L.jx[k - 1][j][lane];
                jyt += L.jy[k - 1][j][lane];
            }
            L.tot[k - 1][0][lane] = frcp(rtot);
            L.tot[k - 1][1][lane] = jxt;
            L.tot[k - 1][2][lane] = jyt;
        }
        __syncthreads();
        double xsum = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) xsum += L.xs[k][j][lane];
        const MixCoef m = mix_coef(C, RT, C->invRT, rtt, eta, xsum, bad);
        L.eos[k][0][lane] = m.c1;
        L.eos[k][1][lane] = m.c2a;
        L.eos[k][2][lane] = m.c2b;
        L.eos[k][3][lane] = m.c3b;
        L.eos[k][4][lane] = mix_lambda(C, eta);
        __syncthreads();
        __syncthreads();
        flag_status(sm->status, bad);
        return;
    }

    const int comp = wave;
    const int nx = sm->nx, ny = sm->ny;
    const char *bsrc = (const char *)(par ? sm->buf[1] : sm->buf[0]);
    char *bdst = (char *)(par ? sm->buf[0] : sm->buf[1]);
    const PopLayout<ST> P(NC, 9, nx, ny);
    // periodic images without a division: the rows and columns of an item lie
    // within a few periods, and few grids are narrower than a strip
    int xc = it.x0 - 2 + lane;
    xc = xc < 0 ? xc + nx : xc;
    while (__any(xc < 0 || xc >= nx)) xc = xc < 0 ? xc + nx : (xc >= nx ? xc - nx : xc);
    auto wrap = [&](int v) {
        while (v < 0) v += ny;
        while (v >= ny) v -= ny;
        return v;
    };
    // this lane's value of a row: uniform row address, 32-bit lane offset
    const uint32_t xb = (uint32_t)xc * 8u, xs = (uint32_t)xc * (uint32_t)sizeof(ST);
    const double invM = C->invM[comp], bi = C->b[comp], sqki = C->sqk[comp];

    PopRow<ST> g[R + 4];
#pragma unroll
    for (int q = 0; q < R + 4; ++q) {
        const int w = wrap(it.y0 - 2 + q);
        g[q].r = *(gptr<double>)((gptr<char>)(bsrc + P.rest(w, comp, 0)) + xb);
#pragma unroll
        for (int a = 1; a < 9; ++a)
            g[q].m[a - 1] = *(gptr<ST>)((gptr<char>)(bsrc + P.move(w, comp, a, 0)) + xs);
    }
    double h[R + 4];
#pragma unroll
    for (int q = 0; q < R + 4; ++q) {
        double v[9], jx, jy;
        v[0] = g[q].r;
#pragma unroll
        for (int a = 1; a < 9; ++a) v[a] = (double)g[q].m[a - 1];
        moments_d2q9(v, h[q], jx, jy);
        L.rt[q][comp][lane] = h[q] * invM;
        if (q >= 2 && q < R + 2) {
            L.jx[q - 2][comp][lane] = jx;
            L.jy[q - 2][comp][lane] = jy;
        }
    }
    __syncthreads();
    double S[R + 2];
    {
        cptr<double> arow = C->aij + comp * FUG_MAXC;
#pragma unroll
        for (int k = 0; k < R + 2; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j) acc = fma(arow[j], L.rt[k + 1][j][lane], acc);
            S[k] = acc;
            L.xs[k][comp][lane] = (h[k + 1] * invM) * acc;
        }
    }
    __syncthreads();
    double lap[R + 2], Gx[R], Gy[R];
    {
        Row3 s3[R + 4];
#pragma unroll
        for (int q = 0; q < R + 4; ++q) s3[q] = row3(L.s[q][lane]);
#pragma unroll
        for (int k = 0; k < R + 2; ++k) lap[k] = lap3(s3[k], s3[k + 1], s3[k + 2]);
        Row3 h3[R + 2];
#pragma unroll
        for (int k = 0; k < R + 2; ++k) h3[k] = row3(h[k + 1]);
#pragma unroll
        for (int c = 0; c < R; ++c) grad3(h3[c], h3[c + 1], h3[c + 2], Gx[c], Gy[c]);
    }
    __syncthreads();
    double Fx[R], Fy[R];
    {
        Row3 p3[R + 2];
#pragma unroll
        for (int k = 0; k < R + 2; ++k) {
            const MixCoef m = {L.eos[k][0][lane], L.eos[k][1][lane], L.eos[k][2][lane],
                               L.eos[k][3][lane]};
            const double rti = h[k + 1] * invM;
            const double psi =
                fma(-sqki, lap[k], rt_lnf(m, L.eos[k][4][lane], RT, rti, bi, S[k]));
            if (!(rti > 0.0)) bad |= FUG_ST_NEGATIVE;
            if (!isfinite(psi)) bad |= FUG_ST_NONFINITE;
            p3[k] = row3(psi);
        }
#pragma unroll
        for (int c = 0; c < R; ++c) {
            double gx, gy;
            grad3(p3[c], p3[c + 1], p3[c + 2], gx, gy);
            const double rty = h[c + 2] * invM;
            Fx[c] = -rty * gx;
            Fy[c] = -rty * gy;
            L.F[c][comp][lane] = {Fx[c], Fy[c]};
        }
    }
    __syncthreads();
    const double omega = C->omega, fcoef = C->fcoef, omc = 1.0 - omega;
    const bool outl = lane >= 2 && lane < 62 && (it.x0 + lane - 2) < nx;
    const int xm = xc == 0 ? nx - 1 : xc - 1, xp = xc == nx - 1 ? 0 : xc + 1;
#pragma unroll
    for (int c = 0; c < R; ++c) {
        if (c >= it.rows) break;
        double Fsx = 0.0, Fsy = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const double2 f = L.F[c][j][lane];
            Fsx += f.x;
            Fsy += f.y;
        }
        const double inv_rho = L.tot[c][0][lane];
        const double ux = fma(0.5, Fsx, L.tot[c][1][lane]) * inv_rho;
        const double uy = fma(0.5, Fsy, L.tot[c][2][lane]) * inv_rho;
        const double orho = omega * h[c + 2];
        const PopRow<ST> &go = g[c + 2];
        ST t[8];
        double rest;
        if constexpr (sizeof(ST) == 4) {
            rest = h[c + 2] - collide_moving_f32<true>(orho, fcoef, omc, ux, uy, Fx[c], Fy[c],
                                                       Gx[c], Gy[c], go.m, t);
        } else {
            collide_d2q9(orho, fcoef, ux, uy, Fx[c], Fy[c], Gx[c], Gy[c], t, rest);
            rest = fma(omc, go.r, rest);
#pragma unroll
            for (int m = 0; m < 8; ++m) t[m] = fma(omc, go.m[m], t[m]);
        }
        if (outl) {
            const int yw = it.y0 + c, ym = yw == 0 ? ny - 1 : yw - 1,
                      yp = yw + 1 == ny ? 0 : yw + 1;
            *(gmptr<double>)((gmptr<char>)(bdst + P.rest(yw, comp, 0)) + xb) = rest;
#pragma unroll
            for (int a = 1; a < 9; ++a) {
                const int ex = D2Q9::ex(a), ey = D2Q9::ey(a);
                const uint32_t xd = (uint32_t)(ex > 0 ? xp : (ex < 0 ? xm : xc));
                const int yd = ey > 0 ? yp : (ey < 0 ? ym : yw);
                *(gmptr<ST>)((gmptr<char>)(bdst + P.move(yd, comp, a, 0)) +
                             xd * (uint32_t)sizeof(ST)) = t[a - 1];
            }
        }
    }
    flag_status(sm->status, bad);
}

template <int NC, typename ST, int R>
hipError_t launch_t(const FusedTable &t, int flip, hipStream_t st) {
    hipLaunchKernelGGL((k_fused_block<NC, ST, R>), dim3(t.nitems), dim3(64 * (NC + R + 2)), 0, st,
                       t, flip);
    return hipGetLastError();
}

template <int NC>
hipError_t launch_nc(bool fp32, const FusedTable &t, int flip, hipStream_t st) {
    if (t.rows == 1)
        return fp32 ? launch_t<NC, float, 1>(t, flip, st) : launch_t<NC, double, 1>(t, flip, st);
    return fp32 ? launch_t<NC, float, 2>(t, flip, st) : launch_t<NC, double, 2>(t, flip, st);
}

}  // namespace block

hipError_t launch_fused_block(int ncomp, bool fp32, const FusedTable &t, int flip, hipStream_t st) {
    switch (ncomp) {
        case 1: return block::launch_nc<1>(fp32, t, flip, st);
        case 2: return block::launch_nc<2>(fp32, t, flip, st);
        case 3: return block::launch_nc<3>(fp32, t, flip, st);
        case 4: return block::launch_nc<4>(fp32, t, flip, st);
        case 5: return block::launch_nc<5>(fp32, t, flip, st);
        case 6: return block::launch_nc<6>(fp32, t, flip, st);
        case 7: return block::launch_nc<7>(fp32, t, flip, st);
        case 8: return block::launch_nc<8>(fp32, t, flip, st);
        case 9: return block::launch_nc<9>(fp32, t, flip, st);
        case 10: return block::launch_nc<10>(fp32, t, flip, st);
        default: return hipErrorInvalidValue;
    }
}
