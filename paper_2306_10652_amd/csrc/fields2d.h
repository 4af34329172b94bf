// D2Q9 steps at tau = 1 in field form (gfx950): the steps of a run between
// its first and its last, without populations in memory.
//
// At tau = 1 the collision drops the old populations (Eq. (1a) with
// omega = 1): they enter a step only through rho_i and j.  A run of n steps
// therefore reads its populations once (k_field_moments: rho_i, j and
// s = sum sqrt(kappa_j) rt_j), then carries rho_i, j and s from step to step
// and writes the populations of the state it ends in with its last step.  A
// step is two kernels:
//
//   k_field_eos   psi_i = RT ln f_i - sqrt(kappa_i) lap s and 1/rho, one
//                 thread per site over all components;
//   k_field_step  F_i, G_i, u, the collision, and the streaming sums: the
//                 nine populations that arrive at a site are added up in
//                 registers (rho_i, j) instead of being stored.
//
// A step moves (N + 1 + 1) + (N + 1) field values per site in the first
// kernel and (2N + 3) + (N + 3) in the second, 5N + 9 = 59 for ten
// components, where the fused kernels move 18 N = 180 population values
// (FP32 storage: 100 in the same unit).  All terms come from the functions
// the fused kernels use, and the populations enter the sums rounded to the
// storage type and in direction order: the state is bitwise theirs.
//
// Measured, us a step (fused kernel before): 1024^2 x 10 332 -> 121 FP64,
// 252 -> 123 FP32 storage; 512^2 x 10 103 -> 39; 200^2 x 10 26.9 -> 17.6;
// 1024^2 x 3 116 -> 52.
#pragma once

#include "fused_common.h"

namespace fields {

using namespace fused;

constexpr int TPB = 256;

// The arrays of one simulation (FieldSim): two sets of rho_i, s and j that
// the steps alternate between, psi_i and 1/rho.  With `wide` all of them lie
// in the population buffer that the run does not read (parity ^ 1), the
// components ld apart; else set 0 and psi are the workspace fields.
struct View {
    double *rho[2], *s[2], *j[2], *psi, *ir;
    int64_t ld;
};

template <class FS>
__device__ __forceinline__ View field_view(const FS &f, int flip, int N, int D) {
    View v;
    const int64_t ld = f.ld;
    double *b = (double *)(((f.parity ^ flip) & 1) ? f.buf[0] : f.buf[1]);
    v.ld = ld;
    if (f.wide) {
        v.rho[0] = b;
        v.rho[1] = b + N * ld;
        v.psi = b + 2 * N * ld;
        b += 3 * N * ld;
        v.s[0] = b;
        v.s[1] = b + ld;
        v.ir = b + 2 * ld;
        v.j[0] = b + 3 * ld;
        v.j[1] = b + (3 + D) * ld;
    } else {
        v.rho[0] = f.rho;
        v.rho[1] = b;
        v.psi = f.psi;
        v.s[0] = f.s;
        v.s[1] = b + N * ld;
        v.ir = b + (N + 1) * ld;
        v.j[0] = f.j;
        v.j[1] = f.u;
    }
    return v;
}

// A table entry by scalar loads.
__device__ __forceinline__ FieldSim load_sim(const FieldSim *tab, int k) {
    cptr<FieldSim> p = (cptr<FieldSim>)tab + k;
    FieldSim f;
    f.c = p->c;
    f.buf[0] = p->buf[0];
    f.buf[1] = p->buf[1];
    f.rho = p->rho;
    f.psi = p->psi;
    f.s = p->s;
    f.j = p->j;
    f.u = p->u;
    f.status = p->status;
    f.ld = p->ld;
    f.parity = p->parity;
    f.wide = p->wide;
    f.nx = p->nx;
    f.ny = p->ny;
    return f;
}

// The simulation of site block `blk` (table: members cumulative in `end`),
// and the block's index within it.
__device__ __forceinline__ FieldSim block_sim(const FieldSim *tab, int nm, const FieldSim &one,
                                              int64_t &blk) {
    if (nm == 0) return one;
    int lo = 0, hi = nm - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (((cptr<FieldSim>)tab)[mid].end > blk)
            hi = mid;
        else
            lo = mid + 1;
    }
    if (lo) blk -= ((cptr<FieldSim>)tab)[lo - 1].end;
    return load_sim(tab, lo);
}

// rho_i, j and s of the populations in memory -> set 0.  Bound by the
// population reads (each once).
template <typename ST>
__global__ __launch_bounds__(TPB) void k_field_moments(const FieldSim *tab, int nm, FieldSim one,
                                                       int flip) {
    int64_t blk = blockIdx.x;
    const FieldSim f = block_sim(tab, nm, one, blk);
    cptr<SimConst> C = (cptr<SimConst>)f.c;
    const int N = C->N, nx = f.nx;
    const uint32_t ns = (uint32_t)nx * (uint32_t)f.ny;
    const uint32_t s = (uint32_t)blk * TPB + threadIdx.x;
    if (s >= ns) return;
    const View v = field_view(f, flip, N, 2);
    const void *g = ((f.parity ^ flip) & 1) ? f.buf[1] : f.buf[0];
    const PopLayout<ST> P(N, 9, nx, f.ny);
    const uint32_t row = s / (uint32_t)nx;
    const int x = (int)(s - row * (uint32_t)nx);
    double jxt = 0.0, jyt = 0.0, sv = 0.0;
#pragma unroll 2
    for (int i = 0; i < N; ++i) {
        double p[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) p[a] = ld_pop<ST>(g, P, row, i, a, x);
        double rho, jx, jy;
        moments_d2q9(p, rho, jx, jy);
        v.rho[0][(int64_t)i * v.ld + s] = rho;
        jxt += jx;
        jyt += jy;
        sv = fma(C->sqk[i], rho * C->invM[i], sv);
    }
    v.s[0][s] = sv;
    v.j[0][s] = jxt;
    v.j[0][v.ld + s] = jyt;
}

// psi_i and 1/rho of set `set`.  One thread per site with every component in
// registers: the N x N mixing sums, N + 2 logarithms and the reciprocals are
// independent chains of one thread, there is no exchange between threads,
// and s is read with its eight neighbours (cache hits).  Bound by VALU work:
// 1330 instructions a wavefront for ten components, 900 of them logarithms;
// 48 us for 1024^2 x 10 (36 us of issue, 193 MB), 20.5 us x 3.  Slower: 64
// registers for eight wavefronts a SIMD (60 us, spills), persistent
// workgroups that load a site ahead (56 to 60 us), components split over
// workgroups on small grids (200^2 x 10: 17.6 us a step -> 19.6 and more, as
// every group repeats the N x N sums).
template <int NC>
__global__ __launch_bounds__(TPB) void k_field_eos(const FieldSim *tab, int nm, FieldSim one,
                                                   int flip, int set) {
    int64_t blk = blockIdx.x;
    const FieldSim f = block_sim(tab, nm, one, blk);
    cptr<SimConst> C = (cptr<SimConst>)f.c;
    const int nx = f.nx, ny = f.ny;
    const uint32_t ns = (uint32_t)nx * (uint32_t)ny;
    const uint32_t s = (uint32_t)blk * TPB + threadIdx.x;
    if (s >= ns) return;
    const View v = field_view(f, flip, NC, 2);
    const double *rho = set ? v.rho[1] : v.rho[0];
    const double *sf = set ? v.s[1] : v.s[0];
    double rt[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) rt[i] = rho[(int64_t)i * v.ld + s];
    double lap;
    {
        const uint32_t y = s / (uint32_t)nx, x = s - y * (uint32_t)nx;
        const uint32_t xw = x == 0 ? nx - 1 : x - 1, xe = x + 1 == (uint32_t)nx ? 0 : x + 1;
        const uint32_t r0 = y * nx, rs = (y == 0 ? ny - 1 : y - 1) * nx,
                       rn = (y + 1 == (uint32_t)ny ? 0 : y + 1) * nx;
        const Row3 S = {sf[rs + xw], sf[rs + x], sf[rs + xe]};
        const Row3 M = {sf[r0 + xw], sf[r0 + x], sf[r0 + xe]};
        const Row3 N = {sf[rn + xw], sf[rn + x], sf[rn + xe]};
        lap = lap3(S, M, N);
    }
    uint32_t bad = 0;
    double rtt = 0.0, eta = 0.0, rtot = 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        rt[i] *= C->invM[i];
        if (!(rt[i] > 0.0)) bad |= FUG_ST_NEGATIVE;
        rtt += rt[i];
        eta = fma(C->b[i], rt[i], eta);
        rtot = fma(C->M[i], rt[i], rtot);
    }
    double S[NC], xsum = 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) acc = fma(C->aij[i * FUG_MAXC + j], rt[j], acc);
        S[i] = acc;
        xsum += rt[i] * acc;
    }
    const double RT = C->RT;
    const MixCoef m = mix_coef(C, RT, C->invRT, rtt, eta, xsum, bad);
    const double lam = mix_lambda(C, eta);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const double psi = fma(-C->sqk[i], lap, rt_lnf(m, lam, RT, rt[i], C->b[i], S[i]));
        if (!isfinite(psi)) bad |= FUG_ST_NONFINITE;
        v.psi[(int64_t)i * v.ld + s] = psi;
    }
    v.ir[s] = frcp(rtot);
    flag_status(f.status, bad);
}

// Two helper wavefronts beside the N component wavefronts of a step's
// workgroup: one sums the forces and forms u, one adds up and stores the
// output row.
constexpr int HELPERS = 2;

template <int NC, bool LAST>
struct StepLds {
    double2 F[2][NC][64];   // F_i of row r - 1, slot r & 1
    double2 u[2][64];       // u of row r - 1, slot r & 1
    double2 q0[2][NC][64];  // new rho_i, j_x,i of row r - 3, slot r & 1
    double q1[2][NC][64];   // new j_y,i
};
template <int NC>
struct StepLds<NC, true> {
    double2 F[2][NC][64];
    double2 u[2][64];
};

// One step from (rho_i, psi_i, j, 1/rho) of set `set`: to (rho_i, j, s) of
// the other set, or (LAST) to the populations of the new state.
//
// Work item and lanes as in the fused kernels: a 64-column strip with 60
// output columns, marching up `rows` rows, one wavefront per component.  Per
// lead row r, with one workgroup barrier:
//      (components)  F_i, G_i of row r - 1 from the rows r - 2 .. r; F_i -> LDS
//   -- barrier r --
//      (helper 0)    u of row r - 1 -> LDS
//      (components)  collide row r - 2; add its populations to the sums of
//                    rows r - 3 .. r - 1 (x neighbours by lane shifts); the
//                    sums of row r - 3 are complete -> LDS
//      (helper 1)    rho_i, j, s of row r - 4 -> memory
// so every exchange has a whole row's time to arrive.  The component
// wavefronts only load and helper 1 only stores (loads and stores in flight
// share one counter: a wavefront with both can only wait for all of them);
// rows are requested three ahead.  72 us for 1024^2 x 10 in 74-row items (252
// workgroups, one per CU, 302 MB and halos at 4.6 TB/s).  Slower: F_i of the
// next row after the barrier, beside the collision (85 -> 88 us in 96-row
// items); rows requested six ahead (no change, three components 80 -> 96).
template <int NC, typename ST, bool LAST>
__global__ __launch_bounds__(64 * (NC + HELPERS)) void k_field_step(
    const FieldSim *tab, FieldSim one, const FusedItem *items, int nitems, int strips, int rows_,
    int flip, int set) {
    __shared__ StepLds<NC, LAST> L;
    FusedItem it;
    FieldSim f;
    if (items) {
        cptr<FusedItem> p = (cptr<FusedItem>)items + blockIdx.x;
        it = {p->sim, p->x0, p->y0, p->rows};
        if (it.sim < 0) return;
        f = load_sim(tab, it.sim);
    } else {
        f = one;
        const int per = gridDim.x / 8;
        const int li = (blockIdx.x % 8) * per + blockIdx.x / 8;
        if (li >= nitems) return;
        it.x0 = (li % strips) * FUSED_OUT;
        it.y0 = (li / strips) * rows_;
        it.rows = min(rows_, f.ny - it.y0);
    }
    cptr<SimConst> C = (cptr<SimConst>)f.c;
    const int nx = f.nx, ny = f.ny;
    const View v = field_view(f, flip, NC, 2);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int xc = (it.x0 - 2 + lane) % nx;
    if (xc < 0) xc += nx;
    const bool outl = lane >= 2 && lane < 62 && (it.x0 + lane - 2) < nx;
    constexpr int H = LAST ? 1 : 2;      // halo rows of psi_i and rho_i
    const int y0 = it.y0, rbeg = y0 - H, rload = y0 + it.rows - 1 + H;
    const int rcol = y0 + it.rows + H;   // last lead row that collides
    const int rend = LAST ? rcol : rcol + 1;
    auto wrap = [&](int q) {
        q %= ny;
        return q < 0 ? q + ny : q;
    };
    auto next = [&](int w) { return w + 1 == ny ? 0 : w + 1; };
    // this lane's value of a row (uniform row address, 32-bit lane offset)
    const uint32_t xb = (uint32_t)xc * 8u;
    auto at = [&](gptr<double> row) { return *(gptr<double>)((gptr<char>)row + xb); };

    if (wave == NC) {
        // helper 0: u(y) = (j + F/2) / rho for y = r - 1
        gptr<double> jx = (gptr<double>)(set ? v.j[1] : v.j[0]);
        gptr<double> jy = jx + v.ld, ir = (gptr<double>)v.ir;
        struct In {
            double jx, jy, ir;
        } a, b;
        auto load = [&](In &q, int w) {
            const int64_t row = (int64_t)w * nx;
            q = {at(jx + row), at(jy + row), at(ir + row)};
        };
        int w = wrap(rbeg - 1);
        load(a, w);
        w = next(w);
        load(b, w);
        auto lead = [&](int r, In &q) {
            __syncthreads();
            double Fx = 0.0, Fy = 0.0;
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const double2 t = L.F[r & 1][i][lane];
                Fx += t.x;
                Fy += t.y;
            }
            L.u[r & 1][lane] = {fma(0.5, Fx, q.jx) * q.ir, fma(0.5, Fy, q.jy) * q.ir};
            w = next(w);
            load(q, w);
        };
        for (int r = rbeg; r <= rend; r += 2) {
            lead(r, a);
            if (r + 1 > rend) break;
            lead(r + 1, b);
        }
        return;
    }
    if (wave > NC) {
        // helper 1: the output row of lead row r - 1
        if constexpr (LAST) {
            for (int r = rbeg; r <= rend; ++r) __syncthreads();
        } else {
            double *rho = set ? v.rho[0] : v.rho[1];
            double *jd = set ? v.j[0] : v.j[1];
            double *sd = set ? v.s[0] : v.s[1];
            auto put = [&](double *row, double q) { *(gmptr<double>)((gmptr<char>)row + xb) = q; };
            int64_t o = (int64_t)y0 * nx;
            for (int r = rbeg; r <= rend; ++r) {
                __syncthreads();
                if (r < y0 + 4) continue;   // uniform
                double2 q0[NC];
                double q1[NC];
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    q0[i] = L.q0[(r - 1) & 1][i][lane];
                    q1[i] = L.q1[(r - 1) & 1][i][lane];
                }
                double sv = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    sv = fma(C->sqk[i], q0[i].x * C->invM[i], sv);
                    jx += q0[i].y;
                    jy += q1[i];
                }
                if (outl) {
#pragma unroll
                    for (int i = 0; i < NC; ++i) put(rho + (int64_t)i * v.ld + o, q0[i].x);
                    put(sd + o, sv);
                    put(jd + o, jx);
                    put(jd + v.ld + o, jy);
                }
                o += nx;
            }
        }
        return;
    }

    // component wavefronts
    const int comp = wave;
    const double invM = C->invM[comp];
    gptr<double> hsrc = (gptr<double>)(set ? v.rho[1] : v.rho[0]) + (int64_t)comp * v.ld;
    gptr<double> psrc = (gptr<double>)v.psi + (int64_t)comp * v.ld;
    struct In {
        double h, p;
    } X, Y, Z;
    auto load = [&](In &q, int w) {
        // in program order, so every wait on a row counts the rows after it
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const int64_t row = (int64_t)w * nx;
        q.h = at(hsrc + row);
        q.p = at(psrc + row);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    int lr = rbeg, lw = wrap(rbeg);     // last row requested and its wrapped index
    auto request = [&](In &q) {
        if (lr < rload) {               // past the item's last row: that row again
            ++lr;
            lw = next(lw);
        }
        load(q, lw);
    };
    load(X, lw);
    request(Y);
    request(Z);

    const Row3 zero = {0.0, 0.0, 0.0};
    Row3 h0 = zero, h1 = zero, h2 = zero, p0 = zero, p1 = zero, p2 = zero;
    struct Site {
        double rho, Fx, Fy, Gx, Gy;
    } A = {0.0, 0.0, 0.0, 0.0, 0.0}, B = A;
    // sums on their way: part = v0 + .. + v3, d13 = v1 - v3 and (n2, n5, n6)
    // of the row below the one to be collided; (m2, m5, m6) going up to that
    // row itself
    double part = 0.0, d13 = 0.0;
    ST n2 = 0, n5 = 0, n6 = 0, m2 = 0, m5 = 0, m6 = 0;

    // populations and their new rows (LAST)
    char *bdst = (char *)(((f.parity ^ flip) & 1) ? f.buf[1] : f.buf[0]);
    const PopLayout<ST> P(NC, 9, nx, ny);
    int yc = 0;                          // wrapped row that is collided (LAST)
    if constexpr (LAST) yc = y0;

    auto shl = [](ST q, bool left) -> ST {   // value of the west / east lane
        if constexpr (sizeof(ST) == 4) {
            const int b = __float_as_int(q);
            return __int_as_float(left ? __builtin_amdgcn_mov_dpp(b, 0x138, 0xf, 0xf, true)
                                       : __builtin_amdgcn_mov_dpp(b, 0x130, 0xf, 0xf, true));
        } else {
            return left ? from_left(q) : from_right(q);
        }
    };

    auto lead = [&](int r, In &cur, const Row3 &hs, const Row3 &hc, Row3 &hn, const Row3 &ps,
                    const Row3 &pc, Row3 &pn, const Site &old, Site &now) {
        hn = row3(cur.h);
        pn = row3(cur.p);
        request(cur);
        {
            double gx, gy;
            grad3(ps, pc, pn, gx, gy);
            grad3(hs, hc, hn, now.Gx, now.Gy);
            now.rho = hc.c;
            const double rty = hc.c * invM;
            now.Fx = -rty * gx;
            now.Fy = -rty * gy;
            L.F[r & 1][comp][lane] = {now.Fx, now.Fy};
        }
        __syncthreads();
        if (r < rbeg + 3 || r > rcol) return;
        const double2 u = L.u[(r - 1) & 1][lane];
        ST t[8];
        double rest;
        if constexpr (sizeof(ST) == 4) {
            rest = old.rho - collide_moving_f32<false>(old.rho, 0.5, 0.0, u.x, u.y, old.Fx, old.Fy,
                                                       old.Gx, old.Gy, t, t);
        } else {
            collide_d2q9(old.rho, 0.5, u.x, u.y, old.Fx, old.Fy, old.Gx, old.Gy, t, rest);
        }
        if constexpr (LAST) {
            if (outl) {
                const int xw = xc == 0 ? nx - 1 : xc - 1, xe = xc + 1 == nx ? 0 : xc + 1;
                const int ys = yc == 0 ? ny - 1 : yc - 1, yn = next(yc);
                *(double *)(bdst + P.rest(yc, comp, xc)) = rest;
#pragma unroll
                for (int a = 1; a < 9; ++a) {
                    const int ex = D2Q9::ex(a), ey = D2Q9::ey(a);
                    const int xd = ex > 0 ? xe : (ex < 0 ? xw : xc);
                    const int yd = ey > 0 ? yn : (ey < 0 ? ys : yc);
                    *(ST *)(bdst + P.move(yd, comp, a, xd)) = t[a - 1];
                }
            }
            yc = next(yc);
        } else {
            const ST v1 = shl(t[0], true), v3 = shl(t[2], false), v7 = shl(t[6], false),
                     v8 = shl(t[7], true);
            const double d4 = (double)t[3], d5 = (double)n5, d6 = (double)n6, d7 = (double)v7,
                         d8 = (double)v8;
            const double rn = (((part + d4) + d5) + d6) + d7 + d8;
            const double e57 = d5 - d7;
            L.q0[r & 1][comp][lane] = {rn, (d13 + e57) + (d8 - d6)};
            L.q1[r & 1][comp][lane] = (((double)n2 - d4) + e57) + (d6 - d8);
            part = ((rest + (double)v1) + (double)m2) + (double)v3;
            d13 = (double)v1 - (double)v3;
            n2 = m2;
            n5 = m5;
            n6 = m6;
            m2 = t[1];
            m5 = shl(t[4], true);
            m6 = shl(t[5], false);
        }
    };
    for (int r = rbeg; r <= rend; r += 6) {
        lead(r, X, h0, h1, h2, p0, p1, p2, A, B);
        if (r + 1 > rend) break;
        lead(r + 1, Y, h1, h2, h0, p1, p2, p0, B, A);
        if (r + 2 > rend) break;
        lead(r + 2, Z, h2, h0, h1, p2, p0, p1, A, B);
        if (r + 3 > rend) break;
        lead(r + 3, X, h0, h1, h2, p0, p1, p2, B, A);
        if (r + 4 > rend) break;
        lead(r + 4, Y, h1, h2, h0, p1, p2, p0, A, B);
        if (r + 5 > rend) break;
        lead(r + 5, Z, h2, h0, h1, p2, p0, p1, B, A);
    }
}

// The same for few components by single wavefronts: lanes and rows of a work
// item as above, every component in one wavefront, which collides row r - 1
// as soon as row r is there.  No exchange between wavefronts and none that
// only helps (two of the five that three components take above); two to four
// of them to a SIMD, bound by memory where the grid fills them (1024^2 x 3:
// 160 MB with its halos in 30 us).  Rows are held without their lane shifts,
// which are taken where they are used: 220 registers instead of 276 for three
// components in FP64.  Which of the two is faster depends on how the rows
// divide, so the tuner times both.  Step kernel above / this, us a step with
// the EOS kernel: 48 grids of 64^2 ... 256^2 x 3 in FP32 storage 84 / 76,
// 512^2 x 1 16.1 / 14.5, 1024^2 x 3 52 / 50.6, 512^2 x 3 22.9 / 23.5,
// 1024^2 x 2 38.5 / 42; with four components 56 / 78.  Taken back: the EOS
// in the same wavefront (no psi_i in memory, one launch): 48 grids 77,
// 1024^2 x 3 slower than both.
template <int NC, typename ST>
__global__ __launch_bounds__(64, NC == 1 ? 4 : NC == 2 ? 3 : 2) void k_field_single(const FieldSim *tab, FieldSim one,
                                                   const FusedItem *items, int nitems, int strips,
                                                   int rows_, int flip, int set) {
    FusedItem it;
    FieldSim f;
    if (items) {
        cptr<FusedItem> p = (cptr<FusedItem>)items + blockIdx.x;
        it = {p->sim, p->x0, p->y0, p->rows};
        if (it.sim < 0) return;
        f = load_sim(tab, it.sim);
    } else {
        f = one;
        const int per = gridDim.x / 8;
        const int li = (blockIdx.x % 8) * per + blockIdx.x / 8;
        if (li >= nitems) return;
        it.x0 = (li % strips) * FUSED_OUT;
        it.y0 = (li / strips) * rows_;
        it.rows = min(rows_, f.ny - it.y0);
    }
    cptr<SimConst> C = (cptr<SimConst>)f.c;
    const int nx = f.nx, ny = f.ny;
    const View v = field_view(f, flip, NC, 2);
    const int lane = threadIdx.x;
    int xc = (it.x0 - 2 + lane) % nx;
    if (xc < 0) xc += nx;
    const bool outl = lane >= 2 && lane < 62 && (it.x0 + lane - 2) < nx;
    const int y0 = it.y0, rbeg = y0 - 2, rend = y0 + it.rows + 1;
    auto wrap = [&](int q) {
        q %= ny;
        return q < 0 ? q + ny : q;
    };
    auto next = [&](int w) { return w + 1 == ny ? 0 : w + 1; };
    const uint32_t xb = (uint32_t)xc * 8u;
    auto at = [&](gptr<double> row) { return *(gptr<double>)((gptr<char>)row + xb); };
    auto put = [&](double *row, double q) { *(gmptr<double>)((gmptr<char>)row + xb) = q; };
    gptr<double> rho = (gptr<double>)(set ? v.rho[1] : v.rho[0]), psi = (gptr<double>)v.psi;
    gptr<double> jx = (gptr<double>)(set ? v.j[1] : v.j[0]), ir = (gptr<double>)v.ir;
    double *rhod = set ? v.rho[0] : v.rho[1];
    double *jd = set ? v.j[0] : v.j[1];
    double *sd = set ? v.s[0] : v.s[1];

    // row r of rho_i and psi_i, row r - 1 of j and 1/rho
    struct In {
        double h[NC], p[NC], jx, jy, ir;
    } X, Y, Z;
    int lr = rbeg, lw = wrap(rbeg), lv = wrap(rbeg - 1);
    auto load = [&](In &q) {
        // in program order, so every wait on a row counts the rows after it
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const int64_t o = (int64_t)lw * nx, m = (int64_t)lv * nx;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            q.h[i] = at(rho + (int64_t)i * v.ld + o);
            q.p[i] = at(psi + (int64_t)i * v.ld + o);
        }
        q.jx = at(jx + m);
        q.jy = at(jx + v.ld + m);
        q.ir = at(ir + m);
        if (lr < rend) {                // past the item's last row: that row again
            ++lr;
            lv = lw;
            lw = next(lw);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    load(X);
    load(Y);
    load(Z);

    auto shl = [](ST q, bool left) -> ST {   // value of the west / east lane
        if constexpr (sizeof(ST) == 4) {
            const int b = __float_as_int(q);
            return __int_as_float(left ? __builtin_amdgcn_mov_dpp(b, 0x138, 0xf, 0xf, true)
                                       : __builtin_amdgcn_mov_dpp(b, 0x130, 0xf, 0xf, true));
        } else {
            return left ? from_left(q) : from_right(q);
        }
    };
    struct Rows {
        double h[NC], p[NC];
    } R0 = {}, R1 = {}, R2 = {};
    // sums on their way, as above
    double part[NC] = {}, d13[NC] = {};
    ST n2[NC] = {}, n5[NC] = {}, n6[NC] = {}, m2[NC] = {}, m5[NC] = {}, m6[NC] = {};
    int64_t o = (int64_t)y0 * nx;

    auto lead = [&](int r, In &cur, const Rows &S, const Rows &M, Rows &T) {
        double jxr = cur.jx, jyr = cur.jy, irr = cur.ir;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            T.h[i] = cur.h[i];
            T.p[i] = cur.p[i];
        }
        load(cur);
        if (r < rbeg + 2) return;
        double Fx[NC], Fy[NC], Gx[NC], Gy[NC], sx = 0.0, sy = 0.0;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            double gx, gy;
            grad3(S.p[i], M.p[i], T.p[i], gx, gy);
            grad3(S.h[i], M.h[i], T.h[i], Gx[i], Gy[i]);
            const double rty = M.h[i] * C->invM[i];
            Fx[i] = -rty * gx;
            Fy[i] = -rty * gy;
            sx += Fx[i];
            sy += Fy[i];
        }
        const double ux = fma(0.5, sx, jxr) * irr, uy = fma(0.5, sy, jyr) * irr;
        double rn[NC], jxt = 0.0, jyt = 0.0, sv = 0.0;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const double h = M.h[i];
            ST t[8];
            double rest;
            if constexpr (sizeof(ST) == 4) {
                rest = h - collide_moving_f32<false>(h, 0.5, 0.0, ux, uy, Fx[i], Fy[i], Gx[i],
                                                     Gy[i], t, t);
            } else {
                collide_d2q9(h, 0.5, ux, uy, Fx[i], Fy[i], Gx[i], Gy[i], t, rest);
            }
            const ST v1 = shl(t[0], true), v3 = shl(t[2], false), v7 = shl(t[6], false),
                     v8 = shl(t[7], true);
            const double d4 = (double)t[3], d5 = (double)n5[i], d6 = (double)n6[i],
                         d7 = (double)v7, d8 = (double)v8;
            rn[i] = (((part[i] + d4) + d5) + d6) + d7 + d8;
            const double e57 = d5 - d7;
            jxt += (d13[i] + e57) + (d8 - d6);
            jyt += (((double)n2[i] - d4) + e57) + (d6 - d8);
            sv = fma(C->sqk[i], rn[i] * C->invM[i], sv);
            part[i] = ((rest + (double)v1) + (double)m2[i]) + (double)v3;
            d13[i] = (double)v1 - (double)v3;
            n2[i] = m2[i];
            n5[i] = m5[i];
            n6[i] = m6[i];
            m2[i] = t[1];
            m5[i] = shl(t[4], true);
            m6[i] = shl(t[5], false);
        }
        if (r < y0 + 2) return;
        if (outl) {
#pragma unroll
            for (int i = 0; i < NC; ++i) put(rhod + (int64_t)i * v.ld + o, rn[i]);
            put(sd + o, sv);
            put(jd + o, jxt);
            put(jd + v.ld + o, jyt);
        }
        o += nx;
    };
    for (int r = rbeg; r <= rend; r += 3) {
        lead(r, X, R0, R1, R2);
        if (r + 1 > rend) break;
        lead(r + 1, Y, R1, R2, R0);
        if (r + 2 > rend) break;
        lead(r + 2, Z, R2, R0, R1);
    }
}

template <int NC>
hipError_t eos_nc(const FieldRun &q, int set, hipStream_t st) {
    hipLaunchKernelGGL((k_field_eos<NC>), dim3((unsigned)q.blocks), dim3(TPB), 0, st, q.tab, q.nm,
                       q.one, q.flip, set);
    return hipGetLastError();
}

template <int NC, typename ST, bool LAST>
hipError_t step_nc(const FieldRun &q, int set, hipStream_t st) {
    const int grid = q.items ? q.nitems : (q.nitems + 7) / 8 * 8;
    hipLaunchKernelGGL((k_field_step<NC, ST, LAST>), dim3(grid), dim3(64 * (NC + HELPERS)), 0, st,
                       q.tab, q.one, q.items, q.nitems, q.strips, q.rows, q.flip, set);
    return hipGetLastError();
}

// Components up to which a step may be taken by single wavefronts.
constexpr int SINGLE_COMP = 3;

template <int NC, typename ST>
hipError_t single_nc(const FieldRun &q, int set, hipStream_t st) {
    const int grid = q.items ? q.nitems : (q.nitems + 7) / 8 * 8;
    hipLaunchKernelGGL((k_field_single<NC, ST>), dim3(grid), dim3(64), 0, st, q.tab, q.one,
                       q.items, q.nitems, q.strips, q.rows, q.flip, set);
    return hipGetLastError();
}

template <int NC>
hipError_t step_sel(const FieldRun &q, bool fp32, bool last, int set, hipStream_t st) {
    if constexpr (NC <= SINGLE_COMP)
        if (q.single && !last)
            return fp32 ? single_nc<NC, float>(q, set, st) : single_nc<NC, double>(q, set, st);
    if (fp32)
        return last ? step_nc<NC, float, true>(q, set, st) : step_nc<NC, float, false>(q, set, st);
    return last ? step_nc<NC, double, true>(q, set, st) : step_nc<NC, double, false>(q, set, st);
}

template <int NC>
int occ_nc(bool single) {
    const void *k = (const void *)k_field_step<NC, double, false>;
    if constexpr (NC <= SINGLE_COMP)
        if (single) k = (const void *)k_field_single<NC, double>;
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &nb, k, single ? 64 : 64 * (NC + HELPERS), 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}

}  // namespace fields

int field_max_comp() { return 10; }

hipError_t launch_field_moments2d(const FieldRun &q, bool fp32, hipStream_t st) {
    if (fp32)
        hipLaunchKernelGGL((fields::k_field_moments<float>), dim3((unsigned)q.blocks), dim3(fields::TPB), 0, st,
                           q.tab, q.nm, q.one, q.flip);
    else
        hipLaunchKernelGGL((fields::k_field_moments<double>), dim3((unsigned)q.blocks), dim3(fields::TPB), 0, st,
                           q.tab, q.nm, q.one, q.flip);
    return hipGetLastError();
}

#define FIELD_BY_N(call)                   \
    switch (ncomp) {                       \
        case 1: return call(1);            \
        case 2: return call(2);            \
        case 3: return call(3);            \
        case 4: return call(4);            \
        case 5: return call(5);            \
        case 6: return call(6);            \
        case 7: return call(7);            \
        case 8: return call(8);            \
        case 9: return call(9);            \
        case 10: return call(10);          \
    }

hipError_t launch_field_eos2d(const FieldRun &q, int ncomp, int set, hipStream_t st) {
#define EOS(n) fields::eos_nc<n>(q, set, st)
    FIELD_BY_N(EOS)
#undef EOS
    return hipErrorInvalidValue;
}

hipError_t launch_field_step2d(const FieldRun &q, int ncomp, bool fp32, bool last, int set,
                               hipStream_t st) {
#define STEP(n) fields::step_sel<n>(q, fp32, last, set, st)
    FIELD_BY_N(STEP)
#undef STEP
    return hipErrorInvalidValue;
}

int field_single_comp() { return fields::SINGLE_COMP; }

int field_blocks_per_cu2d(int ncomp, bool single) {
#define OCC(n) fields::occ_nc<n>(single)
    FIELD_BY_N(OCC)
#undef OCC
    return 1;
}
