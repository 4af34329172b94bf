// D3Q19 steps at tau = 1 in field form (gfx950): the steps of a run between
// its first and its last, without populations in memory.
//
// As on D2Q9 (fields2d.h), the collision at tau = 1 needs rho_i and j of the
// old populations and nothing else, so a run reads its populations once
// (moments and interface passes of the multi-pass kernels), carries rho_i, s
// and j from step to step, and writes the populations of the state it ends
// in (collision pass).  Between them a step is
//
//   velocity pass   u from psi_i, rho_i, j
//   k_stream3       F_i, G_i, collision, and the sums of the nineteen
//                   populations that arrive at a site (rho_i, s, j)
//   k_eos3          psi_i of the new state
//
// which moves 11 N + 24 field values per site where the multi-pass step
// moves 38 N population values and 6 N + 14 field values.  The terms, their
// roundings and the orders of summation are those of the multi-pass kernels:
// bitwise the same state.
//
// Measured on 128^3, N = 10 (us a step, multi-pass before): FP64 1875 ->
// 956 ... 983 (velocity 125, k_stream3 730, k_eos3 106), FP32 storage 1211 ->
// 889 ... 906 (128, 654, 106); 75 64 50, N = 9: 256 -> 127 and 153 -> 122.  What bounds
// k_stream3 is VALU work (64 % busy with 2 to 3 wavefronts a SIMD, 2.7 GB at
// 3.6 TB/s): 430 to 490 instructions a plane of a wavefront, of which the
// rims of its tiles waste a quarter to a third.  The rim planes, which only
// hand five populations into the chunk, once took all of that (75 64 50 FP32
// storage 139 us, 50 120 24 FP64 129 -> 109).  Taken back: the plane loop
// unrolled by three to spare the copies of the ring of planes (FP64 232
// registers, FP32 55 spills); three wavefronts a SIMD in FP64 (168 registers,
// 15 spills: 128^3 956 -> 936, but 100^3 448 -> 522).
#pragma once

#include <type_traits>

#include "fused_common.h"
#include "generic_tiles.h"

namespace fields3 {

using fused::cptr;
using fused::from_left;
using fused::from_right;
using fused::gmptr;
using fused::gptr;

// psi_i of the state (rho_i, s): ln f_i and interface term with the
// operations of the moments and interface passes.  One thread per site,
// every component in registers.
template <int NC>
__global__ __launch_bounds__(TPB) void k_eos3(GenMember g) {
#pragma clang fp contract(off)
    cptr<SimConst> C = (cptr<SimConst>)g.c;
    const int nx = C->nx, ny = C->ny, nz = C->nz;
    const int64_t ns = C->nsites;
    const int64_t s64 = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (s64 >= ns) return;
    const uint32_t s = (uint32_t)s64;
    double rt[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) rt[i] = g.rho_f[(int64_t)i * ns + s];
    double lap;
    {
        const uint32_t row = s / (uint32_t)nx;
        const int x = (int)(s - row * (uint32_t)nx), z = (int)(row / (uint32_t)ny),
                  y = (int)(row - (uint32_t)z * (uint32_t)ny);
        const int xs[3] = {x == 0 ? nx - 1 : x - 1, x, x + 1 == nx ? 0 : x + 1};
        const int ys[3] = {y == 0 ? ny - 1 : y - 1, y, y + 1 == ny ? 0 : y + 1};
        const int zs[3] = {z == 0 ? nz - 1 : z - 1, z, z + 1 == nz ? 0 : z + 1};
        const double sc = g.s_f[s];
        double acc = 0.0;
#pragma unroll
        for (int a = 1; a < D3Q19::Q; ++a) {
            const int64_t nb = (int64_t)xs[D3Q19::ex(a) + 1] +
                               (int64_t)nx * ((int64_t)ys[D3Q19::ey(a) + 1] +
                                              (int64_t)ny * zs[D3Q19::ez(a) + 1]);
            acc = fma(D3Q19::w(a), g.s_f[nb] - sc, acc);
        }
        lap = 6.0 * acc;
    }
    uint32_t bad = 0;
    double rtt = 0.0, eta = 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        rtt = fma(rt[i], C->invM[i], rtt);
        rt[i] *= C->invM[i];
        if (!(rt[i] > 0.0)) bad |= FUG_ST_NEGATIVE;
        eta = fma(C->b[i], rt[i], eta);
    }
    const double inv_rt = 1.0 / rtt;
    double S[NC], am = 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) acc = fma(rt[j], C->aij[i * FUG_MAXC + j], acc);
        S[i] = acc * inv_rt;
        am = fma(rt[i] * inv_rt, S[i], am);
    }
    const double RT = C->RT;
    const double ome = 1.0 - eta;
    if (!(ome > 0.0)) bad |= FUG_ST_COVOLUME;
    const double inv_bm = 1.0 / (eta / rtt);
    const double den = fma(C->ew * eta, eta, fma(C->eu, eta, 1.0));
    const double zm1 = eta / ome - (am * rtt) / (RT * den);
    const double lhat =
        C->eos == 2 ? eta : log(fma(C->d1, eta, 1.0) / fma(C->d2, eta, 1.0)) * C->dk;
    const double lam_c = lhat * inv_bm, pref = log(RT / ome);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const double bi_bm = C->b[i] * inv_bm;
        const double X = fma(bi_bm, zm1, log(rt[i]) + pref);
        const double Y = fma(-am, bi_bm, 2.0 * S[i]);
        const double lnf = fma(RT, X, -(lam_c * Y));
        if (!isfinite(lnf)) bad |= FUG_ST_NONFINITE;
        g.psi_f[(int64_t)i * ns + s] = fma(-C->sqk[i], lap, lnf);
    }
    flag_status(g.status, bad);
}

// One plane of a field at a lane: own row and the rows south and north of
// it.  Its lane shifts are taken where they are used: kept, they cost 16
// registers and 1 to 2 % of the step (128^3 x 10: 965 us FP64, 905 FP32
// storage, against 956 and 889).
struct Plane {
    double s, c, n;
    __device__ __forceinline__ double w() const { return from_left(c); }
    __device__ __forceinline__ double e() const { return from_right(c); }
};

// Lattice gradient in pairwise-difference form, the operations of
// lattice_grad: planes below (b), own (o), above (t).
__device__ __forceinline__ void grad19(const Plane &b, const Plane &o, const Plane &t, double &gx,
                                       double &gy, double &gz) {
#pragma clang fp contract(off)
    constexpr double w1 = 1.0 / 18.0, w2 = 1.0 / 36.0;
    const double d1 = o.e() - o.w(), d3 = o.n - o.s, d5 = t.c - b.c;
    const double d7 = from_right(o.n) - from_left(o.s), d9 = from_right(o.s) - from_left(o.n);
    const double d11 = t.e() - b.w(), d13 = b.e() - t.w(), d15 = t.n - b.s, d17 = b.n - t.s;
    gx = fma(w2, d13, fma(w2, d11, fma(w2, d9, fma(w2, d7, w1 * d1))));
    gy = fma(w2, d17, fma(w2, d15, fma(-w2, d9, fma(w2, d7, w1 * d3))));
    gz = fma(-w2, d17, fma(w2, d15, fma(-w2, d13, fma(w2, d11, w1 * d5))));
    gx *= 3.0;
    gy *= 3.0;
    gz *= 3.0;
}

// One step from the fields of `cur` (rho_i, psi_i, u) to those of `nxt`
// (rho_i, s, j).
//
// A workgroup owns a tile of W - 4 columns and R - 2 rows (R = its wavefronts
// times 64 / W) and marches up the planes of a chunk, component after
// component: the sums over components (j, s) are then taken in order, each
// thread adding to what it wrote for the component before.  A thread holds
// three planes of rho_i and psi_i at its (x, y) and the rows beside it, so
// the gradients need only lane shifts; of the populations of a plane the ten
// that move in y go through LDS (their move in x comes with the address),
// those that move in z wait in registers, and every site is collided once
// but for the tile's rim.
template <typename ST, int WAVES>
__global__ __launch_bounds__(64 * WAVES, sizeof(ST) == 4 ? 3 : 2) void k_stream3(
    GenMember gc, GenMember gn, Tiles3 T) {
    constexpr int nth = 64 * WAVES;
    __shared__ ST ex[2][10][nth];
    // neighbouring tiles on one XCD (workgroups go to the eight in turn)
    const int per = (int)gridDim.x / 8;
    const int u = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (u >= T.tx * T.ty * T.tz) return;
    const int W = T.W, sh = 31 - __clz(W), R = nth >> sh;
    const int x0 = (u % T.tx) * (W - 4), y0 = (u / T.tx % T.ty) * (R - 2),
              z0 = (u / (T.tx * T.ty)) * T.zc;
    cptr<SimConst> C = (cptr<SimConst>)gc.c;
    const int N = C->N, nx = C->nx, ny = C->ny, nz = C->nz;
    const int64_t ns = C->nsites, plane = (int64_t)nx * ny;
    const int nzc = min(T.zc, nz - z0);
    const int t = (int)threadIdx.x, row = t >> sh, lx = t & (W - 1);
    auto wrap = [](int v, int n) {
        while (__any(v < 0 || v >= n)) v = v < 0 ? v + n : (v >= n ? v - n : v);
        return v;
    };
    const int x = wrap(x0 - 2 + lx, nx), y = wrap(y0 - 1 + row, ny);
    const int ys = y == 0 ? ny - 1 : y - 1, yn = y + 1 == ny ? 0 : y + 1;
    // byte offsets within a plane
    const uint32_t oc = ((uint32_t)y * (uint32_t)nx + (uint32_t)x) * 8u,
                   os = ((uint32_t)ys * (uint32_t)nx + (uint32_t)x) * 8u,
                   on = ((uint32_t)yn * (uint32_t)nx + (uint32_t)x) * 8u;
    const bool outv = lx >= 2 && lx < W - 2 && row >= 1 && row < R - 1;
    const bool active = outv && x0 + lx - 2 < nx && y0 + row - 1 < ny;
    auto at = [](const double *p, uint32_t o) {
        return *(gptr<double>)((gptr<char>)(gptr<double>)p + o);
    };
    auto put = [](double *p, uint32_t o, double v) {
        *(gmptr<double>)((gmptr<char>)(gmptr<double>)p + o) = v;
    };
    auto zwrap = [&](int z) {
        while (z < 0) z += nz;
        while (z >= nz) z -= nz;
        return z;
    };
    // value that arrives from the west / east lane
    auto shx = [](ST v, bool left) -> ST {
        if constexpr (sizeof(ST) == 4) {
            const int b = __float_as_int(v);
            return __int_as_float(left ? __builtin_amdgcn_mov_dpp(b, 0x138, 0xf, 0xf, true)
                                       : __builtin_amdgcn_mov_dpp(b, 0x130, 0xf, 0xf, true));
        } else {
            return left ? from_left(v) : from_right(v);
        }
    };
    int buf = 0;
    for (int i = 0; i < N; ++i) {
        const double *rho = gc.rho_f + (int64_t)i * ns, *psi = gc.psi_f + (int64_t)i * ns;
        const double invM = C->invM[i], sqk = C->sqk[i];
        struct Raw {
            double hs, hc, hn, ps, pc, pn;
        };
        auto load = [&](int z) -> Raw {
            const double *r = rho + plane * zwrap(z), *p = psi + plane * zwrap(z);
            return {at(r, os), at(r, oc), at(r, on), at(p, os), at(p, oc), at(p, on)};
        };
        Raw q = load(z0 - 2);
        Plane hb{q.hs, q.hc, q.hn}, pb{q.ps, q.pc, q.pn};
        q = load(z0 - 1);
        Plane ho{q.hs, q.hc, q.hn}, po{q.ps, q.pc, q.pn};
        q = load(z0);
        // sums on their way to plane z - 1 (done but for what comes down
        // from plane z) and populations going up to plane z
        double r5 = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
        ST v7 = 0, v8 = 0, v9 = 0, v10 = 0, v11 = 0, v14 = 0, v15 = 0, v18 = 0;
        ST u5 = 0, u11 = 0, u14 = 0, u15 = 0, u18 = 0;
        // the rim planes (z0 - 1, below, and z0 + nzc, above) give the
        // chunk the five populations that move into it and nothing else
        auto step = [&](int z, auto below, auto above) {
            constexpr bool BELOW = decltype(below)::value, ABOVE = decltype(above)::value;
            const Plane ht{q.hs, q.hc, q.hn}, pt{q.ps, q.pc, q.pn};
            const int64_t zo = plane * zwrap(z);
            const double ux = at(gc.u_f + zo, oc), uy = at(gc.u_f + ns + zo, oc),
                         uz = at(gc.u_f + 2 * ns + zo, oc);
            if constexpr (!ABOVE) q = load(z + 2);
            // j of the components before, and s for plane z - 1
            double Jx = 0.0, Jy = 0.0, Jz = 0.0, sv = 0.0;
            if (!BELOW && !ABOVE && i > 0) {
                Jx = at(gn.j_f + zo, oc);
                Jy = at(gn.j_f + ns + zo, oc);
                Jz = at(gn.j_f + 2 * ns + zo, oc);
            }
            if (!BELOW && i > 0 && z > z0) sv = at(gn.s_f + plane * (z - 1), oc);
            double gx, gy, gz, Gx, Gy, Gz;
            grad19(pb, po, pt, gx, gy, gz);
            grad19(hb, ho, ht, Gx, Gy, Gz);
            const double r = ho.c, rt = r * invM;
            ST A[D3Q19::Q];
            const double rest = collide_tau1<D3Q19, ST>(
                r, ux, uy, uz, -rt * gx, -rt * gy, -rt * gz, Gx, Gy, Gz,
                [&](int a, ST v) { A[a] = v; });
            hb = ho;
            ho = ht;
            pb = po;
            po = pt;
            // the populations that move in y, by direction (those of them
            // that move into the chunk)
            ST *e = ex[buf][0];
            buf ^= 1;
            constexpr int dir[10] = {3, 4, 7, 8, 9, 10, 15, 18, 16, 17};
            constexpr int from = BELOW ? 6 : (ABOVE ? 8 : 0), to = BELOW ? 8 : 10;
#pragma unroll
            for (int d = from; d < to; ++d) e[d * nth + t] = A[dir[d]];
            A[1] = shx(A[1], true);
            A[2] = shx(A[2], false);
            A[11] = shx(A[11], true);
            A[12] = shx(A[12], false);
            A[13] = shx(A[13], true);
            A[14] = shx(A[14], false);
            __syncthreads();
            if (outv) {
#pragma unroll
                for (int d = from; d < to; ++d)
                    A[dir[d]] = e[d * nth + t - D3Q19::ey(dir[d]) * W - D3Q19::ex(dir[d])];
            }
            if (!BELOW && z > z0 && active) {
                double rn = r5;
                rn += (double)A[6];
                rn += (double)v7;
                rn += (double)v8;
                rn += (double)v9;
                rn += (double)v10;
                rn += (double)v11;
                rn += (double)A[12];
                rn += (double)A[13];
                rn += (double)v14;
                rn += (double)v15;
                rn += (double)A[16];
                rn += (double)A[17];
                rn += (double)v18;
                jx = ((jx - (double)A[12]) + (double)A[13]) - (double)v14;
                jy = ((jy - (double)A[16]) + (double)A[17]) - (double)v18;
                jz = jz - (double)A[6];
                jz = ((jz + (double)v11) - (double)A[12]) - (double)A[13];
                jz = ((jz + (double)v14) + (double)v15) - (double)A[16];
                jz = (jz - (double)A[17]) + (double)v18;
                const int64_t zd = plane * (z - 1);
                put(gn.rho_f + (int64_t)i * ns + zd, oc, rn);
                put(gn.s_f + zd, oc, fma(sqk, rn * invM, sv));
                put(gn.j_f + zd, oc, jx);
                put(gn.j_f + ns + zd, oc, jy);
                put(gn.j_f + 2 * ns + zd, oc, jz);
            }
            if constexpr (!BELOW && !ABOVE) {
                r5 = rest;
                r5 += (double)A[1];
                r5 += (double)A[2];
                r5 += (double)A[3];
                r5 += (double)A[4];
                r5 += (double)u5;
                jx = ((Jx + (double)A[1]) - (double)A[2]) + (double)A[7];
                jx = ((jx - (double)A[8]) + (double)A[9]) - (double)A[10];
                jx += (double)u11;
                jy = ((Jy + (double)A[3]) - (double)A[4]) + (double)A[7];
                jy = ((jy - (double)A[8]) - (double)A[9]) + (double)A[10];
                jy += (double)u15;
                jz = Jz + (double)u5;
                v7 = A[7];
                v8 = A[8];
                v9 = A[9];
                v10 = A[10];
                v11 = u11;
                v14 = u14;
                v15 = u15;
                v18 = u18;
            }
            if constexpr (!ABOVE) {
                u5 = A[5];
                u11 = A[11];
                u14 = A[14];
                u15 = A[15];
                u18 = A[18];
            }
        };
        step(z0 - 1, std::true_type{}, std::false_type{});
        for (int z = z0; z < z0 + nzc; ++z) step(z, std::false_type{}, std::false_type{});
        step(z0 + nzc, std::false_type{}, std::true_type{});
    }
}

template <typename ST, int WAVES>
hipError_t stream_t(const FieldRun3 &q, int set, hipStream_t st) {
    hipLaunchKernelGGL((k_stream3<ST, WAVES>), dim3((unsigned)q.nitems), dim3(64 * WAVES), 0, st,
                       q.f[set], q.f[set ^ 1], q.tiles);
    return hipGetLastError();
}

template <typename ST>
hipError_t stream(const FieldRun3 &q, int set, hipStream_t st) {
    switch (q.waves) {
        case 4: return stream_t<ST, 4>(q, set, st);
        case 8: return stream_t<ST, 8>(q, set, st);
        case 12:
            if constexpr (sizeof(ST) == 4) return stream_t<ST, 12>(q, set, st);
    }
    return hipErrorInvalidValue;
}

template <typename ST, int WAVES>
int stream_blocks() {
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &nb, (const void *)k_stream3<ST, WAVES>, 64 * WAVES, 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}

template <int NC>
hipError_t eos(const FieldRun3 &q, int set, hipStream_t st) {
    hipLaunchKernelGGL((k_eos3<NC>), dim3(nblocks(q.ns)), dim3(TPB), 0, st, q.f[set]);
    return hipGetLastError();
}

void velocity(const FieldRun3 &q, int set, hipStream_t st) {
    const GenMember &g = q.f[set];
    hipLaunchKernelGGL((k_velocity_t<D3Q19>), dim3(unit_blocks(q.total[1])), dim3(TPB), 0, st,
                       g.c, g.rho_f, g.psi_f, g.j_f, g.u_f);
}

}  // namespace fields3

int field3_blocks_per_cu(bool fp32, int waves) {
    switch (waves) {
        case 4: return fp32 ? fields3::stream_blocks<float, 4>() : fields3::stream_blocks<double, 4>();
        case 8: return fp32 ? fields3::stream_blocks<float, 8>() : fields3::stream_blocks<double, 8>();
        default: return fields3::stream_blocks<float, 12>();
    }
}

hipError_t launch_field_moments3(const FieldRun3 &q, bool fp32, hipStream_t st) {
    const dim3 nb(nblocks(q.ns));
    const GenMember &g = q.f[0];
    if (fp32)
        hipLaunchKernelGGL((k_moments_eos<D3Q19, float>), nb, dim3(TPB), 0, st, g.c,
                           g.buf[g.parity], g.rho_f, g.psi_f, g.s_f, g.j_f, g.status);
    else
        hipLaunchKernelGGL((k_moments_eos<D3Q19, double>), nb, dim3(TPB), 0, st, g.c,
                           g.buf[g.parity], g.rho_f, g.psi_f, g.s_f, g.j_f, g.status);
    hipLaunchKernelGGL((k_interface<D3Q19>), nb, dim3(TPB), 0, st, g.c, g.s_f, g.psi_f);
    return hipGetLastError();
}

hipError_t launch_field_step3(const FieldRun3 &q, int ncomp, bool fp32, int set, hipStream_t st) {
    fields3::velocity(q, set, st);
    const hipError_t e =
        fp32 ? fields3::stream<float>(q, set, st) : fields3::stream<double>(q, set, st);
    if (e != hipSuccess) return e;
    switch (ncomp) {
        case 1: return fields3::eos<1>(q, set ^ 1, st);
        case 2: return fields3::eos<2>(q, set ^ 1, st);
        case 3: return fields3::eos<3>(q, set ^ 1, st);
        case 4: return fields3::eos<4>(q, set ^ 1, st);
        case 5: return fields3::eos<5>(q, set ^ 1, st);
        case 6: return fields3::eos<6>(q, set ^ 1, st);
        case 7: return fields3::eos<7>(q, set ^ 1, st);
        case 8: return fields3::eos<8>(q, set ^ 1, st);
        case 9: return fields3::eos<9>(q, set ^ 1, st);
        case 10: return fields3::eos<10>(q, set ^ 1, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_field_last3(const FieldRun3 &q, bool fp32, int set, hipStream_t st) {
    fields3::velocity(q, set, st);
    const dim3 cb(unit_blocks(q.total[2]));
    const GenMember &g = q.f[set];
    // the populations go to the buffer the run started from
    if (fp32)
        hipLaunchKernelGGL((k_collide_t<D3Q19, float, false>), cb, dim3(TPB), 0, st, g.c, nullptr,
                           g.buf[g.parity], g.rho_f, g.psi_f, g.u_f);
    else
        hipLaunchKernelGGL((k_collide_t<D3Q19, double, false>), cb, dim3(TPB), 0, st, g.c, nullptr,
                           g.buf[g.parity], g.rho_f, g.psi_f, g.u_f);
    return hipGetLastError();
}
