// LDS-tiled kernels of the nDGP adjoint solve (J^T mu = f, see mg_adj_tiled.h)
// on levels with at least 128 cells per side.
//
// With F' = dK/dSigma of a cell (the one array kept per level besides the
// linearisation point phi), the Jacobian's coefficients are products of F' and
// second differences of phi, so the kernel forms, per cell and plane,
//   face colour o:    W_a = mu - h^2 (2 F' c3h4) (3 A_a - A_x - A_y - A_z) mu,  a = x, y, z
//   target colour c:  E_ab = -h^2 (2 F' c8h4) N_ab mu,                   ab = xy, xz, yz
// and a target cell's sum is
//   S = sum of W_a over its six face neighbours (W_x at p +- x, ...)
//     + sum of +-E_ab over its edge neighbours (+ at p-x-y and p+x+y, - at the others),
// S = faces - h^2 G in the notation of k_adj_tiled.
//
// The march is that of the sweep kernel (mg_sweep.h): a block of 512 threads
// owns 64 packed columns x 8 rows, a wave per row, and a thread forms the
// products of its own column.  phi of the target colour is staged (12 rows x
// 66 columns) and each plane is read once per column, 9 values: the x and y
// neighbours of the face-colour cell (their sums are A_x and A_y, their
// differences the parts of N_xz and N_yz of the target cells one plane above
// and below), the own value (A_z of those planes) and four corners (N_xy).
// W_z stays with its column in a register; the other five products pass through
// LDS, double-buffered, so that one barrier separates the steps.  The products
// of the rows above and below the tile are formed by waves 0 and 1, those of
// the columns beside it by 20 lanes of wave 2, from the ring of phi planes.
// Step kp: read phi of plane kp, form the products of plane kp - 1, sum those
// of plane kp - 2, which completes the target cells of plane kp - 3.
// Per cell and colour pass 28 B: mu of both colours, phi of the target
// colour, F' of both colours, f and the new value.
// At 512^3 a colour pass takes 747 us (5.0 TB/s of those 28 B, 6.0 with the
// halo: HBM bounds it) and a residual + restriction 796 us; forming each
// product where it is staged, with phi read from a ring of 12 x 68 planes and
// two barriers a plane, they took 1150 and 1193 us.  84 to 104 VGPRs: two
// blocks a CU; 11 LDS reads and 5 writes a column and plane.
#pragma once
#include "mg_adj_tiled.h"
#include "mg_sweep.h"

namespace mgk {

// What a column keeps of a phi plane.
struct PhiZ {   // for the products of the planes above and below
    double dx, dy, own;
};
struct PhiXy {   // for the plane's own products
    double ax, ay, nxy;
};

template <int MODE, bool REDUCE>
__global__ __launch_bounds__(SNT)
__attribute__((amdgpu_waves_per_eu(4))) void k_adj_dgp(AdjLevel L, int c, double *out,
                                                       double *out2, const double *fptr,
                                                       double fscale, double *ru0, double *ru1,
                                                       double *rd0, double *rd1, double *partials,
                                                       TileGeom G) {
    __shared__ __align__(16) double sP[4][SSLOT];   // phi_c: slot k & 3
    __shared__ double sWx[2][TY * TXH], sXz[2][TY * TXH];   // rows 0 .. TY - 1
    __shared__ double sWy[2][TPLANE], sXy[2][TPLANE], sYz[2][TPLANE];   // rows -1 .. TY
    __shared__ double sR[2][MODE == ADJ_RESID ? SNT / 2 : 1];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = (int)(blk % G.ntx);
    const int by = (int)((blk / G.ntx) % G.nty);
    const int bz = (int)(blk / ((size_t)G.ntx * G.nty));
    const int m0 = bx * TX, j0 = by * TY, k0 = bz * G.kz, k1 = k0 + G.kz;   // kz is even
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double *Mo = c ? L.u0 : L.u1, *Mc = c ? L.u1 : L.u0;
    const double *Ko = L.kp[c ^ 1], *Kc = L.kp[c], *Pc = L.lin[c], *F = c ? L.f1 : L.f0;
    const double fs = uniform(fptr ? fscale * (*fptr) : 0.0), inv_h2 = uniform(1.0 / L.h2);
    const double w3 = uniform(-2.0 * L.c3h4 * L.h2), w8 = uniform(-2.0 * L.c8h4 * L.h2);

    SweepStage<double> S;
    S.init(tid, j0, m0, L.logn, L.lognh);
    constexpr int VW0 = SweepStage<double>::V0 / 64;
    auto fetch = [&](int k) {
        const char *p = reinterpret_cast<const char *>(Pc) + plane_off<double>(k, L.logn, L.lognh) + S.g;
        if (w >= VW0)
            S.va[0] = *reinterpret_cast<const SweepStage<double>::Vec *>(p);
        else if (w == 0 && lane < 2 * SROWS)
            S.va[0][0] = *reinterpret_cast<const double *>(p);
    };
    auto store = [&](int k) {
        double *s = sP[k & 3] + 1;
        if (w >= VW0)
            *reinterpret_cast<SweepStage<double>::Vec *>(s + S.l) = S.va[0];
        else if (w == 0 && lane < 2 * SROWS)
            s[S.l] = S.va[0][0];
    };

    // own column and the extra one of waves 0..2 (see k_sweep_tiled)
    int o = (w + 2) * TXH + 1 + lane;
    unsigned coff = cell_off<double>(j0 + w, m0 + lane, L.lognh);
    const int ye = w == 0 ? -1 : w == 1 ? TY : (lane >> 1) - 1;
    const int qe = w < 2 ? 1 + lane : (lane & 1) ? TXH - 1 : 0;
    const bool extra = w < 2 || (w == 2 && lane < 2 * TYH);
    int oe = extra ? (ye + 2) * TXH + qe : o;
    unsigned coffe =
        cell_off<double>((j0 + ye) & (L.n - 1), (m0 - 1 + qe) & ((1 << L.lognh) - 1), L.lognh);

    // mu and F' of a column's two cells, one plane ahead
    struct Cell {
        double mo, ko, mc, kc;
    };
    auto load_cell = [&](Cell &q, size_t pl, unsigned off) {
        q.mo = ld(Mo, pl, off);
        q.ko = ld(Ko, pl, off);
        q.mc = ld(Mc, pl, off);
        q.kc = ld(Kc, pl, off);
    };
    // ox: o + the x parity of the face-colour cell in the plane read (its x
    // neighbours are ox and ox - 1); oc: o + that of the target-colour cell
    auto read_z = [](const double *P, int oo, int ox) {
        return PhiZ{P[ox] - P[ox - 1], P[oo + TXH] - P[oo - TXH], P[oo]};
    };
    auto read_xy = [](const double *P, int oo, int ox, int oc) {
        return PhiXy{P[ox] + P[ox - 1], P[oo + TXH] + P[oo - TXH],
                     (P[oc + TXH] - P[oc + TXH - 1]) - (P[oc - TXH] - P[oc - TXH - 1])};
    };

    Cell cn = {}, ce = {};
    PhiZ Z[2] = {};
    double fn = 0.0, wz = 0.0, acc = 0.0, up = 0.0;
    double un = 0.0;   // mu of the next target cell (not PASS)
    double bs1 = 0.0, bs2 = 0.0, rr = 0.0, rm = 0.0;

    // restriction of the plane pair that the previous step closed (kp odd: its
    // planes are kp - 5 and kp - 4): the odd rows' sums are in sR
    auto pair_combine = [&](int K) __attribute__((always_inline)) {
        if (!(w & 1)) {
            int ln = lane;
            asm("" : "+v"(ln), "+s"(K));
            const int lnc = L.logn - 1, I = m0 + ln, J = (j0 + w) >> 1;
            const size_t cidx =
                ((size_t)K << (2 * lnc - 1)) + ((size_t)J << (lnc - 1)) + (size_t)(I >> 1);
            const bool odd = (I + J + K) & 1;
            double *pr = (odd ? rd1 : rd0) + cidx, *pu = (odd ? ru1 : ru0) + cidx;
            const double sr = rr + sR[0][(w >> 1) * 64 + ln], su = rm + sR[1][(w >> 1) * 64 + ln];
            if (c == 0) {   // raw sums of the 4 colour-0 children
                *pr = sr;
                *pu = su;
            } else {        // add the 4 colour-1 children: the 8-cell mean
                *pr = 0.125 * (*pr + sr);
                *pu = 0.125 * (*pu + su);
            }
        }
        rr = rm = 0.0;
    };

    // target cell of plane T: sum is S of the header, f its right-hand side, u its mu;
    // pair: T is odd
    auto finish = [&](double sum, double f, double u, int T, auto pair) __attribute__((always_inline)) {
        constexpr bool PAIR = decltype(pair)::value;
        const size_t pl = plane_off<double>(T, L.logn, L.lognh);
        if constexpr (MODE == ADJ_PASS) {
            const double nv = (sum - L.h2 * (f + fs)) * (1.0 / 6.0);
            __builtin_nontemporal_store(nv, ptr(out, pl, coff));
            if (REDUCE) bs1 += nv;
        } else {
            const double d = (sum - 6.0 * u) * inv_h2 - f;
            if constexpr (MODE == ADJ_RESID) {
                if (REDUCE) {
                    bs1 += d;
                    bs2 += d * d;
                }
                rr += d;
                rm += u;
                if (PAIR && (w & 1)) {   // closes a plane pair
                    sR[0][(w >> 1) * 64 + lane] = rr;
                    sR[1][(w >> 1) * 64 + lane] = rm;
                }
            } else {
                *ptr(out, pl, coff) = d;
                *ptr(out2, pl, coff) = u;
            }
        }
    };

    auto step = [&](int kp, auto par, auto full) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        constexpr bool FULL = decltype(full)::value;
        // opaque copies: see k_sweep_tiled
        asm("" : "+v"(o), "+v"(oe), "+v"(coff), "+v"(coffe), "+v"(S.g), "+v"(S.l));
        if (FULL || kp <= k1) store(kp + 1);
        if (FULL || kp < k1) fetch(kp + 2);
        if constexpr (MODE == ADJ_RESID && PAR == 1) {
            if (FULL || kp >= k0 + 5) pair_combine((kp - 4) >> 1);
        }
        // x parity of the target-colour cell of row w in plane kp is
        // (w + kp + c) & 1; the face-colour cell has its complement, and the
        // parities swap from plane to plane
        const int pt = (w + PAR + c) & 1, oc = o + pt, of = o + 1 - pt;
        // The parts of a step one after the other (interleaved, they do not
        // fit 128 registers), each followed by the loads that it needs in the
        // next step.  First the sums of plane kp - 2 (target parity of plane kp).
        __builtin_amdgcn_sched_barrier(0);
        if (FULL || (kp >= k0 + 1 && kp <= k1 + 2)) {
            const double *Wx = sWx[PAR] - 2 * TXH, *Xz = sXz[PAR] - 2 * TXH;
            const double *Wy = sWy[PAR] - TXH, *Xy = sXy[PAR] - TXH, *Yz = sYz[PAR] - TXH;
            const double ge = (Xz[of - 1] - Xz[of]) + (Yz[o - TXH] - Yz[o + TXH]);
            if (FULL || kp >= k0 + 3)
                finish(acc + (wz - ge), fn, un, kp - 3, std::bool_constant<PAR == 0>{});
            acc = up + ((Wx[oc] + Wx[oc - 1]) + (Wy[o + TXH] + Wy[o - TXH])) +
                  ((Xy[oc - TXH - 1] + Xy[oc + TXH]) - (Xy[oc + TXH - 1] + Xy[oc - TXH]));
            up = wz + ge;
            // formed here: sunk to their use in the next step, they would keep
            // every product read above in a register
            asm volatile("" : "+v"(acc), "+v"(up));
            if constexpr (MODE == ADJ_RESID) asm volatile("" : "+v"(rr), "+v"(rm));
            if constexpr (REDUCE) asm volatile("" : "+v"(bs1), "+v"(bs2));
        }
        if (FULL || (kp >= k0 + 2 && kp <= k1 + 1)) {
            const size_t pl = plane_off<double>(kp - 2, L.logn, L.lognh);
            fn = ld_once(F, pl, coff);
            if (MODE != ADJ_PASS) un = ld(Mc, pl, coff);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (FULL || kp <= k1 + 1) {
            const double *P0 = sP[kp & 3] + 1, *P1 = sP[(kp - 1) & 3] + 1,
                         *P2 = sP[(kp - 2) & 3] + 1;
            const size_t pl = plane_off<double>(kp, L.logn, L.lognh);
            const bool next = FULL || (kp >= k0 - 1 && kp <= k1);
            const PhiZ z = read_z(P0, o, of);
            if (FULL || kp >= k0) {   // products of plane kp - 1 (parities swapped)
                const PhiXy q = read_xy(P1, o, oc, of);
                const double az = z.own + Z[PAR].own, sum = q.ax + q.ay + az;
                const double a = w3 * cn.ko * cn.mo, e = w8 * cn.kc * cn.mc;
                wz = fma(a, 3.0 * az - sum, cn.mo);
                sWx[1 - PAR][o - 2 * TXH] = fma(a, 3.0 * q.ax - sum, cn.mo);
                sWy[1 - PAR][o - TXH] = fma(a, 3.0 * q.ay - sum, cn.mo);
                sXy[1 - PAR][o - TXH] = e * q.nxy;
                sXz[1 - PAR][o - 2 * TXH] = e * (z.dx - Z[PAR].dx);
                sYz[1 - PAR][o - TXH] = e * (z.dy - Z[PAR].dy);
            }
            if (next) load_cell(cn, pl, coff);
            Z[PAR] = z;
            __builtin_amdgcn_sched_barrier(0);
            if (w < 3) {
                if (extra) {
                    if (FULL || kp >= k0) {
                        const int pe = (ye + PAR + c) & 1;
                        const PhiZ za = read_z(P0, oe, oe + 1 - pe), zb = read_z(P2, oe, oe + 1 - pe);
                        const PhiXy qx = read_xy(P1, oe, oe + pe, oe + 1 - pe);
                        const double az = za.own + zb.own, sum = qx.ax + qx.ay + az;
                        const double a = w3 * ce.ko * ce.mo, e = w8 * ce.kc * ce.mc;
                        sXy[1 - PAR][oe - TXH] = e * qx.nxy;
                        if (w < 2) {
                            sWy[1 - PAR][oe - TXH] = fma(a, 3.0 * qx.ay - sum, ce.mo);
                            sYz[1 - PAR][oe - TXH] = e * (za.dy - zb.dy);
                        } else if ((unsigned)ye < (unsigned)TY) {
                            sWx[1 - PAR][oe - 2 * TXH] = fma(a, 3.0 * qx.ax - sum, ce.mo);
                            sXz[1 - PAR][oe - 2 * TXH] = e * (za.dx - zb.dx);
                        }
                    }
                    if (next) load_cell(ce, pl, coffe);
                }
            }
        }
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    fetch(k0 - 2);
    store(k0 - 2);
    fetch(k0 - 1);
    __syncthreads();
    int kp = k0 - 2;
    auto edge = [&](int end) __attribute__((always_inline)) {
#pragma unroll 1
        for (; kp < end; kp += 2) {
            step(kp, even, std::false_type{});
            step(kp + 1, odd, std::false_type{});
        }
    };
    edge(k0 + 4);
#pragma unroll 1
    for (; kp + 1 < k1; kp += 2) {
        step(kp, even, std::true_type{});
        step(kp + 1, odd, std::true_type{});
    }
    edge(k1 + 3);
    if (REDUCE) block_sum2<SNT>(bs1, bs2, partials, blk);
}

}  // namespace mgk
