// One red-black sweep (colour-0 pass, then colour-1 pass) of a level in a
// single launch, for levels with at least 128 cells per side.
//
// Two launches of the colour pass read both colours of the field twice:
// 2 x 16 B per cell in FP64.  Here a block marches through its z-chunk with
// the colour-1 update two planes behind the colour-0 update, so the field
// and delta are read once and written once: 24 B per cell.
//
// A block owns a tile of 64 packed columns x 8 rows, one wave per row.
// Colour-1 cells at the tile's edge need new colour-0 values outside it, so
// the colour-0 update also covers the rows above and below the tile (waves 0
// and 1) and the cell beside each row's end that the colour-1 cells reach
// (lanes 0..19 of wave 2); 12 rows x 66 columns of the old field are staged
// per plane.
//
// A plane is read from LDS once per column.  What a cell needs of the planes
// above and below is its own column of the opposite colour and the x and y
// differences of its own colour there (the xz and yz cross terms), and since
// the packed parity of a column alternates from plane to plane, the
// differences that the cells of planes k - 1 and k + 1 need of plane k are the
// same ones.  A thread therefore carries them in registers (ColRead) instead
// of reading three staged planes per cell, which also keeps the ring of
// staged planes short enough for two blocks of 512 threads per CU.
//
// Step kp (after one barrier) reads plane kp, finishes the colour-0 cells of
// plane kp - 1 and the colour-1 cells of plane kp - 3, writes the staged
// values of plane kp + 1 and starts the loads of plane kp + 2.
//
// At 512^3 FP64 a sweep takes 600 us, 5.4 TB/s of its 24 B per cell (830 us as
// two colour passes): HBM bounds it.  FP32, 400 us, is bound by instruction
// issue: its vector instructions fill 80% of the cycles.  The prolongation adds
// 115 us (210 us before a coarse plane's in-plane part was kept for the fine
// planes that it serves).  Registers are what two blocks per CU leave short (128
// a thread): nDGP uses 98 to 127, Kmouflage 113 to 128 (its prolongation sweep of a
// coarse level spills one, 8 bytes a thread): see the opaque copies and pins below.
#pragma once
#include <type_traits>
#include "mg_tiled.h"

namespace mgk {

constexpr int SNT = 512;              // threads: a wave per tile row
constexpr int SROWS = TY + 4;         // staged rows -2 .. TY + 1
constexpr int SPLANE = SROWS * TXH;   // 792 values per staged plane
constexpr int SSLOT = SPLANE + 2;     // one value before (vector alignment) and one after
static_assert(SNT == 64 * TY, "one wave per tile row");

// Coarse values around a tile for the prolongation: columns m0 - 2 .. m0 + 65
// (a packed column holds the two children of one coarse column) and coarse
// rows j0/2 - 2 .. j0/2 + 5, one per wave.
constexpr int SCW = TX + 4, SCH = SROWS / 2 + 2, SCPLANE = SCW * SCH;
static_assert(SCH * 64 == SNT, "one wave per coarse row");

// Planes whose loads are in flight during a step.  Two for FP32: with one, the
// two resident blocks of a CU have 20 KB of loads outstanding, too little for
// the latency of HBM (FP64: 40 KB).
template <typename R>
constexpr int prefetch() { return sizeof(R) == 4 ? 2 : 1; }

// Staging of a plane of both colours: 16-byte vectors of the 64 interior
// columns by the last NV threads, the two halo columns by the first 24.
template <typename R>
struct SweepStage {
    static constexpr int VW = 16 / sizeof(R);       // values per vector
    static constexpr int VPR = TX / VW;             // vectors per row
    static constexpr int NV = SROWS * VPR;          // 384 (FP64), 192 (FP32)
    static constexpr int V0 = SNT - NV;             // first vector thread
    static_assert(V0 >= 64 && V0 % 64 == 0 && 2 * SROWS <= 64, "staging split");
    typedef R Vec __attribute__((ext_vector_type(VW)));
    static constexpr int PF = prefetch<R>();
    unsigned g;   // byte offset inside a plane
    int l;        // value offset inside a plane view
    Vec va[PF], vb[PF];   // planes in flight: plane k in k % PF
    __device__ __forceinline__ void init(int tid, int j0, int m0, int logn, int lognh) {
        const unsigned jm = (1u << logn) - 1, mm = (1u << lognh) - 1;
        int r, q;
        unsigned m;
        if (tid >= V0) {
            r = (tid - V0) / VPR;
            const int i = (tid - V0) % VPR;
            q = 1 + VW * i;
            m = (unsigned)(m0 + VW * i);
        } else {
            const int side = tid & 1;
            r = tid < 2 * SROWS ? tid >> 1 : 0;
            q = side ? TXH - 1 : 0;
            m = (unsigned)(side ? m0 + TX : m0 - 1) & mm;
        }
        g = ((((unsigned)(j0 - 2 + r) & jm) << lognh) + m) * (unsigned)sizeof(R);
        l = r * TXH + q;
    }
    __device__ __forceinline__ void fetch(const R *A, const R *B, size_t pl, int slot, int w,
                                          int lane) {
        Vec &a = va[slot % PF], &b = vb[slot % PF];
        const char *pa = reinterpret_cast<const char *>(A) + pl + g;
        const char *pb = reinterpret_cast<const char *>(B) + pl + g;
        if (w >= V0 / 64) {
            a = *reinterpret_cast<const Vec *>(pa);
            b = *reinterpret_cast<const Vec *>(pb);
        } else if (w == 0 && lane < 2 * SROWS) {
            a[0] = *reinterpret_cast<const R *>(pa);
            b[0] = *reinterpret_cast<const R *>(pb);
        }
    }
    // Add the prolonged coarse correction to the fetched values of a plane k
    // (odd: k & 1).  The 27/9/3/1 weights factor into 9, 3, 3, 1 in the plane
    // and 3, 1 between the planes; FP32 rounds in this order in every kernel.
    // A coarse plane's in-plane part (x: per value and x parity) serves four
    // fine planes: it is formed when the first of them, an odd one, is staged
    // and kept in registers (xo: the coarse plane below, xn: the newest).
    R xo[VW][2], xn[VW][2];
    // e: the coarse plane; ec, ed: offsets there of the own coarse row and of
    // its neighbour on the row's side (ed > ec: the row is odd)
    template <int N>
    __device__ __forceinline__ void inplane(const R *e, int ec, int ed) {
        const R w9 = (R)(9.0 / 16.0), w3 = (R)(3.0 / 16.0), w1 = (R)(1.0 / 16.0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const R c = w9 * e[ec + i], d = e[ed + i];
            xo[i][0] = xn[i][0];
            xo[i][1] = xn[i][1];
            xn[i][0] = fma(w1, e[ed + i - 1], fma(w3, d, fma(w3, e[ec + i - 1], c)));
            xn[i][1] = fma(w1, e[ed + i + 1], fma(w3, d, fma(w3, e[ec + i + 1], c)));
        }
    }
    __device__ __forceinline__ void inplane(const R *e, int ec, int ed, int w, int lane) {
        if (w >= V0 / 64)
            inplane<VW>(e, ec, ed);
        else if (w == 0 && lane < 2 * SROWS)
            inplane<1>(e, ec, ed);
    }
    __device__ __forceinline__ void correct(int ec, int ed, bool odd) {
        Vec &a = va[odd % PF], &b = vb[odd % PF];
        const bool p0 = (ed > ec) != odd;   // x parity of the colour-0 values
#pragma unroll
        for (int i = 0; i < VW; ++i) {
            R v[2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
                v[q] = odd ? fma((R)0.75, xo[i][q], (R)0.25 * xn[i][q])
                           : fma((R)0.25, xo[i][q], (R)0.75 * xn[i][q]);
            a[i] += p0 ? v[1] : v[0];
            b[i] += p0 ? v[0] : v[1];
        }
    }
    // sa, sb: the slots' plane views (slot base + 1)
    __device__ __forceinline__ void store(R *sa, R *sb, int slot, int w, int lane) const {
        const Vec &a = va[slot % PF], &b = vb[slot % PF];
        if (w >= V0 / 64) {
            if constexpr (sizeof(R) == 8) {
                *reinterpret_cast<Vec *>(sa + l) = a;
                *reinterpret_cast<Vec *>(sb + l) = b;
            } else {   // rows start 8 bytes off a 16-byte boundary in places
                *reinterpret_cast<float2 *>(sa + l) = make_float2(a[0], a[1]);
                *reinterpret_cast<float2 *>(sa + l + 2) = make_float2(a[2], a[3]);
                *reinterpret_cast<float2 *>(sb + l) = make_float2(b[0], b[1]);
                *reinterpret_cast<float2 *>(sb + l + 2) = make_float2(b[2], b[3]);
            }
        } else if (w == 0 && lane < 2 * SROWS) {
            sa[l] = a[0];
            sb[l] = b[0];
        }
    }
};

// What a column takes from one plane: the x and y neighbours of its own
// colour (for the cross terms of the cells one plane above and below), its
// own column of the opposite colour, and the in-plane combinations of its
// own cell there.  FP32 keeps the four neighbours themselves, so that the
// cross terms are summed in the order of the colour pass and the results are
// its results to the bit; FP64 keeps their differences.
template <typename R>
struct ZEdge {
    R xp, xm, yp, ym;
};
template <>
struct ZEdge<double> {
    double x, y;
};
__device__ __forceinline__ void zedge(ZEdge<float> &e, float xp, float xm, float yp, float ym) {
    e = {xp, xm, yp, ym};
}
__device__ __forceinline__ void zedge(ZEdge<double> &e, double xp, double xm, double yp,
                                      double ym) {
    e = {xp - xm, yp - ym};
}
__device__ __forceinline__ void zcross(const ZEdge<float> &p, const ZEdge<float> &m, float &nxz,
                                       float &nyz) {
    nxz = (p.xp + m.xm) - (m.xp + p.xm);
    nyz = (p.yp + m.ym) - (m.yp + p.ym);
}
__device__ __forceinline__ void zcross(const ZEdge<double> &p, const ZEdge<double> &m,
                                       double &nxz, double &nyz) {
    nxz = p.x - m.x;
    nyz = p.y - m.y;
}

template <typename R>
struct ZPart {   // of a plane above or below the cell
    ZEdge<R> e;
    R b;
    // A: own colour, B: opposite colour (plane views); o: the column's offset,
    // ox: of the right one of its two x neighbours in A, o or o + 1
    __device__ __forceinline__ void read(const R *A, const R *B, int o, int ox) {
        zedge(e, A[ox], A[ox - 1], A[o + TXH], A[o - TXH]);
        b = B[o];
    }
};
template <typename R>
struct XyPart {   // of the cell's own plane
    R ax, ay, ex, ey, nxy, u;
    __device__ __forceinline__ void read(const R *A, const R *B, int o, int ox) {
        const R xp = B[ox], xm = B[ox - 1], yp = B[o + TXH], ym = B[o - TXH];
        ax = xp + xm;
        ay = yp + ym;
        ex = xp - xm;
        ey = yp - ym;
        nxy = (A[ox + TXH] + A[ox - TXH - 1]) - (A[ox - TXH] + A[ox + TXH - 1]);
        u = A[o];
    }
};
template <typename R>
__device__ __forceinline__ CombT<R> col_comb(const ZPart<R> &above, const XyPart<R> &c,
                                             const ZPart<R> &below) {
    CombT<R> s;
    s.ax = c.ax;
    s.ay = c.ay;
    s.az = above.b + below.b;
    s.ex = c.ex;
    s.ey = c.ey;
    s.ez = above.b - below.b;
    s.nxy = c.nxy;
    zcross(above.e, below.e, s.nxz, s.nyz);
    return s;
}

// PROLONG: the coarse level, whose correction is u - Ru.  SOURCE: where the
// level's FAS source goes (s0, s1), and the shift of its restricted residual
// (null: 0).
template <typename R>
struct SweepArgs {
    const R *u0, *u1, *r0, *r1;
    R *s0, *s1;
    const double *shift;
};

// PROLONG: the sweep starts from the prolonged field (first post-smoothing
// sweep): the coarse correction is added while the planes are staged.
// SOURCE: the sweep of a coarse level that follows a restriction.  The level's
// field is R u (L.u) and L.f is R d; the launch forms S = L(R u) - (R d -
// shift) from the planes that it stages anyway, stores it and takes it as the
// right-hand side, so that R u is not copied and S not read back (256^3 FP64:
// 48 B per cell less).  S goes to other arrays than R d: blocks read R d of
// their neighbours' cells.
template <int OP, typename R, bool HASF, bool PROLONG, bool SOURCE = false>
__global__ __launch_bounds__(SNT)
__attribute__((amdgpu_waves_per_eu(4))) void k_sweep_tiled(Mod M, LvlT<R> L, R *__restrict__ out0,
                                                           R *__restrict__ out1,
                                                           SweepArgs<R> K, const double *fptr,
                                                           double fscale,
                                                           unsigned long long *clamp,
                                                           TileGeom G) {
    // ring of staged planes: slot k & 3 holds plane k of colours 0 and 1
    __shared__ __align__(16) R sS[4][2][SSLOT];
    __shared__ R sC[2][TPLANE];   // new colour-0 values, rows -1 .. TY
    // the coarse correction; CARRY: its in-plane part is kept in registers and
    // one coarse plane is staged; FP64 Kmouflage and Newton have none to spare
    // (carried, Kmouflage spills 60 bytes a thread: 125 -> 158 us at 256^3) and
    // form it for every fine plane from a ring of coarse planes
    constexpr bool CARRY = OP == OP_DGP || OP == OP_POISSON || sizeof(R) == 4;
    __shared__ R sE[PROLONG && !CARRY ? 4 : 1][PROLONG ? SCPLANE : 1];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = (int)(blk % G.ntx);
    const int by = (int)((blk / G.ntx) % G.nty);
    const int bz = (int)(blk / ((size_t)G.ntx * G.nty));
    const int m0 = bx * TX, j0 = by * TY, k0 = bz * G.kz, k1 = k0 + G.kz;   // kz is even
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const R fs = uniform((R)(fptr ? fscale * (*fptr) : 0.0));
    static_assert(!SOURCE || (HASF && !PROLONG), "the source is the right-hand side");
    const R shift = uniform((R)(SOURCE && K.shift ? *K.shift : 0.0));
    const R inv_h2 = uniform((R)(1.0 / L.h2));
    SweepStage<R> S;
    S.init(tid, j0, m0, L.logn, L.lognh);
    constexpr int PF = prefetch<R>();
    auto fetch = [&](int k, int par) __attribute__((always_inline)) {   // par: k & 1
        S.fetch(L.u0, L.u1, plane_off<R>(k, L.logn, L.lognh), par, w, lane);
    };

    // coarse correction: a wave loads the first 64 columns of its coarse row,
    // and wave 1, which stages no fine values, the last 4 of all rows (through
    // its staging registers).  Offsets carry the colour of (X + Y) in bit 0.
    R cu = 0, cr = 0;
    unsigned cg = 0;
    int eo = 0;   // offset of the staged value's coarse row; bit 16: odd fine row
    const int lnc = L.logn - 1, ncm = (1 << lnc) - 1;
    if constexpr (PROLONG) {
        auto coff_of = [&](int row, int col) {
            const int X = (m0 - 2 + col) & ncm, Y = ((j0 >> 1) - 2 + row) & ncm;
            return ((((unsigned)Y << (lnc - 1)) + (unsigned)(X >> 1)) * (unsigned)sizeof(R)) |
                   (unsigned)((X + Y) & 1);
        };
        cg = coff_of(w, lane);
        const int r = S.l / TXH, q = S.l - r * TXH;
        eo = (((r >> 1) + 1) * SCW + q + 1) | ((r & 1) << 16);
        if (w == 1) {
            S.g = coff_of((lane >> 2) & 7, TX + (lane & 3));
            S.l = ((lane >> 2) & 7) * SCW + TX + (lane & 3);
        }
    }
    auto cload = [&](unsigned g, int Z, R &u, R &r) {
        const size_t off = (((size_t)(Z & ncm) << (2 * lnc - 1)) * sizeof(R)) + (g & ~1u);
        const bool odd = (g ^ (unsigned)Z) & 1u;
        u = *reinterpret_cast<const R *>(reinterpret_cast<const char *>(odd ? K.u1 : K.u0) + off);
        r = *reinterpret_cast<const R *>(reinterpret_cast<const char *>(odd ? K.r1 : K.r0) + off);
    };
    auto cfetch = [&](int Z) {
        if constexpr (PROLONG) {
            cload(cg, Z, cu, cr);
            if (w == 1 && lane < 4 * SCH) {
                R u, r;
                cload(S.g, Z, u, r);
                S.va[0][0] = u;
                S.vb[0][0] = r;
            }
        }
    };
    auto cplane = [&](int Z) { return sE[CARRY ? 0 : Z & 3]; };
    auto cstore = [&](int Z) {
        if constexpr (PROLONG) {
            R *E = cplane(Z);
            E[w * SCW + lane] = cu - cr;
            if (w == 1 && lane < 4 * SCH) E[S.l] = S.va[0][0] - S.vb[0][0];
        }
    };
    // the fetched plane k (par: k & 1) into its ring slot
    auto stage = [&](int k, auto par) __attribute__((always_inline)) {
        constexpr int odd = decltype(par)::value;
        if constexpr (PROLONG) {
            const int Z = (k + 1) >> 1;
            const int ec = eo & 0xffff, ed = ec - SCW + (eo >> 16) * (2 * SCW);
            if (!CARRY) {
#pragma unroll
                for (int i = 0; i < SweepStage<R>::VW; ++i) S.xn[i][0] = S.xn[i][1] = 0;
                S.inplane(cplane(Z - 1), ec, ed, w, lane);
            }
            if (odd || !CARRY) S.inplane(cplane(Z), ec, ed, w, lane);
            if (w >= SweepStage<R>::V0 / 64 || w == 0) S.correct(ec, ed, odd);
        }
        S.store(sS[k & 3][0] + 1, sS[k & 3][1] + 1, odd, w, lane);
    };

    // own column: row w, packed column lane
    int o = (w + 2) * TXH + 1 + lane;
    const unsigned coff0 = cell_off<R>(j0 + w, m0, L.lognh);
    // extra colour-0 column of waves 0..2
    const int ye = w == 0 ? -1 : w == 1 ? TY : (lane >> 1) - 1;
    const int qe = w < 2 ? 1 + lane : (lane & 1) ? TXH - 1 : 0;
    const bool extra = w < 2 || (w == 2 && lane < 2 * TYH);
    int oe = extra ? (ye + 2) * TXH + qe : o;
    unsigned coffe =
        cell_off<R>((j0 + ye) & (L.n - 1), (m0 - 1 + qe) & ((1 << L.lognh) - 1), L.lognh);

    ZPart<R> P[2] = {}, Q[2] = {};   // colour 0 and colour 1: the last two planes
    XyPart<R> q = {};                // colour 1: the last plane
    // delta and f: colour 0 (own and extra) and colour 1, plane k in k % PF
    R d0n[PF] = {}, dxn[PF] = {}, d1n[PF] = {}, f0n[PF] = {}, fxn[PF] = {}, f1n[PF] = {};
    unsigned nclamp = 0;
    XyPart<R> qs = {};               // SOURCE: the same, of the old field
    R Qs[2] = {};
    auto source = [&](const CombT<R> &s, R u, R delta, R rd) {
        return (s.faces() - (R)6 * u) * inv_h2 -
               tiled_term<OP, R>(M, L, s, delta, s.faces(), u, (unsigned long long *)nullptr) -
               (rd - shift);
    };
    auto update = [&](const CombT<R> &s, R u, R delta, R f, bool count) {
        unsigned neg = 0;
        const R nv = tiled_update<OP, R>(M, L, s, delta, s.faces(), u, f + fs, &neg);
        if (count) nclamp += neg;
        return nv;
    };
    // One step; PAR = kp & 1.  FULL: a step with all its parts (planes
    // k0 + 3 .. k1 - 1), free of branches on kp.
    auto step = [&](int kp, auto par, auto full) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        constexpr bool FULL = decltype(full)::value;
        // opaque copies: the addresses derived from them are formed again in
        // every step instead of being kept in registers for the whole march
        asm("" : "+v"(o), "+v"(oe), "+v"(coffe), "+v"(S.g), "+v"(S.l));
        if constexpr (PROLONG) asm("" : "+v"(eo), "+v"(cg));
        const unsigned coff = coff0 + (unsigned)(o - ((w + 2) * TXH + 1)) * (unsigned)sizeof(R);
        if (FULL || kp <= k1) stage(kp + 1, std::integral_constant<int, 1 - PAR>{});
        if (FULL || kp + PF <= k1) fetch(kp + 1 + PF, (PAR + 1 + PF) & 1);
        // coarse plane (kp >> 1) + 2, first needed for plane kp + 3 (PAR = 0)
        if constexpr (PROLONG && PAR == 0) {
            if (FULL || kp <= k1 - 2) cfetch((kp >> 1) + 2);
        }
        if constexpr (PROLONG && PAR == 1) {
            if (FULL || kp <= k1 - 1) cstore((kp + 3) >> 1);
        }
        // delta and f of a cell: loaded PF steps ahead once this step's are
        // used (colour 0 of plane kp - 1, colour 1 of plane kp - 3)
        constexpr int SL = (1 - PAR) % PF;
        R &d0 = d0n[SL], &dx = dxn[SL], &d1 = d1n[SL], &f0 = f0n[SL], &fx = fxn[SL], &f1 = f1n[SL];
        const size_t pl0 = plane_off<R>(kp - 1 + PF, L.logn, L.lognh);
        const bool next0 = FULL || (kp >= k0 - PF && kp <= k1 + 1 - PF);
        // plane views: kp and the two below it
        const R *A0 = sS[kp & 3][0] + 1, *A1 = sS[(kp - 1) & 3][0] + 1,
                *A2 = sS[(kp - 2) & 3][0] + 1;
        // x parity of a colour-0 column of row w in plane kp is (w + kp) & 1;
        // its complement holds for colour 0 in plane kp - 1 and for colour 1
        // in plane kp - 2
        const int ox = o + ((w + PAR + 1) & 1), oy = o + ((w + PAR) & 1);
        const int t = kp - 1;
        if (FULL || kp <= k1 + 1) {
            ZPart<R> a;
            a.read(A0, A0 + SSLOT, o, ox);
            if (FULL || kp >= k0) {
                const bool own = FULL || (t >= k0 && t < k1);
                XyPart<R> c;
                c.read(A1, A1 + SSLOT, o, ox);
                const CombT<R> s = col_comb(a, c, P[PAR]);
                if (SOURCE) {
                    f0 = source(s, c.u, d0, f0);
                    if (own) *ptr(K.s0, plane_off<R>(t, L.logn, L.lognh), coff) = f0;
                }
                const R nv = update(s, c.u, d0, f0, own);
                sC[1 - PAR][o - TXH] = nv;
                if (own)
                    __builtin_nontemporal_store(nv, ptr(out0, plane_off<R>(t, L.logn, L.lognh),
                                                        coff));
            }
            if (next0) {
                d0 = ld(L.d0, pl0, coff);
                if (HASF) f0 = ld(L.f0, pl0, coff);
            }
            P[PAR] = a;
            if (w < 3) {
                if (extra) {
                    if (FULL || kp >= k0) {
                        const int oex = oe + ((ye + PAR + 1) & 1);
                        ZPart<R> ae, be;
                        XyPart<R> c;
                        ae.read(A0, A0 + SSLOT, oe, oex);
                        be.read(A2, A2 + SSLOT, oe, oex);
                        c.read(A1, A1 + SSLOT, oe, oex);
                        const CombT<R> s = col_comb(ae, c, be);
                        if (SOURCE) fx = source(s, c.u, dx, fx);
                        sC[1 - PAR][oe - TXH] = update(s, c.u, dx, fx, false);
                    }
                    if (next0) {
                        dx = ld(L.d0, pl0, coffe);
                        if (HASF) fx = ld(L.f0, pl0, coffe);
                    }
                }
            }
        }
        if (FULL || (kp >= k0 + 1 && kp <= k1 + 2)) {
            const R *B = A2 + SSLOT, *C = sC[PAR] - TXH;
            ZPart<R> a;
            a.read(B, C, o, oy);
            if (FULL || kp >= k0 + 3) {
                const CombT<R> s = col_comb(a, q, Q[PAR]);
                if (SOURCE) {   // the old field: other face neighbours
                    CombT<R> z = s;
                    z.ax = qs.ax;
                    z.ay = qs.ay;
                    z.ex = qs.ex;
                    z.ey = qs.ey;
                    z.az = A2[o] + Qs[PAR];
                    z.ez = A2[o] - Qs[PAR];
                    f1 = source(z, q.u, d1, f1);
                    *ptr(K.s1, plane_off<R>(kp - 3, L.logn, L.lognh), coff) = f1;
                }
                const R nv = update(s, q.u, d1, f1, true);
                __builtin_nontemporal_store(nv, ptr(out1, plane_off<R>(kp - 3, L.logn, L.lognh),
                                                    coff));
            }
            if (FULL || (kp >= k0 + 3 - PF && kp <= k1 + 2 - PF)) {
                const size_t pl = plane_off<R>(kp - 3 + PF, L.logn, L.lognh);
                d1 = ld_once(L.d1, pl, coff);
                if (HASF) f1 = ld_once(L.f1, pl, coff);
            }
            Q[PAR] = a;
            q.read(B, C, o, ox);
            // formed here: sunk to their use in the next step, they would keep
            // every value read in a register
            asm volatile("" : "+v"(q.ax), "+v"(q.ay), "+v"(q.nxy));
            if constexpr (OP == OP_KMO) asm volatile("" : "+v"(q.ex), "+v"(q.ey));
            if constexpr (SOURCE) {
                Qs[PAR] = A2[o];
                const R xp = A2[ox], xm = A2[ox - 1], yp = A2[o + TXH], ym = A2[o - TXH];
                qs.ax = xp + xm;
                qs.ay = yp + ym;
                qs.ex = xp - xm;
                qs.ey = yp - ym;
                asm volatile("" : "+v"(qs.ax), "+v"(qs.ay));
                if constexpr (OP == OP_KMO) asm volatile("" : "+v"(qs.ex), "+v"(qs.ey));
            }
        }
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    fetch(k0 - 2, 0);
    if (PF == 2) fetch(k0 - 1, 1);
    if constexpr (PROLONG) {
#pragma unroll
        for (int z = -2; z <= 0; ++z) {
            cfetch((k0 >> 1) + z);
            cstore((k0 >> 1) + z);
            __syncthreads();
            if (CARRY && z < 0) {
                const int ec = eo & 0xffff, ed = ec - SCW + (eo >> 16) * (2 * SCW);
                S.inplane(sE[0], ec, ed, w, lane);
                __syncthreads();
            }
        }
    }
    stage(k0 - 2, even);
    fetch(k0 - 2 + PF, PF & 1);
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
    for (; kp + PF < k1; kp += 2) {
        step(kp, even, std::true_type{});
        step(kp + 1, odd, std::true_type{});
    }
    edge(k1 + 3);
    if (clamp && nclamp) atomicAdd(clamp, (unsigned long long)nclamp);
}

}  // namespace mgk
