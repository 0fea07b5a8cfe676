// Residual + restriction (see k_resid_restrict) on levels with at least 128
// cells per side.
//
// A block of 512 threads owns 64 packed columns x 8 rows, a wave per row, and
// marches through its z-chunk.  A thread computes both cells of its column and
// reads a staged plane once, nine values per colour: the x and y neighbours of
// a column in one colour are the face neighbours of the other colour's cell in
// the same plane and the cross-term neighbours of the own colour's cells one
// plane above and below, because the packed parity alternates with the colour
// and with the plane.  The rest of a stencil is carried in registers from the
// two planes before, so two staged planes (one read, one written) and one
// barrier a step are enough.
//
// Step kp (after one barrier) reads plane kp, evaluates the cells of plane
// kp - 1, writes the staged values of plane kp + 1 and starts the loads of
// plane kp + 2 (FP32: kp + 3).  The waves of odd rows pass their residuals through LDS to the
// wave of the row below, which adds the eight children of a coarse cell in
// the order of k_resid_restrict and stores it one step later.
//
// 512^3 FP64: 495 us, 4.9 TB/s of its 18 B per cell (560 us with three staged
// planes, two barriers a plane and 38 LDS reads for two cells); FP32 355 to 380
// us, 3.3 TB/s (405 us), bound by instruction issue; 256^3 Kmouflage 88 -> 70 us.
#pragma once
#include "mg_sweep.h"

namespace mgk {

// Staging of a plane (rows -1 .. TY of 66 columns) of both colours: pairs of
// the 64 interior columns by waves 3 .. 7, the two halo columns by 20 lanes of
// wave 0.
template <typename R>
struct RowStage {
    static constexpr int PF = prefetch<R>();
    static constexpr int V0 = SNT - TYH * (TX / 2);   // first pair thread
    static_assert(V0 >= 64 && V0 % 64 == 0 && 2 * TYH <= 64, "staging split");
    typedef R Vec __attribute__((ext_vector_type(2)));
    unsigned g;   // byte offset inside a plane
    int l;        // value offset inside a plane view
    Vec va[PF], vb[PF];   // planes in flight: plane k in k % PF
    __device__ __forceinline__ void init(int tid, int j0, int m0, int logn, int lognh) {
        const unsigned jm = (1u << logn) - 1, mm = (1u << lognh) - 1;
        int r, q;
        unsigned m;
        if (tid >= V0) {
            r = (tid - V0) / (TX / 2);
            const int i = (tid - V0) % (TX / 2);
            q = 1 + 2 * i;
            m = (unsigned)(m0 + 2 * i);
        } else {
            const int side = tid & 1;
            r = tid < 2 * TYH ? tid >> 1 : 0;
            q = side ? TXH - 1 : 0;
            m = (unsigned)(side ? m0 + TX : m0 - 1) & mm;
        }
        g = ((((unsigned)(j0 - 1 + r) & jm) << lognh) + m) * (unsigned)sizeof(R);
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
        } else if (w == 0 && lane < 2 * TYH) {
            a[0] = *reinterpret_cast<const R *>(pa);
            b[0] = *reinterpret_cast<const R *>(pb);
        }
    }
    // sa, sb: the slots' plane views (slot base + 1)
    __device__ __forceinline__ void store(R *sa, R *sb, int slot, int w, int lane) const {
        const Vec &a = va[slot % PF], &b = vb[slot % PF];
        if (w >= V0 / 64) {
            *reinterpret_cast<Vec *>(sa + l) = a;
            *reinterpret_cast<Vec *>(sb + l) = b;
        } else if (w == 0 && lane < 2 * TYH) {
            sa[l] = a[0];
            sb[l] = b[0];
        }
    }
};

// What a column takes of one colour of a plane.  FP32 keeps the neighbours
// themselves: its Laplacian is summed in double, its term in float.
template <typename R>
struct RowCol {
    R xp, xm, yp, ym, own, nxy;
    __device__ __forceinline__ void read(const R *A, int o, int ox, int oy) {
        xp = A[ox];
        xm = A[ox - 1];
        yp = A[o + TXH];
        ym = A[o - TXH];
        own = A[o];
        nxy = (A[oy + TXH] + A[oy - TXH - 1]) - (A[oy - TXH] + A[oy + TXH - 1]);
    }
    __device__ __forceinline__ void pin() { asm volatile("" : "+v"(nxy)); }
    __device__ __forceinline__ ZEdge<R> edge() const { return {xp, xm, yp, ym}; }
    __device__ __forceinline__ double faces(double z) const {
        return ((double)xp + (double)xm) + ((double)yp + (double)ym) + z;
    }
    __device__ __forceinline__ void faces(CombT<R> &s) const {
        s.ax = xp + xm;
        s.ay = yp + ym;
        s.ex = xp - xm;
        s.ey = yp - ym;
    }
};
template <>
struct RowCol<double> {
    double ax, ay, ex, ey, own, nxy;
    __device__ __forceinline__ void read(const double *A, int o, int ox, int oy) {
        const double xp = A[ox], xm = A[ox - 1], yp = A[o + TXH], ym = A[o - TXH];
        ax = xp + xm;
        ay = yp + ym;
        ex = xp - xm;
        ey = yp - ym;
        own = A[o];
        nxy = (A[oy + TXH] + A[oy - TXH - 1]) - (A[oy - TXH] + A[oy + TXH - 1]);
    }
    // formed here: sunk to their use in the next step, they would keep every
    // value read in a register
    __device__ __forceinline__ void pin() {
        asm volatile("" : "+v"(ax), "+v"(ay), "+v"(ex), "+v"(ey), "+v"(nxy));
    }
    __device__ __forceinline__ ZEdge<double> edge() const { return {ex, ey}; }
    __device__ __forceinline__ double faces(double z) const { return ax + ay + z; }
    __device__ __forceinline__ void faces(CombT<double> &s) const {
        s.ax = ax;
        s.ay = ay;
        s.ex = ex;
        s.ey = ey;
    }
};
template <typename R>
struct RowZ {   // kept of the plane before
    ZEdge<R> e;
    R own;
};

// kz counts coarse planes.  HASF: the level has a right-hand side f (every
// level but the finest).  REDUCE: block sums of the residual and its square.
// WG: also store g = -d of every fine cell in FP32 (g0/g1, the packed colours;
// the outer step of the defect-correction solve).
template <int OP, bool REDUCE, bool HASF, typename R, bool WG = false>
__global__ __launch_bounds__(SNT)
__attribute__((amdgpu_waves_per_eu(4))) void k_resid_tiled(Mod M, LvlT<R> L, const double *fptr,
                                                           double fscale, R *ru0, R *ru1, R *rd0,
                                                           R *rd1, double *partials,
                                                           unsigned long long *clamp, TileGeom G,
                                                           float *g0 = nullptr,
                                                           float *g1 = nullptr) {
    __shared__ __align__(16) R sS[2][2][TSLOT];   // plane k in slot k & 1
    // residuals (d0, d1) and u0 + u1 of the odd rows
    __shared__ double sD[2][3][SNT / 2];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = (int)(blk % G.ntx);
    const int by = (int)((blk / G.ntx) % G.nty);
    const int bz = (int)(blk / ((size_t)G.ntx * G.nty));
    const int m0 = bx * TX, j0 = by * TY, k0 = 2 * bz * G.kz, k1 = k0 + 2 * G.kz;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double fs = uniform(fptr ? fscale * (*fptr) : 0.0), inv_h2 = uniform(1.0 / L.h2);
    RowStage<R> S;
    S.init(tid, j0, m0, L.logn, L.lognh);
    constexpr int PF = prefetch<R>();
    // par: k & 1
    auto fetch = [&](int k, int par) __attribute__((always_inline)) {
        S.fetch(L.u0, L.u1, plane_off<R>(k, L.logn, L.lognh), par, w, lane);
    };
    auto store = [&](int par) __attribute__((always_inline)) {
        S.store(sS[par][0] + 1, sS[par][1] + 1, par, w, lane);
    };

    int o = (w + 1) * TXH + 1 + lane;
    unsigned coff = cell_off<R>(j0 + w, m0 + lane, L.lognh);
    RowCol<R> C[2] = {};   // plane kp - 1
    RowZ<R> B[2] = {};     // plane kp - 2
    R dn[PF][2] = {}, fn[PF][2] = {};   // delta, f of plane k in k % PF
    double su = 0.0, sd = 0.0, acc1 = 0.0, acc2 = 0.0;
    unsigned nclamp = 0;

    auto step = [&](int kp, auto par, auto full) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        constexpr bool FULL = decltype(full)::value;
        asm("" : "+v"(o), "+v"(coff), "+v"(S.g), "+v"(S.l));
        if (FULL || kp < k1) store(1 - PAR);
        if (FULL || kp + PF < k1) fetch(kp + 1 + PF, (PAR + 1 + PF) & 1);
        R *dc = dn[(1 - PAR) % PF], *fc = fn[(1 - PAR) % PF];
        const int p = (w + PAR) & 1;
        if (!(w & 1)) {   // even rows: the odd row's children of plane kp - 2
            const int s = (w >> 1) * 64 + lane;
            if (FULL || kp >= k0 + 2) {
                sd += sD[1 - PAR][0][s];
                sd += sD[1 - PAR][1][s];
                su += sD[1 - PAR][2][s];
                if (PAR == 1) {
                    const int K = (kp - 2) >> 1, I = m0 + lane, J = (j0 + w) >> 1;
                    const int lnc = L.logn - 1;
                    const size_t cidx =
                        ((size_t)K << (2 * lnc - 1)) + ((size_t)J << (lnc - 1)) + (size_t)(I >> 1);
                    const int ccol = (I + J + K) & 1;
                    (ccol ? ru1 : ru0)[cidx] = (R)(0.125 * su);
                    (ccol ? rd1 : rd0)[cidx] = (R)(0.125 * sd);
                    su = 0.0;
                    sd = 0.0;
                }
            }
        }
        if (FULL || kp <= k1) {
            // colour-1 neighbours lie at p in the own plane (seen from colour 0)
            RowCol<R> N[2];
            N[0].read(sS[PAR][0] + 1, o, o + (1 - p), o + p);
            N[1].read(sS[PAR][1] + 1, o, o + p, o + (1 - p));
            N[0].pin();
            N[1].pin();
            if (FULL || kp > k0) {
                double d[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const double u = (double)C[c].own;
                    const double f = (HASF ? (double)fc[c] : 0.0) + fs;
                    const double faces =
                        C[1 - c].faces((double)N[1 - c].own + (double)B[1 - c].own);
                    unsigned neg = 0;
                    if constexpr (OP == OP_POISSON && sizeof(R) == 4) {
                        d[c] = (faces - 6.0 * u) * inv_h2 - M.s * (double)dc[c] - f;
                    } else {
                        CombT<R> s;
                        C[1 - c].faces(s);
                        s.az = N[1 - c].own + B[1 - c].own;
                        s.ez = N[1 - c].own - B[1 - c].own;
                        s.nxy = C[c].nxy;
                        zcross(N[c].edge(), B[c].e, s.nxz, s.nyz);
                        d[c] = (faces - 6.0 * u) * inv_h2 -
                               (double)tiled_term<OP, R>(M, L, s, dc[c], (R)faces, (R)u, &neg) - f;
                    }
                    nclamp += neg;
                    if (REDUCE) {
                        acc1 += d[c];
                        acc2 += d[c] * d[c];
                    }
                    if (WG)
                        *ptr(c ? g1 : g0, plane_off<float>(kp - 1, L.logn, L.lognh),
                             cell_off<float>(j0 + w, m0 + lane, L.lognh)) = (float)(-d[c]);
                }
                if (w & 1) {
                    const int s = (w >> 1) * 64 + lane;
                    sD[PAR][0][s] = d[0];
                    sD[PAR][1][s] = d[1];
                    sD[PAR][2][s] = (double)C[0].own + (double)C[1].own;
                } else {
                    sd += d[0];
                    sd += d[1];
                    su += (double)C[0].own + (double)C[1].own;
                }
            }
            const int kd = kp - 1 + PF;
            if (FULL || (kd >= k0 && kd < k1)) {
                const size_t pl = plane_off<R>(kd, L.logn, L.lognh);
                dc[0] = ld_once(L.d0, pl, coff);
                dc[1] = ld_once(L.d1, pl, coff);
                if (HASF) {
                    fc[0] = ld_once(L.f0, pl, coff);
                    fc[1] = ld_once(L.f1, pl, coff);
                }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                B[c].e = C[c].edge();
                B[c].own = C[c].own;
                C[c] = N[c];
            }
        }
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    fetch(k0 - 1, 1);
    if (PF == 2) fetch(k0, 0);
    store(1);
    fetch(k0 - 1 + PF, (1 + PF) & 1);
    __syncthreads();
    step(k0 - 1, odd, std::false_type{});
    int kp = k0;
    auto edge = [&](int end) __attribute__((always_inline)) {
#pragma unroll 1
        for (; kp < end; kp += 2) {
            step(kp, even, std::false_type{});
            step(kp + 1, odd, std::false_type{});
        }
    };
    edge(k0 + 2);
#pragma unroll 1
    for (; kp + 1 + PF < k1; kp += 2) {
        step(kp, even, std::true_type{});
        step(kp + 1, odd, std::true_type{});
    }
    edge(k1 + 2);
    if (clamp && nclamp) atomicAdd(clamp, (unsigned long long)nclamp);
    if (REDUCE) block_sum2<SNT>(acc1, acc2, partials, blk);
}

}  // namespace mgk
