// Kernels of the FAS multigrid solve.  See mg_device.h for the storage
// layout.  Every kernel is one thread per cell (or per coarse cell), 256
// threads per block, with the block index remapped so that each of the 8
// XCDs works on a contiguous z-slab (its halo rows stay in its own L2).
// R is the storage type (double, or float for the FP32 phase of the mixed
// solve); the adjoint operator exists for double only.
#pragma once
#include "mg_device.h"

namespace mgk {

constexpr int TPB = 256;

// device scalar slots (one small array in the workspace)
enum {
    S_MU = 0,      // finest right-hand side mu = mean L(phi), lagged
    S_SHIFT = 1,   // mean change of the finest residual since mu was last set
    S_EPS2 = 2,    // squared RMS of the last reduced residual
    S_MEAN = 3,    // mean of the last summed field
    S_CSUM0 = 4,   // adjoint, tiled finest level: sum of mu over colour 0
    S_CSUM1 = 5,   // ... over colour 1 (each refreshed by the last kernel that wrote the colour)
    S_MU64 = 6,    // defect correction: the FP64 field's bordering scalar (S_MU is the inner one)
    S_EPS64 = 7,   // defect correction: squared RMS of the FP64 finest residual
    S_NSCAL = 16
};

enum { OP_DGP = MODEL_DGP, OP_KMO = MODEL_KMO, OP_POISSON = MODEL_POISSON, OP_ADJ = 3,
       OP_NEWTON = 4 };

// OP_NEWTON: the nDGP equation in its quadratic form eq:dgp_quadratic_eom,
// divided by alpha, L_N = D + 2 D^2 / (3 alpha) - Sigma / alpha with D the
// 7-point Laplacian (centre included), relaxed by the generic Newton-Gauss-
// Seidel step of eq:relaxation_iteration,
//   u <- u - (L_N - f) / (dL_N/du),  dL_N/du = -(6/h^2)(1 + 4 D / (3 alpha)).
// A comparator for the closed-form update: same fixed point on the physical
// branch.  cell_term returns Sigma / alpha; newton_term adds the D part.
template <typename T>
__device__ __forceinline__ T newton_term(const Mod &M, T sigma_over_alpha, T D) {
    return sigma_over_alpha - (T)(2.0 / (3.0 * M.alpha)) * D * D;
}
template <typename T>
__device__ __forceinline__ T newton_update(const Mod &M, T u, T faces, T sig, T f, T h2) {
    const T D = (faces - (T)6 * u) / h2;
    const T r = D - newton_term<T>(M, sig, D) - f;
    const T dL = -((T)6 / h2) * ((T)1 + (T)(4.0 / (3.0 * M.alpha)) * D);
    return u - r / dL;
}

// Blocks are dispatched round-robin over the 8 XCDs; hand XCD x the x-th
// contiguous eighth of the logical tiles.
__device__ __forceinline__ size_t xcd_block(unsigned b, unsigned nb) {
    if (nb & 7u) return b;
    return (size_t)(b & 7u) * (nb >> 3) + (b >> 3);
}

// Adjoint coefficient arrays of one level: for every cell m the derivative of
// its model term K_m with respect to the 6 face neighbours (x+ x- y+ y- z+ z-)
// and the 3 edge pairs (the (+,+)/(-,-) corners carry +e, the (+,-)/(-,+)
// corners -e).
struct Coefs {
    const double *c[9][2];
};

// Sum of the six face values and the non-Laplacian term at the cell of
// colour c, packed (m, j, k), in arithmetic type T.
template <int OP, typename T, typename R>
__device__ __forceinline__ T cell_term(const Mod &M, const LvlT<R> &L, const Coefs &Cf, int c,
                                       int m, int j, int k, T &faces, unsigned long long *clamp) {
    const R *A = c ? L.u1 : L.u0;
    const R *B = c ? L.u0 : L.u1;
    if (OP == OP_NEWTON) {
        const NbT<T> s = load_nb<T, R>(A, B, c, m, j, k, L.n, L.logn, L.lognh);
        faces = (s.xp + s.xm) + (s.yp + s.ym) + (s.zp + s.zm);
        const R *D = c ? L.d1 : L.d0;
        const T delta = (T)D[prow(j, k, L.logn, L.lognh) + m];
        (void)clamp;
        return dgp_sigma_over_alpha<T>(M, L, s, delta);
    } else if (OP != OP_ADJ) {
        const NbT<T> s = load_nb<T, R>(A, B, c, m, j, k, L.n, L.logn, L.lognh);
        faces = (s.xp + s.xm) + (s.yp + s.ym) + (s.zp + s.zm);
        const R *D = c ? L.d1 : L.d0;
        const T delta = (T)D[prow(j, k, L.logn, L.lognh) + m];
        return model_term<OP == OP_ADJ ? OP_DGP : OP, T>(M, L, s, delta, clamp);
    } else {
        // (J^T mu)_p = lap(mu)_p - sum over the neighbours q of p of
        // dK_q/dphi_p mu_q.  The face neighbour at p - x carries its x+
        // coefficient, the one at p + x its x- coefficient; edge corners carry
        // +e_xy at p-x-y and p+x+y, -e_xy at p-x+y and p+x-y.
        const int nm1 = L.n - 1, hm1 = (L.n >> 1) - 1;
        const int p = (j + k + c) & 1;
        const int mp = (m + p) & hm1, mm = (m + p - 1) & hm1;
        const int jp = (j + 1) & nm1, jm = (j - 1) & nm1;
        const int kp = (k + 1) & nm1, km = (k - 1) & nm1;
        const int ln = L.logn, lh = L.lognh;
        const size_t r00 = prow(j, k, ln, lh);
        const size_t rp0 = prow(jp, k, ln, lh), rm0 = prow(jm, k, ln, lh);
        const size_t r0p = prow(j, kp, ln, lh), r0m = prow(j, km, ln, lh);
        const size_t rpp = prow(jp, kp, ln, lh), rmm = prow(jm, km, ln, lh);
        const size_t rpm = prow(jp, km, ln, lh), rmp = prow(jm, kp, ln, lh);
        const int o = c ^ 1;
        const size_t ixp = r00 + mp, ixm = r00 + mm, iyp = rp0 + m, iym = rm0 + m,
                     izp = r0p + m, izm = r0m + m;
        const T vxp = B[ixp], vxm = B[ixm], vyp = B[iyp], vym = B[iym], vzp = B[izp],
                vzm = B[izm];
        faces = (vxp + vxm) + (vyp + vym) + (vzp + vzm);
        T g = Cf.c[0][o][ixm] * vxm + Cf.c[1][o][ixp] * vxp + Cf.c[2][o][iym] * vym
            + Cf.c[3][o][iyp] * vyp + Cf.c[4][o][izm] * vzm + Cf.c[5][o][izp] * vzp;
        const double *exy = Cf.c[6][c], *exz = Cf.c[7][c], *eyz = Cf.c[8][c];
        g += (exy[rm0 + mm] * A[rm0 + mm] + exy[rp0 + mp] * A[rp0 + mp])
           - (exy[rp0 + mm] * A[rp0 + mm] + exy[rm0 + mp] * A[rm0 + mp]);
        g += (exz[r0m + mm] * A[r0m + mm] + exz[r0p + mp] * A[r0p + mp])
           - (exz[r0p + mm] * A[r0p + mm] + exz[r0m + mp] * A[r0m + mp]);
        g += (eyz[rmm + m] * A[rmm + m] + eyz[rpp + m] * A[rpp + m])
           - (eyz[rmp + m] * A[rmp + m] + eyz[rpm + m] * A[rpm + m]);
        (void)clamp;
        return g;
    }
}

template <typename T, typename R>
__device__ __forceinline__ T rhs_at(const LvlT<R> &L, int c, size_t idx, const double *fptr,
                                    double fscale) {
    const R *fa = c ? L.f1 : L.f0;
    T f = fa ? (T)fa[idx] : (T)0;
    if (fptr) f += (T)(fscale * (*fptr));
    return f;
}

// One colour pass: every cell of colour c gets the exact solution of its own
// equation (faces - 6 u)/h^2 - K = f given its neighbours.
template <int OP, typename R>
__global__ __launch_bounds__(TPB) void k_pass(Mod M, LvlT<R> L, Coefs Cf, int c,
                                              R *__restrict__ out, const double *fptr,
                                              double fscale, unsigned long long *clamp) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    const size_t half = (size_t)1 << (3 * L.logn - 1);
    if (t >= half) return;
    const int m = (int)(t & ((1u << L.lognh) - 1));
    const int j = (int)((t >> L.lognh) & (L.n - 1));
    const int k = (int)(t >> (L.lognh + L.logn));
    R faces;
    const R K = cell_term<OP, R, R>(M, L, Cf, c, m, j, k, faces, clamp);
    const R f = rhs_at<R, R>(L, c, t, fptr, fscale);
    if constexpr (OP == OP_NEWTON)
        out[t] = newton_update<R>(M, (c ? L.u1 : L.u0)[t], faces, K, f, (R)L.h2);
    else
        out[t] = (faces - (R)L.h2 * (K + f)) * (R)(1.0 / 6.0);
}

// Deterministic block sum of two values into partials[2*blk .. 2*blk+1].
template <int NT = TPB>
__device__ __forceinline__ void block_sum2(double a, double b, double *partials, size_t blk) {
    __shared__ double sa[NT / 64], sb[NT / 64];
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sa[w] = a;
        sb[w] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double x = 0.0, y = 0.0;
        for (int q = 0; q < NT / 64; ++q) {
            x += sa[q];
            y += sb[q];
        }
        partials[2 * blk] = x;
        partials[2 * blk + 1] = y;
    }
}

// Residual d = (faces - 6u)/h^2 - K - f (double arithmetic) of every cell,
// restricted (8-cell mean) together with u.  With REDUCE the block sums of d
// and d^2 go to partials (finest level: norm and mean).  A block takes 32
// coarse cells, a thread one child: waves 0 and 1 the four children of colour
// 0 of 16 coarse cells each, waves 2 and 3 those of colour 1 (the colour, and
// with it every array, is uniform in a wave).  The means are then summed child
// by child in a fixed order.  These levels (<= 64^3) are bound by latency: one
// thread per coarse cell, its eight children one after the other, took 10.4 us
// at 32^3 and 64^3.
template <int OP, bool REDUCE, typename R>
__global__ __launch_bounds__(TPB) void k_resid_restrict(Mod M, LvlT<R> L, Coefs Cf,
                                                        const double *fptr, double fscale, R *ru0,
                                                        R *ru1, R *rd0, R *rd1, double *partials,
                                                        unsigned long long *clamp) {
    __shared__ double sd[8][32], su[8][32];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = w >> 1, cell = (w & 1) * 16 + (lane & 15);
    // children of colour 0: 0, 3, 5, 6; of colour 1: 1, 2, 4, 7 (bits x, y, z)
    const int qb = lane >> 4, q = qb < 2 ? (col ? 1 + qb : 3 * qb) : (col ? 3 * qb - 2 : 3 + qb);
    const int lnc = L.logn - 1, nc = 1 << lnc;
    const size_t t = blk * 32 + cell;
    auto coords = [&](size_t tc, int &I, int &J, int &K) {
        I = (int)(tc & (nc - 1));
        J = (int)((tc >> lnc) & (nc - 1));
        K = (int)(tc >> (2 * lnc));
    };
    int I, J, K;
    coords(t, I, J, K);
    const int j = 2 * J + ((q >> 1) & 1), k = 2 * K + (q >> 2);
    const double inv_h2 = 1.0 / L.h2;
    double faces;
    double term = cell_term<OP, double, R>(M, L, Cf, col, I, j, k, faces, clamp);
    const size_t idx = prow(j, k, L.logn, L.lognh) + I;
    const double u = (double)(col ? L.u1 : L.u0)[idx];
    if constexpr (OP == OP_NEWTON) term = newton_term(M, term, (faces - 6.0 * u) * inv_h2);
    const double d = (faces - 6.0 * u) * inv_h2 - term - rhs_at<double, R>(L, col, idx, fptr, fscale);
    sd[q][cell] = d;
    su[q][cell] = u;
    __syncthreads();
    if (threadIdx.x < 32) {
        const size_t tc = blk * 32 + threadIdx.x;
        coords(tc, I, J, K);
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a += sd[e][threadIdx.x];
            b += su[e][threadIdx.x];
        }
        const int ccol = (I + J + K) & 1;
        const size_t cidx = ((size_t)K << (2 * lnc - 1)) + ((size_t)J << (lnc - 1)) + (I >> 1);
        (ccol ? ru1 : ru0)[cidx] = (R)(0.125 * b);
        (ccol ? rd1 : rd0)[cidx] = (R)(0.125 * a);
    }
    if (REDUCE) block_sum2(d, d * d, partials, blk);
}

// Starting value of the finest level's bordering scalar mu: the mean of
// L(phi) - f over 64 cells spread over the mesh (one wave).  The finest
// residual is reduced in one pass, eps^2 = <d^2> - <d>^2, which cancels when
// |<d>| is many orders above eps.  A call's first residual evaluation would
// otherwise see mu = 0 and <d> = the whole mean of L(phi); started from this
// estimate, its <d> is of the order of the residual's spread, and its update
// mu += <d> gives the mean over all cells as before.
template <int OP, typename R>
__global__ __launch_bounds__(64) void k_mu_estimate(Mod M, LvlT<R> L, Coefs Cf, double *mu) {
    const int t = threadIdx.x;
    const int c = t & 1;
    const int m = (t * 5) & ((L.n >> 1) - 1);
    const int j = (t * 7 + 1) & (L.n - 1);
    const int k = (t * 11 + 2) & (L.n - 1);
    double faces;
    double term = cell_term<OP, double, R>(M, L, Cf, c, m, j, k, faces, nullptr);
    const size_t idx = prow(j, k, L.logn, L.lognh) + m;
    const double D = (faces - 6.0 * (double)(c ? L.u1 : L.u0)[idx]) / L.h2;
    if constexpr (OP == OP_NEWTON) term = newton_term(M, term, D);
    double d = D - term - rhs_at<double, R>(L, c, idx, nullptr, 0.0);
    for (int off = 32; off > 0; off >>= 1) d += __shfl_down(d, off, 64);
    if (t == 0) *mu = d * (1.0 / 64.0);
}

// FAS source on the coarse level: S = L^H(R u) - (R d - shift), written over
// the restricted residual; the coarse unknown starts from R u.
template <int OP, typename R>
__device__ __forceinline__ void dev_coarse_source(const Mod &M, const LvlT<R> &Lc, const Coefs &Cf,
                                                  R *s0, R *s1, R *u0, R *u1, double shift, int c,
                                                  size_t tt) {
    const int m = (int)(tt & ((1u << Lc.lognh) - 1));
    const int j = (int)((tt >> Lc.lognh) & (Lc.n - 1));
    const int k = (int)(tt >> (Lc.lognh + Lc.logn));
    double faces;
    double term = cell_term<OP, double, R>(M, Lc, Cf, c, m, j, k, faces, nullptr);
    const R ru = (c ? Lc.u1 : Lc.u0)[tt];
    if constexpr (OP == OP_NEWTON) term = newton_term(M, term, (faces - 6.0 * (double)ru) / Lc.h2);
    R *S = c ? s1 : s0;
    const double rd = (double)S[tt] - shift;
    S[tt] = (R)((faces - 6.0 * (double)ru) / Lc.h2 - term - rd);
    (c ? u1 : u0)[tt] = ru;
}

// u_fine += P(uc - rc) with the cell-centred trilinear weights 27/9/3/1 (/64).
template <typename R>
__device__ __forceinline__ void dev_prolong(R *f0, R *f1, int logn, const R *uc0, const R *uc1,
                                            const R *rc0, const R *rc1, size_t t) {
    const int n = 1 << logn, lognh = logn - 1;
    const size_t half = (size_t)1 << (3 * logn - 1);
    if (t >= 2 * half) return;
    const int c = t >= half;
    const size_t tt = t - (c ? half : 0);
    const int m = (int)(tt & ((1u << lognh) - 1));
    const int j = (int)((tt >> lognh) & (n - 1));
    const int k = (int)(tt >> (lognh + logn));
    const int p = (j + k + c) & 1;   // i = 2m + p, parent I = m
    const int lnc = logn - 1, ncm1 = (1 << lnc) - 1;
    const int I = m, J = j >> 1, K = k >> 1;
    const int di = p ? 1 : -1, dj = (j & 1) ? 1 : -1, dk = (k & 1) ? 1 : -1;
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int a = q & 1, b = (q >> 1) & 1, cc = q >> 2;
        const int I2 = (I + a * di) & ncm1, J2 = (J + b * dj) & ncm1, K2 = (K + cc * dk) & ncm1;
        const size_t idx = ((size_t)K2 << (2 * lnc - 1)) + ((size_t)J2 << (lnc - 1)) + (I2 >> 1);
        const double v = ((I2 + J2 + K2) & 1) ? ((double)uc1[idx] - (double)rc1[idx])
                                              : ((double)uc0[idx] - (double)rc0[idx]);
        const double w = (a ? 1.0 : 3.0) * (b ? 1.0 : 3.0) * (cc ? 1.0 : 3.0);
        acc += w * v;
    }
    R *f = c ? f1 : f0;
    f[tt] = (R)((double)f[tt] + acc * (1.0 / 64.0));
}

template <typename R>
__global__ __launch_bounds__(TPB) void k_prolong(R *f0, R *f1, int logn, const R *uc0,
                                                 const R *uc1, const R *rc0, const R *rc1) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    dev_prolong<R>(f0, f1, logn, uc0, uc1, rc0, rc1, t);
}

// 8-cell mean of a packed field (density hierarchy, linearisation points).
template <typename R>
__global__ __launch_bounds__(TPB) void k_restrict(const R *f0, const R *f1, int logn, R *c0,
                                                  R *c1) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    const int lnc = logn - 1, nc = 1 << lnc;
    if (t >= ((size_t)1 << (3 * lnc))) return;
    const int I = (int)(t & (nc - 1)), J = (int)((t >> lnc) & (nc - 1)), K = (int)(t >> (2 * lnc));
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int a = q & 1, b = (q >> 1) & 1, cc = q >> 2;
        const int j = 2 * J + b, k = 2 * K + cc;
        const size_t idx = ((size_t)k << (2 * logn - 1)) + ((size_t)j << (logn - 1)) + I;
        s += ((a + b + cc) & 1) ? (double)f1[idx] : (double)f0[idx];
    }
    const size_t cidx = ((size_t)K << (2 * lnc - 1)) + ((size_t)J << (lnc - 1)) + (I >> 1);
    (((I + J + K) & 1) ? c1 : c0)[cidx] = (R)(0.125 * s);
}

// natural [z][y][x] -> packed colours (optionally minus a device scalar),
// converting the element type
template <typename Rin, typename Rout>
__global__ __launch_bounds__(TPB) void k_pack(const Rin *nat, int logn, Rout *c0, Rout *c1,
                                              const double *shift) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    if (t >= ((size_t)1 << (3 * logn))) return;
    const int n = 1 << logn;
    const int i = (int)(t & (n - 1)), j = (int)((t >> logn) & (n - 1)), k = (int)(t >> (2 * logn));
    const size_t idx = ((size_t)k << (2 * logn - 1)) + ((size_t)j << (logn - 1)) + (i >> 1);
    const double v = (double)nat[t] - (shift ? *shift : 0.0);
    (((i + j + k) & 1) ? c1 : c0)[idx] = (Rout)v;
}

// k_pack of a finest level's field and its restriction to the next level
// (k_restrict of the stored values) in one pass: a thread takes the 2 x 2 x 2
// cells of a coarse cell.  512^3 FP64: 417 us for 386 + 238 us.
template <typename Rin, typename R>
__global__ __launch_bounds__(TPB) void k_pack_restrict(const Rin *nat, int logn, R *f0, R *f1,
                                                       R *c0, R *c1) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    const int lnc = logn - 1, nc = 1 << lnc;
    if (t >= ((size_t)1 << (3 * lnc))) return;
    const int I = (int)(t & (nc - 1)), J = (int)((t >> lnc) & (nc - 1)), K = (int)(t >> (2 * lnc));
    R v[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const size_t row = ((size_t)(2 * K + (q >> 1)) << (2 * logn)) +
                           ((size_t)(2 * J + (q & 1)) << logn) + (size_t)(2 * I);
        v[2 * q] = (R)nat[row];
        v[2 * q + 1] = (R)nat[row + 1];
    }
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int p = (q ^ (q >> 1)) & 1;   // colour of the first cell
        const size_t idx = ((size_t)(2 * K + (q >> 1)) << (2 * logn - 1)) +
                           ((size_t)(2 * J + (q & 1)) << lnc) + (size_t)I;
        f0[idx] = v[2 * q + p];
        f1[idx] = v[2 * q + 1 - p];
        s += (double)v[2 * q];
        s += (double)v[2 * q + 1];
    }
    const size_t cidx = ((size_t)K << (2 * lnc - 1)) + ((size_t)J << (lnc - 1)) + (I >> 1);
    (((I + J + K) & 1) ? c1 : c0)[cidx] = (R)(0.125 * s);
}

// packed colours -> natural (optionally minus a device scalar)
template <typename Rin, typename Rout>
__global__ __launch_bounds__(TPB) void k_unpack(const Rin *c0, const Rin *c1, int logn,
                                                Rout *nat, const double *shift) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    if (t >= ((size_t)1 << (3 * logn))) return;
    const int n = 1 << logn;
    const int i = (int)(t & (n - 1)), j = (int)((t >> logn) & (n - 1)), k = (int)(t >> (2 * logn));
    const size_t idx = ((size_t)k << (2 * logn - 1)) + ((size_t)j << (logn - 1)) + (i >> 1);
    const double v = (double)(((i + j + k) & 1) ? c1 : c0)[idx];
    nat[t] = (Rout)(v - (shift ? *shift : 0.0));
}

// element-wise conversion between precisions (same packed layout)
template <typename Rin, typename Rout>
__global__ __launch_bounds__(TPB) void k_convert(const Rin *a, Rout *b, size_t n) {
    const size_t t = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (t < n) b[t] = (Rout)a[t];
}

// Block sums of a (and a^2) over up to two arrays laid end to end.
template <typename R>
__global__ __launch_bounds__(TPB) void k_sum(const R *a0, const R *a1, size_t nhalf,
                                             double *partials) {
    // grid-stride: a fixed grid for a given size keeps the order deterministic
    const size_t stride = (size_t)gridDim.x * TPB;
    double v = 0.0, v2 = 0.0;
    for (size_t t = (size_t)blockIdx.x * TPB + threadIdx.x; t < nhalf; t += stride) {
        const double x = (double)a0[t];
        v += x;
        v2 += x * x;
    }
    if (a1) {
        for (size_t t = (size_t)blockIdx.x * TPB + threadIdx.x; t < nhalf; t += stride) {
            const double x = (double)a1[t];
            v += x;
            v2 += x * x;
        }
    }
    block_sum2(v, v2, partials, blockIdx.x);
}

// Finalise a reduction.  mode 0: residual of the finest level with lagged mu
// (mu += mean, shift = mean, eps2 = variance); mode 1: plain mean into
// S_MEAN; mode 2: adjoint residual r = d - kappa*mean(mu) with mean(mu) in
// S_MEAN (shift = 0, eps2 = mean r^2); mode 3: the sum of one colour (colour)
// of the adjoint field into S_CSUM0 + colour, and S_MEAN = the mean of both
// colours' sums; mode 4: both colours' sums at once (first and second
// components); mode 5: mode 0 for the FP64 residual of the defect-correction
// solve (S_MU64 and S_EPS64).  Summation order is fixed.
//
// host: pinned host memory (or null).  The residual's scalars are stored there
// too, then seq into host[S_NSCAL - 1]: the host waits for that number, with
// no copy or event on the stream (they cost 14 us per cycle of a 32^3 solve).

// Sums of the nblocks pairs of block sums, by NT threads of a block (all call
// it); the result is valid in thread 0.
template <int NT>
__device__ __forceinline__ void sum_partials(const double *partials, size_t nblocks, double &x,
                                             double &y) {
    __shared__ double sa[NT / 64], sb[NT / 64];
    double a = 0.0, b = 0.0;
    for (size_t q = threadIdx.x; q < nblocks; q += NT) {
        a += partials[2 * q];
        b += partials[2 * q + 1];
    }
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sa[threadIdx.x >> 6] = a;
        sb[threadIdx.x >> 6] = b;
    }
    __syncthreads();
    x = y = 0.0;
    if (threadIdx.x == 0) {
        for (int q = 0; q < NT / 64; ++q) {
            x += sa[q];
            y += sb[q];
        }
    }
}

// Scalars of a finest residual from its sums x (of d) and y (of d^2): modes 0,
// 2 and 5 of k_finalize (one thread).
__device__ __forceinline__ void residual_scalars(double x, double y, double ncells, double *scal,
                                                 int mode, double kappa, double *host,
                                                 unsigned long long seq) {
    const double mean = x / ncells, msq = y / ncells;
    const int imu = mode == 5 ? S_MU64 : S_MU, ieps = mode == 5 ? S_EPS64 : S_EPS2;
    double v, mu = 0.0;
    if (mode == 2) {
        const double km = kappa * scal[S_MEAN];
        scal[S_SHIFT] = 0.0;
        v = msq - 2.0 * km * mean + km * km;
    } else {
        mu = scal[imu] + mean;
        scal[imu] = mu;
        if (mode == 0) scal[S_SHIFT] = mean;
        v = msq - mean * mean;
    }
    v = v < 0.0 ? 0.0 : v;   // keeps NaN
    scal[ieps] = v;
    if (host) {
        host[imu] = mu;
        host[ieps] = v;
        __hip_atomic_store(reinterpret_cast<unsigned long long *>(host) + S_NSCAL - 1, seq,
                           __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ __launch_bounds__(1024) void k_finalize(const double *partials, size_t nblocks,
                                                   double ncells, double *scal, int mode,
                                                   double kappa, int colour = 0,
                                                   double *host = nullptr,
                                                   unsigned long long seq = 0) {
    double x, y;
    sum_partials<1024>(partials, nblocks, x, y);
    if (threadIdx.x == 0) {
        if (mode == 1) {
            scal[S_MEAN] = x / ncells;
        } else if (mode == 3) {
            scal[S_CSUM0 + colour] = x;
            scal[S_MEAN] = (scal[S_CSUM0] + scal[S_CSUM1]) / ncells;
        } else if (mode == 4) {
            scal[S_CSUM0] = x;
            scal[S_CSUM1] = y;
            scal[S_MEAN] = (x + y) / ncells;
        } else {
            residual_scalars(x, y, ncells, scal, mode, kappa, host, seq);
        }
    }
}

// A finest residual's reduction carried into the next launch (the coarse
// source or the tail), which then needs no k_finalize before it (mode 0, up to
// 512 block sums: finest levels <= 64^3).  Every block sums the partials,
// block 0 stores the scalars.
struct Pending {
    const double *partials;   // null: the scalars are stored already
    unsigned nb;
    double ncells;
    double *scal, *host;
    unsigned long long seq;
};
// The shift of the coarse source (S_SHIFT); every thread of the block calls it.
template <int NT>
__device__ __forceinline__ double pending_shift(const Pending &P, bool store) {
    __shared__ double shift;
    double x, y;
    sum_partials<NT>(P.partials, P.nb, x, y);
    if (threadIdx.x == 0) {
        shift = x / P.ncells;
        if (store) residual_scalars(x, y, P.ncells, P.scal, 0, 0.0, P.host, P.seq);
    }
    __syncthreads();
    return shift;
}

__global__ void k_fill(double *a, size_t n, double v) {
    const size_t t = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (t < n) a[t] = v;
}

__global__ void k_fill_u64(unsigned long long *a, size_t n) {
    const size_t t = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (t < n) a[t] = 0ull;
}

// Residual r = (faces - 6u)/h^2 - term - f at every cell, packed output (double).
template <int OP>
__global__ __launch_bounds__(TPB) void k_residual(Mod M, Lvl L, Coefs Cf, const double *fptr,
                                                  double fscale, double *r0, double *r1,
                                                  unsigned long long *clamp) {
    const size_t t = xcd_block(blockIdx.x, gridDim.x) * TPB + threadIdx.x;
    const size_t half = (size_t)1 << (3 * L.logn - 1);
    if (t >= 2 * half) return;
    const int c = t >= half;
    const size_t tt = t - (c ? half : 0);
    const int m = (int)(tt & ((1u << L.lognh) - 1));
    const int j = (int)((tt >> L.lognh) & (L.n - 1));
    const int k = (int)(tt >> (L.lognh + L.logn));
    double faces;
    double term = cell_term<OP, double, double>(M, L, Cf, c, m, j, k, faces, clamp);
    const double u = (c ? L.u1 : L.u0)[tt];
    if constexpr (OP == OP_NEWTON) term = newton_term(M, term, (faces - 6.0 * u) / L.h2);
    (c ? r1 : r0)[tt] = (faces - 6.0 * u) / L.h2 - term
                      - rhs_at<double, double>(L, c, tt, fptr, fscale);
}

template <int OP, typename R>
__global__ __launch_bounds__(TPB) void k_coarse_source(Mod M, LvlT<R> Lc, Coefs Cf, R *s0, R *s1,
                                                       R *u0, R *u1, const double *shift,
                                                       Pending P) {
    const size_t blk = xcd_block(blockIdx.x, gridDim.x), t = blk * TPB + threadIdx.x;
    const double sh = P.partials ? pending_shift<TPB>(P, blk == 0) : shift ? *shift : 0.0;
    const size_t half = (size_t)1 << (3 * Lc.logn - 1);
    if (t >= 2 * half) return;
    const int c = t >= half;
    dev_coarse_source<OP, R>(M, Lc, Cf, s0, s1, u0, u1, sh, c, t - (c ? half : 0));
}

// ---------------------------------------------------------------- coarse tail
// All levels from 16^3 down to 4^3 in one workgroup: the sub-cycle (smoothing,
// residual + restriction, coarse source, recursion, prolongation) runs with
// barriers between phases instead of one launch per phase.  A colour pass
// first computes every new value of the colour into registers, then writes
// them in place after a barrier, so all cells see the pre-pass state.
//
// One workgroup uses one of the 256 CUs, so what bounds the tail is the
// latency of its serial phases.  Level sizes are compile-time constants (the
// coarsest level is 4^3), and every phase gives each thread a single cell at
// a time: the residual is evaluated per fine cell into LDS and summed over
// the 8 children afterwards (a thread that evaluated the 8 children of its
// coarse cell one after the other kept at most half of the threads busy).
constexpr int TAIL_THREADS = 1024;
constexpr int TAIL_MAX_N = 16;   // <= 2048 cells per colour: 2 per thread
constexpr int TAIL_MAX_LEVELS = 3;

template <typename R>
struct TailLv {
    LvlT<R> L;      // u, d and f (the FAS source, workspace: written by the tail)
    R *ru0, *ru1;   // R u of the finer level
};

template <typename R>
struct TailArgs {
    int nlev, nu1, nu2, nuc;
    int cycle;   // 0 V, 1 F, 2 W
    // the first level's coarse source is formed here (V-cycles, whose tail
    // runs once per source): f then holds R d and u starts from R u
    bool source;
    const double *shift;   // of that source (null: 0), or pending
    Pending pend;
    TailLv<R> lv[TAIL_MAX_LEVELS];
    Coefs cf[TAIL_MAX_LEVELS];
};

// LDS layout, in order: per level u, f (and d, or for the adjoint the
// coefficient arrays of the levels below 16^3), R u below the first level;
// then the residuals (FP64) of the first level's cells.
template <int OP>
__host__ __device__ constexpr int tail_level_arrays(int logn, bool first) {
    // half-level arrays: u 2, f 2, d 2 or 18 coefficient halves, R u 2
    return 4 + (OP == OP_ADJ ? (logn < 4 ? 18 : 0) : 2) + (first ? 0 : 2);
}
// Values before level lv (of nl).
template <int OP>
__host__ __device__ constexpr int tail_offset(int nl, int lv) {
    int tot = 0;
    for (int q = 0; q < lv; ++q) {
        const int logn = 1 + nl - q;
        tot += tail_level_arrays<OP>(logn, q == 0) * (1 << (3 * logn - 1));
    }
    return tot;
}
template <int OP, typename R>
__host__ __device__ constexpr int tail_lds_bytes(int nl) {
    const int tot = tail_offset<OP>(nl, nl);
    return tot * (int)sizeof(R) + (nl > 1 ? (1 << (3 * (nl + 1))) * (int)sizeof(double) : 0);
}

// The thread index, opaque to the compiler: the addresses of a phase are formed
// in that phase.  (Formed for all phases ahead of their loops they do not fit
// the 128 registers of a 1024-thread block: 500 bytes per lane of scratch.)
__device__ __forceinline__ int tail_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

template <int LOGN>
__device__ __forceinline__ void tail_cell(int t, int &m, int &j, int &k) {
    m = t & ((1 << (LOGN - 1)) - 1);
    j = (t >> (LOGN - 1)) & ((1 << LOGN) - 1);
    k = t >> (2 * LOGN - 1);
}

// New value of the cell of colour c at packed index t.
template <int OP, int LOGN, typename R>
__device__ __forceinline__ R tail_new(const Mod &M, const LvlT<R> &L, const Coefs &Cf, int c,
                                      int t) {
    int m, j, k;
    tail_cell<LOGN>(t, m, j, k);
    R faces;
    const R K = cell_term<OP, R, R>(M, L, Cf, c, m, j, k, faces, nullptr);
    const R f = (c ? L.f1 : L.f0)[t];
    if constexpr (OP == OP_NEWTON)
        return newton_update<R>(M, (c ? L.u1 : L.u0)[t], faces, K, f, (R)L.h2);
    else
        return (faces - (R)L.h2 * (K + f)) * (R)(1.0 / 6.0);
}

template <int OP, int LOGN, typename R>
__device__ __forceinline__ void tail_sweeps(const Mod &M, const LvlT<R> &L, const Coefs &Cf,
                                            int count) {
    constexpr int HALF = 1 << (3 * LOGN - 1), CNT = (HALF + TAIL_THREADS - 1) / TAIL_THREADS;
#pragma unroll 1
    for (int s = 0; s < count; ++s) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            R nv[CNT];
            const int tid = tail_tid();
#pragma unroll
            for (int q = 0; q < CNT; ++q) {
                const int t = tid + q * TAIL_THREADS;
                if (HALF % TAIL_THREADS == 0 || t < HALF)
                    nv[q] = tail_new<OP, LOGN, R>(M, L, Cf, c, t);
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < CNT; ++q) {
                const int t = tid + q * TAIL_THREADS;
                if (HALF % TAIL_THREADS == 0 || t < HALF) (c ? L.u1 : L.u0)[t] = nv[q];
            }
            __syncthreads();
        }
    }
}

// The sweeps of the 4^3 level (32 cells per colour) on the first wavefront
// alone: a lane per cell, and no workgroup barrier between passes.  A
// wavefront's LDS reads and writes take effect in program order, so every
// read of a pass precedes its writes and follows the previous pass's writes,
// as in tail_sweeps.
template <int OP, typename R>
__device__ __forceinline__ void tail_sweeps_wave(const Mod &M, const LvlT<R> &L, const Coefs &Cf,
                                                 int count) {
    if (threadIdx.x < 32) {
        int t = threadIdx.x;
        if constexpr (OP == OP_ADJ) {
#pragma unroll 1
            for (int s = 0; s < count; ++s) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    t = tail_tid();   // 18 coefficients per pass: no room for kept addresses
                    const R nv = tail_new<OP, 2, R>(M, L, Cf, c, t);
                    __builtin_amdgcn_wave_barrier();
                    (c ? L.u1 : L.u0)[t] = nv;
                    __builtin_amdgcn_wave_barrier();
                }
            }
        } else {
            // A pass waits for the face values that the previous pass wrote;
            // its own colour's cross differences are two passes old and are
            // read ahead, beside the previous pass.
            int m, j, k;
            tail_cell<2>(t, m, j, k);
            const R d[2] = {L.d0[t], L.d1[t]}, f[2] = {L.f0[t], L.f1[t]};
            NbT<R> s[2];
            load_cross(s[0], L.u0, 0, m, j, k, 4, 2, 1);
#pragma unroll 1
            for (int q = 0; q < count; ++q) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    R *u = c ? L.u1 : L.u0;
                    const R *o = c ? L.u0 : L.u1;
                    load_faces(s[c], o, c, m, j, k, 4, 2, 1);
                    load_cross(s[c ^ 1], o, c ^ 1, m, j, k, 4, 2, 1);
                    const R faces = (s[c].xp + s[c].xm) + (s[c].yp + s[c].ym) +
                                    (s[c].zp + s[c].zm);
                    R nv;
                    if constexpr (OP == OP_NEWTON)
                        nv = newton_update<R>(M, u[t], faces,
                                              dgp_sigma_over_alpha<R>(M, L, s[c], d[c]), f[c],
                                              (R)L.h2);
                    else
                        nv = (faces - (R)L.h2 * (model_term<OP, R>(
                                                     M, L, s[c], d[c],
                                                     (unsigned long long *)nullptr) +
                                                 f[c])) *
                             (R)(1.0 / 6.0);
                    __builtin_amdgcn_wave_barrier();
                    u[t] = nv;
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    }
    __syncthreads();
}

// FAS transfer to the next tail level: residual of every cell (double) into
// res, 8-cell means R u and R d, coarse source S = L(R u) - R d, u = R u.
template <int OP, int LOGN, typename R>
__device__ __forceinline__ void tail_restrict(const Mod &M, const LvlT<R> &L, const Coefs &Cf,
                                              const LvlT<R> &Lc, const Coefs &Cc, R *ru0, R *ru1,
                                              double *res) {
    constexpr int HALF = 1 << (3 * LOGN - 1), CNT = (HALF + TAIL_THREADS - 1) / TAIL_THREADS;
    constexpr int LC = LOGN - 1, NC3 = 1 << (3 * LC);
    const double inv_h2 = 1.0 / L.h2;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int tid = tail_tid();
#pragma unroll
        for (int q = 0; q < CNT; ++q) {
            const int t = tid + q * TAIL_THREADS;
            if (HALF % TAIL_THREADS == 0 || t < HALF) {
                int m, j, k;
                tail_cell<LOGN>(t, m, j, k);
                double faces;
                double term = cell_term<OP, double, R>(M, L, Cf, c, m, j, k, faces, nullptr);
                const double u = (double)(c ? L.u1 : L.u0)[t];
                if constexpr (OP == OP_NEWTON)
                    term = newton_term(M, term, (faces - 6.0 * u) * inv_h2);
                res[c * HALF + t] = (faces - 6.0 * u) * inv_h2 - term - (double)(c ? L.f1 : L.f0)[t];
            }
        }
    }
    __syncthreads();
    const int t = tail_tid();
    static_assert(NC3 <= TAIL_THREADS, "one coarse cell per thread");
    R *S0 = const_cast<R *>(Lc.f0), *S1 = const_cast<R *>(Lc.f1);
    if (t < NC3) {
        const int I = t & ((1 << LC) - 1), J = (t >> LC) & ((1 << LC) - 1), K = t >> (2 * LC);
        double sd = 0.0, su = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int a = q & 1, b = (q >> 1) & 1, cc = q >> 2, col = (a + b + cc) & 1;
            const int idx = ((2 * K + cc) << (2 * LOGN - 1)) + ((2 * J + b) << (LOGN - 1)) + I;
            sd += res[col * HALF + idx];
            su += (double)(col ? L.u1 : L.u0)[idx];
        }
        const int cidx = (K << (2 * LC - 1)) + (J << (LC - 1)) + (I >> 1);
        const bool odd = (I + J + K) & 1;
        (odd ? ru1 : ru0)[cidx] = (R)(0.125 * su);
        (odd ? S1 : S0)[cidx] = (R)(0.125 * sd);
    }
    __syncthreads();
    if (t < NC3) {
        LvlT<R> Lr = Lc;
        Lr.u0 = ru0;
        Lr.u1 = ru1;
        constexpr int HC = NC3 / 2;
        auto source = [&](int c, int tt) __attribute__((always_inline)) {
            dev_coarse_source<OP, R>(M, Lr, Cc, S0, S1, Lc.u0, Lc.u1, 0.0, c, (size_t)tt);
        };
        if constexpr (OP == OP_ADJ) {   // the coefficient pointers need a constant colour
            if (t < HC)
                source(0, t);
            else
                source(1, t - HC);
        } else {
            source(t >= HC, t & (HC - 1));
        }
    }
    __syncthreads();
}

// u_fine += P(uc - rc) (see dev_prolong; u: both colours, one after the
// other), from the correction e in natural order.
template <int LOGN, typename R>
__device__ __forceinline__ void tail_prolong(R *u, const R *uc0, const R *uc1, const R *rc0,
                                             const R *rc1, double *e) {
    constexpr int LC = LOGN - 1, NCM = (1 << LC) - 1, HALF = 1 << (3 * LOGN - 1);
    const int t = tail_tid();
    if (t < (1 << (3 * LC))) {
        const int I = t & NCM, J = (t >> LC) & NCM, K = t >> (2 * LC), i = t >> 1;
        e[t] = ((I + J + K) & 1) ? (double)uc1[i] - (double)rc1[i]
                                 : (double)uc0[i] - (double)rc0[i];
    }
    __syncthreads();
    constexpr int CNT = 2 * HALF < TAIL_THREADS ? 1 : 2 * HALF / TAIL_THREADS;
#pragma unroll
    for (int q = 0; q < CNT; ++q) {
        const int tt = t + q * TAIL_THREADS, c = tt >= HALF;
        if (CNT > 1 || tt < 2 * HALF) {
            int m, j, k;
            tail_cell<LOGN>(tt & (HALF - 1), m, j, k);
            const int p = (j + k + c) & 1;   // i = 2m + p, parent I = m
            const int I2 = (m + (p ? 1 : -1)) & NCM;
            const int J = j >> 1, J2 = (J + ((j & 1) ? 1 : -1)) & NCM;
            const int K = k >> 1, K2 = (K + ((k & 1) ? 1 : -1)) & NCM;
            double acc = 0.0;
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                const int a = o & 1, b = (o >> 1) & 1, cc = o >> 2;
                const double w = (a ? 1.0 : 3.0) * (b ? 1.0 : 3.0) * (cc ? 1.0 : 3.0);
                acc += w * e[((((cc ? K2 : K) << LC) + (b ? J2 : J)) << LC) + (a ? I2 : m)];
            }
            u[tt] = (R)((double)u[tt] + acc * (1.0 / 64.0));
        }
    }
    __syncthreads();
}

// Tail level LV of a launch with its fields in LDS.
template <int OP, int NL, int LV, typename R>
struct TailView {
    static constexpr int LOGN = 1 + NL - LV, HALF = 1 << (3 * LOGN - 1);
    LvlT<R> L;
    R *f0, *f1, *d0, *d1, *ru0, *ru1;   // d0: also the first LDS coefficient array
    Coefs cf;
    __device__ __forceinline__ TailView(const TailArgs<R> &A, R *lds) {
        R *p = lds + tail_offset<OP>(NL, LV);
        L = A.lv[LV].L;
        L.n = 1 << LOGN;
        L.logn = LOGN;
        L.lognh = LOGN - 1;
        L.u0 = p;
        L.u1 = p + HALF;
        L.f0 = f0 = p + 2 * HALF;
        L.f1 = f1 = p + 3 * HALF;
        L.d0 = d0 = p + 4 * HALF;
        L.d1 = d1 = p + 5 * HALF;
        ru0 = p + (tail_level_arrays<OP>(LOGN, true)) * HALF;
        ru1 = ru0 + HALF;
        if constexpr (OP == OP_ADJ) {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    cf.c[i][c] = LOGN < 4 ? (const double *)(d0 + (2 * i + c) * HALF)
                                          : A.cf[LV].c[i][c];
            }
        }
    }
    // The level's inputs, through registers: every load of a launch's levels
    // is in flight before the first is waited for.
    static constexpr int NIN = (OP == OP_ADJ ? (LOGN < 4 ? 18 : 0) : 2) + (LV == 0 ? 4 : 0);
    static constexpr int CNT = (HALF + TAIL_THREADS - 1) / TAIL_THREADS;
    struct In {
        R v[NIN > 0 ? NIN * CNT : 1];
    };
    static __device__ __forceinline__ const R *source(const TailArgs<R> &A, int i) {
        const LvlT<R> &G = A.lv[LV].L;
        constexpr int NF = LV == 0 ? 4 : 0;
        if (i < NF)
            return i == 0   ? (A.source ? A.lv[LV].ru0 : G.u0)
                   : i == 1 ? (A.source ? A.lv[LV].ru1 : G.u1)
                   : i == 2 ? G.f0
                            : G.f1;
        if (OP != OP_ADJ) return i == NF ? G.d0 : G.d1;
        return (const R *)A.cf[LV].c[(i - NF) >> 1][(i - NF) & 1];
    }
    __device__ __forceinline__ void fetch(const TailArgs<R> &A, In &in) const {
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            const R *src = source(A, i);
#pragma unroll
            for (int q = 0; q < CNT; ++q) {
                const int t = threadIdx.x + q * TAIL_THREADS;
                if (HALF % TAIL_THREADS == 0 || t < HALF) in.v[i * CNT + q] = src[t];
            }
        }
    }
    __device__ __forceinline__ void store(const In &in) const {
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            // the first level's u and f lead its arrays, the rest starts at d0
            R *dst = L.u0 + (LV == 0 ? i : i + 4) * HALF;
#pragma unroll
            for (int q = 0; q < CNT; ++q) {
                const int t = threadIdx.x + q * TAIL_THREADS;
                if (HALF % TAIL_THREADS == 0 || t < HALF) dst[t] = in.v[i * CNT + q];
            }
        }
    }
};

// One cycle (0 V, 1 F, 2 W) on tail level LV, recursing at compile time.
template <int OP, int NL, int LV, typename R>
__device__ __forceinline__ void tail_cycle(const Mod &M, const TailArgs<R> &A, R *lds, int type) {
    const TailView<OP, NL, LV, R> T(A, lds);
    constexpr int LOGN = 1 + NL - LV;
    if constexpr (LV == NL - 1) {
        tail_sweeps_wave<OP, R>(M, T.L, T.cf, A.nuc);
    } else {
        const TailView<OP, NL, LV + 1, R> Tc(A, lds);
        tail_sweeps<OP, LOGN, R>(M, T.L, T.cf, A.nu1);
        tail_restrict<OP, LOGN, R>(M, T.L, T.cf, Tc.L, Tc.cf, Tc.ru0, Tc.ru1,
                                   reinterpret_cast<double *>(lds + tail_offset<OP>(NL, NL)));
        // F: a coarse F-cycle, then a coarse V-cycle; W: two coarse W-cycles
        const int visits = type == 0 ? 1 : 2;
#pragma unroll 1
        for (int v = 0; v < visits; ++v)
            tail_cycle<OP, NL, LV + 1, R>(M, A, lds, type == 1 && v == 1 ? 0 : type);
        tail_prolong<LOGN, R>(T.L.u0, Tc.L.u0, Tc.L.u1, Tc.ru0, Tc.ru1,
                              reinterpret_cast<double *>(lds + tail_offset<OP>(NL, NL)));
        tail_sweeps<OP, LOGN, R>(M, T.L, T.cf, A.nu2);
    }
}

// The tail levels live in LDS for the whole sub-cycle: their fields are
// copied in, the sub-cycle runs on LDS, and the first level's u goes back.
template <int OP, int NL, typename R>
__global__ __launch_bounds__(TAIL_THREADS) void k_tail(Mod M, TailArgs<R> A) {
    extern __shared__ double lds_raw[];
    R *lds = reinterpret_cast<R *>(lds_raw);
    const TailView<OP, NL, 0, R> T(A, lds);
    {
        const TailView<OP, NL, (NL > 1 ? 1 : 0), R> T1(A, lds);
        const TailView<OP, NL, (NL > 2 ? 2 : 0), R> T2(A, lds);
        typename decltype(T)::In in0;
        typename decltype(T1)::In in1;
        typename decltype(T2)::In in2;
        T.fetch(A, in0);
        if constexpr (NL > 1) T1.fetch(A, in1);
        if constexpr (NL > 2) T2.fetch(A, in2);
        T.store(in0);
        if constexpr (NL > 1) T1.store(in1);
        if constexpr (NL > 2) T2.store(in2);
    }
    __syncthreads();
    if (A.source) {
        const double shift = A.pend.partials ? pending_shift<TAIL_THREADS>(A.pend, true)
                             : A.shift       ? *A.shift
                                             : 0.0;
        constexpr int HALF = decltype(T)::HALF, CNT = decltype(T)::CNT;
        const int tid = tail_tid();
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int q = 0; q < CNT; ++q) {
                const int t = tid + q * TAIL_THREADS;
                if (HALF % TAIL_THREADS == 0 || t < HALF)
                    dev_coarse_source<OP, R>(M, T.L, T.cf, T.f0, T.f1, T.L.u0, T.L.u1, shift, c,
                                             (size_t)t);
            }
        }
        __syncthreads();
    }
    tail_cycle<OP, NL, 0, R>(M, A, lds, A.cycle);
    // u0 and u1 lie one after the other in LDS
    constexpr int half0 = 1 << (3 * (1 + NL) - 1);
    for (int t = threadIdx.x; t < half0; t += TAIL_THREADS) {
        const R a = T.L.u0[t], b = T.L.u1[t];
        A.lv[0].L.u0[t] = a;
        A.lv[0].L.u1[t] = b;
    }
}

}  // namespace mgk
