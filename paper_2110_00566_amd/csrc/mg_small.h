// Fused kernels of the levels between the single-workgroup tail and the
// LDS-tiled levels (32^3 and 64^3, and finest levels of 8^3 and 16^3): a sweep
// with the residual + restriction that follows it (way down), and the
// prolongation with the sweep that follows it (way up).
//
// These levels hold a few MB at most; a launch of one colour pass there takes
// 4 us, nearly all of it launch and load latency.  A block therefore takes a
// cube of 8^3 cells and recomputes what it needs of the cells around it: on
// the way down it stages the field with a halo of 3, updates colour 0 on a
// halo of 2 and colour 1 on a halo of 1 and evaluates the residual of its own
// cells; on the way up it stages the prolonged field with a halo of 2.  The
// recomputed values are those of the neighbouring blocks to the bit.  One
// launch instead of three each way; 512 threads, one cell per thread and
// phase in most phases.
#pragma once
#include "mg_kernels.h"

namespace mgk {

constexpr int SMT = 512;   // threads
constexpr int SMC = 8;     // cells per side of a block's cube

// A cube of LDS values of W cells per side around the block's cells (halo H).
template <typename R, int H>
struct SmallCube {
    static constexpr int W = SMC + 2 * H, CELLS = W * W * W;
    static __device__ __forceinline__ int at(int x, int y, int z) { return (z * W + y) * W + x; }
    template <typename T>
    static __device__ __forceinline__ NbT<T> nb(const R *u, int o) {
        constexpr int Y = W, Z = W * W;
        NbT<T> s;
        s.xp = (T)u[o + 1];
        s.xm = (T)u[o - 1];
        s.yp = (T)u[o + Y];
        s.ym = (T)u[o - Y];
        s.zp = (T)u[o + Z];
        s.zm = (T)u[o - Z];
        s.nxy = ((T)u[o + Y + 1] + (T)u[o - Y - 1]) - ((T)u[o - Y + 1] + (T)u[o + Y - 1]);
        s.nxz = ((T)u[o + Z + 1] + (T)u[o - Z - 1]) - ((T)u[o - Z + 1] + (T)u[o + Z - 1]);
        s.nyz = ((T)u[o + Z + Y] + (T)u[o - Z - Y]) - ((T)u[o - Z + Y] + (T)u[o + Z - Y]);
        return s;
    }
};

// The block's corner and the level's index arithmetic.
struct SmallTile {
    int i0, j0, k0, nm, logn;
    __device__ __forceinline__ SmallTile(size_t blk, int n, int logn_) : nm(n - 1), logn(logn_) {
        const int lt = logn - 3, m = (1 << lt) - 1;
        i0 = ((int)blk & m) * SMC;
        j0 = ((int)(blk >> lt) & m) * SMC;
        k0 = (int)(blk >> (2 * lt)) * SMC;
    }
    // packed index and colour of the cell at cube offsets x, y, z (from the corner)
    __device__ __forceinline__ int packed(int x, int y, int z, int &c) const {
        const int i = (i0 + x) & nm, j = (j0 + y) & nm, k = (k0 + z) & nm;
        c = (i + j + k) & 1;
        return (k << (2 * logn - 1)) + (j << (logn - 1)) + (i >> 1);
    }
};

// Colour pass of colour C on the cells up to HALO cells outside the block, in
// the staged cube u: every new value is formed before the first is stored.
// Own cells are written to out.
template <int OP, typename R, int H, int C, int HALO>
__device__ __forceinline__ void small_pass(const Mod &M, const LvlT<R> &L, const SmallTile &B,
                                           R *u, R fs, R *out, unsigned long long *clamp) {
    using Q = SmallCube<R, H>;
    constexpr int S = SMC + 2 * HALO, HR = S / 2, N = HR * S * S;
    constexpr int CNT = (N + SMT - 1) / SMT;
    R nv[CNT];
    int off[CNT];
#pragma unroll
    for (int r = 0; r < CNT; ++r) {
        const int t = threadIdx.x + r * SMT;
        off[r] = -1;
        if (t < N) {
            const int y = (t / HR) % S - HALO, z = t / (HR * S) - HALO;
            const int x = 2 * (t % HR) - HALO + ((C + HALO + y + z) & 1);
            const int o = Q::at(x + H, y + H, z + H);
            int c;
            const int idx = B.packed(x, y, z, c);
            const bool own = HALO == 0 || ((unsigned)x < SMC && (unsigned)y < SMC && (unsigned)z < SMC);
            const NbT<R> s = Q::template nb<R>(u, o);
            const R faces = (s.xp + s.xm) + (s.yp + s.ym) + (s.zp + s.zm);
            const R delta = (C ? L.d1 : L.d0)[idx];
            const R *fa = C ? L.f1 : L.f0;
            const R f = (fa ? fa[idx] : (R)0) + fs;
            if constexpr (OP == OP_NEWTON)
                nv[r] = newton_update<R>(M, u[o], faces, dgp_sigma_over_alpha<R>(M, L, s, delta), f,
                                         (R)L.h2);
            else
                nv[r] = (faces - (R)L.h2 * (model_term<OP, R>(M, L, s, delta, own ? clamp : nullptr) +
                                            f)) *
                        (R)(1.0 / 6.0);
            off[r] = o;
            if (own) out[idx] = nv[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < CNT; ++r)
        if (off[r] >= 0) u[off[r]] = nv[r];
    __syncthreads();
}

// Sweep, then residual (double) and restriction of the swept field: u -> out0,
// out1; R u and R d to the coarse level; REDUCE: block sums of d and d^2.
template <int OP, bool REDUCE, typename R>
__global__ __launch_bounds__(SMT) void k_small_down(Mod M, LvlT<R> L, R *out0, R *out1,
                                                    const double *fptr, R *ru0, R *ru1, R *rd0,
                                                    R *rd1, double *partials,
                                                    unsigned long long *clamp) {
    constexpr int H = 3;
    using Q = SmallCube<R, H>;
    __shared__ R u[Q::CELLS];
    __shared__ double sd[SMC * SMC * SMC];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const SmallTile B(blk, L.n, L.logn);
    const R fs = (R)(fptr ? *fptr : 0.0);
#pragma unroll
    for (int r = 0; r < (Q::CELLS + SMT - 1) / SMT; ++r) {
        const int t = threadIdx.x + r * SMT;
        if (t < Q::CELLS) {
            int c;
            const int idx = B.packed(t % Q::W - H, (t / Q::W) % Q::W - H, t / (Q::W * Q::W) - H, c);
            u[t] = (c ? L.u1 : L.u0)[idx];
        }
    }
    __syncthreads();
    small_pass<OP, R, H, 0, 2>(M, L, B, u, fs, out0, clamp);
    small_pass<OP, R, H, 1, 1>(M, L, B, u, fs, out1, clamp);
    const int t = threadIdx.x, x = t & 7, y = (t >> 3) & 7, z = t >> 6;
    const int o = Q::at(x + H, y + H, z + H);
    int c;
    const int idx = B.packed(x, y, z, c);
    const double inv_h2 = 1.0 / L.h2;
    const Nb s = Q::template nb<double>(u, o);
    const double faces = (s.xp + s.xm) + (s.yp + s.ym) + (s.zp + s.zm), uv = (double)u[o];
    const double delta = (double)(c ? L.d1 : L.d0)[idx];
    double term;
    if constexpr (OP == OP_NEWTON)
        term = newton_term(M, dgp_sigma_over_alpha<double>(M, L, s, delta),
                           (faces - 6.0 * uv) * inv_h2);
    else
        term = model_term<OP, double>(M, L, s, delta, clamp);
    const double d = (faces - 6.0 * uv) * inv_h2 - term - rhs_at<double, R>(L, c, idx, fptr, 1.0);
    sd[t] = d;
    __syncthreads();
    if (t < 64) {
        const int X = t & 3, Y = (t >> 2) & 3, Z = t >> 4;
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int fx = 2 * X + (q & 1), fy = 2 * Y + ((q >> 1) & 1), fz = 2 * Z + (q >> 2);
            a += sd[(fz * SMC + fy) * SMC + fx];
            b += (double)u[Q::at(fx + H, fy + H, fz + H)];
        }
        const int I = (B.i0 >> 1) + X, J = (B.j0 >> 1) + Y, K = (B.k0 >> 1) + Z;
        const int lnc = L.logn - 1, cidx = (K << (2 * lnc - 1)) + (J << (lnc - 1)) + (I >> 1);
        const bool odd = (I + J + K) & 1;
        (odd ? ru1 : ru0)[cidx] = (R)(0.125 * b);
        (odd ? rd1 : rd0)[cidx] = (R)(0.125 * a);
    }
    if (REDUCE) block_sum2<SMT>(d, d * d, partials, blk);
}

// Prolongation of the coarse correction (see dev_prolong) and one sweep of
// the corrected field: u -> out0, out1.
template <int OP, typename R>
__global__ __launch_bounds__(SMT) void k_small_up(Mod M, LvlT<R> L, R *out0, R *out1, const R *uc0,
                                                  const R *uc1, const R *rc0, const R *rc1,
                                                  const double *fptr, unsigned long long *clamp) {
    constexpr int H = 2;
    using Q = SmallCube<R, H>;
    constexpr int CW = SMC / 2 + 4;   // coarse cells -2 .. SMC/2 + 1
    static_assert(CW * CW * CW == SMT, "one coarse value per thread");
    __shared__ R u[Q::CELLS];
    __shared__ double e[CW * CW * CW];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const SmallTile B(blk, L.n, L.logn);
    const R fs = (R)(fptr ? *fptr : 0.0);
    constexpr int CNT = (Q::CELLS + SMT - 1) / SMT;
    R v[CNT];
#pragma unroll
    for (int r = 0; r < CNT; ++r) {
        const int t = threadIdx.x + r * SMT;
        if (t < Q::CELLS) {
            int c;
            const int idx = B.packed(t % Q::W - H, (t / Q::W) % Q::W - H, t / (Q::W * Q::W) - H, c);
            v[r] = (c ? L.u1 : L.u0)[idx];
        }
    }
    {
        const int t = threadIdx.x, lnc = L.logn - 1, ncm = (1 << lnc) - 1;
        const int I = ((B.i0 >> 1) - 2 + t % CW) & ncm, J = ((B.j0 >> 1) - 2 + (t / CW) % CW) & ncm,
                  K = ((B.k0 >> 1) - 2 + t / (CW * CW)) & ncm;
        const int idx = (K << (2 * lnc - 1)) + (J << (lnc - 1)) + (I >> 1);
        e[t] = ((I + J + K) & 1) ? (double)uc1[idx] - (double)rc1[idx]
                                 : (double)uc0[idx] - (double)rc0[idx];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < CNT; ++r) {
        const int t = threadIdx.x + r * SMT;
        if (t < Q::CELLS) {
            // cube coordinates start at an even cell: cell x has the coarse
            // column x / 2 + 1 of e and its neighbour on the cell's side
            const int x = t % Q::W, y = (t / Q::W) % Q::W, z = t / (Q::W * Q::W);
            const int X = (x >> 1) + 1, Y = (y >> 1) + 1, Z = (z >> 1) + 1;
            const int X2 = X + ((x & 1) ? 1 : -1), Y2 = Y + ((y & 1) ? 1 : -1),
                      Z2 = Z + ((z & 1) ? 1 : -1);
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int a = q & 1, b = (q >> 1) & 1, cc = q >> 2;
                const double w = (a ? 1.0 : 3.0) * (b ? 1.0 : 3.0) * (cc ? 1.0 : 3.0);
                acc += w * e[((cc ? Z2 : Z) * CW + (b ? Y2 : Y)) * CW + (a ? X2 : X)];
            }
            u[t] = (R)((double)v[r] + acc * (1.0 / 64.0));
        }
    }
    __syncthreads();
    small_pass<OP, R, H, 0, 1>(M, L, B, u, fs, out0, clamp);
    small_pass<OP, R, H, 1, 0>(M, L, B, u, fs, out1, clamp);
}

}  // namespace mgk
