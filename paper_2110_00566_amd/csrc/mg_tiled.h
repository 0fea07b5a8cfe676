// LDS-tiled versions of the kernels that touch every finest-level cell
// (colour pass, prolongation, coarse source), for levels with at least 128
// cells per side.  The smoothing sweeps of the solves are in mg_sweep.h, the
// residual + restriction in mg_resid.h.
//
// A block owns a tile of TX = 64 packed x-columns (one wave wide) and TY = 8
// rows and marches through a z-chunk.  The planes it needs are staged once in
// LDS (tile plus a one-cell halo, periodic wrap) in a small ring, and the next
// plane is prefetched into registers while the current one is computed, so
// each global value is read about once per block instead of once per
// neighbouring thread.  Consecutive logical blocks are neighbours in y; the XCD
// remapping keeps a whole z-slab on one XCD so y-halos are L2 hits.
#pragma once
#include "mg_kernels.h"

namespace mgk {

constexpr int TX = 64, TY = 8, TXH = TX + 2, TYH = TY + 2;
constexpr int TPLANE = TXH * TYH;   // 660 values per staged plane
constexpr int TLOADS = (TPLANE + TPB - 1) / TPB;

struct TileGeom {
    int ntx, nty, kz;   // tiles in x, tiles in y, planes per block
};

// Byte offsets for the marching kernels: a thread's positions inside a z-plane
// are fixed for the whole march, so their offsets are computed once (32 bit)
// and each plane adds one uniform (scalar) base.
template <typename R>
__device__ __forceinline__ unsigned stage_off(int e, int j0, int m0, int logn, int lognh) {
    const int r = e / TXH, q = e - r * TXH;
    const unsigned j = (unsigned)(j0 - 1 + r) & ((1u << logn) - 1);
    const unsigned m = (unsigned)(m0 - 1 + q) & ((1u << lognh) - 1);
    return ((j << lognh) + m) * (unsigned)sizeof(R);
}
template <typename R>
__device__ __forceinline__ unsigned cell_off(int j, int m, int lognh) {
    return (((unsigned)j << lognh) + (unsigned)m) * (unsigned)sizeof(R);
}
template <typename R>
__device__ __forceinline__ size_t plane_off(int k, int logn, int lognh) {
    return ((size_t)((unsigned)k & ((1u << logn) - 1)) << (logn + lognh)) * sizeof(R);
}
template <typename R>
__device__ __forceinline__ R ld(const R *base, size_t plane, unsigned off) {
    return *reinterpret_cast<const R *>(reinterpret_cast<const char *>(base) + plane + off);
}
// A cell's own delta and f are read once per launch: non-temporal loads
// keep them from displacing the staged planes' halo rows in the caches.
template <typename R>
__device__ __forceinline__ R ld_once(const R *base, size_t plane, unsigned off) {
    return __builtin_nontemporal_load(
        reinterpret_cast<const R *>(reinterpret_cast<const char *>(base) + plane + off));
}
template <typename R>
__device__ __forceinline__ R *ptr(R *base, size_t plane, unsigned off) {
    return reinterpret_cast<R *>(reinterpret_cast<char *>(base) + plane + off);
}

// Staging of one z-plane (tile plus halo: TYH rows of TXH values) of two
// arrays of a level into LDS.  A staged plane starts one value into its LDS
// slot of TSLOT values.  FP64: each row's 64 interior values are read as 32
// 16-byte vectors (rows start on 512-byte boundaries of the level's arrays)
// and land on 16-byte LDS addresses (slot base + 8 + 528 r + 16 i); the two
// halo columns are single values.  320 vectors + 20 halo values: every thread
// takes one vector, then threads 0..63 one more and threads 64..83 a halo
// value.  FP32: one value per load.
constexpr int TSLOT = TPLANE + 2;

template <typename R>
struct Stage2 {
    unsigned soff[TLOADS];
    R ra[TLOADS], rb[TLOADS];
    __device__ __forceinline__ void init(int tid, int j0, int m0, int logn, int lognh) {
#pragma unroll
        for (int q = 0; q < TLOADS; ++q) soff[q] = stage_off<R>(tid + q * TPB, j0, m0, logn, lognh);
    }
    __device__ __forceinline__ void fetch(const R *A, const R *B, size_t pl, int tid) {
#pragma unroll
        for (int q = 0; q < TLOADS; ++q) {
            if (tid + q * TPB < TPLANE) {
                ra[q] = ld(A, pl, soff[q]);
                rb[q] = ld(B, pl, soff[q]);
            }
        }
    }
    // sa, sb: the slots' plane views (slot base + 1)
    __device__ __forceinline__ void store(R *sa, R *sb, int tid) const {
#pragma unroll
        for (int q = 0; q < TLOADS; ++q) {
            const int e = tid + q * TPB;
            if (e < TPLANE) {
                sa[e] = ra[q];
                sb[e] = rb[q];
            }
        }
    }
};

// FP32: 16 vectors of 4 values per row (160 per plane) and 20 halo values,
// one per thread; a vector lands in LDS as two 8-byte halves (a staged row
// starts 8 bytes off a 16-byte boundary in every other slot and row).
template <>
struct Stage2<float> {
    static constexpr int NV = TYH * (TX / 4);   // 160 vectors per plane
    static_assert(NV + 2 * TYH <= TPB, "staging split");
    unsigned g;   // byte offset inside a plane
    int l;        // value offset inside a plane view
    float4 a, b;
    __device__ __forceinline__ void init(int tid, int j0, int m0, int logn, int lognh) {
        const unsigned jm = (1u << logn) - 1, mm = (1u << lognh) - 1;
        if (tid < NV) {
            const int r = tid >> 4, i = tid & 15;
            g = ((((unsigned)(j0 - 1 + r) & jm) << lognh) + (unsigned)(m0 + 4 * i)) * 4u;
            l = r * TXH + 1 + 4 * i;
        } else {
            const int h = tid < NV + 2 * TYH ? tid - NV : 0, r = h >> 1, side = h & 1;
            const unsigned m = (unsigned)(side ? m0 + TX : m0 - 1) & mm;
            g = ((((unsigned)(j0 - 1 + r) & jm) << lognh) + m) * 4u;
            l = r * TXH + (side ? TXH - 1 : 0);
        }
    }
    __device__ __forceinline__ void fetch(const float *A, const float *B, size_t pl, int tid) {
        const char *pa = reinterpret_cast<const char *>(A) + pl + g;
        const char *pb = reinterpret_cast<const char *>(B) + pl + g;
        if (tid < NV) {
            a = *reinterpret_cast<const float4 *>(pa);
            b = *reinterpret_cast<const float4 *>(pb);
        } else if (tid < NV + 2 * TYH) {
            a.x = *reinterpret_cast<const float *>(pa);
            b.x = *reinterpret_cast<const float *>(pb);
        }
    }
    __device__ __forceinline__ void store(float *sa, float *sb, int tid) const {
        if (tid < NV) {
            *reinterpret_cast<float2 *>(sa + l) = make_float2(a.x, a.y);
            *reinterpret_cast<float2 *>(sa + l + 2) = make_float2(a.z, a.w);
            *reinterpret_cast<float2 *>(sb + l) = make_float2(b.x, b.y);
            *reinterpret_cast<float2 *>(sb + l + 2) = make_float2(b.z, b.w);
        } else if (tid < NV + 2 * TYH) {
            sa[l] = a.x;
            sb[l] = b.x;
        }
    }
};

template <>
struct Stage2<double> {
    static constexpr int NV = TYH * (TX / 2);   // 320 vectors per plane
    static_assert(TPB == 256 && NV - TPB == 64 && 2 * TYH <= TPB - 64, "staging split");
    unsigned g0, g1;   // byte offsets inside a plane
    int l0, l1;        // value offsets inside a plane view
    double2 a0, a1, b0, b1;
    double ha, hb;
    __device__ __forceinline__ void init(int tid, int j0, int m0, int logn, int lognh) {
        const unsigned jm = (1u << logn) - 1, mm = (1u << lognh) - 1;
        {
            const int r = tid >> 5, i = tid & 31;
            g0 = ((((unsigned)(j0 - 1 + r) & jm) << lognh) + (unsigned)(m0 + 2 * i)) * 8u;
            l0 = r * TXH + 1 + 2 * i;
        }
        if (tid < 64) {
            const int r = 8 + (tid >> 5), i = tid & 31;
            g1 = ((((unsigned)(j0 - 1 + r) & jm) << lognh) + (unsigned)(m0 + 2 * i)) * 8u;
            l1 = r * TXH + 1 + 2 * i;
        } else {
            const int h = tid < 64 + 2 * TYH ? tid - 64 : 0, r = h >> 1, side = h & 1;
            const unsigned m = (unsigned)(side ? m0 + TX : m0 - 1) & mm;
            g1 = ((((unsigned)(j0 - 1 + r) & jm) << lognh) + m) * 8u;
            l1 = r * TXH + (side ? TXH - 1 : 0);
        }
    }
    __device__ __forceinline__ void fetch(const double *A, const double *B, size_t pl, int tid) {
        const char *a = reinterpret_cast<const char *>(A) + pl;
        const char *b = reinterpret_cast<const char *>(B) + pl;
        a0 = *reinterpret_cast<const double2 *>(a + g0);
        b0 = *reinterpret_cast<const double2 *>(b + g0);
        if (tid < 64) {
            a1 = *reinterpret_cast<const double2 *>(a + g1);
            b1 = *reinterpret_cast<const double2 *>(b + g1);
        } else if (tid < 64 + 2 * TYH) {
            ha = *reinterpret_cast<const double *>(a + g1);
            hb = *reinterpret_cast<const double *>(b + g1);
        }
    }
    __device__ __forceinline__ void store(double *sa, double *sb, int tid) const {
        *reinterpret_cast<double2 *>(sa + l0) = a0;
        *reinterpret_cast<double2 *>(sb + l0) = b0;
        if (tid < 64) {
            *reinterpret_cast<double2 *>(sa + l1) = a1;
            *reinterpret_cast<double2 *>(sb + l1) = b1;
        } else if (tid < 64 + 2 * TYH) {
            sa[l1] = ha;
            sb[l1] = hb;
        }
    }
};

// Stencil of the cell at local (r, q) (halo-shifted tile coordinates) with
// packed-x parity p, from staged planes: B = opposite colour at plane k,
// A = own colour at k-1 / k / k+1, Bz = opposite colour at k-1 / k+1.
template <typename T, typename R>
__device__ __forceinline__ NbT<T> lds_nb(const R *Am, const R *A0, const R *Ap, const R *B0,
                                         const R *Bm, const R *Bp, int r, int q, int p) {
    const int qp = q + p, qm = q + p - 1;
    const int o = r * TXH, op = (r + 1) * TXH, om = (r - 1) * TXH;
    NbT<T> s;
    s.xp = (T)B0[o + qp];
    s.xm = (T)B0[o + qm];
    s.yp = (T)B0[op + q];
    s.ym = (T)B0[om + q];
    s.zp = (T)Bp[o + q];
    s.zm = (T)Bm[o + q];
    s.nxy = ((T)A0[op + qp] + (T)A0[om + qm]) - ((T)A0[om + qp] + (T)A0[op + qm]);
    s.nxz = ((T)Ap[o + qp] + (T)Am[o + qm]) - ((T)Am[o + qp] + (T)Ap[o + qm]);
    s.nyz = ((T)Ap[op + q] + (T)Am[om + q]) - ((T)Am[op + q] + (T)Ap[om + q]);
    return s;
}

// Non-Laplacian term of the tiled kernels at a cell with face sum faces and
// centre value u.  OP_NEWTON (the Newton-GS comparator) works on the
// quadratic form: Sigma/alpha - 2 D^2/(3 alpha), D = (faces - 6u)/h^2.
template <int OP, typename T, typename L_, typename S_, typename Clamp>
__device__ __forceinline__ T tiled_term(const Mod &M, const L_ &L, const S_ &s, T delta, T faces,
                                        T u, Clamp *clamp) {
    if constexpr (OP == OP_NEWTON)
        return newton_term<T>(M, dgp_sigma_over_alpha<T>(M, L, s, delta),
                              (faces - (T)6 * u) / (T)L.h2);
    else
        return model_term<OP, T>(M, L, s, delta, clamp);
}

// New value of a cell in a colour pass: the closed-form update, or for
// OP_NEWTON the Newton-Gauss-Seidel step on the quadratic form.
template <int OP, typename R, typename L_, typename S_, typename Clamp>
__device__ __forceinline__ R tiled_update(const Mod &M, const L_ &L, const S_ &s, R delta,
                                          R faces, R u, R f, Clamp *clamp) {
    if constexpr (OP == OP_NEWTON) {
        return newton_update<R>(M, u, faces, dgp_sigma_over_alpha<R>(M, L, s, delta), f,
                                (R)L.h2);
    } else {
        const R K = model_term<OP, R>(M, L, s, delta, clamp);
        return (faces - (R)L.h2 * (K + f)) * (R)(1.0 / 6.0);
    }
}

// One colour pass (see k_pass) on an LDS-staged tile.
template <int OP>
__global__ __launch_bounds__(TPB) void k_pass_tiled(Mod M, Lvl L, int c, double *__restrict__ out,
                                                    TileGeom G) {
    __shared__ __align__(16) double sA[3][TSLOT], sB[3][TSLOT];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = (int)(blk % G.ntx);
    const int by = (int)((blk / G.ntx) % G.nty);
    const int bz = (int)(blk / ((size_t)G.ntx * G.nty));
    const int m0 = bx * TX, j0 = by * TY, k0 = bz * G.kz;
    const double *A = c ? L.u1 : L.u0;
    const double *B = c ? L.u0 : L.u1;
    const double *D = c ? L.d1 : L.d0;
    const double *F = c ? L.f1 : L.f0;
    const int tid = threadIdx.x, tx = tid & 63, ty = tid >> 6;
    unsigned coff[2];
    Stage2<double> S;
    S.init(tid, j0, m0, L.logn, L.lognh);
#pragma unroll
    for (int h = 0; h < 2; ++h) coff[h] = cell_off<double>(j0 + ty + 4 * h, m0 + tx, L.lognh);
    auto fetch = [&](int k) { S.fetch(A, B, plane_off<double>(k, L.logn, L.lognh), tid); };
    auto store = [&](int slot) { S.store(sA[slot] + 1, sB[slot] + 1, tid); };
    // own cells' delta and f, one plane ahead
    double dn[2], fn[2];
    auto fetch_cells = [&](int k) {
        const size_t pl = plane_off<double>(k, L.logn, L.lognh);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            dn[h] = ld_once(D, pl, coff[h]);
            fn[h] = ld_once(F, pl, coff[h]);
        }
    };
    // slot of plane k: (k - k0 + 1) mod 3
    fetch(k0 - 1);
    store(0);
    fetch(k0);
    store(1);
    fetch(k0 + 1);
    fetch_cells(k0);
    for (int k = k0; k < k0 + G.kz; ++k) {
        const int sm = (k - k0) % 3, s0 = (k - k0 + 1) % 3, sp = (k - k0 + 2) % 3;
        store(sp);
        const double d0 = dn[0], d1 = dn[1], f0 = fn[0], f1 = fn[1];
        __syncthreads();
        if (k + 2 <= k0 + G.kz) fetch(k + 2);
        if (k + 1 < k0 + G.kz) fetch_cells(k + 1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = ty + 4 * h;
            const int j = j0 + row;
            const int p = (j + k + c) & 1;
            const Nb s = lds_nb<double, double>(sA[sm] + 1, sA[s0] + 1, sA[sp] + 1, sB[s0] + 1,
                                                sB[sm] + 1, sB[sp] + 1, row + 1, tx + 1, p);
            const double faces = (s.xp + s.xm) + (s.yp + s.ym) + (s.zp + s.zm);
            unsigned neg = 0;
            const double nv =
                tiled_update<OP, double>(M, L, s, h ? d1 : d0, faces,
                                         sA[s0][1 + (row + 1) * TXH + tx + 1], h ? f1 : f0, &neg);
            // streamed: the next reader is a later launch
            __builtin_nontemporal_store(nv, ptr(out, plane_off<double>(k, L.logn, L.lognh),
                                                coff[h]));
        }
        __syncthreads();
    }
}

// u_fine += P(uc - rc) (see k_prolong) with the coarse difference staged in
// LDS: 66 coarse columns x 6 coarse rows, ring of 3 coarse planes.  REDUCE:
// block sums of the corrected colour-0 and colour-1 values into partials.
// RC: storage type of the coarse level (the defect-correction cycles
// prolong an FP64 coarse correction into an FP32 finest level).
template <typename R, bool REDUCE = false, typename RC = R>
__global__ __launch_bounds__(TPB) void k_prolong_tiled(R *f0, R *f1, int logn, const RC *uc0,
                                                       const RC *uc1, const RC *rc0, const RC *rc1,
                                                       TileGeom G, double *partials = nullptr) {
    constexpr int CR = TY / 2 + 2;   // coarse rows staged
    constexpr int CPL = TXH * CR;    // 396 values per coarse plane
    __shared__ double sE[3][CPL];
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = (int)(blk % G.ntx);
    const int by = (int)((blk / G.ntx) % G.nty);
    const int bz = (int)(blk / ((size_t)G.ntx * G.nty));
    const int m0 = bx * TX, j0 = by * TY, K0 = bz * G.kz;   // kz counts coarse planes
    const int lnc = logn - 1, ncm1 = (1 << lnc) - 1;
    const int lognh = logn - 1;
    const int tid = threadIdx.x;
    double re[2];
    auto fetch = [&](int K) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + q * TPB;
            if (e < CPL) {
                const int r = e / TXH, cI = e - r * TXH;
                const int I = (m0 - 1 + cI) & ncm1;
                const int J = ((j0 >> 1) - 1 + r) & ncm1;
                const int Kw = K & ncm1;
                const size_t idx = ((size_t)Kw << (2 * lnc - 1)) + ((size_t)J << (lnc - 1)) + (I >> 1);
                re[q] = ((I + J + Kw) & 1) ? ((double)uc1[idx] - (double)rc1[idx])
                                           : ((double)uc0[idx] - (double)rc0[idx]);
            }
        }
    };
    auto store = [&](int slot) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + q * TPB;
            if (e < CPL) sE[slot][e] = re[q];
        }
    };
    // slot of coarse plane K: (K - K0 + 1) mod 3
    fetch(K0 - 1);
    store(0);
    fetch(K0);
    store(1);
    fetch(K0 + 1);
    double bsum[2] = {0.0, 0.0};
    for (int K = K0; K < K0 + G.kz; ++K) {
        store((K - K0 + 2) % 3);
        __syncthreads();
        if (K + 2 <= K0 + G.kz) fetch(K + 2);
        // 2 fine planes x 8 rows x 64 columns x 2 colours = 2048 cells, 8 per thread
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const int cell = tid + h * TPB;
            const int tx = cell & 63, row = (cell >> 6) & 7, c = (cell >> 9) & 1, kk = cell >> 10;
            const int k = 2 * K + kk, j = j0 + row, m = m0 + tx;
            const int p = (j + k + c) & 1;
            const int di = p ? 1 : -1, dj = (j & 1) ? 1 : -1, dk = kk ? 1 : -1;
            const int lc = tx + 1, lr = (j >> 1) - (j0 >> 1) + 1;
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int a = q & 1, b = (q >> 1) & 1, cc = q >> 2;
                const int slot = (K + cc * dk - K0 + 1 + 3) % 3;
                const double w = (a ? 1.0 : 3.0) * (b ? 1.0 : 3.0) * (cc ? 1.0 : 3.0);
                acc += w * sE[slot][(lr + b * dj) * TXH + lc + a * di];
            }
            const size_t idx = prow(j, k, logn, lognh) + m;
            R *f = c ? f1 : f0;
            const R nv = (R)((double)f[idx] + acc * (1.0 / 64.0));
            f[idx] = nv;
            if (REDUCE) bsum[c] += (double)nv;
        }
        __syncthreads();
    }
    if (REDUCE) block_sum2(bsum[0], bsum[1], partials, blk);
}

// FAS source on a coarse level (see k_coarse_source) on an LDS-staged tile:
// S = L(R u) - (R d - shift) at both colours, written over R d, and u = R u.
template <int OP, typename R>
__global__ __launch_bounds__(TPB) void k_coarse_source_tiled(Mod M, LvlT<R> Lc, R *s0, R *s1,
                                                             R *u0, R *u1, const double *shift,
                                                             TileGeom G) {
    __shared__ __align__(16) R sA[3][TSLOT], sB[3][TSLOT];   // colour 0 / colour 1 of R u
    const size_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = (int)(blk % G.ntx);
    const int by = (int)((blk / G.ntx) % G.nty);
    const int bz = (int)(blk / ((size_t)G.ntx * G.nty));
    const int m0 = bx * TX, j0 = by * TY, k0 = bz * G.kz;
    const int tid = threadIdx.x, tx = tid & 63, ty = tid >> 6;
    const double sh = shift ? *shift : 0.0;
    unsigned coff[2];
    Stage2<R> S2;
    S2.init(tid, j0, m0, Lc.logn, Lc.lognh);
#pragma unroll
    for (int h = 0; h < 2; ++h) coff[h] = cell_off<R>(j0 + ty + 4 * h, m0 + tx, Lc.lognh);
    auto fetch = [&](int k) { S2.fetch(Lc.u0, Lc.u1, plane_off<R>(k, Lc.logn, Lc.lognh), tid); };
    auto store = [&](int slot) { S2.store(sA[slot] + 1, sB[slot] + 1, tid); };
    fetch(k0 - 1);
    store(0);
    fetch(k0);
    store(1);
    fetch(k0 + 1);
    for (int k = k0; k < k0 + G.kz; ++k) {
        const int sm = (k - k0) % 3, sz = (k - k0 + 1) % 3, sp = (k - k0 + 2) % 3;
        store(sp);
        __syncthreads();
        if (k + 2 <= k0 + G.kz) fetch(k + 2);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int row = ty + 4 * (h & 1), c = h >> 1;
            const int j = j0 + row;
            const int p = (j + k + c) & 1;
            const R *Am = (c ? sB[sm] : sA[sm]) + 1;
            const R *A0 = (c ? sB[sz] : sA[sz]) + 1;
            const R *Ap = (c ? sB[sp] : sA[sp]) + 1;
            const R *Bm = (c ? sA[sm] : sB[sm]) + 1;
            const R *B0 = (c ? sA[sz] : sB[sz]) + 1;
            const R *Bp = (c ? sA[sp] : sB[sp]) + 1;
            const Nb s = lds_nb<double, R>(Am, A0, Ap, B0, Bm, Bp, row + 1, tx + 1, p);
            const size_t pl = plane_off<R>(k, Lc.logn, Lc.lognh);
            const unsigned o = coff[h & 1];
            const R ru = A0[(row + 1) * TXH + tx + 1];
            const double faces = (s.xp + s.xm) + (s.yp + s.ym) + (s.zp + s.zm);
            const double delta = (double)ld_once(c ? Lc.d1 : Lc.d0, pl, o);
            R *S = ptr(c ? s1 : s0, pl, o);
            const double rd = (double)ld_once(c ? s1 : s0, pl, o) - sh;
            *S = (R)((faces - 6.0 * (double)ru) / Lc.h2
                     - tiled_term<OP, double>(M, Lc, s, delta, faces, (double)ru,
                                                (unsigned long long *)nullptr) - rd);
            *ptr(c ? u1 : u0, pl, o) = ru;
        }
        __syncthreads();
    }
}

}  // namespace mgk
