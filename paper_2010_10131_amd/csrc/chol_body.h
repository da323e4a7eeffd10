// Small FP64 Cholesky factorization + in-place triangular inverse for one
// workgroup (used by the Cholesky-QR of the ALS branch and of the subspace
// iteration eigensolver, and by the batched eigensolver).
#pragma once
#include "common.h"
#include <type_traits>

namespace sth {

// One workgroup of NTH threads (a multiple of 64, at least 256), n <= 128,
// everything in LDS (dynamic LDS of chol_lds_bytes(n)).
//
// G (n x n, symmetric, ldg) + shift_rel * trace(G) / n * I = L L^T.  The
// matrix is padded with an identity block to np = 16 * ceil(n / 16), so that
// every block is a full 16 x 16 tile (the padded factor is diag(L, I)).
// Right-looking on the augmented matrix [A | I] in 16-column panels, so that
// row block K of L^{-1} is final with panel K.  Per panel:
//   * diagonal block: one wave factors it and inverts it in one stream of
//     instructions.  Row l of the block is in lane l of the even 16-lane rows,
//     column l of D^{-1} in lane l of the odd ones: both take the step
//     a_c -= L(c, J) a_J, with column J of L as an FP64 DPP operand;
//   * panel: P(B) = A(B, K) D^{-T} below it (kept in its own buffer) and
//     L^{-1}(K, J) = D^{-1} W(K, J) left of it, nb - 1 products of 16 x 16 tiles
//     on the FP64 matrix cores;
//   * trailing update A(B, C) -= P(B) P(C)^T and W(B, J) -= P(B) L^{-1}(K, J) on
//     the matrix cores.  W(B, J) (J <= K) lies where L(B, J) was.  The first wave
//     updates the next diagonal block and goes on to factor it while the others
//     do the rest: two barriers per panel.
// L^{-1} is left in LDS (lower tiles; the upper ones hold other things); with
// SWEEP (below) R = L^T (upper, may be NULL) and Rinv = L^{-T} (upper) are written,
// n x n.  A non-positive pivot sets flag[0] = 2 and is
// replaced by a tiny positive one so that the run continues.
//
// Bound by the serial chain of the diagonal blocks.  Against the form with lane
// reads for the broadcasts, the library's rsqrt, the inversion of L as a second
// sweep and five barriers per panel, order 16 went from 9.6 to 5.6 us, order 80
// from 43 to 15 us, order 128 from 75 to 25 us.
//
// L lives in LDS with an odd leading dimension, so that walking a row and
// walking a column are both free of bank conflicts; a constant one, so that every
// offset within a tile is an immediate (a lone wave is bound by its instructions).
constexpr int CB = 16;
constexpr int CLD = 129;

__host__ __device__ inline int chol_np(int64_t n) { return (int)((n + CB - 1) / CB * CB); }

// Dynamic LDS of chol_body: L (CLD x np) and the panel P (CLD x CB).
__host__ __device__ inline size_t chol_lds_bytes(int64_t n) {
    return (size_t)CLD * (chol_np(n) + CB) * 8;
}

// v of lane `src` of the wave (uniform)
__device__ __forceinline__ double chol_lane(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}
// Every lane: v of the lane of the even 16-lane row of its pair of rows.
__device__ __forceinline__ double chol_even_row(double v) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]);
}
// a_c -= src(lane N + c of each 16-lane row) * m, c < 4 (FP64 DPP broadcast; the
// s_nop keeps the two wait states a DPP read needs after a VALU write)
template <int N>
__device__ __forceinline__ void chol_bc4(double &a0, double &a1, double &a2, double &a3, double src, double m) {
    asm("s_nop 1\n"
        "v_fmac_f64_dpp %0, -%4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %1, -%4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %2, -%4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %3, -%4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3)
        : "v"(src), "v"(m), "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3));
}
template <int N>
__device__ __forceinline__ void chol_bc1(double &a, double src, double m) {
    asm("s_nop 1\n v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
        : "+v"(a)
        : "v"(src), "v"(m), "n"(N));
}
// a[c] -= src(lane c) * m for c = C .. 15
template <int C>
__device__ __forceinline__ void chol_bc(double (&a)[CB], double src, double m) {
    if constexpr (C < CB) {
        if constexpr (C % 4 == 0) {
            chol_bc4<C>(a[C], a[C + 1], a[C + 2], a[C + 3], src, m);
            chol_bc<C + 4>(a, src, m);
        } else {
            chol_bc1<C>(a[C], src, m);
            chol_bc<C + 1>(a, src, m);
        }
    }
}

// Column steps J.. of a 16 x 16 block: a is row l of the block (even 16-lane
// rows, piv = l) or column l of its factor's inverse, begun as e_l (odd rows,
// piv < 0).  REPAIR replaces non-positive pivots by tiny; without it bad only
// tells that there was one.
template <bool REPAIR, int J>
__device__ __forceinline__ void chol_block(double (&a)[CB], int piv, double tiny, bool &bad) {
    if constexpr (J < CB) {
        double d = chol_lane(a[J], J);
        const bool neg = !(d > 0.0);
        bad |= neg;
        if constexpr (REPAIR) {
            d = neg ? tiny : d;
            if (piv == J) a[J] = d;
        }
        const double col = chol_even_row(a[J]);
        // 1 / sqrt(d): the hardware estimate with one third-order step
        double rd = __builtin_amdgcn_rsq(d);
        const double e = fma(-d * rd, rd, 1.0);
        rd = fma(rd * e, fma(0.375, e, 0.5), rd);
        a[J] *= rd;
        chol_bc<J + 1>(a, col * rd, a[J]);
        chol_block<REPAIR, J + 1>(a, piv, tiny, bad);
    }
}

// Barrier that orders LDS only: the stores of finished tiles to global memory
// stay in flight across it (nothing here reads them back).
__device__ __forceinline__ void chol_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// SWEEP (the batched eigensolver and the ALS branch): L^{-1} from L afterwards,
// block column by block column from the last one,
// L^{-1}(B, K) = -(sum_{J in (K, B]} L^{-1}(B, J) L(J, K)) D_K^{-1}.
// Where a mode keeps more vectors than the product of the other ranks gives its
// unfolding signal, the surplus eigenvectors lie in the noise, and which ones come
// out hangs on the last bits of L^{-1}; ALS sweeps on FP32 data carry such bits on.
// Both keep the order of operations that their results have had.  Order 80: 19 us
// in place of 15.
template <int NTH, bool SWEEP = false>
__device__ __forceinline__ void chol_body(const double *__restrict__ G, int n, int64_t ldg,
                                          double shift_rel, double *__restrict__ Rout,
                                          double *__restrict__ Rinv, int64_t *__restrict__ flag) {
    constexpr int NW = NTH / 64;
    constexpr int LC = 128 / NW;   // columns per wave at most
    extern __shared__ __align__(16) double s_l[];  // L, column-major, leading dimension ld
    const int np = chol_np(n), nb = np / CB;
    double *s_p = s_l + np * CLD;   // panel P
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tr = lane & 15, tg = lane >> 4;   // matrix-core tile coordinates
    const int rc = tr + CLD * tg;   // element (row tr, column tg) of a tile
    const int cr = tg + CLD * tr;   // element (row tg, column tr)

    // lower triangle of G padded with the identity: every load issued before the
    // first is stored
    {
        double v[LC][2];
#pragma unroll
        for (int u = 0; u < LC; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = wave + NW * u, i = lane + 64 * h;
                v[u][h] = i == j ? 1.0 : 0.0;
                if (64 * h < n && j < n && i < n && i >= j) v[u][h] = G[i + ldg * j];
            }
#pragma unroll
        for (int u = 0; u < LC; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = wave + NW * u, i = lane + 64 * h;
                if (j < np && i < np) s_l[i + CLD * j] = v[u][h];
            }
    }
    __syncthreads();
    double tiny = 0.0;
    bool bad = false;
    // a 16 x 16 identity beside the first diagonal block (the panel's place when
    // that is the only block): the odd rows' start of every block
    const int ident = CLD * CB;
    if (wave == 0) {
        double t = 0.0;
        for (int i = lane; i < n; i += 64) t += s_l[i + CLD * i];
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
        if (shift_rel != 0.0)
            for (int i = lane; i < n; i += 64) s_l[i + CLD * i] += shift_rel * t / n;
        tiny = 1e-300 + 1e-30 * fabs(t);
#pragma unroll
        for (int v = 0; v < 4; ++v) s_l[ident + cr + 4 * v] = tg + 4 * v == tr ? 1.0 : 0.0;
    } else {
        // the triangle outside R, but for the diagonal blocks
        for (int j = wave - 1; j < n; j += NW - 1)
            for (int i = (j / CB + 1) * CB + lane; i < n; i += 64) {
                if (SWEEP && Rout) Rout[i + n * j] = 0.0;
            }
    }
    // tile c -= P(b) X (c begun as 0 where fresh): X(k, j) = x[XK k + XJ j]
    auto update = [&](int b, double *c, bool fresh, const double *x, auto xt) {
        constexpr bool XT = decltype(xt)::value;
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        if (!fresh)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] = c[cr + 4 * v];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-s_p[CB * b + rc + 4 * kk * CLD],
                                                       XT ? x[rc + 4 * kk * CLD] : x[cr + 4 * kk], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) c[cr + 4 * v] = acc[v];
    };
    // acc = D^{-1} X with D^{-1} in the diagonal block dk
    auto solve = [&](const double *dk, const double *x, auto xt) {
        constexpr bool XT = decltype(xt)::value;
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(dk[rc + 4 * kk * CLD], XT ? x[rc + 4 * kk * CLD] : x[cr + 4 * kk],
                                                       acc, 0, 0, 0);
        return acc;
    };
    using TransX = std::true_type;
    using PlainX = std::false_type;
    for (int kb = 0; kb < nb; ++kb) {
        const int k0 = kb * CB, kp = kb - 1;
        double *dk = s_l + k0 + CLD * k0;
        if (wave == 0) {
            // the diagonal block, with the previous panel's update
            if (kb) update(kb, dk, false, s_p + k0, TransX());
            const bool even = (tg & 1) == 0;
            const double *src = even ? dk : s_l + ident;
            double a[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) a[c] = src[tr + CLD * c];
            bool neg = false;
            chol_block<false, 0>(a, tr, tiny, neg);
            if (neg) {   // repeated with the pivots replaced
                bad = true;
#pragma unroll
                for (int c = 0; c < CB; ++c) a[c] = src[tr + CLD * c];
                chol_block<true, 0>(a, even ? tr : -1, tiny, neg);
            }
            if (tg == 1) {   // column tr of D^{-1}
#pragma unroll
                for (int c = 0; c < CB; ++c) dk[c + CLD * tr] = c >= tr ? a[c] : 0.0;
            }
            if (SWEEP && Rout && tg == 0 && k0 + tr < n) {
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    if (k0 + c < n) Rout[k0 + c + n * (k0 + tr)] = c <= tr ? a[c] : 0.0;
            }
        } else if (kb) {
            // the rest of the previous panel's update: lower tiles of A, then W
            const int nt = nb - kb, na = nt * (nt + 1) / 2;
            for (int q = wave; q < na + (SWEEP ? 0 : nt * kb); q += NW - 1) {
                if (q < na) {
                    int bi = 0;
                    while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
                    const int bj = kb + q - bi * (bi + 1) / 2;
                    bi += kb;
                    update(bi, s_l + CB * (bi + CLD * bj), false, s_p + CB * bj, TransX());
                } else {
                    const int bi = kb + (q - na) % nt, bj = (q - na) / nt;
                    update(bi, s_l + CB * (bi + CLD * bj), bj == kp, s_l + CB * (kp + CLD * bj), PlainX());
                }
            }
        }
        chol_sync();
        // P(b)^T = D^{-1} A(b, K)^T for b > kb, L^{-1}(K, b) = D^{-1} W(K, b) for b < kb
        for (int q = (SWEEP ? kb : 0) + wave; q < nb - 1; q += NW) {
            const bool below = q >= kb;
            const int i0 = CB * (below ? q + 1 : q);
            f64x4 acc;
            if (below) {
                acc = solve(dk, s_l + i0 + CLD * k0, TransX());
#pragma unroll
                for (int v = 0; v < 4; ++v) s_p[i0 + rc + 4 * v * CLD] = acc[v];
                if constexpr (SWEEP) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) s_l[i0 + CLD * k0 + rc + 4 * v * CLD] = acc[v];
                }
            } else {
                acc = solve(dk, s_l + k0 + CLD * i0, PlainX());
#pragma unroll
                for (int v = 0; v < 4; ++v) s_l[k0 + CLD * i0 + cr + 4 * v] = acc[v];
            }
            if (SWEEP && Rout) {   // R(K, b)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (i0 + tr < n && k0 + tg + 4 * v < n) Rout[k0 + tg + 4 * v + n * (i0 + tr)] = acc[v];
            }
        }
        chol_sync();
    }
    if (bad && flag) flag[0] = 2;
    if constexpr (SWEEP) {
        for (int kb = nb - 1; kb >= 0; --kb) {
            const int k0 = CB * kb;
            const double *dk = s_l + k0 + CLD * k0;
            for (int bi = kb + 1 + wave; bi < nb; bi += NW) {   // the sums, in the panel's place
                f64x4 acc = {0.0, 0.0, 0.0, 0.0};
                for (int bj = kb + 1; bj <= bi; ++bj)
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s_l[CB * (bi + CLD * bj) + rc + 4 * kk * CLD],
                                                                   s_l[CB * bj + CLD * k0 + cr + 4 * kk], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) s_p[CB * bi + cr + 4 * v] = acc[v];
            }
            chol_sync();
            for (int bi = kb + 1 + wave; bi < nb; bi += NW) {
                f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-s_p[CB * bi + rc + 4 * kk * CLD], dk[cr + 4 * kk], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) s_l[CB * bi + CLD * k0 + cr + 4 * v] = acc[v];
            }
            chol_sync();
        }
        for (int j = wave; j < n; j += NW)
            for (int i = lane; i < n; i += 64) Rinv[i + n * j] = i <= j ? s_l[j + CLD * i] : 0.0;
    }
}

}  // namespace sth
