// FP64 symmetric eigensolver for the EIG branch of Alg. 2: the R_n leading
// eigenvectors of the mode-n Gram matrix.
//
// Routes (eig_launch):
//   * eig_leading up to order 128: two-sided cyclic Jacobi with a parallel
//     (round-robin) ordering in one 512-thread workgroup, A and V in LDS when
//     they fit (jacobi_*_kernel; relative accuracy, sweep cap reported).
//   * decompositions up to order 128, and every order where the subspace
//     iteration does not apply: the direct solver of teig_body.h
//     (tridiagonalization, bisection, inverse iteration) in one workgroup.
//   * above order 128 with a block p = R + 16 (rounded to 8) <= 128: subspace
//     iteration Q <- orth(S Q) from a seeded Gaussian block (2 products when
//     S carries single-precision rounding, 3 for FP64 data; orth = shifted
//     Cholesky-QR, see orth()), Rayleigh-Ritz with the direct solver on
//     T = Q^T S Q, then a residual test: the R Ritz pairs are accepted when
//     every ||S u - theta u|| <= max(16 sqrt(n) eps, u_S) |theta_1|, i.e. when
//     they are exact eigenpairs of a perturbation of S no larger than that of
//     a backward-stable direct solver or than the rounding S already carries
//     (u_S: the unit roundoff of the products that formed S, eps for FP64
//     products, 2^-24 for FP32 and bf16x6, 2^-17 for bf16x3).  A failed test
//     runs a second round (2 more products and Rayleigh-Ritz from the same
//     basis); when that fails too, the direct solver runs on S itself.  Every
//     launch after the first round is gated on the device by the residuals
//     (it returns at once when they passed), so the whole solve is one
//     fixed, capturable sequence, and the result is the leading eigenpairs
//     on every spectrum, with or without a gap after R.
//
// Selection: eigenvalues in descending order, the R leading eigenvectors
// signed so that their entry of largest magnitude is positive (first index
// on ties).
#include "chol_body.h"
#include "common.h"
#include "eig_body.h"
#include "internal.h"
#include "teig_body.h"

namespace sth {

template <bool ALDS, bool VLDS>
__global__ __launch_bounds__(EIG_THREADS) void jacobi_kernel(const double *__restrict__ S, int n,
                                                             int R, double *__restrict__ Ag,
                                                             double *__restrict__ Vg,
                                                             double *__restrict__ U,
                                                             double *__restrict__ lam, double tol,
                                                             int max_sweeps,
                                                             int64_t *__restrict__ flag) {
    jacobi_body<ALDS, VLDS>(S, n, R, Ag, Vg, U, lam, tol, max_sweeps, flag);
}

template <bool VLDS>
__global__ __launch_bounds__(EIG_THREADS) void jacobi_small_kernel(const double *__restrict__ S, int n,
                                                                   int R, double *__restrict__ Vg,
                                                                   double *__restrict__ U,
                                                                   double *__restrict__ lam, double tol,
                                                                   int max_sweeps,
                                                                   int64_t *__restrict__ flag) {
    jacobi_small_body<VLDS>(S, n, R, Vg, U, lam, tol, max_sweeps, flag);
}

// SMALL: n <= TE_LDS_N (teig_small); ZLDS: see teig_body
template <bool SMALL, bool ZLDS>
__global__ __launch_bounds__(TE_T) void teig_kernel(const double *__restrict__ S, int64_t lds, int n, int R,
                                                   double *__restrict__ U, int64_t ldu,
                                                   double *__restrict__ lam, int sign_rule, TeScratch sc,
                                                   int64_t *__restrict__ flag, const double *__restrict__ chk,
                                                   double chk_tol, int64_t *__restrict__ count) {
    // gated on a residual test (chk): runs only when some chk[r] exceeds
    // chk_tol * chk[R] or is not finite; count records that it ran
    if (!gate_open(chk, R, chk_tol)) return;
    if (chk && count && threadIdx.x == 0) *count += 1;
    if constexpr (SMALL) teig_small(S, lds, n, R, U, ldu, lam, sign_rule != 0, sc, flag);
    else teig_body<ZLDS>(S, lds, n, R, U, ldu, lam, sign_rule != 0, sc, flag);
}

// ---- subspace-iteration products: one 16 x 16 tile of C per workgroup on
// the FP64 matrix cores, the waves splitting the contraction in steps of 16
// (lane group g takes 4 g .. 4 g + 3 of a step, so that an operand walked along
// the contraction is read in whole 128-byte lines), their partial tiles summed
// in LDS in a fixed order.  Out-of-range rows and columns read clamped addresses
// and use zeros.  All take a gate (see gate_open).  They are bound by the
// latency of a wave's successive steps, not by the matrix cores: hence many
// waves per tile, 16- and 32-byte loads and two steps in flight.  n = 512, p = 80:
// S Q 5.6 us and Q^T Q 6.4 us, against 7.2 and 9.6 with four waves per tile and
// 8-byte loads, one step at a time (an empty launch in the same trace: 4.4).
constexpr int SI_NN_T = 512, SI_TN_T = 1024;

// four consecutive elements along the contraction
template <bool CONTIG>
__device__ __forceinline__ void si_load4(double (&v)[4], const double *p, int64_t stride) {
    if constexpr (CONTIG) __builtin_memcpy(v, p, 32);
    else
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p[stride * u];
}

// acc = sum over k < kmax of a(k) b(k), this wave's share; pa and pb point at
// this lane's row and column, sa and sb are their strides along k (1 where CA,
// CB1).  Two steps' loads are in flight.
template <bool CA, bool CB1>
__device__ __forceinline__ f64x4 si_tile(const double *pa, int64_t sa, bool rok, const double *pb, int64_t sb,
                                         bool cok, int kmax, int wave, int nw, int tg) {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int s0 = 32 * wave; s0 < kmax; s0 += 32 * nw) {
        double a[2][4], b[2][4];
        if (s0 + 32 <= kmax) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int kk = s0 + 16 * h + 4 * tg;
                si_load4<CA>(a[h], pa + sa * kk, sa);
                si_load4<CB1>(b[h], pb + sb * kk, sb);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (!rok) a[h][u] = 0.0;
                    if (!cok) b[h][u] = 0.0;
                }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int kk = s0 + 16 * h + 4 * tg + u;
                    const bool ok = kk < kmax;
                    const int kc = ok ? kk : 0;
                    a[h][u] = pa[sa * kc];
                    b[h][u] = pb[sb * kc];
                    if (!(ok && rok)) a[h][u] = 0.0;
                    if (!(ok && cok)) b[h][u] = 0.0;
                }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[h][u], b[h][u], acc, 0, 0, 0);
    }
    return acc;
}

// The summed tile: thread tid < 256 gets the element of tile row
// (tid >> 4 & 3) + 4 (tid >> 6), column tid & 15.
template <int NW>
__device__ __forceinline__ double si_sum(double (&s_acc)[NW][256], f64x4 acc, int wave, int lane, int tid) {
#pragma unroll
    for (int v = 0; v < 4; ++v) s_acc[wave][64 * v + lane] = acc[v];
    __syncthreads();
    double c = 0.0;
    if (tid < 256)
#pragma unroll
        for (int w = 0; w < NW; ++w) c += s_acc[w][tid];
    return c;
}

// Z (n x q) = S Q.
__global__ __launch_bounds__(SI_NN_T) void si_sq_kernel(int n, int q, const double *__restrict__ S,
                                                       const double *__restrict__ Q, int64_t ldq,
                                                       double *__restrict__ Z, int64_t ldz,
                                                       const double *__restrict__ gate, int gate_R,
                                                       double gate_tol) {
    if (!gate_open(gate, gate_R, gate_tol)) return;
    constexpr int NW = SI_NN_T / 64;
    __shared__ double s_acc[NW][256];
    const int mt = (n + 15) >> 4;
    const int bi = blockIdx.x % mt, bj = blockIdx.x / mt;
    const int i0 = bi << 4, j0 = bj << 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tr = lane & 15, tg = lane >> 4;
    const int ia = min(i0 + tr, n - 1), jb = min(j0 + tr, q - 1);
    // D(row = column of Q, col = row of S): the stores run along the rows
    const f64x4 acc = si_tile<true, false>(Q + ldq * jb, 1, j0 + tr < q, S + ia, n, i0 + tr < n, n, wave, NW, tg);
    const double z = si_sum<NW>(s_acc, acc, wave, lane, tid);
    const int col = j0 + tg + 4 * wave, row = i0 + tr;
    if (tid < 256 && row < n && col < q) Z[row + ldz * col] = z;
}

// C = 1.5 A - 0.5 A B, one Newton-Schulz step toward orthonormal columns
// (A m x q, B = A^T A).
__global__ __launch_bounds__(SI_NN_T) void si_ns_kernel(int m, int q, const double *__restrict__ A, int64_t lda,
                                                       const double *__restrict__ B, double *__restrict__ C,
                                                       const double *__restrict__ gate, int gate_R,
                                                       double gate_tol) {
    if (!gate_open(gate, gate_R, gate_tol)) return;
    constexpr int NW = SI_NN_T / 64;
    __shared__ double s_acc[NW][256];
    const int mt = (m + 15) >> 4;
    const int bi = blockIdx.x % mt, bj = blockIdx.x / mt;
    const int i0 = bi << 4, j0 = bj << 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tr = lane & 15, tg = lane >> 4;
    const int ia = min(i0 + tr, m - 1), jb = min(j0 + tr, q - 1);
    const f64x4 acc = si_tile<true, false>(B + (int64_t)q * jb, 1, j0 + tr < q, A + ia, lda, i0 + tr < m, q, wave, NW, tg);
    const double c = si_sum<NW>(s_acc, acc, wave, lane, tid);
    const int col = j0 + tg + 4 * wave, row = i0 + tr;
    if (tid < 256 && row < m && col < q) C[row + lda * col] = 1.5 * A[row + lda * col] - 0.5 * c;
}

// C (p x q) = A^T B with A (k x p), B (k x q).  SYM: B = A, only the tiles
// on and below the diagonal are formed and each is written to both halves.
template <bool SYM>
__global__ __launch_bounds__(SI_TN_T) void si_tn_kernel(int p, int q, int k, const double *__restrict__ A, int64_t lda,
                                                       const double *__restrict__ B, int64_t ldb,
                                                       double *__restrict__ C, int64_t ldc,
                                                       const double *__restrict__ gate, int gate_R,
                                                       double gate_tol) {
    if (!gate_open(gate, gate_R, gate_tol)) return;
    constexpr int NW = SI_TN_T / 64;
    __shared__ double s_acc[NW][256];
    int bi, bj;
    if (SYM) {
        const int t = blockIdx.x;
        bi = 0;
        while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
        bj = t - bi * (bi + 1) / 2;
    } else {
        const int pt = (p + 15) >> 4;
        bi = blockIdx.x % pt;
        bj = blockIdx.x / pt;
    }
    const int i0 = bi << 4, j0 = bj << 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tr = lane & 15, tg = lane >> 4;
    const int ia = min(i0 + tr, p - 1), jb = min(j0 + tr, q - 1);
    const f64x4 acc = si_tile<true, true>(A + lda * ia, 1, i0 + tr < p, B + ldb * jb, 1, j0 + tr < q, k, wave, NW, tg);
    const double c = si_sum<NW>(s_acc, acc, wave, lane, tid);
    const int row = i0 + tg + 4 * wave, col = j0 + tr;
    if (tid < 256 && row < p && col < q) {
        C[row + ldc * col] = c;
        if (SYM && bi != bj) C[col + ldc * row] = c;
    }
}

// Q = A R^{-1} with G (+ shift) = R^T R (chol_body), A and Q n x p, p <= 128.
// Every workgroup factors G for itself and takes 16 rows of A, which it has
// loaded before: the redundant factorizations run side by side, where a
// factorization in one workgroup and a product after it cost another launch and
// the trip of R^{-1} through memory (n = 512, p = 80: 16.5 us, against 15 + 7).
constexpr int SI_CQ_T = 512;
__global__ __launch_bounds__(SI_CQ_T) void si_cholqr_kernel(int n, int p, const double *__restrict__ A, int64_t lda,
                                                           const double *__restrict__ G, double shift_rel,
                                                           double *__restrict__ Q, int64_t *__restrict__ flag,
                                                           const double *__restrict__ gate, int gate_R,
                                                           double gate_tol) {
    if (!gate_open(gate, gate_R, gate_tol)) return;
    constexpr int NW = SI_CQ_T / 64, AV = CB * 128 / SI_CQ_T;
    extern __shared__ __align__(16) double s_l[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tr = lane & 15, tg = lane >> 4;
    const int i0 = CB * blockIdx.x, np = chol_np(p);
    double av[AV];   // row tid & 15, column (tid >> 4) + 32 u
#pragma unroll
    for (int u = 0; u < AV; ++u) {
        const int i = i0 + (tid & 15), k = (tid >> 4) + SI_CQ_T / 16 * u;
        av[u] = i < n && k < p ? A[i + lda * k] : 0.0;
    }
    chol_body<SI_CQ_T>(G, p, p, shift_rel, nullptr, nullptr, blockIdx.x == 0 ? flag : nullptr);
    // the panel's place is free now: A(i, k) = s_a[k + CLD i]; R^{-1}(k, j) = L^{-1}(j, k)
    double *s_a = s_l + np * CLD;
#pragma unroll
    for (int u = 0; u < AV; ++u) {
        const int k = (tid >> 4) + SI_CQ_T / 16 * u;
        if (k < np) s_a[k + CLD * (tid & 15)] = av[u];
    }
    __syncthreads();
    for (int j0 = CB * wave; j0 < np; j0 += CB * NW) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = 0; k0 <= j0; k0 += CB)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int k = k0 + 4 * kk + tg;
                // D(row = j, col = i): stores run along the rows of A
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s_l[j0 + tr + CLD * k], s_a[k + CLD * tr], acc, 0, 0, 0);
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = j0 + tg + 4 * v;
            if (j < p && i0 + tr < n) Q[i0 + tr + lda * j] = acc[v];
        }
    }
}

// Rayleigh-Ritz finish, one workgroup per Ritz vector r:
//   U(:, r) = Q W(:, r), then the sign rule on it;
//   res[r] = ||Z W(:, r) - theta_r U(:, r)|| with Z = S Q (the Ritz residual);
//   lam[r] = theta_r; res[R] = |theta_1| (workgroup 0); res2 (may be null)
//   gets the same values.  Gated (see gate_open); gate must not be res.
// Bound by what one CU reads (Q and Z whole): two rows per 16-byte load and 16
// loads in flight, 9.7 us at n = 512, p = 80 (16.4 with 8-byte loads).
constexpr int RR_T = 512, RR_W = RR_T / 64;
__global__ __launch_bounds__(RR_T) void rr_finish_kernel(const double *__restrict__ Q, const double *__restrict__ Zs,
                                                        int n, int p, const double *__restrict__ W,
                                                        const double *__restrict__ th, int R,
                                                        double *__restrict__ U, double *__restrict__ lam,
                                                        double *__restrict__ res, double *__restrict__ res2,
                                                        const double *__restrict__ gate, double gate_tol) {
    if (!gate_open(gate, R, gate_tol)) return;
    const int r = blockIdx.x, tid = threadIdx.x;
    __shared__ double s_w[SI_BLOCK_MAX];
    __shared__ double s_ss[RR_W], s_bv[RR_W], s_vv[RR_W];
    __shared__ int s_bi[RR_W];
    __shared__ double s_sign, s_half[4][256];
    for (int k = tid; k < p; k += RR_T) s_w[k] = W[k + (int64_t)p * r];
    __syncthreads();
    const double t = th[r];
    double ss = 0.0, best = -1.0, bval = 0.0;
    int arg = 0;
    // two rows per thread in 16-byte loads, the two halves of the workgroup
    // splitting the contraction
    const int half = tid >> 8, kh = (p + 1) >> 1, kb = half * kh, ke = min(p, kb + kh);
    for (int r0 = 0; r0 < n; r0 += 512) {
        const int i = r0 + 2 * (tid & 255);
        const int ic = min(i, n - 2);   // n > 128
        double u[2] = {0.0, 0.0}, z[2] = {0.0, 0.0};
        if (i < n)
            for (int k0 = kb; k0 < ke; k0 += 8) {
                double qv[8][2], zv[8][2];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const int64_t o = ic + (int64_t)n * min(k0 + c, ke - 1);
                    __builtin_memcpy(qv[c], Q + o, 16);
                    __builtin_memcpy(zv[c], Zs + o, 16);
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const double w = k0 + c < ke ? s_w[k0 + c] : 0.0;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        u[h] += qv[c][h] * w;
                        z[h] += zv[c][h] * w;
                    }
                }
            }
        __syncthreads();   // s_half is free
        if (half) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s_half[2 * h][tid & 255] = u[h];
                s_half[2 * h + 1][tid & 255] = z[h];
            }
        }
        __syncthreads();
        if (!half)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // rows ic and ic + 1: only those not taken by another thread
                const int row = ic + h;
                if (i >= n || row < i || row >= n) continue;
                const double uu = u[h] + s_half[2 * h][tid], d = z[h] + s_half[2 * h + 1][tid] - t * uu;
                ss += d * d;
                U[row + (int64_t)n * r] = uu;
                if (fabs(uu) > best) {
                    best = fabs(uu);
                    arg = row;
                    bval = uu;
                }
            }
    }
    for (int o = 32; o > 0; o >>= 1) {
        ss += __shfl_xor(ss, o);
        const double b2 = __shfl_xor(best, o), v2 = __shfl_xor(bval, o);
        const int a2 = __shfl_xor(arg, o);
        if (b2 > best || (b2 == best && a2 < arg)) {
            best = b2;
            arg = a2;
            bval = v2;
        }
    }
    if ((tid & 63) == 0) {
        s_ss[tid >> 6] = ss;
        s_bv[tid >> 6] = best;
        s_bi[tid >> 6] = arg;
        s_vv[tid >> 6] = bval;
    }
    __syncthreads();
    if (tid == 0) {
        double tot = 0.0, b = s_bv[0], v = s_vv[0];
        int a = s_bi[0];
        for (int w = 0; w < RR_W; ++w) tot += s_ss[w];
        for (int w = 1; w < RR_W; ++w)
            if (s_bv[w] > b || (s_bv[w] == b && s_bi[w] < a)) {
                b = s_bv[w];
                a = s_bi[w];
                v = s_vv[w];
            }
        s_sign = v < 0.0 ? -1.0 : 1.0;
        res[r] = sqrt(tot);
        if (res2) res2[r] = res[r];
        if (lam) lam[r] = t;
        if (r == 0) {
            res[R] = fabs(t);
            if (res2) res2[R] = fabs(t);
        }
    }
    __syncthreads();
    if (s_sign < 0.0)
        for (int i = tid; i < n; i += RR_T) U[i + (int64_t)n * r] = -U[i + (int64_t)n * r];
}

namespace {

int64_t si_block(int64_t n, int64_t R) { return si_block_host(n, R); }

// The subspace iteration applies above order 128 when its block fits and
// leaves a guard (p < n) and R is within the Gram's rank bound.
bool use_si(int64_t n, int64_t R, int64_t rank_bound) {
    const int64_t p = si_block(n, R);
    return n > EIG_DIRECT_MAX && p <= SI_BLOCK_MAX && p < n && R <= rank_bound;
}

// residual test of the Ritz pairs: ||S u - theta u|| <= max(SI_RES_C sqrt(n) eps, u_S) |theta_1|
constexpr double SI_RES_C = 16.0;
// iterations of the first round: 2 when S carries single-precision rounding
// (u_S >= 2^-24: the test is that loose), 3 for FP64 data; the gated second
// round adds SI_ITERS_MORE
constexpr int SI_ITERS_LOOSE = 2, SI_ITERS_FP64 = 3, SI_ITERS_MORE = 2;

struct SiWs {
    double *Q, *Z, *Z2, *G, *T, *W, *th, *res, *res2;
    double *te;   // teig scratch of the p x p Rayleigh-Ritz problem
    double *fb;   // teig scratch of the direct solve of S (fallback)
};

size_t jacobi_ws(int64_t n) { return (size_t)(256 + 2 * n * n * sizeof(double)); }

SiWs si_layout(char *ws, int64_t n, int64_t p, int64_t R) {
    SiWs w;
    double *d = (double *)(ws + 256);
    w.Q = d; d += n * p;
    w.Z = d; d += n * p;
    w.Z2 = d; d += n * p;
    w.G = d; d += p * p;
    w.T = d; d += p * p;
    w.W = d; d += p * p;
    w.th = d; d += p;
    w.res = d; d += p + 1;
    w.res2 = d; d += p + 1;
    w.te = d; d += teig_scratch_doubles(p, R, true);
    w.fb = d;
    return w;
}

size_t si_bytes(int64_t n, int64_t p, int64_t R) {
    return 256 + (size_t)(3 * n * p + 3 * p * p + 3 * p + 2) * 8 + teig_scratch_doubles(p, R, true) * 8 +
           teig_scratch_doubles(n, R, n <= TE_LDS_N) * 8 + 256;
}

size_t teig_bytes(int64_t n, int64_t R) { return 256 + teig_scratch_doubles(n, R, n <= TE_LDS_N) * 8; }

hipError_t si_sq(int n, int q, const double *S, const double *Q, int64_t ldq, double *Z, int64_t ldz,
                 const double *gate, int gR, double gtol, hipStream_t s) {
    const dim3 grid((unsigned)(((n + 15) / 16) * ((q + 15) / 16)));
    hipLaunchKernelGGL(si_sq_kernel, grid, dim3(SI_NN_T), 0, s, n, q, S, Q, ldq, Z, ldz, gate, gR, gtol);
    return hipGetLastError();
}

hipError_t si_tn(bool sym, int p, int q, int k, const double *A, int64_t lda, const double *B, int64_t ldb,
                 double *C, int64_t ldc, const double *gate, int gR, double gtol, hipStream_t s) {
    const int pt = (p + 15) / 16, qt = (q + 15) / 16;
    if (sym)
        hipLaunchKernelGGL((si_tn_kernel<true>), dim3((unsigned)(pt * (pt + 1) / 2)), dim3(SI_TN_T), 0, s, p, q, k, A,
                           lda, B, ldb, C, ldc, gate, gR, gtol);
    else
        hipLaunchKernelGGL((si_tn_kernel<false>), dim3((unsigned)(pt * qt)), dim3(SI_TN_T), 0, s, p, q, k, A, lda, B,
                           ldb, C, ldc, gate, gR, gtol);
    return hipGetLastError();
}

struct Gate {
    const double *res;
    int R;
    double tol;
};

// Cholesky-QR of the n x p matrix A into Q: G = A^T A (+ shift), G = R^T R,
// Q = A R^{-1}; shift_rel > 0 gives the shifted first pass of the shifted
// Cholesky-QR3 scheme (stable for condition numbers up to ~1/eps).
hipError_t cholqr_pass(const double *A, double *Q, int n, int p, double shift_rel, SiWs &w, int64_t *flag,
                       const Gate &g, hipStream_t s) {
    hipError_t e;
    if ((e = si_tn(true, p, p, n, A, n, A, n, w.G, p, g.res, g.R, g.tol, s))) return e;
    const size_t lds = chol_lds_bytes(p);
    if (lds > 64 * 1024)
        if ((e = hipFuncSetAttribute((const void *)si_cholqr_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds))) return e;
    hipLaunchKernelGGL(si_cholqr_kernel, dim3((unsigned)((n + CB - 1) / CB)), dim3(SI_CQ_T), lds, s, n, p, A, (int64_t)n,
                       (const double *)w.G, shift_rel, Q, flag, g.res, g.R, g.tol);
    return hipGetLastError();
}

enum OrthKind { ORTH_MID, ORTH_QR3, ORTH_NS };

// Orthonormalization of the iterate A (overwritten) into Q:
//   ORTH_MID: the shifted pass and one plain pass; the intermediate bases
//     only need to be well conditioned (the shifted pass alone leaves them
//     too ill-conditioned for the next product's orthonormalization);
//   ORTH_QR3: shifted Cholesky-QR3, orthonormal to working accuracy for
//     condition numbers up to ~1/eps;
//   ORTH_NS: the shifted pass, one plain pass and one Newton-Schulz step
//     (the two passes leave ||Q^T Q - I|| far below 1, the step squares it),
//     for Grams that carry single-precision rounding.
hipError_t orth(double *A, double *Q, int n, int p, OrthKind kind, SiWs &w, int64_t *flag, const Gate &g,
                hipStream_t s) {
    hipError_t e;
    const double shift = 11.0 * ((double)n * p + (double)p * (p + 1)) * 1.1102230246251565e-16;
    if ((e = cholqr_pass(A, w.Z2, n, p, shift * p, w, flag, g, s))) return e;   // trace/p * p = trace
    if (kind == ORTH_MID) return cholqr_pass(w.Z2, Q, n, p, 0.0, w, flag, g, s);
    if ((e = cholqr_pass(w.Z2, A, n, p, 0.0, w, flag, g, s))) return e;
    if (kind == ORTH_QR3) return cholqr_pass(A, Q, n, p, 0.0, w, flag, g, s);
    if ((e = si_tn(true, p, p, n, A, n, A, n, w.G, p, g.res, g.R, g.tol, s))) return e;
    hipLaunchKernelGGL(si_ns_kernel, dim3((unsigned)(((n + 15) / 16) * ((p + 15) / 16))), dim3(SI_NN_T), 0, s, n, p,
                       (const double *)A, n, (const double *)w.G, Q, g.res, g.R, g.tol);
    return hipGetLastError();
}

hipError_t jacobi_launch(int64_t n, int64_t R, const double *S, double *U, double *lam, double tol,
                         int max_sweeps, void *ws, int64_t *flag, hipStream_t s) {
    double *Ag = (double *)((char *)ws + 256);
    double *Vg = Ag + n * n;
    const size_t mat = (size_t)n * n * sizeof(double);
    const size_t budget = EIG_LDS_AV;
    if (n <= 2 * JS_MAXM) {
        // A in LDS; V too when both fit (V in the workspace otherwise)
        const bool vl = jacobi_small_lds(n, true) <= budget;
        const size_t lds = jacobi_small_lds(n, vl);
        if (vl) {
            if (hipError_t ea = hipFuncSetAttribute((const void *)jacobi_small_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) return ea;
            hipLaunchKernelGGL(jacobi_small_kernel<true>, dim3(1), dim3(EIG_THREADS), lds, s, S, (int)n, (int)R, Ag, U, lam, tol, max_sweeps, flag);
        } else {
            if (hipError_t ea = hipFuncSetAttribute((const void *)jacobi_small_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) return ea;
            hipLaunchKernelGGL(jacobi_small_kernel<false>, dim3(1), dim3(EIG_THREADS), lds, s, S, (int)n, (int)R, Ag, U, lam, tol, max_sweeps, flag);
        }
    } else if (2 * mat <= budget) {
        auto k = jacobi_kernel<true, true>;
        if (hipError_t ea = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(2 * mat))) return ea;
        hipLaunchKernelGGL(k, dim3(1), dim3(EIG_THREADS), 2 * mat, s, S, (int)n, (int)R, Ag, Vg, U, lam, tol, max_sweeps, flag);
    } else if (mat <= budget) {
        auto k = jacobi_kernel<true, false>;
        if (hipError_t ea = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)mat)) return ea;
        hipLaunchKernelGGL(k, dim3(1), dim3(EIG_THREADS), mat, s, S, (int)n, (int)R, Ag, Vg, U, lam, tol, max_sweeps, flag);
    } else {
        hipLaunchKernelGGL((jacobi_kernel<false, false>), dim3(1), dim3(EIG_THREADS), 0, s, S, (int)n, (int)R, Ag, Vg, U, lam, tol, max_sweeps, flag);
    }
    return hipGetLastError();
}

template <bool SMALL, bool ZLDS>
hipError_t teig_go(const double *S, int64_t lds, int64_t n, int64_t R, double *U, int64_t ldu, double *lam,
                   bool sign_rule, TeScratch sc, int64_t *flag, const double *chk, double chk_tol, int64_t *count,
                   size_t lds_b, hipStream_t s) {
    auto k = teig_kernel<SMALL, ZLDS>;
    if (hipError_t ea = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_b))
        return ea;
    hipLaunchKernelGGL(k, dim3(1), dim3(TE_T), lds_b, s, S, lds, (int)n, (int)R, U, ldu, lam, sign_rule ? 1 : 0, sc,
                       flag, chk, chk_tol, count);
    return hipGetLastError();
}

}  // namespace

// Direct solver (teig_body.h) on the n x n matrix S; scratch holds
// teig_bytes(n, R).
hipError_t teig_launch(const double *S, int64_t lds, int64_t n, int64_t R, double *U, int64_t ldu, double *lam,
                       bool sign_rule, void *scratch, int64_t *flag, const double *chk, double chk_tol,
                       int64_t *count, hipStream_t s) {
    const TeScratch sc = teig_scratch_layout((double *)scratch, n, R, n <= TE_LDS_N);
    const size_t lb = teig_lds_bytes(n, R);
    if (n <= TE_LDS_N) return teig_go<true, true>(S, lds, n, R, U, ldu, lam, sign_rule, sc, flag, chk, chk_tol, count, lb, s);
    return teig_z_fits(n, R) ? teig_go<false, true>(S, lds, n, R, U, ldu, lam, sign_rule, sc, flag, chk, chk_tol, count, lb, s)
                             : teig_go<false, false>(S, lds, n, R, U, ldu, lam, sign_rule, sc, flag, chk, chk_tol, count, lb, s);
}

size_t eig_ws_bytes(int64_t n) {
    // every R <= n: the direct solver, the subspace iteration, or Jacobi
    size_t b = std::max(jacobi_ws(n), teig_bytes(n, n));
    for (int64_t R = 1; R <= n; ++R)
        if (use_si(n, R, n)) b = std::max(b, si_bytes(n, si_block(n, R), R));
    return b;
}

// R leading eigenpairs of the symmetric n x n matrix S (routes: see the top
// of this file).  jacobi_small: eig_leading's route for n <= 128 (Jacobi);
// otherwise the direct solver there.  rank_bound: rank(S) <= rank_bound (the
// subspace block is capped at it, and more vectors than that need the direct
// solver).  s_unit: unit roundoff of the products that formed S (0 when S is
// exact data).
hipError_t eig_launch(int64_t n, int64_t R, const double *S, double *U, double *lam, double tol,
                      int max_sweeps, void *ws, int64_t *flag, hipStream_t s, int64_t rank_bound,
                      bool jacobi_small, double s_unit) {
    if (n <= EIG_DIRECT_MAX) {
        if (jacobi_small) return jacobi_launch(n, R, S, U, lam, tol, max_sweeps, ws, flag, s);
        return teig_launch(S, n, n, R, U, n, lam, true, (char *)ws + 256, flag, nullptr, 0.0, nullptr, s);
    }
    if (!use_si(n, R, rank_bound))
        return teig_launch(S, n, n, R, U, n, lam, true, (char *)ws + 256, flag, nullptr, 0.0, nullptr, s);
    const int64_t p = std::min(si_block(n, R), rank_bound);
    SiWs w = si_layout((char *)ws, n, p, R);
    const int ni = (int)n, pi = (int)p, Ri = (int)R;
    hipError_t e;
    // start block: seeded Gaussian, used as it is (its span is all that
    // matters to the iteration, and an n x p Gaussian is well conditioned)
    if ((e = gaussian_f64(w.Q, n * p, 0x5EED5EEDull, (uint64_t)n * 1000 + p, s))) return e;
    // a Cholesky breakdown inside the iteration (S of rank below p) is not an
    // error of the result: it spoils the Ritz pairs, the residual test then
    // sends the solve on; it is recorded in flag[2] only.  flag[3] counts the
    // second rounds, flag[1] the direct solves of S.
    int64_t *si_flag = flag ? flag + 2 : nullptr;
    const bool loose = s_unit >= 0x1p-24;
    const double tol_res = std::max(SI_RES_C * std::sqrt((double)n) * 2.220446049250313e-16, s_unit);
    // round 0 runs always; round 1 continues from round 0's basis only when
    // a Ritz residual of round 0 fails the test (every launch gated on it)
    for (int round = 0; round < 2; ++round) {
        const Gate g = {round ? w.res : nullptr, Ri, tol_res};
        const int iters = round ? SI_ITERS_MORE : (loose ? SI_ITERS_LOOSE : SI_ITERS_FP64);
        for (int it = 0; it < iters; ++it) {
            if ((e = si_sq(ni, pi, S, w.Q, n, w.Z, n, g.res, g.R, g.tol, s))) return e;
            const OrthKind kind = it + 1 < iters ? ORTH_MID : (loose ? ORTH_NS : ORTH_QR3);
            if ((e = orth(w.Z, w.Q, ni, pi, kind, w, si_flag, g, s))) return e;
        }
        // Rayleigh-Ritz: T = Q^T S Q, its R leading pairs (W, theta), U = Q W
        if ((e = si_sq(ni, pi, S, w.Q, n, w.Z, n, g.res, g.R, g.tol, s))) return e;
        if ((e = si_tn(false, pi, pi, ni, w.Q, n, w.Z, n, w.T, p, g.res, g.R, g.tol, s))) return e;
        if ((e = teig_launch(w.T, p, p, R, w.W, p, w.th, false, w.te, si_flag, g.res, g.tol,
                             round && flag ? flag + 3 : nullptr, s)))
            return e;
        hipLaunchKernelGGL(rr_finish_kernel, dim3((unsigned)R), dim3(RR_T), 0, s, w.Q, w.Z, ni, pi, w.W, w.th, Ri, U,
                           lam, round ? w.res2 : w.res, round ? nullptr : w.res2, g.res, g.tol);
        if ((e = hipGetLastError())) return e;
    }
    // the direct solver on S when the last round's Ritz pairs fail the test
    return teig_launch(S, n, n, R, U, n, lam, true, w.fb, flag, w.res2, tol_res, flag ? flag + 1 : nullptr, s);
}

}  // namespace sth
