// Small dense FP64 linear algebra for the ALS branch (Alg. 3 and the QR of
// Alg. 2) and the FP64 norm reductions (Eq. 1).
//
//   gemm_tn       C = A^T B over a long contraction, split over workgroups
//                 with a fixed-order reduction (deterministic)
//   gemm_nn       C = A op(B) with a short contraction
//   gemm_f64      C = op(A) op(B) in LDS panels (FP32 data)
//   chol_kernel   one workgroup: G (+ shift) = R^T R (Cholesky, R upper),
//                 writes R and R^{-1}; used for the normal equations of
//                 Alg. 3 and for Cholesky-QR
//   sumsq / diff  FP64 sums of squares with per-block partials reduced in a
//                 fixed order
#include "chol_body.h"
#include "common.h"
#include "internal.h"

namespace sth {

// Both products run on the FP64 matrix cores in 16 x 16 tiles and are bound by
// latency at the ALS branch's sizes (R = 10, I = 30648: 2.5 MB and 6 MFLOP).
// The LDS-panel form that served them before took 34 us a call there, padding
// R to 32 and a contraction of R to 128; these take about 5 us.
constexpr int GTN_K = 256;   // contraction per workgroup aimed at (64 per wave)

// C_z = A^T B over the k-slice z: one 16 x 16 tile per workgroup, the four waves
// on interleaved 32-wide steps (lane group g takes 8 consecutive k), their
// partial tiles summed in LDS in wave order.
__global__ __launch_bounds__(256) void gemm_tn_kernel(int m, int n, int k, const double *__restrict__ A, int64_t lda,
                                                     const double *__restrict__ B, int64_t ldb,
                                                     double *__restrict__ C, int64_t ldc, int64_t cz, int kslice) {
    __shared__ f64x4 s_acc[3][64];
    const int mt = (m + 15) >> 4;
    const int i0 = (blockIdx.x % mt) << 4, j0 = (blockIdx.x / mt) << 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tr = lane & 15, tg = lane >> 4;
    const int kend = min(k, (int)(blockIdx.y + 1) * kslice);
    const double *a = A + lda * min(i0 + tr, m - 1), *b = B + ldb * min(j0 + tr, n - 1);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = blockIdx.y * kslice + 32 * wave; k0 < kend; k0 += 128) {
        double x[8], y[8];
        const int kk = k0 + 8 * tg;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int kc = kk + u < kend ? kk + u : kend - 1;
            x[u] = a[kc];
            y[u] = b[kc];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool ok = kk + u < kend;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? x[u] : 0.0, ok ? y[u] : 0.0, acc, 0, 0, 0);
        }
    }
    if (wave > 0) s_acc[wave - 1][lane] = acc;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w) acc += s_acc[w][lane];
    C += cz * blockIdx.y;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = i0 + tg + 4 * v, c = j0 + tr;
        if (r < m && c < n) C[r + ldc * c] = acc[v];
    }
}

// C = the nz partial products (m x n each) summed: four waves on interleaved
// partials of 64 elements, combined in a fixed order
__global__ __launch_bounds__(256) void gemm_reduce_kernel(int m, int n, int nz, const double *__restrict__ part,
                                                         double *__restrict__ C, int64_t ldc) {
    __shared__ double s_sum[4][64];
    const int el = threadIdx.x & 63, ks = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + el;
    const int64_t mn = (int64_t)m * n;
    double acc = 0.0;
    if (e < mn)
#pragma unroll 8
        for (int z = ks; z < nz; z += 4) acc += part[z * mn + e];
    s_sum[ks][el] = acc;
    __syncthreads();
    if (ks == 0 && e < mn) C[e % m + ldc * (e / m)] = (s_sum[0][el] + s_sum[1][el]) + (s_sum[2][el] + s_sum[3][el]);
}

// C (m x n) = A (m x k) op(B), op(B) k x n: one 16 x 16 tile per wave, the four
// waves of a workgroup on consecutive row tiles.
template <bool TB>
__global__ __launch_bounds__(256) void gemm_nn_kernel(int m, int n, int k, const double *__restrict__ A, int64_t lda,
                                                     const double *__restrict__ B, int64_t ldb,
                                                     double *__restrict__ C, int64_t ldc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tr = lane & 15, tg = lane >> 4;
    const int i0 = (blockIdx.x * 4 + wave) << 4, j0 = blockIdx.y << 4;
    if (i0 >= m) return;
    const int ia = min(i0 + tr, m - 1), jb = min(j0 + tr, n - 1);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < k; k0 += 16) {
        double a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int kk = k0 + 4 * u + tg, kc = kk < k ? kk : k - 1;
            a[u] = A[ia + lda * kc];
            b[u] = TB ? B[jb + ldb * kc] : B[kc + ldb * jb];
            if (kk >= k) {
                a[u] = 0.0;
                b[u] = 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = i0 + tg + 4 * v, c = j0 + tr;
        if (r < m && c < n) C[r + ldc * c] = acc[v];
    }
}

namespace {
// k-slices of gemm_tn: about GTN_K values of k per workgroup, at most 64 slices
// and 1024 workgroups
int gemm_tn_splits(int m, int n, int k) {
    const int tiles = ((m + 15) / 16) * ((n + 15) / 16);
    int nz = std::min((k + GTN_K - 1) / GTN_K, 64);
    while (nz > 1 && tiles * nz > 1024) nz = (nz + 1) / 2;
    return std::max(nz, 1);
}
}  // namespace

size_t gemm_tn_ws_bytes(int m, int n, int k) {
    const int nz = gemm_tn_splits(m, n, k);
    return nz > 1 ? (size_t)nz * m * n * sizeof(double) : 0;
}

hipError_t gemm_tn(int m, int n, int k, const double *A, int64_t lda, const double *B, int64_t ldb, double *C,
                   int64_t ldc, void *ws, hipStream_t s) {
    if (m == 0 || n == 0) return hipSuccess;
    int nz = gemm_tn_splits(m, n, k);
    const int kslice = std::max(((k + nz - 1) / nz + 127) / 128 * 128, 128);   // whole steps of the four waves
    nz = std::max(1, (k + kslice - 1) / kslice);
    const dim3 grid((unsigned)(((m + 15) / 16) * ((n + 15) / 16)), (unsigned)nz);
    double *out = nz > 1 ? (double *)ws : C;
    hipLaunchKernelGGL(gemm_tn_kernel, grid, dim3(256), 0, s, m, n, k, A, lda, B, ldb, out, nz > 1 ? m : ldc,
                       (int64_t)m * n, kslice);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nz == 1) return e;
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3((unsigned)(((int64_t)m * n + 63) / 64)), dim3(256), 0, s, m, n, nz,
                       (const double *)ws, C, ldc);
    return hipGetLastError();
}

hipError_t gemm_nn(bool tb, int m, int n, int k, const double *A, int64_t lda, const double *B, int64_t ldb,
                   double *C, int64_t ldc, hipStream_t s) {
    if (m == 0 || n == 0) return hipSuccess;
    const dim3 grid((unsigned)((m + 63) / 64), (unsigned)((n + 15) / 16));
    if (tb)
        hipLaunchKernelGGL(gemm_nn_kernel<true>, grid, dim3(256), 0, s, m, n, k, A, lda, B, ldb, C, ldc);
    else
        hipLaunchKernelGGL(gemm_nn_kernel<false>, grid, dim3(256), 0, s, m, n, k, A, lda, B, ldb, C, ldc);
    return hipGetLastError();
}

// The LDS-panel products, for the ALS branch on FP32 data.  There the bases are
// rounded to the FP32 or bf16 factors of the next product, and the sweeps carry a
// last-bit difference on: one element rounded the other way moves the factors by
// 1e-8 to 1e-7.  These keep the order of operations that the results of FP32 data
// have had; FP64 data takes gemm_tn and gemm_nn (5 us a call for 34).
constexpr int GT = 32;   // gemm tile (rows and columns of C)
constexpr int GK = 128;  // k-extent staged in LDS per step

// C_part[z] (m x n, ldc) = op(A) op(B) over k-slice z.  The skinny products
// of the eigensolver and the ALS branch are latency-bound, so every step
// loads a whole GT x GK panel of each operand with all loads in flight at
// once (coalesced along the contiguous index of each operand), then runs
// GK rank-1 updates from LDS: one global round trip per 128 values of k.
__global__ __launch_bounds__(256) void gemm_f64_kernel(int ta, int tb, int m, int n, int k,
                                                       const double *__restrict__ A,
                                                       int64_t lda, const double *__restrict__ B,
                                                       int64_t ldb, double *__restrict__ C,
                                                       int64_t ldc, int kslice, double *__restrict__ part) {
    extern __shared__ __align__(16) double s_gemm[];
    double *sA = s_gemm;                  // sA[kk * (GT + 1) + r] = op(A)(row0 + r, kc + kk)
    double *sB = s_gemm + GK * (GT + 1);  // sB[kk * (GT + 1) + c] = op(B)(kc + kk, col0 + c)
    constexpr int PER = GT * GK / 256;    // elements of each panel per thread
    const int tid = threadIdx.x;
    const int tx = tid % 16, ty = tid / 16;
    const int row0 = blockIdx.x * GT, col0 = blockIdx.y * GT;
    const int kz = blockIdx.z;
    const int kbeg = kz * kslice, kend = min(k, kbeg + kslice);
    double acc[2][2] = {{0, 0}, {0, 0}};
    for (int kc = kbeg; kc < kend; kc += GK) {
        double ra[PER], rb[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = tid + 256 * u;
            // A panel: contiguous along r (op = A) or along kk (op = A^T)
            int r, kk;
            if (ta) { kk = e % GK; r = e / GK; } else { r = e % GT; kk = e / GT; }
            int gr = row0 + r, gk = kc + kk;
            ra[u] = (gr < m && gk < kend) ? (ta ? A[gk + lda * gr] : A[gr + lda * gk]) : 0.0;
            // B panel: contiguous along kk (op = B) or along c (op = B^T)
            int cc, kb;
            if (tb) { cc = e % GT; kb = e / GT; } else { kb = e % GK; cc = e / GK; }
            int gc = col0 + cc, gk2 = kc + kb;
            rb[u] = (gc < n && gk2 < kend) ? (tb ? B[gc + ldb * gk2] : B[gk2 + ldb * gc]) : 0.0;
        }
        __syncthreads();  // the previous step's reads of the panels are done
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = tid + 256 * u;
            int r, kk;
            if (ta) { kk = e % GK; r = e / GK; } else { r = e % GT; kk = e / GT; }
            sA[kk * (GT + 1) + r] = ra[u];
            int cc, kb;
            if (tb) { cc = e % GT; kb = e / GT; } else { kb = e % GK; cc = e / GK; }
            sB[kb * (GT + 1) + cc] = rb[u];
        }
        __syncthreads();
        const int kn = min(GK, kend - kc);
#pragma unroll 8
        for (int kk = 0; kk < kn; ++kk) {
            const double a0 = sA[kk * (GT + 1) + tx], a1 = sA[kk * (GT + 1) + tx + 16];
            const double b0 = sB[kk * (GT + 1) + ty], b1 = sB[kk * (GT + 1) + ty + 16];
            acc[0][0] += a0 * b0;
            acc[1][0] += a1 * b0;
            acc[0][1] += a0 * b1;
            acc[1][1] += a1 * b1;
        }
    }
    for (int x = 0; x < 2; ++x)
        for (int y = 0; y < 2; ++y) {
            int r = row0 + tx + 16 * x, c = col0 + ty + 16 * y;
            if (r < m && c < n) {
                if (part) part[(int64_t)kz * m * n + r + (int64_t)m * c] = acc[x][y];
                else C[r + ldc * c] = acc[x][y];
            }
        }
}

constexpr size_t GEMM_LDS = (size_t)2 * GK * (GT + 1) * sizeof(double);

__global__ void gemm_f64_reduce_kernel(int m, int n, int nz, const double *__restrict__ part,
                                       double *__restrict__ C, int64_t ldc) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)m * n) return;
    int r = (int)(e % m), c = (int)(e / m);
    double s = 0.0;
    for (int z = 0; z < nz; ++z) s += part[(int64_t)z * m * n + e];
    C[r + ldc * c] = s;
}

size_t gemm_ws_bytes(int m, int n, int k) {
    int nz = gemm_splits(m, n, k);
    return nz > 1 ? (size_t)nz * m * n * sizeof(double) : 0;
}

// k-slices: one LDS step (GK values of k) per workgroup where the tile count
// leaves the chip idle, at most 32 slices.
int gemm_splits(int m, int n, int k) {
    const int tiles = ((m + GT - 1) / GT) * ((n + GT - 1) / GT);
    if (tiles >= 256) return 1;
    int nz = (k + GK - 1) / GK;
    nz = std::min(nz, 32);
    while (nz > 1 && tiles * nz > 1024) nz = (nz + 1) / 2;
    return std::max(nz, 1);
}

hipError_t gemm_f64(int ta, int tb, int m, int n, int k, const double *A, int64_t lda, const double *B,
                    int64_t ldb, double *C, int64_t ldc, void *ws, hipStream_t s) {
    if (m == 0 || n == 0) return hipSuccess;
    int nz = gemm_splits(m, n, k);
    int kslice = (k + nz - 1) / nz;
    kslice = (kslice + GT - 1) / GT * GT;
    if (kslice == 0) kslice = GT;
    nz = std::max(1, (k + kslice - 1) / kslice);
    dim3 grid((m + GT - 1) / GT, (n + GT - 1) / GT, nz);
    double *part = nz > 1 ? (double *)ws : nullptr;
    hipError_t ea = hipFuncSetAttribute((const void *)gemm_f64_kernel,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)GEMM_LDS);
    if (ea != hipSuccess) return ea;
    hipLaunchKernelGGL(gemm_f64_kernel, grid, dim3(256), GEMM_LDS, s, ta, tb, m, n, k, A, lda, B,
                       ldb, C, ldc, kslice, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nz == 1) return e;
    int64_t tot = (int64_t)m * n;
    hipLaunchKernelGGL(gemm_f64_reduce_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, m,
                       n, nz, part, C, ldc);
    return hipGetLastError();
}

constexpr int CHOL_THREADS = 512;

__global__ __launch_bounds__(CHOL_THREADS) void chol_kernel(const double *__restrict__ G, int n,
                                                            int64_t ldg, double shift_rel,
                                                            double *__restrict__ Rout,
                                                            double *__restrict__ Rinv,
                                                            int64_t *__restrict__ flag) {
    chol_body<CHOL_THREADS, true>(G, n, ldg, shift_rel, Rout, Rinv, flag);
}

hipError_t chol_launch(const double *G, int n, int64_t ldg, double shift_rel, double *R,
                       double *Rinv, int64_t *flag, hipStream_t s) {
    const size_t lds = chol_lds_bytes(n);
    if (lds > 64 * 1024)
        if (hipError_t ea = hipFuncSetAttribute((const void *)chol_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) return ea;
    hipLaunchKernelGGL(chol_kernel, dim3(1), dim3(CHOL_THREADS), lds, s, G, n, ldg, shift_rel, R, Rinv, flag);
    return hipGetLastError();
}

// ------------------------------------------------------------- norms ----

template <typename T>
__global__ __launch_bounds__(256) void sumsq_kernel(const T *__restrict__ x, const T *__restrict__ y,
                                                    int64_t count, double *__restrict__ part) {
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256) {
        double v = (double)x[e];
        if (y) v -= (double)y[e];
        s += v * v;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    __shared__ double sw[4];
    if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((sw[0] + sw[1]) + sw[2]) + sw[3];
}

__global__ void sum_parts_kernel(const double *__restrict__ part, int n, double *__restrict__ out,
                                 int64_t *__restrict__ flag) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += part[i];
    *out = s;
    if (flag && !(fabs(s) <= 1.7e308)) flag[0] = 3;  // NaN or Inf
}

hipError_t sumsq_launch(int dtype, const void *x, const void *y, int64_t count, double *out,
                        double *part, int64_t *flag, hipStream_t s) {
    int nb = (int)std::min<int64_t>(SUMSQ_BLOCKS, std::max<int64_t>(1, (count + 255) / 256));
    if (dtype == DT_F64)
        hipLaunchKernelGGL(sumsq_kernel<double>, dim3(nb), dim3(256), 0, s, (const double *)x,
                           (const double *)y, count, part);
    else
        hipLaunchKernelGGL(sumsq_kernel<float>, dim3(nb), dim3(256), 0, s, (const float *)x,
                           (const float *)y, count, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_parts_kernel, dim3(1), dim3(64), 0, s, part, nb, out, flag);
    return hipGetLastError();
}

// --------------------------------------------------------------- misc ----

__global__ void fill_f64_kernel(double *p, int64_t n, double v) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = v;
}

hipError_t fill_f64(double *p, int64_t n, double v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

__global__ void copy_f64_kernel(const double *src, double *dst, int64_t n) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) dst[e] = src[e];
}

hipError_t copy_f64(const double *src, double *dst, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

__global__ void zero_bytes_kernel(uint32_t *p, int64_t nwords) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nwords) p[e] = 0u;
}

hipError_t zero_words(void *p, int64_t nwords, hipStream_t s) {
    if (nwords <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_bytes_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, s,
                       (uint32_t *)p, nwords);
    return hipGetLastError();
}

// Gaussian initial guess (ALS L_0, subspace-iteration start block).
__global__ void gaussian_kernel(double *p, int64_t n, uint64_t seed, uint64_t stream) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    p[e] = gaussian_value(seed, stream, (uint64_t)e);
}

hipError_t gaussian_f64(double *p, int64_t n, uint64_t seed, uint64_t stream, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gaussian_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, seed, stream);
    return hipGetLastError();
}

}  // namespace sth
