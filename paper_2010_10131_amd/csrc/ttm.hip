// Matricization-free mode-n TTM on the gfx950 matrix cores.
//
// Computes, for a column-major tensor viewed as (L, K, M) along mode n
// (L = product of the dims before n, M = product after), the mode-n product
// with the transpose of a K x Rout factor V (Eq. 2; the core update of
// Alg. 2 and the expansion step of the Tucker reconstruction):
//
//     Z(a, r, b) = sum_k V(k, r) * Y(a, k, b)          (Z is (L, Rout, M))
//
// The loops are split at mode n into "inside" (a), "along" (k) and
// "outside" (b) as in Sec. V / Fig. 4; the (a, b) pairs are the rows of one
// GEMM with K-long rows that are strided by L in memory.  Nothing is
// transposed or copied.
//
// Design (MI355X): the kernel is HBM-bound for bf16x3 and for small Rout, so
// each Y element is read from HBM exactly once, straight into the lane that
// feeds it to the matrix cores (no LDS round trip for Y):
//   * a wave owns NT row tiles of 16 rows and RTB r-tiles of 16 columns;
//   * per 32-wide chunk of k a lane loads the 8 consecutive k of its row
//     (two 16-byte loads when L = 1, 8 strided loads otherwise), splits them
//     once into the requested precision and multiplies them against every
//     r-tile of the factor;
//   * the factor is pre-split by ttm_prep_u into matrix-core-ready 16-byte
//     quads and staged once per workgroup in LDS (read from L2 when it does
//     not fit), so the only HBM traffic is one read of Y and one write of Z;
//   * the next chunk's loads are issued before the current chunk's
//     matrix-core work (register double buffering).
#include "common.h"
#include "internal.h"
#include "ttm_body.h"

#include <mutex>

namespace sth {

// V (K x Rout) -> quads [c][rt][q][lane] (16 bytes each), zero padded.
// transpose = 0: V = U with U (K x Rout) column-major.
// transpose = 1: V = U^T with U (Rout x K) column-major.
template <int PREC>
__global__ void ttm_prep_u_kernel(const double *__restrict__ U, int64_t K, int64_t Rout,
                                  int transpose, uint4 *__restrict__ out, int nchunks,
                                  int ntiles) {
    constexpr int NQ = Frag<PREC>::NQ;
    int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t total = (int64_t)nchunks * ntiles * 64;
    if (gid >= total) return;
    int lane = (int)(gid % 64);
    int64_t blk = gid / 64;  // c * ntiles + rt
    int rt = (int)(blk % ntiles);
    int c = (int)(blk / ntiles);
    int g = lane / 16;
    int64_t r = (int64_t)rt * 16 + lane % 16;
    double x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        int64_t k = (int64_t)c * KC + 8 * g + j;
        double v = 0.0;
        if (k < K && r < Rout) v = transpose ? U[r + Rout * k] : U[k + K * r];
        x[j] = v;
    }
    FragQ<PREC> f;
    make_frag(x, f.f);
#pragma unroll
    for (int q = 0; q < NQ; ++q) out[(blk * NQ + q) * 64 + lane] = f.q[q];
}

template <typename T, int PREC, int NT, int RTB, bool CONTIG, bool ULDS, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void ttm_kernel(
    const T *__restrict__ Y, const uint4 *__restrict__ Uq, T *__restrict__ Z, int64_t L, int64_t K,
    int64_t Rout, int64_t P, int nchunks, int ntiles, int64_t nrowblocks) {
    ttm_body<T, PREC, NT, RTB, CONTIG, ULDS, WAVES>(Y, Uq, Z, L, K, Rout, P, nchunks, ntiles,
                                                    nrowblocks, blockIdx.x, gridDim.x, blockIdx.y);
}

// The TTM fused with the error sums of a reconstruction (nothing stored):
// per-workgroup sums of (X - Z)^2 and X^2 into epart.
template <typename T, int PREC, int NT, int RTB, bool CONTIG, bool ULDS, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void ttm_err_kernel(
    const T *__restrict__ Y, const uint4 *__restrict__ Uq, const T *__restrict__ X, int64_t L, int64_t K,
    int64_t Rout, int64_t P, int nchunks, int ntiles, int64_t nrowblocks, double *__restrict__ epart) {
    ttm_body<T, PREC, NT, RTB, CONTIG, ULDS, WAVES, 1, false, true>(Y, Uq, nullptr, L, K, Rout, P, nchunks, ntiles,
                                                                   nrowblocks, blockIdx.x, gridDim.x, blockIdx.y,
                                                                   X, epart);
}

// out[0], out[1] = the sums of the n (d, x) pairs: 256 threads each sum a
// strided subset in order, then a fixed tree
__global__ __launch_bounds__(256) void sum_pairs_kernel(const double *__restrict__ part, int64_t n,
                                                        double *__restrict__ out) {
    __shared__ double sa[256], sb[256];
    double a = 0.0, b = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        a += part[2 * i];
        b += part[2 * i + 1];
    }
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sa[threadIdx.x] += sa[threadIdx.x + o];
            sb[threadIdx.x] += sb[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = sa[0];
        out[1] = sb[0];
    }
}

template <typename T, int PREC, int NCH, int WAVES, bool ERR>
__global__ __launch_bounds__(64 * WAVES) void ttm_expand_kernel(
    const T *__restrict__ Y, const uint4 *__restrict__ Uq, T *__restrict__ Z, int64_t L, int64_t K, int64_t Rout,
    int64_t P, int nchunks, int ntiles, int rtn, int64_t nblocks, int64_t sa, int64_t sb,
    const T *__restrict__ X, double *__restrict__ epart) {
    ttm_expand_body<T, PREC, NCH, WAVES, ERR>(Y, Uq, Z, L, K, Rout, P, nchunks, ntiles, rtn, nblocks, sa, sb, X,
                                              epart);
}

template <typename T, int PREC, int RTB, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void ttm_stream_kernel(
    const T *__restrict__ Y, const uint4 *__restrict__ Uq, T *__restrict__ Z, int64_t L, int64_t K, int64_t Rout,
    int64_t P, int nchunks, int ntiles, int64_t nblocks, int64_t sa, int64_t sb) {
    ttm_stream_body<T, PREC, RTB, WAVES>(Y, Uq, Z, L, K, Rout, P, nchunks, ntiles, nblocks, sa, sb);
}

template <int PREC, int NT, int CPW, bool FULL>
__global__ __launch_bounds__(64 * KS_WAVES) void ttm_ks_kernel(
    const float *__restrict__ Y, const uint4 *__restrict__ Uq, float *__restrict__ Z, int64_t K,
    int64_t Rout, int64_t P, int nchunks, int ntiles, int64_t nblocks) {
    ttm_ks_body<PREC, NT, CPW, false, FULL>(Y, Uq, Z, K, Rout, P, nchunks, ntiles, nblocks, blockIdx.x,
                                            gridDim.x, blockIdx.y);
}

// Long contraction over few rows (FP64 products): the general kernel gives a
// wave 16 NT rows and the whole of K, so a first mode of 30648 entries over
// 2256 rows ran on 9 workgroups (2.2 ms for 553 MB).  Here the eight waves of
// a workgroup share 16 rows: wave w takes the chunks w, w + 8, ... (the
// workgroup streams 2 KB of each row per pass), with the next two chunks of
// rows and factor in flight, and the eight partial tiles are summed in LDS in
// wave order.  Bound by HBM with one workgroup on each of 141 of the 256 CUs:
// 2187 -> 190 us (2.9 TB/s).  FP64 accumulation only: an FP32 sum over K keeps its order.
constexpr int KW_WAVES = 8;
template <typename T, int RTB, bool CONTIG>
__global__ __launch_bounds__(64 * KW_WAVES) void ttm_kw_kernel(const T *__restrict__ Y, const uint4 *__restrict__ Uq,
                                                              T *__restrict__ Z, int64_t L, int64_t K,
                                                              int64_t Rout, int64_t P, int nchunks, int ntiles) {
    constexpr int NQ = Frag<P_FP64>::NQ;
    __shared__ f64x4 s_acc[KW_WAVES - 1][RTB][64];
    if (CONTIG) L = 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4;
    const int rt0 = blockIdx.y * RTB;
    const int64_t p = (int64_t)blockIdx.x * 16 + (lane & 15);
    const int64_t pc = p < P ? p : P - 1, b = pc / L, a = pc - b * L;
    const int64_t base = a + L * K * b;
    f64x4 acc[RTB];
#pragma unroll
    for (int rt = 0; rt < RTB; ++rt) acc[rt] = f64x4{0, 0, 0, 0};
    T x[2][8];
    FragQ<P_FP64> u[2][RTB];
    auto load = [&](int c, T (&xs)[8], FragQ<P_FP64> (&us)[RTB]) {
        ttm_load_chunk<T, CONTIG>(Y, base, L, K, (int64_t)c * KC + 8 * g, xs);
#pragma unroll
        for (int rt = 0; rt < RTB; ++rt) {
            const int rtg = rt0 + rt < ntiles ? rt0 + rt : ntiles - 1;
            const uint4 *src = Uq + (((int64_t)c * ntiles + rtg) * NQ) * 64 + lane;
#pragma unroll
            for (int q = 0; q < NQ; ++q) us[rt].q[q] = src[q * 64];
        }
    };
    auto multiply = [&](const T (&xs)[8], const FragQ<P_FP64> (&us)[RTB]) {
        Frag<P_FP64> yb;
        make_frag(xs, yb);
#pragma unroll
        for (int rt = 0; rt < RTB; ++rt) mma_frag(us[rt].f, yb, acc[rt]);
    };
    int c = wave;
    if (c < nchunks) load(c, x[0], u[0]);
    if (c + KW_WAVES < nchunks) load(c + KW_WAVES, x[1], u[1]);
    for (; c < nchunks; c += 2 * KW_WAVES) {
        multiply(x[0], u[0]);
        if (c + 2 * KW_WAVES < nchunks) load(c + 2 * KW_WAVES, x[0], u[0]);
        if (c + KW_WAVES < nchunks) {
            multiply(x[1], u[1]);
            if (c + 3 * KW_WAVES < nchunks) load(c + 3 * KW_WAVES, x[1], u[1]);
        }
    }
    if (wave > 0)
#pragma unroll
        for (int rt = 0; rt < RTB; ++rt) s_acc[wave - 1][rt][lane] = acc[rt];
    __syncthreads();
    if (wave > 0 || p >= P) return;
    const int64_t zoff = a + L * Rout * b;
#pragma unroll
    for (int rt = 0; rt < RTB; ++rt) {
#pragma unroll
        for (int w = 0; w < KW_WAVES - 1; ++w) acc[rt] += s_acc[w][rt][lane];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t r = (int64_t)(rt0 + rt) * 16 + drow<P_FP64>(g, v);
            if (r < Rout) Z[zoff + L * r] = (T)acc[rt][v];
        }
    }
}

// Scratch for callers that cannot allocate (ttm_mode_n_noalloc): the
// pre-split factor of one call lives here instead of in a caller workspace.
// Each device that runs the library holds its own copy until the process
// ends.  Host code must never pass `scratch` itself to a kernel (on the host
// it names a stand-in, not a device address); it uses the address that
// ttm_scratch_ptr() looked up for the current device.
constexpr size_t TTM_SCRATCH_BYTES = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[TTM_SCRATCH_BYTES];

// ---------------------------------------------------------------- host ----

size_t ttm_prep_bytes(int64_t K, int64_t Rout, int prec) {
    int64_t nchunks = (K + KC - 1) / KC;
    int64_t ntiles = (Rout + 15) / 16;
    return (size_t)(nchunks * ntiles * 64 * 16 * prec_nq(prec));
}

size_t ttm_scratch_bytes() { return TTM_SCRATCH_BYTES; }

// Device address of `scratch` on the current device, looked up once per
// device with that device current and kept for later calls.
hipError_t ttm_scratch_ptr(void **out) {
    static std::mutex mu;
    static void *addr[64] = {nullptr};
    *out = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

hipError_t ttm_prep_u(const double *U, int64_t K, int64_t Rout, int transpose, int prec,
                      void *out, hipStream_t s) {
    int nchunks = (int)((K + KC - 1) / KC);
    int ntiles = (int)((Rout + 15) / 16);
    int64_t total = (int64_t)nchunks * ntiles * 64;
    dim3 grid((unsigned)((total + 255) / 256));
    uint4 *o = (uint4 *)out;
    switch (prec) {
        case P_FP64: hipLaunchKernelGGL(ttm_prep_u_kernel<P_FP64>, grid, dim3(256), 0, s, U, K, Rout, transpose, o, nchunks, ntiles); break;
        case P_FP32: hipLaunchKernelGGL(ttm_prep_u_kernel<P_FP32>, grid, dim3(256), 0, s, U, K, Rout, transpose, o, nchunks, ntiles); break;
        case P_BF16X3: hipLaunchKernelGGL(ttm_prep_u_kernel<P_BF16X3>, grid, dim3(256), 0, s, U, K, Rout, transpose, o, nchunks, ntiles); break;
        default: hipLaunchKernelGGL(ttm_prep_u_kernel<P_BF16X6>, grid, dim3(256), 0, s, U, K, Rout, transpose, o, nchunks, ntiles); break;
    }
    return hipGetLastError();
}

namespace {

constexpr int TTM_WAVES = 8;
constexpr size_t TTM_LDS_MAX = 144 * 1024;
constexpr int64_t TTM_ERR_WGS = 1024;   // fused error sums: workgroups per r-block at most (few partial sums)

template <typename T, int PREC, int NT, int RTB, bool CONTIG, bool ULDS>
hipError_t launch_ttm_t(const T *Y, const uint4 *Uq, T *Z, int64_t L, int64_t K, int64_t Rout,
                        int64_t M, hipStream_t s) {
    const int64_t P = L * M;
    const int nchunks = (int)((K + KC - 1) / KC);
    const int ntiles = (int)((Rout + 15) / 16);
    const int nrb = (ntiles + RTB - 1) / RTB;
    const int64_t nrowblocks = (P + 16 * NT - 1) / (16 * NT);
    const size_t lds = ULDS ? (size_t)nchunks * RTB * Frag<PREC>::NQ * 64 * 16 : 0;
    int64_t wgs = (nrowblocks + TTM_WAVES - 1) / TTM_WAVES;
    const int per_cu = ULDS ? (int)std::max<size_t>(1, std::min<size_t>(2, (160 * 1024) / std::max<size_t>(lds, 1))) : 2;
    const int64_t cap = (int64_t)device_cu_count() * per_cu;
    if (ULDS && wgs > cap) wgs = cap;  // persistent: amortize the factor staging
    if (wgs < 1) wgs = 1;
    auto kern = ttm_kernel<T, PREC, NT, RTB, CONTIG, ULDS, TTM_WAVES>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs, (unsigned)nrb), dim3(64 * TTM_WAVES), lds, s, Y, Uq,
                       Z, L, K, Rout, P, nchunks, ntiles, nrowblocks);
    return hipGetLastError();
}

template <int PREC, int CPW>
hipError_t launch_ttm_ks(const float *Y, const uint4 *Uq, float *Z, int64_t K, int64_t Rout, int64_t M,
                         hipStream_t s) {
    constexpr int NT = 2;
    const int nchunks = (int)((K + KC - 1) / KC);
    const int ntiles = (int)((Rout + 15) / 16);
    const int nrb = (ntiles + 3) / 4;
    const int64_t nblocks = (M + 16 * NT - 1) / (16 * NT);
    const size_t lds = ttm_ks_lds(NT);
    const int64_t wgs = std::max<int64_t>(1, std::min<int64_t>(nblocks, (int64_t)device_cu_count()));
    // whole chunks for every wave: the branch-free kernel
    auto kern = (K == (int64_t)KS_WAVES * CPW * KC) ? ttm_ks_kernel<PREC, NT, CPW, true>
                                                    : ttm_ks_kernel<PREC, NT, CPW, false>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs, (unsigned)nrb), dim3(64 * KS_WAVES), lds, s, Y, Uq, Z, K,
                       Rout, M, nchunks, ntiles, nblocks);
    return hipGetLastError();
}

// Strided rows in 16-byte vectors: L a multiple of the vector, aligned tensors.
template <typename T>
bool ttm_vec_ok(const void *Y, const void *Z, int64_t L) {
    return L > 1 && L % (16 / (int64_t)sizeof(T)) == 0 &&
           ((reinterpret_cast<uintptr_t>(Y) | reinterpret_cast<uintptr_t>(Z)) & 15) == 0;
}

// Grid of the vector kernels: row blocks of 16 V rows over the waves of at most
// `cap` workgroups, and the (a, b) step from a wave's block to its next.
template <typename T>
struct VecGrid {
    int64_t nblocks, wgs, sa, sb;
    VecGrid(int64_t L, int64_t P, int waves, int64_t cap) {
        constexpr int64_t V = 16 / sizeof(T);
        nblocks = (P + 16 * V - 1) / (16 * V);
        wgs = std::max<int64_t>(1, std::min<int64_t>((nblocks + waves - 1) / waves, cap));
        const int64_t d = wgs * waves * 16 * V;
        sb = d / L;
        sa = d - sb * L;
    }
};

// Chunks whose fragments the expansion kernel keeps in registers (0: too many)
template <typename T, int PREC>
constexpr int expand_chunks() { return PREC == P_FP64 && sizeof(T) == 4 ? 1 : 2; }

// Where the expansion kernel serves: contractions of its chunks, but for FP64 data
// in two chunks between one and eight waves per CU, where the streaming kernel
// spreads the r-tiles better (50 -> 200 over 30400 rows: 37 us, 30), and the
// general kernel's error sums the rows (100^3 from 50^3: 47 us, 42).
template <typename T, int PREC>
bool use_expand(int64_t P, int nchunks) {
    if (nchunks > expand_chunks<T, PREC>()) return false;
    const int64_t cu = device_cu_count(), nblocks = (P + 31) / 32;   // FP64 data: blocks of 32 rows
    return !(sizeof(T) == 8 && nchunks == 2 && nblocks > cu && nblocks < 8 * cu);
}

// The expansion kernel (K <= 64): every r-tile from one read of Y where their
// factor quads fit the LDS, equal ranges of r-tiles otherwise.  ERR: part takes one
// pair of sums per workgroup; *nparts, its length, is set to their number.
template <typename T, int PREC, bool ERR>
hipError_t launch_expand(const T *Y, const uint4 *Uq, T *Z, int64_t L, int64_t K, int64_t Rout, int64_t M,
                         const T *X, double *part, int64_t *nparts, hipStream_t s) {
    constexpr int NQ = Frag<PREC>::NQ;
    const int64_t P = L * M, cu = device_cu_count();
    const int nchunks = (int)((K + KC - 1) / KC), ntiles = (int)((Rout + 15) / 16);
    // Few row blocks (less than eight waves per CU): two waves a workgroup, ranges
    // of r-tiles of at most 32 KB, so that every CU has several workgroups, and
    // enough ranges for eight waves per CU (Y, at most some tens of MB, is read
    // again from the caches).  50 -> 200 over 5000 rows in FP32: 14.4 us with as
    // many tiles in a range as fit, 7.0 so (the general kernel 11.3); 20 -> 336 over
    // 30400: 21.8, 17.1 (19.8).
    const int64_t nblocks = (P + 16 * (16 / sizeof(T)) - 1) / (16 * (16 / sizeof(T)));
    const bool few = nblocks < 8 * cu;
    const int fit = (int)((few ? 32 * 1024 : TTM_LDS_MAX) / ((size_t)nchunks * NQ * 1024));
    const int64_t waves = few ? 2 : TTM_WAVES, max_wgs = ERR ? std::min<int64_t>(4 * cu, TTM_ERR_WGS) : 4 * cu;
    int64_t ranges = few ? std::min<int64_t>(ntiles, 8 * cu / nblocks) : 1;
    if (ERR) ranges = std::max<int64_t>(1, std::min<int64_t>(ranges, *nparts / std::min((nblocks + 1) / 2, max_wgs)));
    int rtn = (int)std::min<int64_t>((ntiles + ranges - 1) / ranges, fit);
    int64_t nrb = (ntiles + rtn - 1) / rtn;
    rtn = (int)((ntiles + nrb - 1) / nrb);
    const size_t lds = (size_t)nchunks * rtn * NQ * 1024;
    const int64_t per_cu = lds <= 72 * 1024 ? 2 : 1;
    const VecGrid<T> vg(L, P, (int)waves, few ? max_wgs : cu * per_cu);
    if (ERR) *nparts = vg.wgs * nrb;
    const dim3 grid((unsigned)vg.wgs, (unsigned)nrb);
    auto go = [&](auto kern) -> hipError_t {
        if (lds > 64 * 1024) {
            hipError_t r = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (r != hipSuccess) return r;
        }
        hipLaunchKernelGGL(kern, grid, dim3((unsigned)(64 * waves)), lds, s, Y, Uq, Z, L, K, Rout, P, nchunks, ntiles, rtn,
                           vg.nblocks, vg.sa, vg.sb, X, part);
        return hipGetLastError();
    };
    if (few) {
        if constexpr (expand_chunks<T, PREC>() == 2) {
            if (nchunks == 2) return go(ttm_expand_kernel<T, PREC, 2, 2, ERR>);
        }
        return go(ttm_expand_kernel<T, PREC, 1, 2, ERR>);
    }
    if constexpr (expand_chunks<T, PREC>() == 2) {
        if (nchunks == 2) return go(ttm_expand_kernel<T, PREC, 2, TTM_WAVES, ERR>);
    }
    return go(ttm_expand_kernel<T, PREC, 1, TTM_WAVES, ERR>);
}

template <typename T, int PREC, int RTB, int WAVES>
hipError_t launch_stream_w(const T *Y, const uint4 *Uq, T *Z, int64_t L, int64_t K, int64_t Rout, int64_t M,
                           hipStream_t s) {
    const int64_t P = L * M;
    const int nchunks = (int)((K + KC - 1) / KC), ntiles = (int)((Rout + 15) / 16);
    const size_t lds = (size_t)nchunks * RTB * Frag<PREC>::NQ * 1024;
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(16 / WAVES, (160 * 1024) / (int64_t)lds));
    const VecGrid<T> vg(L, P, WAVES, (int64_t)device_cu_count() * per_cu);
    auto kern = ttm_stream_kernel<T, PREC, RTB, WAVES>;
    if (lds > 64 * 1024) {
        hipError_t r = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (r != hipSuccess) return r;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)vg.wgs, (unsigned)((ntiles + RTB - 1) / RTB)), dim3(64 * WAVES), lds,
                       s, Y, Uq, Z, L, K, Rout, P, nchunks, ntiles, vg.nblocks, vg.sa, vg.sb);
    return hipGetLastError();
}

// Waves per workgroup of the streaming kernel, 0 where the general kernel (half the
// rows per wave, two workgroups per CU) takes over.  w8 are the workgroups of eight
// waves and all RTB r-tiles, which read Y once:
//   * from half a workgroup per CU on they are the fastest form up to one per CU
//     (512 x 64 in bf16x3, 131 K rows on 255 workgroups: 59 us, 65 in the general
//     kernel, 113 with the r-tiles dealt two by two to four waves, which reads Y
//     twice);
//   * beyond, while the last round of workgroups is full enough: 2200 blocks of 64
//     rows (275 workgroups) in FP32 148 us, general kernel 131; 5000 blocks 221
//     and 221, in bf16x3 154 and 160.  One r-tile gains everywhere;
//   * below, fewer waves and r-tiles spread the rows over the CUs (512 x 16 in
//     FP32, 16 K rows: 39 us in the general kernel, 17).  With several r-tiles that
//     reads Y again for each part, which pays where the products are slow (FP32,
//     512 x 64, 64 K rows: 49.5 us, general 52.4) or Y small; else not (bf16x3,
//     520 blocks of 64 rows: 34 us, 25).
// FP64 products of FP32 data: only where full (300 x 20, 19 K rows: 30 us in four
// waves, 17 in the general kernel) or over few chunks of one r-tile (128 x 16, 16 K
// rows: 8.7 and 9.2 us; 512 x 8, 13 K rows: 35 and 28).
template <typename T, int PREC, int RTB>
int stream_waves(int64_t P, int64_t Rout, int nchunks) {
    constexpr bool WIDEN = PREC == P_FP64 && sizeof(T) == 4;
    constexpr int64_t ROWS = 16 * (16 / sizeof(T));
    const int64_t cu = device_cu_count(), nblocks = (P + ROWS - 1) / ROWS;
    const int64_t nrb = ((Rout + 15) / 16 + RTB - 1) / RTB, w8 = (nblocks + 7) / 8 * nrb;
    if (2 * w8 > cu) {
        if (w8 <= cu) return WIDEN && RTB == 2 ? 0 : 8;
        const bool full = 20 * w8 >= 17 * cu * ((w8 + cu - 1) / cu);
        return full || (RTB == 1 && !WIDEN) ? 8 : 0;
    }
    const int narrow = nblocks >= cu ? 4 : 2;
    if (WIDEN) return RTB == 1 && nchunks <= 4 ? narrow : 0;
    if (RTB == 1 || PREC == P_FP32) return narrow;
    return nblocks < cu || (RTB == 4 && nblocks * nrb <= 2 * cu) ? narrow : 0;
}

template <typename T, int PREC, int RTB>
hipError_t launch_stream(int waves, const T *Y, const uint4 *Uq, T *Z, int64_t L, int64_t K, int64_t Rout, int64_t M,
                         hipStream_t s) {
    if (waves == 8) return launch_stream_w<T, PREC, RTB, 8>(Y, Uq, Z, L, K, Rout, M, s);
    if (waves == 4) return launch_stream_w<T, PREC, (RTB < 2 ? RTB : 2), 4>(Y, Uq, Z, L, K, Rout, M, s);
    return launch_stream_w<T, PREC, 1, 2>(Y, Uq, Z, L, K, Rout, M, s);
}

template <typename T, int PREC, int RTB>
hipError_t launch_ttm_r(const T *Y, const uint4 *Uq, T *Z, int64_t L, int64_t K, int64_t Rout,
                        int64_t M, hipStream_t s) {
    const int nchunks = (int)((K + KC - 1) / KC);
    const size_t lds = (size_t)nchunks * RTB * Frag<PREC>::NQ * 64 * 16;
    const bool contig = (L == 1) && (K % (16 / sizeof(T)) == 0) &&
                        ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
    // contiguous rows of 256 < K <= 512 values in FP32 storage: the K-split
    // kernel (all eight waves busy, whole row blocks streamed)
    if constexpr (sizeof(T) == 4 && (PREC == P_FP32 || PREC == P_BF16X3) && RTB == 4) {
        const int nchunks = (int)((K + KC - 1) / KC);
        if (contig && nchunks > 8 && nchunks <= 16)
            return launch_ttm_ks<PREC, 2>(reinterpret_cast<const float *>(Y), Uq, reinterpret_cast<float *>(Z),
                                          K, Rout, M, s);
    }
    if constexpr (PREC == P_FP64) {
        // few rows and a long contraction: the eight waves of a workgroup split
        // K (at least four chunks each) where the general kernel would leave many
        // CUs without a workgroup (times against it, by its workgroups):
        //   contiguous rows: K = 1000, R = 33 188 0.97, 235 1.26; K = 4000 235 0.90;
        //   strided rows cost the split more (a lane's rows are not whole lines):
        //   K = 1000, R = 100 142 1.07; K = 8000 188 0.96; one range of several
        //   r-tiles, K = 2000 157 0.84, 188 1.04; FP64 data, one r-tile, K = 1000
        //   47 0.80, 94 1.45
        constexpr int NTG = RTB == 1 ? 2 : 1;
        const int64_t P = L * M, ntiles = (Rout + 15) / 16, nrb = (ntiles + RTB - 1) / RTB, cu = device_cu_count();
        const bool many_chunks = nchunks >= 12 * KW_WAVES;
        int64_t limit;   // workgroups of the general kernel, below which the split is taken
        if (contig) limit = many_chunks ? cu : 3 * cu / 4;
        else if (many_chunks) limit = 3 * cu / 4;
        else if (RTB > 1 && nrb == 1) limit = 5 * cu / 8;
        else limit = sizeof(T) == 8 && RTB == 1 && nchunks < 6 * KW_WAVES ? cu / 4 : cu / 2;
        if (nchunks >= 4 * KW_WAVES && (P + 16 * NTG * TTM_WAVES - 1) / (16 * NTG * TTM_WAVES) * nrb < limit) {
            const dim3 grid((unsigned)((P + 15) / 16), (unsigned)nrb);
            if (contig)
                hipLaunchKernelGGL((ttm_kw_kernel<T, RTB, true>), grid, dim3(64 * KW_WAVES), 0, s, Y, Uq, Z, L, K,
                                   Rout, P, nchunks, (int)ntiles);
            else
                hipLaunchKernelGGL((ttm_kw_kernel<T, RTB, false>), grid, dim3(64 * KW_WAVES), 0, s, Y, Uq, Z, L, K,
                                   Rout, P, nchunks, (int)ntiles);
            return hipGetLastError();
        }
    }
    if (ttm_vec_ok<T>(Y, Z, L)) {
        if (use_expand<T, PREC>(L * M, nchunks))
            return launch_expand<T, PREC, false>(Y, Uq, Z, L, K, Rout, M, nullptr, nullptr, nullptr, s);
        // FP64 accumulators of four tiles x four rows do not fit the registers
        if constexpr (!(PREC == P_FP64 && sizeof(T) == 4 && RTB == 4)) {
            const int waves = lds <= TTM_LDS_MAX ? stream_waves<T, PREC, RTB>(L * M, Rout, nchunks) : 0;
            if (waves) return launch_stream<T, PREC, RTB>(waves, Y, Uq, Z, L, K, Rout, M, s);
        }
    }
    // row tiles per wave: keeps a lane under 256 VGPRs (8 waves per workgroup)
    constexpr int NT = (PREC == P_FP64) ? (RTB == 1 ? 2 : 1) : (RTB == 1 ? 4 : 2);
    if (lds <= TTM_LDS_MAX) {
        if (contig) return launch_ttm_t<T, PREC, NT, RTB, true, true>(Y, Uq, Z, L, K, Rout, M, s);
        return launch_ttm_t<T, PREC, NT, RTB, false, true>(Y, Uq, Z, L, K, Rout, M, s);
    }
    if (contig) return launch_ttm_t<T, PREC, NT, RTB, true, false>(Y, Uq, Z, L, K, Rout, M, s);
    return launch_ttm_t<T, PREC, NT, RTB, false, false>(Y, Uq, Z, L, K, Rout, M, s);
}

template <typename T, int PREC>
hipError_t launch_ttm_p(const T *Y, const uint4 *Uq, T *Z, int64_t L, int64_t K, int64_t Rout,
                        int64_t M, hipStream_t s) {
    const int64_t ntiles = (Rout + 15) / 16;
    if (ntiles <= 1) return launch_ttm_r<T, PREC, 1>(Y, Uq, Z, L, K, Rout, M, s);
    if (ntiles <= 2) return launch_ttm_r<T, PREC, 2>(Y, Uq, Z, L, K, Rout, M, s);
    return launch_ttm_r<T, PREC, 4>(Y, Uq, Z, L, K, Rout, M, s);
}

// ---- the TTM fused with the reconstruction error ----

int ttm_err_rtb(int64_t Rout) {
    const int64_t ntiles = (Rout + 15) / 16;
    return ntiles <= 1 ? 1 : (ntiles <= 2 ? 2 : 4);
}

template <typename T, int PREC, int RTB>
hipError_t launch_ttm_err_r(const T *Y, const uint4 *Uq, const T *X, int64_t L, int64_t K, int64_t Rout,
                            int64_t M, double *part, double *out, hipStream_t s) {
    constexpr int NT = (PREC == P_FP64) ? (RTB == 1 ? 2 : 1) : (RTB == 1 ? 4 : 2);
    const int64_t P = L * M;
    const int nchunks = (int)((K + KC - 1) / KC);
    const int ntiles = (int)((Rout + 15) / 16);
    const int nrb = (ntiles + RTB - 1) / RTB;
    const int64_t nrowblocks = (P + 16 * NT - 1) / (16 * NT);
    const size_t lds = (size_t)nchunks * RTB * Frag<PREC>::NQ * 64 * 16;
    const bool ulds = lds <= TTM_LDS_MAX;
    int64_t wgs = std::min<int64_t>(TTM_ERR_WGS, (nrowblocks + TTM_WAVES - 1) / TTM_WAVES);
    if (ulds) {
        const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(2, (160 * 1024) / std::max<size_t>(lds, 1)));
        wgs = std::min<int64_t>(wgs, (int64_t)device_cu_count() * per_cu);
    }
    if (wgs < 1) wgs = 1;
    const bool contig = L == 1;
    hipError_t e;
    auto go = [&](auto kern, size_t lb) -> hipError_t {
        if (lb > 64 * 1024) {
            hipError_t r = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lb);
            if (r != hipSuccess) return r;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)wgs, (unsigned)nrb), dim3(64 * TTM_WAVES), lb, s, Y, Uq, X, L, K,
                           Rout, P, nchunks, ntiles, nrowblocks, part);
        return hipGetLastError();
    };
    if (ulds) e = contig ? go(ttm_err_kernel<T, PREC, NT, RTB, true, true, TTM_WAVES>, lds)
                         : go(ttm_err_kernel<T, PREC, NT, RTB, false, true, TTM_WAVES>, lds);
    else e = contig ? go(ttm_err_kernel<T, PREC, NT, RTB, true, false, TTM_WAVES>, 0)
                    : go(ttm_err_kernel<T, PREC, NT, RTB, false, false, TTM_WAVES>, 0);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_pairs_kernel, dim3(1), dim3(256), 0, s, part, wgs * nrb, out);
    return hipGetLastError();
}

template <typename T, int PREC>
hipError_t launch_ttm_err_p(const T *Y, const uint4 *Uq, const T *X, int64_t L, int64_t K, int64_t Rout,
                            int64_t M, double *part, double *out, hipStream_t s) {
    const int nchunks = (int)((K + KC - 1) / KC);
    // where the factor fits the LDS in one range
    if (ttm_vec_ok<T>(Y, X, L) && use_expand<T, PREC>(L * M, nchunks) &&
        (size_t)nchunks * ((Rout + 15) / 16) * Frag<PREC>::NQ * 1024 <= TTM_LDS_MAX) {
        int64_t np = (int64_t)(ttm_err_part_doubles(Rout) / 2);
        hipError_t e = launch_expand<T, PREC, true>(Y, Uq, nullptr, L, K, Rout, M, X, part, &np, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(sum_pairs_kernel, dim3(1), dim3(256), 0, s, part, np, out);
        return hipGetLastError();
    }
    switch (ttm_err_rtb(Rout)) {
        case 1: return launch_ttm_err_r<T, PREC, 1>(Y, Uq, X, L, K, Rout, M, part, out, s);
        case 2: return launch_ttm_err_r<T, PREC, 2>(Y, Uq, X, L, K, Rout, M, part, out, s);
        default: return launch_ttm_err_r<T, PREC, 4>(Y, Uq, X, L, K, Rout, M, part, out, s);
    }
}

}  // namespace

size_t ttm_err_part_doubles(int64_t Rout) {
    const int64_t ntiles = (Rout + 15) / 16, rtb = ttm_err_rtb(Rout);
    return (size_t)(2 * TTM_ERR_WGS * ((ntiles + rtb - 1) / rtb));
}

hipError_t ttm_err_launch(int dtype, int prec, const void *Y, const void *Uq, const void *X, int64_t L, int64_t K,
                          int64_t Rout, int64_t M, double *part, double *out, hipStream_t s) {
    const uint4 *uq = (const uint4 *)Uq;
    if (dtype == DT_F64)
        return launch_ttm_err_p<double, P_FP64>((const double *)Y, uq, (const double *)X, L, K, Rout, M, part, out, s);
    const float *y = (const float *)Y, *x = (const float *)X;
    switch (prec) {
        case P_FP64: return launch_ttm_err_p<float, P_FP64>(y, uq, x, L, K, Rout, M, part, out, s);
        case P_FP32: return launch_ttm_err_p<float, P_FP32>(y, uq, x, L, K, Rout, M, part, out, s);
        case P_BF16X3: return launch_ttm_err_p<float, P_BF16X3>(y, uq, x, L, K, Rout, M, part, out, s);
        default: return launch_ttm_err_p<float, P_BF16X6>(y, uq, x, L, K, Rout, M, part, out, s);
    }
}

hipError_t ttm_launch(int dtype, int prec, const void *Y, const void *Uq, void *Z, int64_t L,
                      int64_t K, int64_t Rout, int64_t M, hipStream_t s) {
    if (L * M == 0 || Rout == 0) return hipSuccess;
    const uint4 *uq = (const uint4 *)Uq;
    if (dtype == DT_F64) {
        return launch_ttm_p<double, P_FP64>((const double *)Y, uq, (double *)Z, L, K, Rout, M, s);
    }
    const float *y = (const float *)Y;
    float *z = (float *)Z;
    switch (prec) {
        case P_FP64: return launch_ttm_p<float, P_FP64>(y, uq, z, L, K, Rout, M, s);
        case P_FP32: return launch_ttm_p<float, P_FP32>(y, uq, z, L, K, Rout, M, s);
        case P_BF16X3: return launch_ttm_p<float, P_BF16X3>(y, uq, z, L, K, Rout, M, s);
        default: return launch_ttm_p<float, P_BF16X6>(y, uq, z, L, K, Rout, M, s);
    }
}

}  // namespace sth
