// Matricization-free mode-n Gram and TTT on the gfx950 matrix cores.
//
//   S(i, j) = sum_{a, b} A(a, i, b) * B(a, j, b)
//
// with A viewed as (L, IA, M) and B as (L, IB, M) along mode n.  B = A gives
// the Gram matrix Y_(n) Y_(n)^T of the EIG branch (Alg. 2); a different B
// gives the TTT of Eq. 3 (read as a contraction over every mode but n) used
// by the ALS branch.  The contraction runs over the P = L*M rows (a, b) in
// place, as the paper's "series of GEMMs accumulated into one result"
// (Sec. V), without forming X_(n).
//
// Design (MI355X):
//   * output blocks of TB x TB (TB = 32 * WT), 4 waves per workgroup in a
//     2 x 2 arrangement, each wave WT x WT tiles of 16 x 16;
//   * split-K over P: each workgroup owns one output block and one range of
//     rows; blocks of the same row range are mapped to the same XCD so the
//     re-reads of a row range across blocks hit that XCD's L2, not HBM;
//   * per 32-row chunk the workgroup loads its A (and B) slab with coalesced
//     reads (lanes along i when L = 1, along a otherwise), converts every
//     element once to the requested precision and stores it in LDS already
//     in matrix-core fragment layout; the next chunk's loads are in flight
//     while the current chunk is multiplied;
//   * FP32 (or bf16-split) products accumulate in FP32 for FLUSH chunks and
//     are then added into FP64 registers; workgroups write FP64 partial
//     blocks and a second kernel reduces them in a fixed order
//     (deterministic), mirroring the lower triangle for the Gram.
#include "common.h"
#include "gram_body.h"
#include "internal.h"

namespace sth {

template <typename T, int PREC, int WT, bool SYM, bool FIBRES>
__global__ __launch_bounds__(256) void gram_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                   int64_t L, int64_t IA, int64_t IB, int64_t P,
                                                   int64_t kper, int nkc, int nbi, int nbj,
                                                   int nblocks, int64_t total_wg,
                                                   double *__restrict__ partials) {
    gram_body<T, PREC, WT, SYM, FIBRES>(A, B, L, IA, IB, P, kper, nkc, nbi, nbj, nblocks, total_wg,
                                xcd_logical_id(total_wg), partials);
}

// TB = 32 * WT.  With WT = 4 the block runs eight waves of 64 x 32 each
// (2 x 4 grid): a wave's FP32 accumulators and their FP64 partial sums then
// stay in its own registers (four waves of 64 x 64 need more than a wave's
// 256 registers and shuttle them through the accumulation registers every
// chunk); measured on the 512-wide Gram: FP32 products 1.36x, bf16x3 1.5x
// faster than four waves.
template <int PREC, int WT>
constexpr bool gram_l1_eight_waves() { return WT == 4; }

template <int PREC, int WT, bool FULLI>
__global__ __launch_bounds__((gram_l1_eight_waves<PREC, WT>() ? 512 : 256)) void gram_l1_kernel(
    const float *__restrict__ Y, int64_t I, int64_t P, int64_t kper, int nkc, int nblocks,
    int64_t total_wg, double *__restrict__ partials) {
    if constexpr (gram_l1_eight_waves<PREC, WT>())
        gram_l1_body<PREC, 4, 2, 2, 4, FULLI>(Y, I, P, kper, nkc, nblocks, total_wg,
                                                    xcd_logical_id(total_wg), partials);
    else
        gram_l1_body<PREC, WT, WT, 2, 2, FULLI>(Y, I, P, kper, nkc, nblocks, total_wg,
                                                      xcd_logical_id(total_wg), partials);
}

template <int PREC, int CH, bool QUAD, int MS>
__global__ __launch_bounds__(SK_T) void gram_skinny_kernel(const float *__restrict__ Y, int I, int64_t P,
                                                          int nkc, double *__restrict__ partials) {
    gram_skinny_body<PREC, CH, QUAD, MS>(Y, I, P, nkc, blockIdx.x, partials);
}

// ---- FP64 products, I <= 160: the lower triangle in 16 x 16 tiles -----------
// One workgroup per CU walks row blocks of SC rows (dealt round-robin, so that
// the chip streams one region), staged in LDS as they are in memory: i fastest
// when L = 1 (one contiguous run), each column's SC rows otherwise.  The waves
// share the 32 x 32 super tiles of the lower triangle (two of 16 x 16 a side, the
// upper one of a diagonal super tile left out), MS each at most; where there are
// fewer than waves, ks groups of waves split a block's rows and are summed at the
// end.  Two stages of loads are in flight, of at most TRI_STAGE values each: a
// stage costs a barrier and a trip through LDS whatever it holds, so short rows
// take more of them at a time (see tri_sc).  Float data is widened as it is stored
// (widened as it is read, once per tile and step, 160^4's first mode took 3.2 ms:
// the conversions and the products share the FP64 units).
//
// Bound from I of about 100 on by the FP64 matrix cores (64 cycles a 16 x 16 x 4
// product) and the staging that follows a stage's products, below by the reading
// of Y.  160^4's first mode, 4.1 M rows: 2.16 ms (1.6 ms of products on the fullest
// SIMD), 2.45 in the skinny body, whose loading waves widen and sort fragments
// beside their products.  The later modes, I = 160 with L = 16, 256, ..: 290 us
// together, 967 in 128 x 128 blocks, which pad the triangle of 55 tiles to 160.  64^3 double: 8 us a mode, 20 in one block of 64
// and few workgroups.
constexpr int TRI_T = 512, TRI_W = TRI_T / 64;
constexpr int TRI_SC = 32;      // rows of a stage at least
constexpr int TRI_MAXI = 160;   // 15 super tiles: two per wave
constexpr int TRI_STAGE = TRI_MAXI * TRI_SC;   // values of a stage at most

typedef double f64x2 __attribute__((ext_vector_type(2)));

// doubles of a stage (even; reads of the rows beyond I stay within)
__host__ __device__ inline int tri_stage(int I, int sc, bool flat) {
    return flat ? (I * sc + 34) / 2 * 2 : 32 * ((I + 31) / 32) * (sc + 2);
}

template <typename T, int MS, int SC, bool FLAT>
__global__ __launch_bounds__(TRI_T) void gram_tri64_kernel(const T *__restrict__ Y, int64_t L, int I, int64_t P,
                                                          int ks, int nkc, double *__restrict__ partials) {
    constexpr int VE = 16 / sizeof(T);
    constexpr int NV = (TRI_STAGE / VE + TRI_T - 1) / TRI_T;   // 16-byte vectors per thread and stage
    constexpr int LDP = SC + 2;
    typedef T vec_t __attribute__((ext_vector_type(VE)));
    extern __shared__ __align__(16) char s_tri[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tr = lane & 15, tg = lane >> 4;
    const int ns = ((I + 15) / 16 + 1) / 2, nss = ns * (ns + 1) / 2, noff = nss - ns;
    const int gw = TRI_W / ks, wg = wave % gw, gk = wave / gw;   // wave of its group, group
    // element (row i, k of the stage) at i * rs + k * cs
    const int rs = FLAT ? 1 : LDP, cs = FLAT ? I : 1;
    const int stage_e = tri_stage(I, SC, FLAT);
    double *s_st = reinterpret_cast<double *>(s_tri);

    // super tiles off the diagonal first (four products a step), then those on it
    // (three); -1: none
    int q[MS], oa[MS], ob[MS];
    bool diag[MS];
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        const int u = wg + gw * m;
        int bi = 0, bj = 0;
        diag[m] = u >= noff;
        if (u < noff) {   // (1, 0), (2, 0), (2, 1), ..
            bi = 1;
            while (bi * (bi + 1) / 2 <= u) ++bi;
            bj = u - bi * (bi - 1) / 2;
        } else if (u < nss) {
            bi = bj = u - noff;
        }
        q[m] = u < nss ? bi * (bi + 1) / 2 + bj : -1;
        oa[m] = (32 * bi + tr) * rs + tg * cs;
        ob[m] = (32 * bj + tr) * rs + tg * cs;
    }
    f64x4 acc[MS][2][2];
#pragma unroll
    for (int m = 0; m < MS; ++m)
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[m][x >> 1][x & 1] = f64x4{0.0, 0.0, 0.0, 0.0};

    const int64_t nblk = (P + SC - 1) / SC;
    const int kc = blockIdx.x;
    const int nst = kc < nblk ? (int)((nblk - 1 - kc) / nkc + 1) : 0;
    // L > 1: this thread's rows p of a block (the same for all its vectors) and
    // their place in the tensor, carried from stage to stage
    const int vr = SC / VE, pv = VE * (tid % vr), row0 = tid / vr, rstep = TRI_T / vr;
    const int64_t step = (int64_t)SC * nkc, qs = FLAT ? 0 : step / L, r_s = FLAT ? 0 : step - qs * L;
    int64_t pb = 0, pa = 0;
    if (!FLAT) {
        const int64_t p = (int64_t)kc * SC + pv;
        pb = p / L;
        pa = p - pb * L;
    }
    vec_t raws[2][NV];   // two stages in flight
    // the loads alone, unmasked and unconditional (clamped places): a branch or a
    // select here would wait for them before the stage in hand is multiplied.  A
    // thread's vectors past the stage repeat its last one, or row I - 1 (read on, they
    // would fetch other workgroups' rows: 10 times the bytes at I = 16).
    const int64_t count = P * I;
    auto load = [&](int st, vec_t (&raw)[NV]) {
        const int64_t p0 = ((int64_t)st * nkc + kc) * SC, last = min(count, (p0 + SC) * I) - VE;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            if constexpr (FLAT) {
                const int64_t e = p0 * I + VE * (tid + TRI_T * u);
                __builtin_memcpy(&raw[u], Y + min(e, last), 16);
            } else {
                const int row = min(row0 + rstep * u, I - 1);
                __builtin_memcpy(&raw[u], Y + L * row + (p0 + pv < P ? pa + L * I * pb : 0), 16);
            }
        }
        if constexpr (!FLAT) {
            pa += r_s;
            pb += qs;
            if (pa >= L) {
                pa -= L;
                ++pb;
            }
        }
    };
    auto store = [&](int st, vec_t (&raw)[NV]) {
        const int64_t p0 = ((int64_t)st * nkc + kc) * SC;
        double *d = s_st + (st & 1) * stage_e;
        if (p0 + SC > P) {   // the last block of rows: zeroes past the end
#pragma unroll
            for (int u = 0; u < NV; ++u)
#pragma unroll
                for (int c = 0; c < VE; ++c) {
                    if constexpr (FLAT) {
                        const int64_t e = p0 * I + VE * (tid + TRI_T * u) + c;
                        raw[u][c] = e < count ? Y[e] : (T)0;
                    } else if (p0 + pv >= P) raw[u][c] = (T)0;
                }
        }
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int e = VE * (tid + TRI_T * u), row = row0 + rstep * u;
            if (FLAT ? e < I * SC : row < I) {
                double *x = d + (FLAT ? e : row * LDP + pv);
#pragma unroll
                for (int c = 0; c < VE; c += 2)
                    *reinterpret_cast<f64x2 *>(x + c) = f64x2{(double)raw[u][c], (double)raw[u][c + 1]};
            }
        }
    };
    auto compute = [&](int st) {
        const double *d = s_st + (st & 1) * stage_e;
        // the next step's elements are read while one is multiplied
        double a[2][MS][2], b[2][MS][2];
        auto read = [&](int k, double (&x)[MS][2], double (&y)[MS][2]) {
#pragma unroll
            for (int m = 0; m < MS; ++m)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    x[m][h] = d[oa[m] + 16 * h * rs + k * cs];
                    y[m][h] = d[ob[m] + 16 * h * rs + k * cs];
                }
        };
        auto mult = [&](const double (&x)[MS][2], const double (&y)[MS][2]) {
#pragma unroll
            for (int m = 0; m < MS; ++m) {
                if (q[m] < 0) continue;
                acc[m][0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m][0], y[m][0], acc[m][0][0], 0, 0, 0);
                acc[m][1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m][1], y[m][0], acc[m][1][0], 0, 0, 0);
                acc[m][1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m][1], y[m][1], acc[m][1][1], 0, 0, 0);
                if (!diag[m]) acc[m][0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m][0], y[m][1], acc[m][0][1], 0, 0, 0);
            }
        };
        const int dk = 4 * ks;
        read(4 * gk, a[0], b[0]);
        int k = 4 * gk;
        for (; k + dk < SC; k += 2 * dk) {
            read(k + dk, a[1], b[1]);
            mult(a[0], b[0]);
            read(min(k + 2 * dk, SC - 4), a[0], b[0]);
            mult(a[1], b[1]);
        }
        if (k < SC) mult(a[0], b[0]);
    };
    if (nst > 0) {
        load(0, raws[0]);
        load(1, raws[1]);
        store(0, raws[0]);
    }
    __syncthreads();
    for (int st = 0; st < nst; st += 2) {
        load(st + 2, raws[0]);
        compute(st);
        if (st + 1 < nst) store(st + 1, raws[1]);
        __syncthreads();
        if (st + 1 >= nst) break;
        load(st + 3, raws[1]);
        compute(st + 1);
        if (st + 2 < nst) store(st + 2, raws[0]);
        __syncthreads();
    }
    if (ks > 1) {   // the groups' sums, in a fixed order
        f64x4 *s_acc = reinterpret_cast<f64x4 *>(s_tri);
        auto at = [&](int g, int m, int x) { return (((g * gw + wg) * MS + m) * 4 + x) * 64 + lane; };
        if (gk > 0) {
#pragma unroll
            for (int m = 0; m < MS; ++m)
#pragma unroll
                for (int x = 0; x < 4; ++x) s_acc[at(gk - 1, m, x)] = acc[m][x >> 1][x & 1];
        }
        __syncthreads();
        if (gk > 0) return;
        for (int g = 0; g < ks - 1; ++g)
#pragma unroll
            for (int m = 0; m < MS; ++m)
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[m][x >> 1][x & 1] += s_acc[at(g, m, x)];
    }
    // partial super tiles, summed by gram_reduce_kernel<32, true>
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        if (q[m] < 0) continue;
        double *dst = partials + ((int64_t)kc * nss + q[m]) * 1024;
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v) dst[16 * x + tg + 4 * v + 32 * (16 * y + tr)] = acc[m][x][y][v];
    }
}

// Sums the partial blocks over the row ranges and writes the IA x IB result
// (mirroring the lower triangle when SYM).  64 elements per workgroup, each
// summed by four waves over interleaved ranges of partials (8 loads in
// flight per thread), the four sums combined in a fixed order.
template <int TB, bool SYM>
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double *__restrict__ partials, int nkc, int nbi,
                                                          int nblocks, int64_t IA, int64_t IB,
                                                          double *__restrict__ S) {
    const int q = blockIdx.y;
    int bi, bj;
    if (SYM) {
        bi = 0;
        while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
        bj = q - bi * (bi + 1) / 2;
    } else {
        bi = q % nbi;
        bj = q / nbi;
    }
    __shared__ double s_part[4][64];
    const int el = threadIdx.x & 63, ks = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + el;
    const bool ev = e < TB * TB;
    const int ec = ev ? e : 0;
    const int64_t stride = (int64_t)nblocks * TB * TB;
    const double *src = partials + (int64_t)q * TB * TB + ec;
    double acc = 0.0;
    int k = ks;
    for (; k + 28 < nkc; k += 32) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(int64_t)(k + 4 * u) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; k < nkc; k += 4) acc += src[(int64_t)k * stride];
    s_part[ks][el] = acc;
    __syncthreads();
    if (ks != 0 || !ev) return;
    const double sum = (s_part[0][el] + s_part[1][el]) + (s_part[2][el] + s_part[3][el]);
    const int il = e % TB, jl = e / TB;
    const int64_t i = (int64_t)bi * TB + il, j = (int64_t)bj * TB + jl;
    if (i >= IA || j >= IB) return;
    if (SYM && bi == bj && il < jl) return;  // upper part of a diagonal block: mirrored below
    S[i + IA * j] = sum;
    if (SYM && i != j) S[j + IA * i] = sum;
}

// TTT against a narrow second operand (L = 1, IB <= 64, FP64 products): the
// ALS branch's P = Y_(1) Z_(1)^T with a long first mode.  The block kernel pads
// IB to its block edge (10 -> 128 for I = 30648: 556 us for 553 MB).  Here a
// workgroup owns 32 rows of A and every column of B: lane (m, g) of a wave
// loads rows 2 m and 2 m + 1 of column 4 s + g (256 contiguous bytes per 16
// lanes), the even and the odd rows forming two tiles, so that nothing is
// staged in LDS and A is read once; the four waves take interleaved groups of
// columns and sum their tiles in LDS in wave order.  Bound by HBM: 107 us,
// 5.2 TB/s.
// kper: columns per range (blockIdx.y), dst + z IA IB its result.
template <typename T, int NT, bool VEC>
__global__ __launch_bounds__(256) void ttt_narrow_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                        int64_t IA, int IB, int64_t P, int64_t kper,
                                                        double *__restrict__ dst) {
    constexpr int U = 4;   // column groups in flight per wave
    __shared__ f64x4 s_acc[3][2 * NT][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tr = lane & 15, tg = lane >> 4;
    const int64_t i = (int64_t)blockIdx.x * 32 + 2 * tr;
    const int64_t ia = i < IA ? i : IA - 1, ib = i + 1 < IA ? i + 1 : IA - 1;
    const int64_t pend = min(P, (int64_t)(blockIdx.y + 1) * kper);
    f64x4 acc[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[h][t] = f64x4{0, 0, 0, 0};
    for (int64_t p0 = (int64_t)blockIdx.y * kper + 4 * wave; p0 < pend; p0 += 16 * U) {
        double a[U][2], b[U][NT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + 16 * u + tg;
            const bool ok = p < pend;
            const int64_t pc = ok ? p : pend - 1;
            T x0, x1;
            if constexpr (VEC) {   // IA even: a pair of rows is aligned and wholly inside
                typedef T t2 __attribute__((ext_vector_type(2)));
                const t2 x = *reinterpret_cast<const t2 *>(A + IA * pc + (i < IA ? i : IA - 2));
                x0 = x.x;
                x1 = x.y;
            } else {
                x0 = A[IA * pc + ia];
                x1 = A[IA * pc + ib];
            }
            a[u][0] = ok ? (double)x0 : 0.0;
            a[u][1] = ok ? (double)x1 : 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int r = 16 * t + tr;
                const double y = (double)B[(int64_t)IB * pc + (r < IB ? r : IB - 1)];
                b[u][t] = ok ? y : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[0][t] = mma(a[u][0], b[u][t], acc[0][t]);
                acc[1][t] = mma(a[u][1], b[u][t], acc[1][t]);
            }
    }
    if (wave > 0)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t) s_acc[wave - 1][2 * t + h][lane] = acc[h][t];
    __syncthreads();
    if (wave > 0) return;
    dst += (int64_t)blockIdx.y * IA * IB;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int w = 0; w < 3; ++w) acc[h][t] += s_acc[w][2 * t + h][lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = (int64_t)blockIdx.x * 32 + 2 * (tg + 4 * v) + h;
                const int r = 16 * t + tr;
                if (row < IA && r < IB) dst[row + IA * r] = acc[h][t][v];
            }
        }
}

// out = the nz partial results of count elements summed in order
__global__ __launch_bounds__(256) void ttt_sum_kernel(const double *__restrict__ part, int64_t count, int nz,
                                                     double *__restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= count) return;
    double s = 0.0;
#pragma unroll 8
    for (int z = 0; z < nz; ++z) s += part[z * count + e];
    out[e] = s;
}

// ---------------------------------------------------------------- host ----

namespace {

struct GramShape {
    int wt, tb, nbi, nbj, nblocks, nkc;
    int64_t kper;
};

GramShape gram_shape_t(int64_t IA, int64_t IB, int64_t P, bool sym, int64_t target, int wt_max);

GramShape gram_shape(int64_t IA, int64_t IB, int64_t P, bool sym) {
    return gram_shape_t(IA, IB, P, sym, 2 * (int64_t)device_cu_count(), 4);
}

GramShape gram_shape_t(int64_t IA, int64_t IB, int64_t P, bool sym, int64_t target, int wt_max) {
    GramShape g;
    int64_t imax = std::max(IA, IB);
    g.wt = std::min(wt_max, imax > 64 ? 4 : (imax > 32 ? 2 : 1));
    g.tb = 32 * g.wt;
    g.nbi = (int)((IA + g.tb - 1) / g.tb);
    g.nbj = (int)((IB + g.tb - 1) / g.tb);
    g.nblocks = sym ? g.nbi * (g.nbi + 1) / 2 : g.nbi * g.nbj;
    // aim at `target` workgroups (about 2 per CU for one tensor), rows per
    // workgroup >= 512, and partial traffic well below the input traffic
    int64_t nkc = std::max<int64_t>(1, target / g.nblocks);
    int64_t maxk = std::max<int64_t>(1, P / 512);
    nkc = std::min(nkc, maxk);
    int64_t kper = (P + nkc - 1) / nkc;
    kper = (kper + KC - 1) / KC * KC;
    if (kper < KC) kper = KC;
    g.kper = kper;
    g.nkc = (int)std::max<int64_t>(1, (P + kper - 1) / kper);
    return g;
}

// Skinny path geometry: CH chunks of 32 columns per stage, as many as keep
// the loader at one task per thread and two stages within the LDS
// budget; one workgroup per CU (the LDS of a stage), each at least 4 stages.
struct SkShape {
    int ch, nkc;
};

SkShape sk_shape(int prec, int64_t I, int64_t P) {
    SkShape k;
    const int NQ = prec == P_BF16X6 ? 3 : 2;
    const int64_t TBp = 32 * (int64_t)sk_ns(I);
    k.ch = prec == P_BF16X6 ? 4 : 8;   // bf16x6 at 8 chunks would spill registers
    while (k.ch > 1 && (TBp * k.ch > SK_T || 2 * k.ch * NQ * 4 * TBp * 16 > 150 * 1024)) k.ch >>= 1;
    const int64_t cols = 32 * (int64_t)k.ch;
    k.nkc = (int)std::min<int64_t>(device_cu_count(), std::max<int64_t>(1, P / (4 * cols)));
    return k;
}

size_t sk_lds(int prec, int64_t I, int ch) {
    const int NQ = prec == P_BF16X6 ? 3 : 2;
    return (size_t)2 * ch * NQ * 4 * 32 * sk_ns(I) * 16;
}

template <int PREC, int CH>
hipError_t launch_skinny_ch(const float *A, int64_t I, int64_t P, const SkShape &k, double *partials, hipStream_t s) {
    auto kern = I < 4 ? gram_skinny_kernel<PREC, CH, false, 1>
                      : I <= SK_MS1_MAXI ? gram_skinny_kernel<PREC, CH, true, 1> : gram_skinny_kernel<PREC, CH, true, SK_MS>;
    const size_t lds = sk_lds(PREC, I, CH);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)k.nkc), dim3(SK_T), lds, s, A, (int)I, P, k.nkc, partials);
    return hipGetLastError();
}

template <int PREC>
hipError_t launch_skinny(const float *A, int64_t I, int64_t P, double *partials, double *S, hipStream_t s) {
    const SkShape k = sk_shape(PREC, I, P);
    hipError_t e;
    switch (k.ch) {
        case 8:
            if constexpr (PREC != P_BF16X6) {
                e = launch_skinny_ch<PREC, 8>(A, I, P, k, partials, s);
                break;
            }
            [[fallthrough]];
        case 4: e = launch_skinny_ch<PREC, 4>(A, I, P, k, partials, s); break;
        case 2: e = launch_skinny_ch<PREC, 2>(A, I, P, k, partials, s); break;
        default: e = launch_skinny_ch<PREC, 1>(A, I, P, k, partials, s); break;
    }
    if (e != hipSuccess) return e;
    const int NS = sk_ns(I);
    hipLaunchKernelGGL((gram_reduce_kernel<32, true>), dim3((32 * 32 + 63) / 64, NS * (NS + 1) / 2), dim3(256), 0,
                       s, partials, k.nkc, NS, NS * (NS + 1) / 2, I, I, S);
    return hipGetLastError();
}

template <int PREC, int WT>
hipError_t launch_gram_l1(const float *A, int64_t IA, int64_t M, const GramShape &g,
                          double *partials, hipStream_t s) {
    constexpr int TB = 32 * WT;
    const int64_t total = (int64_t)g.nkc * g.nblocks;
    const int64_t per_xcd = (total + 7) / 8;
    const size_t lds = (size_t)2 * 2 * Frag<PREC>::NQ * 4 * TB * 16;
    // I a multiple of the block edge: the full path's loads (blocks of 64 and 128:
    // whole fragment octets per thread); I > SK_MAXI here, so quads fit
    auto kern = IA % TB == 0 ? gram_l1_kernel<PREC, WT, (WT >= 2)> : gram_l1_kernel<PREC, WT, false>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(gram_l1_eight_waves<PREC, WT>() ? 512 : 256), lds, s, A, IA, M, g.kper,
                       g.nkc, g.nblocks, total, partials);
    return hipGetLastError();
}

// The narrow TTT: ranges of columns until about two workgroups per CU (their
// partial results in the block kernel's workspace: g.nkc ranges of at most 128
// columns fit it for any IB <= 64), at least 256 columns each.
template <typename T, int NT>
hipError_t launch_ttt_narrow(const T *A, const T *B, int64_t IA, int64_t IB, int64_t P, const GramShape &g,
                             double *partials, double *S, hipStream_t s) {
    const int64_t rows = (IA + 31) / 32;
    int64_t nz = std::max<int64_t>(1, std::min<int64_t>({(2 * device_cu_count() + rows - 1) / rows, P / 256, g.nkc}));
    const int64_t kper = ((P + nz - 1) / nz + 15) / 16 * 16;
    nz = (P + kper - 1) / kper;
    double *dst = nz > 1 ? partials : S;
    const dim3 grid((unsigned)rows, (unsigned)nz);
    if (IA % 2 == 0 && (reinterpret_cast<uintptr_t>(A) & 15) == 0)
        hipLaunchKernelGGL((ttt_narrow_kernel<T, NT, true>), grid, dim3(256), 0, s, A, B, IA, (int)IB, P, kper, dst);
    else
        hipLaunchKernelGGL((ttt_narrow_kernel<T, NT, false>), grid, dim3(256), 0, s, A, B, IA, (int)IB, P, kper, dst);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nz == 1) return e;
    hipLaunchKernelGGL(ttt_sum_kernel, dim3((unsigned)((IA * IB + 255) / 256)), dim3(256), 0, s, partials, IA * IB,
                       (int)nz, S);
    return hipGetLastError();
}

// Geometry of the triangle kernel: rows per stage, wave groups along the
// contraction (the fewest products per wave, then the fewest groups), workgroups:
// one per CU with at least two stages each.
struct TriShape {
    int ks, ms, sc, nkc;   // wave groups, super tiles per wave, rows per stage, workgroups
    size_t lds;
};

int tri_nkc(int64_t P, int sc) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(device_cu_count(), P / (2 * sc)));
}

// Rows per stage: as many as fill its TRI_STAGE values where every CU still gets two
// stages (32 otherwise, which spreads few rows over more CUs).  512 MB of FP64
// data, L = 1: I = 16 158 us (256 rows a stage; 554 with 32 and the loads past the
// stage, 291 in the block kernel), I = 32 111 us (368, 164), I = 64 171 us (210,
// 190); I = 32, L = 16, 64 MB: 23 us (33, 26).
int tri_sc(int64_t I, int64_t P) {
    for (int sc = 8 * TRI_SC; sc > TRI_SC; sc /= 2)
        if (I * sc <= TRI_STAGE && P >= 2 * (int64_t)sc * device_cu_count()) return sc;
    return TRI_SC;
}

TriShape tri_shape(int64_t I, int64_t P, bool flat) {
    TriShape t;
    const int ns = sk_ns(I), nss = ns * (ns + 1) / 2;
    double best = 1e9;
    for (int ks = 1; ks <= TRI_W; ks *= 2) {
        const int per = (nss + TRI_W / ks - 1) / (TRI_W / ks);
        if (per <= 2 && (double)per / ks < best) {
            best = (double)per / ks;
            t.ks = ks;
            t.ms = per;
        }
    }
    t.sc = tri_sc(I, P);   // above 32 only for I <= 80: one super tile per wave
    t.lds = std::max((size_t)2 * tri_stage((int)I, t.sc, flat) * sizeof(double),
                     (size_t)(t.ks - 1) * (TRI_W / t.ks) * t.ms * 4 * 64 * sizeof(f64x4));
    t.nkc = tri_nkc(P, t.sc);
    return t;
}

template <typename T, int MS, int SC>
hipError_t launch_tri_m(const T *A, int64_t L, int64_t I, int64_t P, const TriShape &t, double *partials, hipStream_t s) {
    auto kern = L == 1 ? gram_tri64_kernel<T, MS, SC, true> : gram_tri64_kernel<T, MS, SC, false>;
    if (t.lds > 64 * 1024)
        if (hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)t.lds)) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)t.nkc), dim3(TRI_T), t.lds, s, A, L, (int)I, P, t.ks, t.nkc, partials);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tri(const T *A, int64_t L, int64_t I, int64_t M, double *partials, double *S, hipStream_t s) {
    const TriShape t = tri_shape(I, L * M, L == 1);
    const int64_t P = L * M;
    hipError_t e;
    switch (t.sc) {
        case 8 * TRI_SC: e = launch_tri_m<T, 1, 8 * TRI_SC>(A, L, I, P, t, partials, s); break;
        case 4 * TRI_SC: e = launch_tri_m<T, 1, 4 * TRI_SC>(A, L, I, P, t, partials, s); break;
        case 2 * TRI_SC: e = launch_tri_m<T, 1, 2 * TRI_SC>(A, L, I, P, t, partials, s); break;
        default:
            e = t.ms == 1 ? launch_tri_m<T, 1, TRI_SC>(A, L, I, P, t, partials, s)
                          : launch_tri_m<T, 2, TRI_SC>(A, L, I, P, t, partials, s);
    }
    if (e != hipSuccess) return e;
    const int ns = sk_ns(I);
    hipLaunchKernelGGL((gram_reduce_kernel<32, true>), dim3(16, ns * (ns + 1) / 2), dim3(256), 0, s, partials, t.nkc, ns,
                       ns * (ns + 1) / 2, I, I, S);
    return hipGetLastError();
}

template <typename T, int PREC, int WT, bool SYM>
hipError_t launch_gram_t(const T *A, const T *B, int64_t L, int64_t IA, int64_t IB, int64_t M,
                         const GramShape &g, double *partials, double *S, hipStream_t s) {
    constexpr int TB = 32 * WT;
    const int64_t P = L * M;
    const int64_t total = (int64_t)g.nkc * g.nblocks;
    const int64_t per_xcd = (total + 7) / 8;
    if constexpr (SYM && PREC == P_FP64) {
        // whole 16-byte vectors along the rows; other L stay with the general kernel
        if (IA <= TRI_MAXI && IA * P >= 64 && (L == 1 || L % (16 / (int64_t)sizeof(T)) == 0)) return launch_tri<T>(A, L, IA, M, partials, S, s);
    }
    if constexpr (SYM && sizeof(T) == 4) {
        if constexpr (PREC != P_FP64) {
            if (L == 1 && IA <= SK_MAXI) return launch_skinny<PREC>(A, IA, M, partials, S, s);
        }
        if (WT >= 2 && L == 1) {
            hipError_t e = launch_gram_l1<PREC, WT>(A, IA, M, g, partials, s);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((gram_reduce_kernel<TB, SYM>), dim3((TB * TB + 63) / 64, g.nblocks),
                               dim3(256), 0, s, partials, g.nkc, g.nbi, g.nblocks, IA, IB, S);
            return hipGetLastError();
        }
    }
    if constexpr (!SYM && sizeof(T) == 8 && WT == 4) {
        // rows beyond one block and few columns of B; FP32 data keeps the block
        // kernel's order of operations (its ALS sweeps round the bases to the
        // next product's factors and carry a last-bit difference on)
        if (L == 1 && IA >= 2 && IB <= 64) {
            if (IB <= 16) return launch_ttt_narrow<T, 1>(A, B, IA, IB, P, g, partials, S, s);
            if (IB <= 32) return launch_ttt_narrow<T, 2>(A, B, IA, IB, P, g, partials, S, s);
            return launch_ttt_narrow<T, 4>(A, B, IA, IB, P, g, partials, S, s);
        }
    }
    const size_t lds = (size_t)2 * Frag<PREC>::NQ * TB * 4 * 16;
    auto kern = gram_kernel<T, PREC, WT, SYM, false>;
    // Long fibres that are not whole octets: two chunks in three or more lie within
    // one and are read as widely as whole ones.  A kernel of its own: the condition,
    // in the kernel of the other L, cost those 4 to 9 percent.  300 rows in bf16x3:
    // L = 1001 194 -> 127 us, 201 133 -> 102, 100 149 -> 117; 64 rows, L = 66 24 ->
    // 26.  FP64 data in blocks of up to 64 gains nothing (64 rows, L = 1001: 34 -> 38).
    if constexpr (sizeof(T) == 4 || WT == 4) {
        if (L % 8 != 0 && L >= 3 * KC) kern = gram_kernel<T, PREC, WT, SYM, true>;
    }
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(256), lds, s, A, B, L, IA, IB, P,
                       g.kper, g.nkc, g.nbi, g.nbj, g.nblocks, total, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gram_reduce_kernel<TB, SYM>), dim3((TB * TB + 63) / 64, g.nblocks),
                       dim3(256), 0, s, partials, g.nkc, g.nbi, g.nblocks, IA, IB, S);
    return hipGetLastError();
}

template <typename T, int PREC, bool SYM>
hipError_t launch_gram_w(const T *A, const T *B, int64_t L, int64_t IA, int64_t IB, int64_t M,
                         const GramShape &g, double *partials, double *S, hipStream_t s) {
    switch (g.wt) {
        case 1: return launch_gram_t<T, PREC, 1, SYM>(A, B, L, IA, IB, M, g, partials, S, s);
        case 2: return launch_gram_t<T, PREC, 2, SYM>(A, B, L, IA, IB, M, g, partials, S, s);
        default: return launch_gram_t<T, PREC, 4, SYM>(A, B, L, IA, IB, M, g, partials, S, s);
    }
}

template <bool SYM>
hipError_t launch_gram_d(int dtype, int prec, const void *A, const void *B, int64_t L, int64_t IA,
                         int64_t IB, int64_t M, const GramShape &g, double *partials, double *S,
                         hipStream_t s) {
    if (dtype == DT_F64)
        return launch_gram_w<double, P_FP64, SYM>((const double *)A, (const double *)B, L, IA, IB, M, g, partials, S, s);
    const float *a = (const float *)A, *b = (const float *)B;
    switch (prec) {
        case P_FP64: return launch_gram_w<float, P_FP64, SYM>(a, b, L, IA, IB, M, g, partials, S, s);
        case P_FP32: return launch_gram_w<float, P_FP32, SYM>(a, b, L, IA, IB, M, g, partials, S, s);
        case P_BF16X3: return launch_gram_w<float, P_BF16X3, SYM>(a, b, L, IA, IB, M, g, partials, S, s);
        default: return launch_gram_w<float, P_BF16X6, SYM>(a, b, L, IA, IB, M, g, partials, S, s);
    }
}

}  // namespace

void gram_geometry(int64_t IA, int64_t IB, int64_t P, bool sym, int64_t target, int wt_max, int *wt,
                   int *nbi, int *nbj, int *nblocks, int *nkc, int64_t *kper) {
    GramShape g = gram_shape_t(IA, IB, P, sym, target, wt_max);
    *wt = g.wt;
    *nbi = g.nbi;
    *nbj = g.nbj;
    *nblocks = g.nblocks;
    *nkc = g.nkc;
    *kper = g.kper;
}

size_t gram_ws_bytes(int64_t IA, int64_t IB, int64_t P, bool sym) {
    GramShape g = gram_shape(IA, IB, P, sym);
    size_t b = (size_t)g.nkc * g.nblocks * g.tb * g.tb * sizeof(double);
    if (sym && IA <= SK_MAXI) {
        // the skinny path (L = 1) and the triangle kernel (FP64 products)
        const int NS = sk_ns(IA);
        int nkc = IA <= TRI_MAXI ? tri_nkc(P, TRI_SC) : 1;
        for (int prec = P_FP32; prec <= P_BF16X6; ++prec) nkc = std::max(nkc, sk_shape(prec, IA, P).nkc);
        b = std::max(b, (size_t)nkc * (NS * (NS + 1) / 2) * 1024 * sizeof(double));
    }
    return b;
}

hipError_t gram_launch(int dtype, int prec, const void *A, const void *B, int64_t L, int64_t IA,
                       int64_t IB, int64_t M, bool sym, double *partials, double *S,
                       hipStream_t s) {
    const int64_t P = L * M;
    if (P == 0) {
        return fill_f64(S, IA * IB, 0.0, s);  // a kernel, so that the call stays graph-capturable
    }
    GramShape g = gram_shape(IA, IB, P, sym);
    if (sym) return launch_gram_d<true>(dtype, prec, A, A, L, IA, IA, M, g, partials, S, s);
    return launch_gram_d<false>(dtype, prec, A, B, L, IA, IB, M, g, partials, S, s);
}

}  // namespace sth
