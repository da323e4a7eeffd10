// Device body of the direct FP64 symmetric eigensolver used for the R
// leading eigenpairs (Alg. 2, EIG branch: the leading eigenvectors of the
// mode-n Gram), run by one 512-thread workgroup:
//
//   1. Householder tridiagonalization A = Q T Q^T.  Step k builds the
//      reflector H_k = I - tau_k v_k v_k^T (v_k(k+1) = 1) from column k and
//      applies it to the trailing block as A <- A - v w^T - w v^T with
//      p = tau A v, w = p - (tau/2)(p^T v) v.  The rank-2 update of step k
//      is folded into the pass that forms p for step k + 1 (one read and one
//      write of the trailing block per step); column k + 1 gets its pending
//      update first so that v_{k+1} is known before that pass.
//   2. Eigenvalues of T by bisection on Sturm counts, the R largest only.
//      The count of eigenvalues below sigma is the number of sign changes in
//      the leading principal minors p_i of T - sigma I, taken with the
//      three-term recurrence p_i = (d_i - sigma) p_{i-1} - e_{i-1}^2 p_{i-2}
//      (no division; every 8 steps the pair is rescaled by a power of two,
//      which keeps every sign).  e^2 is floored at
//      (2^-60 ||T||)^2, so a vanishing minor is never followed by another
//      and counts as positive (the LDL^T count with a negative-zero pivot).
//      Each eigenvalue is searched by a group of
//      lanes, each lane counting at 4 points at once (independent chains),
//      which splits the bracket into (4 x group size + 1) parts per round.
//   3. Eigenvectors of T by inverse iteration: two solves of
//      (T - lambda I) x = b by Gaussian elimination with partial pivoting,
//      from a pseudo-random start vector of each eigenvector's own.
//   4. Orthogonalization: eigenvalues closer than 1e-9 ||T|| form clusters,
//      whose vectors (combinations inside the cluster's eigenspace) are made
//      orthonormal by classical Gram-Schmidt applied twice; then one
//      Newton-Schulz step Z <- Z (3 I - Z^T Z) / 2 on the whole block, on the
//      FP64 matrix cores, removes the O(eps ||T|| / gap) overlaps that
//      inverse iteration leaves between distinct eigenvalues.
//   5. Back-transformation Z <- H_0 H_1 ... H_{n-3} Z.
//   6. Optional sign rule (the entry of largest magnitude of each column is
//      made positive, first index on ties), eigenvalues in descending order.
//
// The matrix is scaled by a power of two so that its largest entry lies in
// [1, 2) (exact; eigenvalues are scaled back).  Accuracy is that of a
// backward-stable method: residuals and departure from orthogonality of
// order eps ||S||, eigenvectors to eps ||S|| / gap.  Non-finite input sets
// flag[0] = 3 and the run still ends with every index in range.
#pragma once
#include "common.h"

#include <type_traits>

namespace sth {

constexpr int TE_T = 512;            // threads per workgroup
constexpr int TE_W = TE_T / 64;      // waves
constexpr int TE_LDS_N = 128;        // up to this order the matrix stays in registers and LDS (teig_small)
constexpr int TE_LDS_BUDGET = 157 * 1024;   // dynamic LDS bytes a teig workgroup may take

// Global scratch of one solve (doubles):
//   Vr  n * n    n <= TE_LDS_N: reflector k in column k (used where they do
//                not fit the LDS)
//   F   3 n R    inverse-iteration factors, [(3 i + c) R + r] (n <= TE_LDS_N:
//                (n + 1) R multipliers, where they do not fit the LDS)
//   G   R * R    Gram of the eigenvector block (Newton-Schulz)
//   Zg  n * R    eigenvector block, row-major (only when it is not in LDS);
//                also the staging buffer of the Newton-Schulz product
//   Ag  n * n    n > TE_LDS_N: working copy of A, then the reflectors
struct TeScratch {
    double *Vr, *F, *G, *Zg, *Ag;
};

__host__ __device__ inline int64_t te_part_doubles(int64_t n) { return 16 * n > 1024 ? 16 * n : 1024; }
__host__ __device__ inline size_t te_big_lds_bytes(int64_t n, int64_t R, bool zlds) {
    return (size_t)((zlds ? n * R : 0) + te_part_doubles(n) + 8 * n + R) * 8 + (size_t)R * 4 + 16;
}
// n > TE_LDS_N: the eigenvector block fits the LDS
__host__ __device__ inline bool teig_z_fits(int64_t n, int64_t R) {
    return te_big_lds_bytes(n, R, true) <= (size_t)TE_LDS_BUDGET;
}
__host__ __device__ inline size_t teig_scratch_doubles(int64_t n, int64_t R, bool alds) {
    return (size_t)((alds ? n * n : 0) + 3 * n * R + R * R + n * R + (alds ? 0 : n * n)) + 64;
}
__host__ __device__ inline TeScratch teig_scratch_layout(double *base, int64_t n, int64_t R, bool alds) {
    TeScratch t;
    double *d = (double *)(((uintptr_t)base + 255) & ~(uintptr_t)255);
    t.Vr = alds ? d : nullptr;
    d += alds ? n * n : 0;
    t.F = d;
    d += 3 * n * R;
    t.G = d;
    d += R * R;
    t.Zg = d;
    d += n * R;
    t.Ag = alds ? nullptr : d;
    return t;
}

// DPP move of both halves of a double (lanes the pattern leaves out read 0)
template <int CTRL, int ROWS>
__device__ __forceinline__ double te_dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
    return __hiloint2double(hi, lo);
}
// Sum over the 64 lanes of a wave, returned in every lane: row_shr 1, 2, 4, 8
// leave each 16-lane row's sum in its last lane, row_bcast 15 and 31 carry
// them into lane 63, read back with readlane (register moves only, no LDS).
__device__ __forceinline__ double te_wave_sum(double v) {
    v += te_dpp<0x111, 0xf>(v);   // row_shr:1
    v += te_dpp<0x112, 0xf>(v);   // row_shr:2
    v += te_dpp<0x114, 0xf>(v);   // row_shr:4
    v += te_dpp<0x118, 0xf>(v);   // row_shr:8
    v += te_dpp<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v += te_dpp<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double te_wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double te_wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}

// value of v in lane src (src uniform across the wave)
__device__ __forceinline__ double te_lane(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

// 1 / x: the hardware reciprocal refined by one Newton step
__device__ __forceinline__ double te_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// Numbers of eigenvalues of the tridiagonal (d, e2 = e^2) below sig[c],
// TE_NC independent counts interleaved: the sign changes of the leading
// principal minors p_i of T - sigma I.  A zero minor counts as positive (the
// LDL^T count with a negative-zero pivot): adding +0 turns -0 into +0, and
// the caller floors e^2 at a tiny positive value so that a zero minor is
// never followed by another.  Every 8 steps the pair (p_{i-1}, p_i) of each
// count is multiplied by the power of two that brings the exponent of the
// larger one to zero (exact, signs kept): the entries of T are at most
// 2 n <= 2^10 after scaling, so the larger one grows by less than 2^22 per step
// and shrinks by less than the e^2 floor (2^-120 ||T||^2) per two steps,
// which keeps every value normal between normalizations.
constexpr int TE_NC = 4;
__device__ __forceinline__ double te_pow2_inv(double m) {
    // 2^-e with e the unbiased exponent of the normal number m > 0
    const int e = (__double2hiint(m) >> 20) & 0x7ff;
    return __hiloint2double((2046 - e) << 20, 0);
}
__device__ __forceinline__ void te_sturm(const double *__restrict__ d, const double *__restrict__ e2, int n,
                                         const double (&sig)[TE_NC], int (&cnt)[TE_NC]) {
    double p0[TE_NC], p1[TE_NC];
#pragma unroll
    for (int c = 0; c < TE_NC; ++c) {
        p0[c] = 1.0;
        p1[c] = (d[0] - sig[c]) + 0.0;
        cnt[c] = (int)((unsigned)__double2hiint(p1[c]) >> 31);
    }
    int i = 1;
    for (; i + 8 <= n; i += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double di = d[i + u], ei = e2[i + u - 1];
#pragma unroll
            for (int c = 0; c < TE_NC; ++c) {
                const double p2 = fma(di - sig[c], p1[c], -ei * p0[c]) + 0.0;
                cnt[c] += (int)((unsigned)(__double2hiint(p2) ^ __double2hiint(p1[c])) >> 31);
                p0[c] = p1[c];
                p1[c] = p2;
            }
        }
#pragma unroll
        for (int c = 0; c < TE_NC; ++c) {
            const double sc = te_pow2_inv(fmax(fabs(p0[c]), fabs(p1[c])));
            p0[c] *= sc;
            p1[c] *= sc;
        }
    }
    for (; i < n; ++i) {
        const double di = d[i], ei = e2[i - 1];
#pragma unroll
        for (int c = 0; c < TE_NC; ++c) {
            const double p2 = fma(di - sig[c], p1[c], -ei * p0[c]) + 0.0;
            cnt[c] += (int)((unsigned)(__double2hiint(p2) ^ __double2hiint(p1[c])) >> 31);
            p0[c] = p1[c];
            p1[c] = p2;
        }
    }
}

// Start vector entry of eigenvector r: uniform in [-1, 1).
__device__ __forceinline__ double te_start(int r, int i) {
    const uint64_t h = splitmix64(0x7E16ull ^ ((uint64_t)(uint32_t)r << 32) ^ (uint64_t)(uint32_t)i);
    return (double)(h >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// ---- orders up to TE_LDS_N: the solver inside registers and LDS ------------
// One workgroup, bound by latency: every phase is a serial chain, so each is
// laid out to shorten its chain rather than to spread the (small) work.
//   1. Tridiagonalization (ts_tridiag): a lead wave derives the vectors of a
//      step, four waves hold the columns in registers.
//   2. Bisection: counts at 256 points bracket every eigenvalue, then a group
//      of lanes per eigenvalue, one point per lane, four waves (one per SIMD).
//   3. Inverse iteration, one lane per vector: the elimination keeps only its
//      multipliers (the pivot choice in the lowest mantissa bit), the rest of
//      U follows from them and T.  The first solve is U x = random, the second
//      is whole.  Meanwhile the idle waves form the factors T_b of the blocked
//      reflectors.
//   4. Clusters by Gram-Schmidt; then each wave takes 16 columns into
//      registers in the matrix cores' result layout, which is also their
//      B-operand layout: the Newton-Schulz step and the back-transformation
//      (I - V_b T_b V_b^T, 16 reflectors at a time) need no barrier and no LDS
//      round trip of Z, only the A operands come from LDS (or, where the
//      reflectors do not fit beside Z and the multipliers, the scratch).
// Cycles at order 80, R = 64, the form with every phase on all eight waves,
// scalar Sturm steps, whole elimination factors in the scratch and unblocked
// reflectors against this one: tridiagonalization 346 k -> 145 k, bisection
// 174 k -> 64 k, inverse iteration 147 k -> 50 k, Newton-Schulz 40 k -> 27 k,
// back-transformation 132 k -> 22 k; 366 -> 138 us (order 64, R = 8: 250 -> 79).
struct TsLayout {
    int ldz, ldv, sld, nb;
    bool fl, vl;               // multipliers, reflectors in LDS
    int off_f, off_v, off_part, off_vec;
    size_t bytes;
};
constexpr int TS_VEC = 4 * TE_LDS_N + 2 * (TE_LDS_N + 32) + 6 * TE_LDS_N;   // doubles of the vectors
__host__ __device__ inline TsLayout ts_layout(int n, int R) {
    TsLayout t;
    t.nb = n > 2 ? (n + 13) / 16 : 1;
    const int part = 256 * t.nb > 1024 ? 256 * t.nb : 1024;
    const int budget = TE_LDS_BUDGET / 8 - part - TS_VEC - 1;
    t.ldz = n * (R | 1) <= budget ? (R | 1) : R;   // odd: columns and rows both free of bank conflicts
    t.sld = n * (n | 1) <= budget ? (n | 1) : n;
    const int z = n * t.ldz, f = (n + 1) * R, v = n * (n | 1), st = n * t.sld;
    t.fl = z + f <= budget;
    t.vl = z + f + v <= budget;
    t.ldv = t.vl ? (n | 1) : n;
    t.off_f = z;
    t.off_v = z + f;
    int main = t.vl ? z + f + v : (t.fl ? z + f : z);
    if (main < st) main = st;
    main += main & 1;          // the vectors are read in 16-byte pairs
    t.off_part = main;
    t.off_vec = main + part;
    t.bytes = (size_t)(main + part + TS_VEC) * 8;
    return t;
}

// two wave sums at once (their chains overlap)
__device__ __forceinline__ void te_wave_sum2(double &a, double &b) {
    a += te_dpp<0x111, 0xf>(a);
    b += te_dpp<0x111, 0xf>(b);
    a += te_dpp<0x112, 0xf>(a);
    b += te_dpp<0x112, 0xf>(b);
    a += te_dpp<0x114, 0xf>(a);
    b += te_dpp<0x114, 0xf>(b);
    a += te_dpp<0x118, 0xf>(a);
    b += te_dpp<0x118, 0xf>(b);
    a += te_dpp<0x142, 0xa>(a);
    b += te_dpp<0x142, 0xa>(b);
    a += te_dpp<0x143, 0xc>(a);
    b += te_dpp<0x143, 0xc>(b);
    a = te_lane(a, 63);
    b = te_lane(b, 63);
}

// 1 / sqrt(x), x a normal number: the hardware estimate with one third-order step
__device__ __forceinline__ double te_rsqrt(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * r, r, 1.0);
    return fma(r * e, fma(0.375, e, 0.5), r);
}

// Four columns of one row slot: a_c -= v w_c + w v_c, y += a_c x_c, with v_c, w_c
// and x_c broadcast from lanes N .. N + 3 of each row of 16 lanes (the only DPP
// control FP64 instructions take; a broadcast through readlane takes two
// instructions and a hazard per operand, 57 cycles a column against 16).  The
// s_nop keeps the two wait states a DPP read needs after a VALU write.
template <int N>
__device__ __forceinline__ void ts_cols4(double &a0, double &a1, double &a2, double &a3, double &y, double rv,
                                         double rw, double rx, double nv, double nw) {
#define TS_F(d, s0, s1, c) "v_fmac_f64_dpp " d ", " s0 ", " s1 " row_newbcast:" c " row_mask:0xf bank_mask:0xf\n"
    asm("s_nop 1\n" TS_F("%0", "%6", "%8", "%10") TS_F("%1", "%6", "%8", "%11") TS_F("%2", "%6", "%8", "%12")
            TS_F("%3", "%6", "%8", "%13") TS_F("%0", "%5", "%9", "%10") TS_F("%1", "%5", "%9", "%11")
                TS_F("%2", "%5", "%9", "%12") TS_F("%3", "%5", "%9", "%13") TS_F("%4", "%7", "%0", "%10")
                    TS_F("%4", "%7", "%1", "%11") TS_F("%4", "%7", "%2", "%12") TS_F("%4", "%7", "%3", "%13")
        : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3), "+v"(y)
        : "v"(rv), "v"(rw), "v"(rx), "v"(nv), "v"(nw), "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3));
#undef TS_F
}
// this lane's H consecutive entries of a vector in LDS (16-byte aligned)
template <int H>
__device__ __forceinline__ void ts_get(const double *s, double (&a)[H]) {
    const int lane = threadIdx.x & 63;
    if constexpr (H == 2) {
        const double2 t = *reinterpret_cast<const double2 *>(s + 2 * lane);
        a[0] = t.x;
        a[1] = t.y;
    } else {
        a[0] = s[lane];
    }
}
template <int H>
__device__ __forceinline__ void ts_put(double *s, const double (&a)[H]) {
    const int lane = threadIdx.x & 63;
    if constexpr (H == 2) *reinterpret_cast<double2 *>(s + 2 * lane) = make_double2(a[0], a[1]);
    else s[lane] = a[0];
}
template <int G, int NG, typename F>
__device__ __forceinline__ void ts_groups(F f) {
    if constexpr (G < NG) {
        if (f(std::integral_constant<int, G>{})) ts_groups<G + 1, NG>(f);
    }
}

// Step 1 for n <= 64 H.  stg: the matrix in LDS (leading dimension sld; the
// mean of the two triangles times sc is reduced); V: column k receives the
// unscaled v_k = x - beta e_{k+1} (zeros above row k + 1), leading dimension
// ldv, and H_k = I - tau_k v_k v_k^T; s_vec 4 * 64 H doubles, part 4 * 64 H.
// Reads stg before its first barrier only, so V may overlap it.
//
// Wave 0 leads: from the partial products and the raw next column it forms
// w and the next column x and hands v, w, x over in LDS; waves 1 .. TW hold
// the columns j = w - 1 (mod TW), lane l the rows H l .. H l + H - 1 of each,
// and apply the update and form the product with x, while the lead derives
// the reflector (norm, beta, tau) of that column.  The product needs only the
// unscaled x: v = x - beta e_{k+1} gives A v = A x - beta A e_{k+1}.  The
// column slots move down by one every TW steps, so that the next column is
// always slot 0 and every register index is static.  (With every wave
// repeating the lead's vector work behind one barrier a step, the lead and
// the column wave on its SIMD slowed each other down: 1500 cycles a step at
// n = 64, 2300 at 80.)
template <int H>
__device__ __forceinline__ void ts_tridiag(const double *stg, int sld, double sc, int n, double *V, int ldv,
                                           double *part, double *s_vec, double *s_d, double *s_e, double *s_tau) {
    constexpr int TW = 4, NQ = 64 * H / TW, ST = 64 * H, NB = NQ / 16;
    const int lane = threadIdx.x & 63;
    const int wv_ = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *const s_v = s_vec, *const s_w = s_vec + ST, *const s_x = s_vec + 2 * ST, *const s_c = s_vec + 3 * ST;
    if (wv_ > TW) {
        __syncthreads();
        __syncthreads();
        for (int k = 0; k + 1 < n; ++k) {
            __syncthreads();
            __syncthreads();
        }
        return;
    }
    if (wv_ == 0) {
        // ---- the lead ----
        double x[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int i = H * lane + h, ic = i < n ? i : n - 1;
            const double c = 0.5 * (stg[ic] + stg[sld * ic]) * sc;
            x[h] = (i > 0 && i < n) ? c : 0.0;
            s_x[i] = x[h];
            if (i == 0) s_d[0] = c;
        }
        __syncthreads();   // stg is read
        __builtin_amdgcn_s_setprio(3);
        double beta, tau, v1;
        // reflector of column k from x (rows > k)
        auto reflect = [&](int k, auto podd) {
            constexpr int h1 = H == 2 && decltype(podd)::value == 0 ? 1 : 0;   // k + 1 odd when k is even
            double sx = 0.0;
#pragma unroll
            for (int h = 0; h < H; ++h)
                if (H * lane + h != k + 1) sx = fma(x[h], x[h], sx);
            const double x0 = te_lane(x[h1], (k + 1) / H);
            sx = te_wave_sum(sx);
            beta = x0;
            tau = 0.0;
            if (sx > 1e-200) {
                const double s2 = fma(x0, x0, sx), nrm = s2 * te_rsqrt(s2);
                beta = x0 >= 0.0 ? -nrm : nrm;
                tau = te_rcp(fma(fabs(x0), nrm, s2));   // 2 / ||v||^2
            }
            v1 = x0 - beta;
        };
        auto step = [&](int k, auto podd) {
            constexpr int h1 = H == 2 && decltype(podd)::value == 0 ? 1 : 0;   // where row k + 1 lives
            const int l1 = (k + 1) / H;
            reflect(k, podd);
            if (lane == 0) {
                s_e[k] = beta;
                s_tau[k] = tau;
            }
            __syncthreads();   // the partial products and the raw column k + 1
            double y[H], c[H], t[TW][H], xy = 0.0;
#pragma unroll
            for (int u = 0; u < TW; ++u) ts_get<H>(part + u * ST, t[u]);
            ts_get<H>(s_c, c);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                y[h] = (t[0][h] + t[1][h]) + (t[2][h] + t[3][h]);
                xy = fma(x[h], y[h], xy);
            }
            const double y0 = te_lane(y[h1], l1), c0 = te_lane(c[h1], l1);
            // v^T A v = x^T y - 2 beta y_0 + beta^2 c_0;  p = tau A v;  w = p - K v
            const double t0 = tau * fma(beta * beta, c0, -2.0 * beta * y0);
            xy = te_wave_sum(xy);
            const double K = 0.5 * tau * fma(tau, xy, t0);
            double w[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int i = H * lane + h;
                const double v = i == k + 1 ? v1 : x[h];
                const double t = fma(-K, v, tau * fma(-beta, c[h], y[h]));
                w[h] = i > k ? t : 0.0;
                x[h] = v;
            }
            ts_put<H>(s_v, x);
            ts_put<H>(s_w, w);
            const double w1 = te_lane(w[h1], l1);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int i = H * lane + h;
                const double t = fma(-v1, w[h], fma(-w1, x[h], c[h]));
                x[h] = i > k + 1 ? t : 0.0;
            }
            ts_put<H>(s_x, x);
            __syncthreads();   // v, w, x handed over
            if (lane == 0) s_d[k + 1] = fma(-2.0 * v1, w1, c0);
        };
        __syncthreads();   // x of column 0
        for (int k = 0;; k += 2) {
            if (k + 1 >= n) break;
            step(k, std::integral_constant<int, 0>{});
            if (k + 2 >= n) break;
            step(k + 1, std::integral_constant<int, 1>{});
        }
        __builtin_amdgcn_s_setprio(0);
        return;
    }
    // ---- the column waves ----
    const int w = wv_ - 1;
    double ar[H][NQ], y[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int i = H * lane + h, ic = i < n ? i : n - 1;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int j = w + TW * q, jc = j < n ? j : n - 1;
            const double a = 0.5 * (stg[ic + sld * jc] + stg[jc + sld * ic]) * sc;
            ar[h][q] = (i < n && j < n) ? a : 0.0;
        }
        y[h] = 0.0;
    }
    __syncthreads();   // stg is read
    __syncthreads();   // x of column 0
    // entries of the vector for column slots 16 b + lane % 16 of block Q; slots
    // past column 64 H - 1 wrap to a finished row, whose entries are zero
    auto rep = [&](const double *vec, int Q, int b) {
        return vec[(w + TW * (Q + 16 * b + (lane & 15))) & (ST - 1)];
    };
    {
        double rx[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) rx[b] = rep(s_x, 0, b);
        ts_groups<0, NQ / 4>([&](auto gc) {
            constexpr int q = 4 * decltype(gc)::value, b = q / 16;
            if (TW * q >= n) return false;
#pragma unroll
            for (int h = 0; h < H; ++h)
                ts_cols4<q % 16>(ar[h][q], ar[h][q + 1], ar[h][q + 2], ar[h][q + 3], y[h], 0.0, 0.0, rx[b], 0.0, 0.0);
            return true;
        });
    }
    auto step = [&](int Q, auto sconst) {
        constexpr int s = decltype(sconst)::value;
        const int k = TW * Q + s;
        ts_put<H>(part + w * ST, y);
        if (w == (s + 1) % TW) {
            double c[H];
#pragma unroll
            for (int h = 0; h < H; ++h) c[h] = ar[h][s == TW - 1 ? 1 : 0];
            ts_put<H>(s_c, c);
        }
        __syncthreads();
        __syncthreads();
        double v[H], wv[H], rv[NB], rw[NB], rx[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            rv[b] = rep(s_v, Q, b);
            rw[b] = rep(s_w, Q, b);
            rx[b] = rep(s_x, Q, b);
        }
        ts_get<H>(s_v, v);
        ts_get<H>(s_w, wv);
#pragma unroll
        for (int h = 0; h < H; ++h) y[h] = 0.0;
        if (w == s) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int i = H * lane + h;
                if (i < n) V[i + (int64_t)ldv * k] = v[h];
            }
        }
        // the rank-2 update and the product with the next column (entries of
        // finished rows are zero in v, w and x); the last step of a block
        // moves the slots down
        constexpr int SH = s == TW - 1 ? 1 : 0;
        ts_groups<0, NQ / 4>([&](auto gc) {
            constexpr int q = 4 * decltype(gc)::value, b = q / 16;
            if (TW * (Q + q) >= n) return false;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                double a0 = ar[h][q], a1 = ar[h][q + 1], a2 = ar[h][q + 2], a3 = ar[h][q + 3];
                ts_cols4<q % 16>(a0, a1, a2, a3, y[h], rv[b], rw[b], rx[b], -v[h], -wv[h]);
                ar[h][q > 0 ? q - SH : 0] = q > 0 || !SH ? a0 : a1;
                ar[h][q + 1 - SH] = a1;
                ar[h][q + 2 - SH] = a2;
                ar[h][q + 3 - SH] = a3;
            }
            return true;
        });
    };
    for (int Q = 0; TW * Q + 1 < n; ++Q) {
        step(Q, std::integral_constant<int, 0>{});
        if (TW * Q + 2 >= n) break;
        step(Q, std::integral_constant<int, 1>{});
        if (TW * Q + 3 >= n) break;
        step(Q, std::integral_constant<int, 2>{});
        if (TW * Q + 4 >= n) break;
        step(Q, std::integral_constant<int, 3>{});
    }
}

// Eight minors from (p0, p1): q_i = (d_i - sigma) q_{i-1} - e_{i-1}^2 q_{i-2}, the
// entries d and -e^2 broadcast from lanes N .. N + 7 of each row of 16 lanes.
// (Read as 16 bytes shared by every lane, a step costs each wave 8 to 16 cycles
// of LDS: 49 cycles a step with four waves, against 27 here.)  -sigma q and d q
// round apart, a change of d_i by at most eps |sigma|.
template <int N>
__device__ __forceinline__ void ts_minors8(double p0, double p1, double (&q)[8], double d, double ne, double ns) {
#define TS_S(o, a, b, c) "v_mul_f64 " o ", %12, " a "\n v_fmac_f64_dpp " o ", %10, " a " row_newbcast:" c \
        " row_mask:0xf bank_mask:0xf\n v_fmac_f64_dpp " o ", %11, " b " row_newbcast:" c " row_mask:0xf bank_mask:0xf\n"
    asm("s_nop 1\n" TS_S("%0", "%9", "%8", "%13") TS_S("%1", "%0", "%9", "%14") TS_S("%2", "%1", "%0", "%15")
            TS_S("%3", "%2", "%1", "%16") TS_S("%4", "%3", "%2", "%17") TS_S("%5", "%4", "%3", "%18")
                TS_S("%6", "%5", "%4", "%19") TS_S("%7", "%6", "%5", "%20")
        : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3]), "=&v"(q[4]), "=&v"(q[5]), "=&v"(q[6]), "=&v"(q[7])
        : "v"(p0), "v"(p1), "v"(d), "v"(ne), "v"(ns), "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3), "n"(N + 4),
          "n"(N + 5), "n"(N + 6), "n"(N + 7));
#undef TS_S
}

// Sturm count at sigma (see te_sturm).  de[i] = (d_i, -e_{i-1}^2), padded by 32
// zero entries: the minors past the last are zero multiples whose signs are
// masked off.  Every lane of the wave must be active.
__device__ __forceinline__ int ts_sturm(const double2 *__restrict__ de, int n, double sigma) {
    const int l16 = threadIdx.x & 15;
    double2 t = de[1 + l16];
    double p0 = 1.0, p1 = de[0].x - sigma;
    unsigned bits = (unsigned)__double2hiint(p1) >> 31;   // bit 0: the sign of the last minor
    int cnt = (int)bits;
    auto half = [&](auto nc, int left) {
        double q[8];
        ts_minors8<decltype(nc)::value>(p0, p1, q, t.x, t.y, -sigma);
        unsigned b = bits;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            b = __builtin_amdgcn_alignbit(b, (unsigned)__double2hiint(q[u]), 31);   // b << 1 | sign
        // the first `left` of these steps exist
        const unsigned m = left >= 8 ? 0xffu : (0xffu << (8 - left)) & 0xffu;
        cnt += __popc((b ^ (b >> 1)) & m);
        bits = b & 1u;
        // power of two from the fourth minor, off the chain (12 steps of growth
        // or decay stay normal)
        const double sc = te_pow2_inv(fmax(fabs(q[2]), fabs(q[3])));
        p0 = q[6] * sc;
        p1 = q[7] * sc;
    };
    for (int i = 1; i < n; i += 16) {
        const double2 tn = de[i + 16 + l16];
        half(std::integral_constant<int, 0>{}, n - i);
        if (i + 8 < n) half(std::integral_constant<int, 8>{}, n - i - 8);
        t = tn;
    }
    return cnt;
}

// keeps both operands of a select evaluated (the compiler would otherwise
// branch around the dearer one, lane by lane)
__device__ __forceinline__ double ts_keep(double v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ double ts_sel(bool c, double a, double b) {
    return __hiloint2double(c ? __double2hiint(a) : __double2hiint(b), c ? __double2loint(a) : __double2loint(b));
}

// Step 3 for vector r: x of (T - lam I) x = b by elimination with partial
// pivoting, twice, x in column r of Z (row stride ldz), the multiplier m_i of
// row i in F (row i + 1, row stride R; row 0 is a zero).  The rows of U follow
// from the multipliers: a row that was not exchanged has the pivot e_i / m_i
// and the entry left by the elimination of the row above, an exchanged one is
// the row (e_i, d_{i+1} - lam, e_{i+1}) of T.  de: d in .x; s_e: e floored
// away from zero, zero past its end; s_re: its reciprocals.  Chunks of rows
// are loaded ahead of the chain.
__device__ __forceinline__ void ts_inverse(const double2 *__restrict__ de, const double *__restrict__ s_e,
                                           const double *__restrict__ s_re, int n, int R, double lm, double tiny,
                                           int r, double *__restrict__ F, double *__restrict__ Z, int ldz,
                                           double *__restrict__ s_inv) {
    constexpr int CH = 8;
    double cd = de[0].x - lm, cu = s_e[0];
    auto eliminate = [&](double dn, double e, double en, double re, double *f) {
        const double nd = dn - lm;
        const bool piv = fabs(cd) < fabs(e);
        const double mp = cd * re, mn = ts_keep(e * te_rcp(cd));
        double ml = ts_sel(piv, mp, mn);
        ml = __hiloint2double(__double2hiint(ml), (__double2loint(ml) & ~1) | (piv ? 1 : 0));
        *f = ml;
        const double u1 = ts_sel(piv, nd, cu), m0 = ts_sel(piv, cu, nd);
        cd = fma(-ml, u1, m0);
        cu = ts_sel(piv, -ml * en, en);
    };
    F[r] = 0.0;
    {
        double *f = F + R + r;
        int i = 0;
        for (; i + CH < n; i += CH, f += CH * R) {
            double d[CH], e[CH + 1], re[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                d[u] = de[i + 1 + u].x;
                e[u] = s_e[i + u];
                re[u] = s_re[i + u];
            }
            e[CH] = s_e[i + CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) eliminate(d[u], e[u], e[u + 1], re[u], f + u * R);
        }
        for (; i + 1 < n; ++i, f += R) eliminate(de[i + 1].x, s_e[i], s_e[i + 1], s_re[i], f);
    }
    if (cd == 0.0) cd = tiny;
    const double rlast = te_rcp(cd);
    double nrm2 = 0.0, x1, x2;
    // x_i from the rows below: y / u0 - (u1 / u0) x_{i+1} - (u2 / u0) x_{i+2}
    auto coef = [&](double ml, double mprev, double e, double en, double re, double dn, double &ru, double &a1,
                    double &a2) {
        const bool piv = __double2loint(ml) & 1, pprev = __double2loint(mprev) & 1;
        ru = ts_sel(piv, re, ml * re);
        const double c = ts_sel(pprev, -mprev * e, e);
        a1 = ts_sel(piv, dn - lm, c) * ru;
        a2 = ts_sel(piv, en, 0.0) * ru;
    };
    auto back = [&](double top, auto rhs) {
        x1 = top * rlast;
        x2 = 0.0;
        Z[(n - 1) * ldz + r] = x1;
        nrm2 = x1 * x1;
        int i = n - 2;
        const double *f = F + (n - 1) * R + r;   // row i
        double *z = Z + i * ldz + r;
        for (; i >= CH - 1; i -= CH, f -= CH * R, z -= CH * ldz) {
            double ml[CH + 1], e[CH + 1], re[CH], d[CH], y[CH], ru[CH], a1[CH], a2[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                ml[u] = f[-u * R];
                e[u + 1] = s_e[i - u];
                re[u] = s_re[i - u];
                d[u] = de[i + 1 - u].x;
                y[u] = rhs(z - u * ldz);
            }
            ml[CH] = f[-CH * R];
            e[0] = s_e[i + 1];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                coef(ml[u], ml[u + 1], e[u + 1], e[u], re[u], d[u], ru[u], a1[u], a2[u]);
                y[u] *= ru[u];
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const double x = fma(-a1[u], x1, fma(-a2[u], x2, y[u]));
                z[-u * ldz] = x;
                nrm2 = fma(x, x, nrm2);
                x2 = x1;
                x1 = x;
            }
        }
        for (; i >= 0; --i, f -= R, z -= ldz) {
            double ru, a1, a2;
            const double y = rhs(z);
            coef(f[0], f[-R], s_e[i], s_e[i + 1], s_re[i], de[i + 1].x, ru, a1, a2);
            const double x = fma(-a1, x1, fma(-a2, x2, y * ru));
            z[0] = x;
            nrm2 = fma(x, x, nrm2);
            x2 = x1;
            x1 = x;
        }
    };
    // first solve: U x = a random vector
    uint32_t rnd = (uint32_t)splitmix64(0x7E16ull ^ (uint64_t)(uint32_t)r);
    auto draw = [&](const double *) {
        rnd = rnd * 1664525u + 1013904223u;
        return (double)(int)(rnd | 1u) * 0x1p-31;
    };
    back(draw(nullptr), draw);
    // second solve: forward substitution of the normalized x, then back
    const double inv = te_rsqrt(nrm2);
    double cb = Z[r] * inv;
    {
        const double *f = F + R + r;
        double *z = Z + r;
        int i = 0;
        auto forward = [&](double ml, double nb, double *out) {
            const bool piv = __double2loint(ml) & 1;
            const double yy = ts_sel(piv, nb, cb), m0 = ts_sel(piv, cb, nb);
            cb = fma(-ml, yy, m0);
            *out = yy;
        };
        for (; i + CH < n; i += CH, f += CH * R, z += CH * ldz) {
            double ml[CH], nb[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                ml[u] = f[u * R];
                nb[u] = z[(u + 1) * ldz] * inv;
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) forward(ml[u], nb[u], z + u * ldz);
        }
        for (; i + 1 < n; ++i, f += R, z += ldz) forward(f[0], z[ldz] * inv, z);
    }
    back(cb, [&](const double *z) { return *z; });
    s_inv[r] = te_rsqrt(nrm2);
}

// T of the 16 reflectors k0 .. k0 + 15 of V by one wave: H_k0 ... H_{k0+15} =
// I - V T V^T with T^{-1} = diag(1 / tau) + the strict upper triangle of V^T V
// (rows and columns of tau = 0 vanish).  Out: T[r + 16 c], 256 doubles of LDS.
__device__ __forceinline__ void ts_block_t(const double *V, int ldv, int n, int k0, const double *s_tau,
                                           double *__restrict__ T) {
    const int lane = threadIdx.x & 63, tr = lane & 15, tg = lane >> 4;
    const int kc = k0 + tr < n - 1 ? k0 + tr : n - 2;
    f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    for (int i0 = k0 & ~7; i0 < n; i0 += 8) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = i0 + 4 * u + tg;
            double a = V[(i < n ? i : n - 1) + (int64_t)ldv * kc];
            if (i >= n) a = 0.0;
            acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, acc[u], 0, 0, 0);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) T[(tg + 4 * v) + 16 * tr] = acc[0][v] + acc[1][v];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // column tr of the inverse, from its diagonal upwards (the four lane
    // groups repeat it); G is read before T is overwritten
    double x[16];
    double tau[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) tau[s] = k0 + s < n - 1 ? s_tau[k0 + s] : 0.0;
#pragma unroll
    for (int s = 15; s >= 0; --s) {
        double t = 0.0;
#pragma unroll
        for (int q = s + 1; q < 16; ++q) t = fma(T[s + 16 * q], x[q], t);   // x is zero past column tr
        x[s] = s == tr ? tau[s] : (s < tr ? -tau[s] * t : 0.0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (tg == 0)
#pragma unroll
        for (int s = 0; s < 16; ++s) T[s + 16 * tr] = x[s];
}

template <bool FL, bool VL>
__device__ void ts_body(const double *__restrict__ S, int64_t lds, int n, int R, double *__restrict__ U,
                        int64_t ldu, double *__restrict__ lam, bool sign_rule, double *scV, double *scF,
                        int64_t *__restrict__ flag) {
    extern __shared__ __align__(16) double te_dyn[];
    __shared__ double s_red[TE_W], s_red2[TE_W];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TsLayout L = ts_layout(n, R);
    const int ldz = L.ldz, ldv = L.ldv;
    double *const stg = te_dyn, *const Z = te_dyn;
    double *const F = FL ? te_dyn + L.off_f : scF;
    double *const V = VL ? te_dyn + L.off_v : scV;
    double *const part = te_dyn + L.off_part;           // partial products, then the T blocks
    double *const s_vec = te_dyn + L.off_vec;                  // 4 TE_LDS_N
    double2 *const s_de = (double2 *)(s_vec + 4 * TE_LDS_N);   // TE_LDS_N + 32 pairs
    double *const s_d = s_vec + 4 * TE_LDS_N + 2 * (TE_LDS_N + 32), *const s_e = s_d + TE_LDS_N, *const s_tau = s_e + TE_LDS_N,
                 *const s_re = s_tau + TE_LDS_N, *const s_lam = s_re + TE_LDS_N, *const s_inv = s_lam + TE_LDS_N;

    // ---- the matrix into LDS, its scale ----------------------------------
    double mx = 0.0;
    int bad = 0;
    if (tid == 0) s_bad = 0;
    for (int j = wave; j < n; j += TE_W)
        for (int i = lane; i < n; i += 64) {
            const double v = S[i + lds * j];
            if (!(fabs(v) <= 1.7976931348623157e308)) bad = 1;
            else mx = fmax(mx, fabs(v));
            stg[i + L.sld * j] = v;
        }
    mx = te_wave_max(mx);
    if (lane == 0) s_red[wave] = mx;
    __syncthreads();
    if (bad) s_bad = 1;
    mx = 0.0;
    for (int w = 0; w < TE_W; ++w) mx = fmax(mx, s_red[w]);
    __syncthreads();
    const bool nonfinite = s_bad != 0;
    if (nonfinite && tid == 0 && flag) flag[0] = 3;
    if (mx == 0.0 && !nonfinite) {   // the zero matrix: e_1 .. e_R
        for (int64_t e = tid; e < (int64_t)n * R; e += TE_T) {
            const int i = (int)(e % n), r = (int)(e / n);
            U[i + ldu * r] = (i == r) ? 1.0 : 0.0;
        }
        if (lam)
            for (int r = tid; r < R; r += TE_T) lam[r] = 0.0;
        return;
    }
    const int sexp = (mx > 0.0 && !nonfinite) ? ilogb(mx) : 0;
    const double sc_in = ldexp(1.0, -sexp), sc_out = ldexp(1.0, sexp);

    // ---- 1. tridiagonalization -------------------------------------------
    if (n <= 64) ts_tridiag<1>(stg, L.sld, sc_in, n, V, ldv, part, s_vec, s_d, s_e, s_tau);
    else ts_tridiag<2>(stg, L.sld, sc_in, n, V, ldv, part, s_vec, s_d, s_e, s_tau);
    __syncthreads();

    // ---- 2. bisection for the R largest eigenvalues ----------------------
    double glo = 1e300, ghi = -1e300;
    if (tid < n) {
        const double r = (tid > 0 ? fabs(s_e[tid - 1]) : 0.0) + (tid + 1 < n ? fabs(s_e[tid]) : 0.0);
        glo = s_d[tid] - r;
        ghi = s_d[tid] + r;
    }
    glo = te_wave_min(glo);
    ghi = te_wave_max(ghi);
    if (lane == 0) {
        s_red[wave] = glo;
        s_red2[wave] = ghi;
    }
    __syncthreads();
    glo = fmin(s_red[0], s_red[1]);
    ghi = fmax(s_red2[0], s_red2[1]);   // n <= 128: two waves
    const double tnorm = fmax(fmax(fabs(glo), fabs(ghi)), 1e-300);
    glo -= 4.0 * 2.220446049250313e-16 * tnorm;
    ghi += 4.0 * 2.220446049250313e-16 * tnorm;
    if (tid < n) {
        // e floored at 2^-60 ||T|| (its sign kept): a change of the off-diagonal
        // below 1e-18 ||T||, far under the eps ||T|| accuracy of the pairs
        const double emin = 0x1p-60 * tnorm;
        double em1 = tid > 0 ? fmax(fabs(s_e[tid - 1]), emin) : 0.0;
        s_de[tid] = make_double2(s_d[tid], -em1 * em1);
        double e0 = tid + 1 < n ? s_e[tid] : 1.0;
        if (!(fabs(e0) >= emin)) e0 = e0 < 0.0 ? -emin : emin;
        s_re[tid] = 1.0 / e0;
        s_inv[tid] = e0;   // moved below, once every thread has read s_e
    } else if (tid < n + 32) {
        s_de[tid] = make_double2(0.0, 0.0);   // read ahead by the counts
    }
    __syncthreads();
    if (tid < n) s_e[tid] = tid + 1 < n ? s_inv[tid] : 0.0;
    // (s_e is read by step 3 only, after the next barrier)
    {
        // four waves, one per SIMD.  First the counts at 256 points of the
        // whole interval, which bracket every eigenvalue at once; then a group
        // of tpe lanes splits one eigenvalue's bracket into tpe + 1 parts
        // per round
        int *const s_cnt = (int *)part;
        constexpr int N0 = 256;
        const double w0 = (ghi - glo) * (1.0 / (N0 + 1));
        if (tid < 256) s_cnt[tid] = ts_sturm(s_de, n, fma(w0, (double)(tid + 1), glo));
        __syncthreads();
        int tpe = 64;
        while (tpe > 1 && tpe * R > 256) tpe >>= 1;
        const int r = tid / tpe, t = lane % tpe, sh = lane & ~(tpe - 1);
        const double step = 1.0 / (double)(tpe + 1);
        const unsigned long long mask = tpe == 64 ? ~0ull : ((1ull << tpe) - 1);
        if (tid < 256) {
            // every lane of a wave stays active until its last group is done:
            // the counts broadcast their operands across lanes
            const int kk = n - 1 - (r < R ? r : R - 1);   // the kk-th smallest, 0-based
            int b0 = 0;                                   // points whose count is at most kk
#pragma unroll
            for (int o = N0 / 2; o > 0; o >>= 1)
                if (s_cnt[b0 + o - 1] <= kk) b0 += o;
            if (b0 == N0 - 1 && s_cnt[N0 - 1] <= kk) b0 = N0;
            double lo = b0 > 0 ? fma(w0, (double)b0, glo) : glo;
            double hi = b0 < N0 ? fma(w0, (double)(b0 + 1), glo) : ghi;
            for (int round = 0; round < 64; ++round) {
                const bool open = hi - lo > 2.220446049250313e-16 * (tnorm + fabs(lo) + fabs(hi));
                if (__ballot(open) == 0) break;
                const double wdt = (hi - lo) * step;
                const int cnt = ts_sturm(s_de, n, fma(wdt, (double)(t + 1), lo));
                const int below = __popcll((__ballot(cnt <= kk) >> sh) & mask);
                const double nlo = below > 0 ? fma(wdt, (double)below, lo) : lo;
                const double nhi = below < tpe ? fma(wdt, (double)(below + 1), lo) : hi;
                lo = open ? nlo : lo;
                hi = open ? nhi : hi;
            }
            if (t == 0 && r < R) s_lam[r] = 0.5 * (lo + hi);
        }
    }
    __syncthreads();

    // ---- 3. inverse iteration; the reflector blocks' T -------------------
    {
        const int nzw = (R + 63) / 64;   // waves with a vector
        if (wave < nzw) {
            if (tid < R) {
                // inside a cluster the shift moves off the eigenvalue: (T - shift)^{-1}
                // then weights the whole eigenspace alike, and the vectors' random
                // starts keep them apart (at the same computed eigenvalue they would
                // all turn into one direction, and Gram-Schmidt would magnify their
                // residuals).  By 32 eps ||T|| where the eigenvalues are equal to
                // rounding, well beyond their spread (100 eigenvalues, three values: the
                // residuals reach 2e-13 ||S||, 1e-10 at 4 eps); else by 4, less than the
                // distances within the cluster
                const double ulp = 2.220446049250313e-16 * tnorm;
                double lm = s_lam[tid];
                const double above = tid > 0 ? s_lam[tid - 1] - lm : HUGE_VAL;
                if (above <= 1e-9 * tnorm) lm += (above <= 8.0 * ulp ? 32.0 : 4.0) * ulp;
                ts_inverse(s_de, s_e, s_re, n, R, lm, ulp, tid, F, Z, ldz, s_inv);
            }
        } else if (n > 2) {
            for (int b = wave - nzw; b < L.nb; b += TE_W - nzw) ts_block_t(V, ldv, n, 16 * b, s_tau, part + 256 * b);
        }
    }
    __syncthreads();
    for (int i = wave; i < n; i += TE_W)
        for (int r = lane; r < R; r += 64) Z[i * ldz + r] *= s_inv[r];
    int close = 0;
    if (tid > 0 && tid < R) close = s_lam[tid - 1] - s_lam[tid] <= 1e-9 * tnorm ? 1 : 0;

    // ---- 4a. clusters: classical Gram-Schmidt twice inside each ----------
    if (__syncthreads_or(close)) {
        double *const s_dot = s_vec;
        int c0 = 0;
        for (int j = 1; j < R; ++j) {
            if (!(s_lam[j - 1] - s_lam[j] <= 1e-9 * tnorm)) {
                c0 = j;
                continue;
            }
            for (int pass = 0; pass < 2; ++pass) {
                for (int i = c0 + wave; i < j; i += TE_W) {
                    double s = 0.0;
                    for (int q = lane; q < n; q += 64) s += Z[q * ldz + i] * Z[q * ldz + j];
                    s = te_wave_sum(s);
                    if (lane == 0) s_dot[i] = s;
                }
                __syncthreads();
                if (tid < n) {
                    double acc = Z[tid * ldz + j];
                    for (int i = c0; i < j; ++i) acc -= s_dot[i] * Z[tid * ldz + i];
                    Z[tid * ldz + j] = acc;
                }
                __syncthreads();
            }
            double s = 0.0;
            for (int q = lane; q < n; q += 64) s += Z[q * ldz + j] * Z[q * ldz + j];
            s = te_wave_sum(s);
            const double inv = s > 0.0 ? 1.0 / sqrt(s) : 1.0;
            __syncthreads();
            if (tid < n) Z[tid * ldz + j] *= inv;
            __syncthreads();
        }
    }

    // ---- 4b. Newton-Schulz, back-transformation, sign, output ------------
    const int nt = (R + 15) / 16, ntr = (n + 15) / 16;
    if (wave < nt) {
        constexpr int MT = TE_LDS_N / 16;
        const int tr = lane & 15, tg = lane >> 4, col = 16 * wave + tr;
        f64x4 z[MT];   // rows 16 t + tg + 4 v of column col
#pragma unroll
        for (int t = 0; t < MT; ++t)
            if (t < ntr)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * t + tg + 4 * v;
                    const double x = Z[(i < n ? i : n - 1) * ldz + (col < R ? col : R - 1)];
                    z[t][v] = (i < n && col < R) ? x : 0.0;
                }
        // this wave's columns of G = Z^T Z, then Z <- 1.5 Z - 0.5 Z G
        f64x4 zn[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t)
            if (t < ntr) zn[t] = 1.5 * z[t];
        for (int c = 0; c < nt; ++c) {
            const int ca = 16 * c + tr;
            const double *za = Z + (ca < R ? ca : R - 1);
            f64x4 g0 = {0.0, 0.0, 0.0, 0.0}, g1 = g0;
#pragma unroll
            for (int t = 0; t < MT; ++t)
                if (t < ntr)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = 16 * t + tg + 4 * v;
                        double a = za[(i < n ? i : n - 1) * ldz];
                        if (ca >= R) a = 0.0;
                        if (v & 1) g1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, z[t][v], g1, 0, 0, 0);
                        else g0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, z[t][v], g0, 0, 0, 0);
                    }
            g0 = -0.5 * (g0 + g1);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 16 * c + tg + 4 * v;
                const double *zk = Z + (k < R ? k : R - 1);   // G is zero there
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    if (t < ntr) {
                        const int i = 16 * t + tr;
                        double a = zk[(i < n ? i : n - 1) * ldz];
                        if (i >= n) a = 0.0;
                        zn[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, g0[v], zn[t], 0, 0, 0);
                    }
            }
        }
        // Z <- (I - V_b T_b V_b^T) Z from the last block of reflectors
        if (n > 2)
            for (int b = L.nb - 1; b >= 0; --b) {
                const int kc = 16 * b + tr < n - 1 ? 16 * b + tr : n - 2;   // columns past the last have no row in T
                const double *vk = V + (int64_t)ldv * kc;
                f64x4 p0 = {0.0, 0.0, 0.0, 0.0}, p1 = p0;
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    if (t >= b && t < ntr)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int i = 16 * t + tg + 4 * v;
                            const double a = vk[i < n ? i : n - 1];   // Z is zero past row n
                            if (v & 1) p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, zn[t][v], p1, 0, 0, 0);
                            else p0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, zn[t][v], p0, 0, 0, 0);
                        }
                p0 += p1;
                f64x4 wv = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    wv = __builtin_amdgcn_mfma_f64_16x16x4f64(part[256 * b + tr + 16 * (tg + 4 * v)], p0[v], wv, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int kv = 16 * b + tg + 4 * v < n - 1 ? 16 * b + tg + 4 * v : n - 2;
                    const double *vr = V + (int64_t)ldv * kv;
#pragma unroll
                    for (int t = 0; t < MT; ++t)
                        if (t >= b && t < ntr) {
                            const int i = 16 * t + tr;
                            double a = -vr[i < n ? i : n - 1];
                            if (i >= n) a = 0.0;
                            zn[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, wv[v], zn[t], 0, 0, 0);
                        }
                }
            }
        // sign rule: the entry of largest magnitude of the column (rows tg +
        // 4 m of this lane, then the four lane groups; first index on ties)
        double best = -1.0, bval = 0.0;
        int arg = 0;
#pragma unroll
        for (int t = 0; t < MT; ++t)
            if (t < ntr)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double a = fabs(zn[t][v]);
                    if (a > best) {
                        best = a;
                        bval = zn[t][v];
                        arg = 16 * t + tg + 4 * v;
                    }
                }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const double b2 = __shfl_xor(best, o), v2 = __shfl_xor(bval, o);
            const int a2 = __shfl_xor(arg, o);
            if (b2 > best || (b2 == best && a2 < arg)) {
                best = b2;
                bval = v2;
                arg = a2;
            }
        }
        const double sg = sign_rule && bval < 0.0 ? -1.0 : 1.0;
        if (col < R) {
#pragma unroll
            for (int t = 0; t < MT; ++t)
                if (t < ntr)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = 16 * t + tg + 4 * v;
                        if (i < n) U[i + ldu * col] = sg * zn[t][v];
                    }
            if (lam && tg == 0) lam[col] = s_lam[col] * sc_out;
        }
    }
}

// R leading eigenpairs for n <= TE_LDS_N (dynamic LDS of ts_layout(n, R).bytes;
// scratch of teig_scratch_doubles(n, R, true) doubles).
__device__ __forceinline__ void teig_small(const double *S, int64_t lds, int n, int R, double *U, int64_t ldu,
                                           double *lam, bool sign_rule, const TeScratch &sc, int64_t *flag) {
    const TsLayout L = ts_layout(n, R);   // uniform
    if (L.vl) ts_body<true, true>(S, lds, n, R, U, ldu, lam, sign_rule, sc.Vr, sc.F, flag);
    else if (L.fl) ts_body<true, false>(S, lds, n, R, U, ldu, lam, sign_rule, sc.Vr, sc.F, flag);
    else ts_body<false, false>(S, lds, n, R, U, ldu, lam, sign_rule, sc.Vr, sc.F, flag);
}

// dynamic LDS of a solve
__host__ __device__ inline size_t teig_lds_bytes(int64_t n, int64_t R) {
    return n <= TE_LDS_N ? ts_layout((int)n, (int)R).bytes : te_big_lds_bytes(n, R, teig_z_fits(n, R));
}

// ---- orders above TE_LDS_N -------------------------------------------------
// R leading eigenpairs of the symmetric n x n matrix S (column-major,
// leading dimension lds; (S + S^T) / 2 is used), n > TE_LDS_N.  U (n x R,
// leading dimension ldu) receives the eigenvectors, lam (R, may be NULL) the
// eigenvalues in descending order.  A lives in the scratch; ZLDS: the
// eigenvector block in LDS (teig_z_fits).
template <bool ZLDS>
__device__ void teig_body(const double *__restrict__ S, int64_t lds, int n, int R, double *__restrict__ U,
                          int64_t ldu, double *__restrict__ lam, bool sign_rule, TeScratch sc,
                          int64_t *__restrict__ flag) {
    extern __shared__ __align__(16) double te_dyn[];
    __shared__ double s_red[TE_W], s_red2[TE_W];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t nn = (int64_t)n * n;
    int64_t main_sz = 0;
    if (ZLDS && (int64_t)n * R > main_sz) main_sz = (int64_t)n * R;
    double *const A = sc.Ag;                            // column-major, leading dimension n
    double *const part = te_dyn + main_sz;              // te_part_doubles(n)
    double *const s_v = part + te_part_doubles(n);      // 2 n (double-buffered reflector)
    double2 *const s_vw = (double2 *)(s_v + 2 * n);     // n pairs (v, w) of the last step
    double *const s_p = s_v + 4 * n;                    // n (p of the last step; later e^2)
    double *const s_d = s_p + n;                        // n
    double *const s_e = s_d + n;                        // n
    double *const s_tau = s_e + n;                      // n
    double *const s_lam = s_tau + n;                    // R
    int *const s_cs = (int *)(s_lam + R);               // R cluster starts
    double *const Z = ZLDS ? te_dyn : sc.Zg;   // row-major n x R (after step 1)
    const double *const Vr = A;   // column k of A holds v_k below the diagonal

    // ---- scale by a power of two, load (S + S^T) / 2 --------------------
    double mx = 0.0;
    int bad = 0;
    for (int64_t e = tid; e < nn; e += TE_T) {
        const double v = S[(e % n) + lds * (e / n)];
        if (!(fabs(v) <= 1.7976931348623157e308)) bad = 1;
        else mx = fmax(mx, fabs(v));
    }
    if (tid == 0) s_bad = 0;
    mx = te_wave_max(mx);
    if (lane == 0) s_red[wave] = mx;
    __syncthreads();
    if (bad) s_bad = 1;
    mx = 0.0;
    for (int w = 0; w < TE_W; ++w) mx = fmax(mx, s_red[w]);
    __syncthreads();
    const bool nonfinite = s_bad != 0;
    if (nonfinite && tid == 0 && flag) flag[0] = 3;
    if (mx == 0.0 && !nonfinite) {   // the zero matrix: e_1 .. e_R
        for (int64_t e = tid; e < (int64_t)n * R; e += TE_T) {
            const int i = (int)(e % n), r = (int)(e / n);
            U[i + ldu * r] = (i == r) ? 1.0 : 0.0;
        }
        if (lam)
            for (int r = tid; r < R; r += TE_T) lam[r] = 0.0;
        return;
    }
    const int sexp = (mx > 0.0 && !nonfinite) ? ilogb(mx) : 0;
    const double sc_in = ldexp(1.0, -sexp), sc_out = ldexp(1.0, sexp);
    for (int64_t e = tid; e < nn; e += TE_T) {
        const int i = (int)(e % n), j = (int)(e / n);
        A[e] = 0.5 * (S[i + lds * j] + S[j + lds * i]) * sc_in;
    }
    __syncthreads();

    // ---- 1. tridiagonalization -------------------------------------------
    {
        // Per step k two barriers: wave 0 first turns the partial sums of step
        // k - 1 into p = tau A v and K = (tau / 2) p^T v, forms (v, w) of step
        // k - 1, updates column k and builds H_k; then every wave applies step
        // k - 1's update to the trailing block and accumulates A v_k.
        constexpr int TU = 4;   // columns per thread whose loads are issued together
        double Kprev = 0.0;
        for (int k = 0; k + 2 < n; ++k) {
            double *const vc = s_v + (k & 1) * n;
            const double *const vp = s_v + ((k & 1) ^ 1) * n;
            if (wave == 0) {
                if (k > 0) {
                    const double taup = s_tau[k - 1];
                    double t = 0.0;
                    for (int i = k + lane; i < n; i += 64) {
                        double sp = 0.0;
#pragma unroll
                        for (int w = 0; w < TE_W; ++w) sp += part[w * n + i];
                        const double p = taup * sp;
                        s_p[i] = p;
                        t += p * vp[i];
                    }
                    Kprev = 0.5 * taup * te_wave_sum(t);
                }
                // (v, w) of step k - 1 for rows >= k, column k with that step's
                // pending update, then H_k
                double sig = 0.0, a0 = 0.0;
                double wpk = 0.0, vpk = 0.0;
                if (k > 0) {
                    vpk = vp[k];
                    wpk = s_p[k] - Kprev * vpk;
                }
                for (int i = k + lane; i < n; i += 64) {
                    double a = A[i + (int64_t)n * k];
                    if (k > 0) {
                        const double vpi = vp[i], wpi = s_p[i] - Kprev * vpi;
                        s_vw[i] = make_double2(vpi, wpi);
                        a -= vpi * wpk + wpi * vpk;
                    }
                    if (i >= k + 2) sig += a * a;
                    if (i == k + lane && lane < 2) a0 = a;
                    part[i] = a;
                }
                sig = te_wave_sum(sig);
                const double akk = te_lane(a0, 0), x0 = te_lane(a0, 1);
                double beta = x0, tau = 0.0, scl = 0.0;
                if (sig > 0.0) {
                    const double nrm = sqrt(x0 * x0 + sig);
                    beta = x0 >= 0.0 ? -nrm : nrm;
                    tau = (beta - x0) / beta;
                    scl = 1.0 / (x0 - beta);
                }
                for (int i = k + 1 + lane; i < n; i += 64) {
                    const double v = (i == k + 1) ? 1.0 : (tau == 0.0 ? 0.0 : part[i] * scl);
                    vc[i] = v;
                    A[i + (int64_t)n * k] = v;   // column k is not read again by the reduction
                }
                if (lane == 0) {
                    s_d[k] = akk;
                    s_e[k] = beta;
                    s_tau[k] = tau;
                }
            }
            __syncthreads();
            // trailing block: pending update of step k - 1, and partial sums of A v_k
            for (int i0 = k + 1; i0 < n; i0 += 64) {
                const int i = i0 + lane;
                if (i < n) {
                    double acc = 0.0;
                    double2 pwi = make_double2(0.0, 0.0);
                    if (k > 0) pwi = s_vw[i];
                    for (int jb = k + 1 + wave; jb < n; jb += TE_W * TU) {
                        double a[TU], vcj[TU];
                        double2 pw[TU];
#pragma unroll
                        for (int u = 0; u < TU; ++u) {
                            const int j = jb + TE_W * u;
                            const int jc = j < n ? j : n - 1;
                            a[u] = A[i + (int64_t)n * jc];
                            vcj[u] = j < n ? vc[jc] : 0.0;
                            pw[u] = (k > 0) ? s_vw[jc] : make_double2(0.0, 0.0);
                        }
#pragma unroll
                        for (int u = 0; u < TU; ++u) {
                            const int j = jb + TE_W * u;
                            if (k > 0) {
                                a[u] -= pwi.x * pw[u].y + pwi.y * pw[u].x;
                                if (j < n) A[i + (int64_t)n * j] = a[u];
                            }
                            acc += a[u] * vcj[u];
                        }
                    }
                    part[wave * n + i] = acc;
                }
            }
            __syncthreads();
        }
        if (wave == 0) {
            // p and K of the last step (n - 3)
            const double taup = s_tau[n - 3];
            const double *vp = s_v + ((n - 3) & 1) * n;
            double t = 0.0;
            for (int i = n - 2 + lane; i < n; i += 64) {
                double sp = 0.0;
#pragma unroll
                for (int w = 0; w < TE_W; ++w) sp += part[w * n + i];
                const double p = taup * sp;
                s_p[i] = p;
                t += p * vp[i];
            }
            Kprev = 0.5 * taup * te_wave_sum(t);
        }
        if (tid == 0) {
            // the last 2 x 2 block with the update of step n - 3
            const double *v = s_v + ((n - 3) & 1) * n;
            const double v1 = v[n - 2], v2 = v[n - 1];
            const double w1 = s_p[n - 2] - Kprev * v1, w2 = s_p[n - 1] - Kprev * v2;
            s_d[n - 2] = A[(n - 2) + (int64_t)n * (n - 2)] - 2.0 * v1 * w1;
            s_e[n - 2] = A[(n - 1) + (int64_t)n * (n - 2)] - (v2 * w1 + w2 * v1);
            s_d[n - 1] = A[(n - 1) + (int64_t)n * (n - 1)] - 2.0 * v2 * w2;
        }
        __syncthreads();
    }

    // ---- 2. bisection for the R largest eigenvalues ----------------------
    double glo = 1e300, ghi = -1e300;
    for (int i = tid; i < n; i += TE_T) {
        const double r = (i > 0 ? fabs(s_e[i - 1]) : 0.0) + (i + 1 < n ? fabs(s_e[i]) : 0.0);
        glo = fmin(glo, s_d[i] - r);
        ghi = fmax(ghi, s_d[i] + r);
    }
    glo = te_wave_min(glo);
    ghi = te_wave_max(ghi);
    if (lane == 0) {
        s_red[wave] = glo;
        s_red2[wave] = ghi;
    }
    __syncthreads();
    glo = s_red[0];
    ghi = s_red2[0];
    for (int w = 1; w < TE_W; ++w) {
        glo = fmin(glo, s_red[w]);
        ghi = fmax(ghi, s_red2[w]);
    }
    const double tnorm = fmax(fmax(fabs(glo), fabs(ghi)), 1e-300);
    glo -= 4.0 * 2.220446049250313e-16 * tnorm;
    ghi += 4.0 * 2.220446049250313e-16 * tnorm;
    {
        // e^2, floored at (2^-60 ||T||)^2: a change of the off-diagonal below
        // 1e-18 ||T||, far under the eps ||T|| accuracy of the eigenvalues
        const double e2min = 0x1p-120 * tnorm * tnorm;
        for (int i = tid; i + 1 < n; i += TE_T) s_p[i] = fmax(s_e[i] * s_e[i], e2min);
    }
    __syncthreads();
    {
        // a group of tpe lanes searches one eigenvalue, TE_NC points per lane:
        // each round splits the bracket into tpe * TE_NC + 1 parts.  Groups
        // cover at most 256 lanes (one wave per SIMD) at a time: more lanes
        // would only add FP64 work per round (the counts, not their latency,
        // bound the search)
        int tpe = 64;
        while (tpe > 1 && tpe * R > 256) tpe >>= 1;   // at most four waves: the counts are FP64-throughput bound
        const int ngroups = TE_T / tpe, g = tid / tpe, t = tid % tpe;
        const double npts1 = (double)(tpe * TE_NC + 1);
        const int rounds_r = (R + ngroups - 1) / ngroups;
        for (int rr = 0; rr < rounds_r; ++rr) {
            const int r = g + rr * ngroups;
            if (r < R) {   // uniform within the group
                const int kk = n - 1 - r;   // the kk-th smallest, 0-based
                double lo = glo, hi = ghi;
                for (int round = 0; round < 64; ++round) {
                    if (!(hi - lo > 2.220446049250313e-16 * (tnorm + fabs(lo) + fabs(hi)))) break;
                    double sig[TE_NC];
                    int cnt[TE_NC];
#pragma unroll
                    for (int c = 0; c < TE_NC; ++c) sig[c] = lo + (hi - lo) * (double)(t * TE_NC + c + 1) / npts1;
                    te_sturm(s_d, s_p, n, sig, cnt);
                    double nlo = -HUGE_VAL, nhi = HUGE_VAL;
#pragma unroll
                    for (int c = 0; c < TE_NC; ++c) {
                        if (cnt[c] <= kk) nlo = fmax(nlo, sig[c]);
                        else nhi = fmin(nhi, sig[c]);
                    }
                    for (int o = 1; o < tpe; o <<= 1) {
                        nlo = fmax(nlo, __shfl_xor(nlo, o));
                        nhi = fmin(nhi, __shfl_xor(nhi, o));
                    }
                    lo = fmax(lo, nlo);
                    hi = fmin(hi, nhi);
                }
                if (t == 0) s_lam[r] = 0.5 * (lo + hi);
            }
        }
    }
    __syncthreads();

    // ---- 3. inverse iteration, one thread per eigenvector ----------------
    {
        const double tiny = 2.220446049250313e-16 * tnorm;
        double *__restrict__ F = sc.F;
        double *__restrict__ Zr = Z;
        for (int r = tid; r < R; r += TE_T) {
            const double lm = s_lam[r];
            double nrm2 = 0.0;
            for (int i = 0; i < n; ++i) {
                const double b = te_start(r, i);
                Zr[(int64_t)i * R + r] = b;
                nrm2 += b * b;
            }
            for (int pass = 0; pass < 2; ++pass) {
                const double inv = te_rcp(sqrt(nrm2));
                // forward elimination with partial pivoting: U rows (1 / u0, u1, u2) to F, y to Z
                double cd = s_d[0] - lm, cu = s_e[0], cb = Zr[r] * inv;
#pragma unroll 4
                for (int i = 0; i + 1 < n; ++i) {
                    const double sub = s_e[i], nd = s_d[i + 1] - lm, nu = i + 2 < n ? s_e[i + 1] : 0.0;
                    const double nb = Zr[(int64_t)(i + 1) * R + r] * inv;
                    double ru0, u1, u2, y;
                    if (fabs(cd) >= fabs(sub)) {
                        if (cd == 0.0) cd = tiny;
                        ru0 = te_rcp(cd);
                        const double ml = sub * ru0;
                        u1 = cu;
                        u2 = 0.0;
                        y = cb;
                        cd = nd - ml * cu;
                        cu = nu;
                        cb = nb - ml * cb;
                    } else {
                        ru0 = te_rcp(sub);
                        const double ml = cd * ru0;
                        u1 = nd;
                        u2 = nu;
                        y = nb;
                        cd = cu - ml * nd;
                        cu = -ml * nu;
                        cb = cb - ml * nb;
                    }
                    F[(int64_t)(3 * i) * R + r] = ru0;
                    F[(int64_t)(3 * i + 1) * R + r] = u1;
                    F[(int64_t)(3 * i + 2) * R + r] = u2;
                    Zr[(int64_t)i * R + r] = y;
                }
                if (cd == 0.0) cd = tiny;
                // back substitution, the factors of 4 rows loaded ahead
                double x1 = cb * te_rcp(cd), x2 = 0.0;
                Zr[(int64_t)(n - 1) * R + r] = x1;
                nrm2 = x1 * x1;
                for (int i0 = n - 2; i0 >= 0; i0 -= 4) {
                    double f0[4], f1[4], f2[4], y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int i = i0 - u >= 0 ? i0 - u : 0;
                        f0[u] = F[(int64_t)(3 * i) * R + r];
                        f1[u] = F[(int64_t)(3 * i + 1) * R + r];
                        f2[u] = F[(int64_t)(3 * i + 2) * R + r];
                        y[u] = Zr[(int64_t)i * R + r];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (i0 - u < 0) break;
                        const double x = (y[u] - f1[u] * x1 - f2[u] * x2) * f0[u];
                        Zr[(int64_t)(i0 - u) * R + r] = x;
                        nrm2 += x * x;
                        x2 = x1;
                        x1 = x;
                    }
                }
            }
            const double inv = te_rcp(sqrt(nrm2));
            for (int i = 0; i < n; ++i) Zr[(int64_t)i * R + r] *= inv;
        }
    }
    __syncthreads();

    // ---- 4a. clusters: classical Gram-Schmidt twice inside each ----------
    if (tid == 0) {
        int cs = 0;
        s_cs[0] = 0;
        for (int r = 1; r < R; ++r) {
            if (!(s_lam[r - 1] - s_lam[r] <= 1e-9 * tnorm)) cs = r;
            s_cs[r] = cs;
        }
    }
    __syncthreads();
    for (int j = 1; j < R; ++j) {
        const int c0 = s_cs[j];
        if (c0 == j) continue;
        for (int pass = 0; pass < 2; ++pass) {
            for (int i = c0 + wave; i < j; i += TE_W) {
                double s = 0.0;
                for (int q = lane; q < n; q += 64) s += Z[(int64_t)q * R + i] * Z[(int64_t)q * R + j];
                s = te_wave_sum(s);
                if (lane == 0) part[i] = s;
            }
            __syncthreads();
            for (int q = tid; q < n; q += TE_T) {
                double acc = Z[(int64_t)q * R + j];
                for (int i = c0; i < j; ++i) acc -= part[i] * Z[(int64_t)q * R + i];
                Z[(int64_t)q * R + j] = acc;
            }
            __syncthreads();
        }
        double s = 0.0;
        for (int q = tid; q < n; q += TE_T) s += Z[(int64_t)q * R + j] * Z[(int64_t)q * R + j];
        s = te_wave_sum(s);
        if (lane == 0) s_red[wave] = s;
        __syncthreads();
        s = 0.0;
        for (int w = 0; w < TE_W; ++w) s += s_red[w];
        const double inv = s > 0.0 ? 1.0 / sqrt(s) : 1.0;
        for (int q = tid; q < n; q += TE_T) Z[(int64_t)q * R + j] *= inv;
        __syncthreads();
    }

    // ---- 4b. one Newton-Schulz step on the FP64 matrix cores -------------
    {
        const int tr = lane & 15, tg = lane >> 4;
        const int nt = (R + 15) / 16, ntr = (n + 15) / 16;
        // G = Z^T Z (tiles bi <= bj, mirrored)
        for (int q = wave; q < nt * (nt + 1) / 2; q += TE_W) {
            int bi = 0;
            while ((bi + 1) * nt - bi * (bi + 1) / 2 <= q) ++bi;
            const int bj = bi + q - (bi * nt - bi * (bi - 1) / 2);
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
            const int ra = 16 * bi + tr, cb = 16 * bj + tr;
            for (int k0 = 0; k0 < n; k0 += 4) {
                const int k = k0 + tg;
                const double a = (ra < R && k < n) ? Z[(int64_t)k * R + ra] : 0.0;
                const double b = (cb < R && k < n) ? Z[(int64_t)k * R + cb] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * bi + tg + 4 * v;
                if (row < R && cb < R) {
                    sc.G[row + (int64_t)R * cb] = acc[v];
                    sc.G[cb + (int64_t)R * row] = acc[v];
                }
            }
        }
        __syncthreads();
        // Znew = 1.5 Z - 0.5 Z G into the staging buffer (row tile per task)
        double *const Zs = ZLDS ? sc.Zg : sc.F;
        for (int q = wave; q < ntr * nt; q += TE_W) {
            const int bi = q / nt, bj = q % nt;
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
            const int ra = 16 * bi + tr, cb = 16 * bj + tr;
            for (int k0 = 0; k0 < R; k0 += 4) {
                const int k = k0 + tg;
                const double a = (ra < n && k < R) ? Z[(int64_t)ra * R + k] : 0.0;
                const double b = (k < R && cb < R) ? sc.G[k + (int64_t)R * cb] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * bi + tg + 4 * v;
                if (row < n && cb < R) Zs[(int64_t)row * R + cb] = 1.5 * Z[(int64_t)row * R + cb] - 0.5 * acc[v];
            }
        }
        __syncthreads();
        for (int64_t e = tid; e < (int64_t)n * R; e += TE_T) Z[e] = Zs[e];
        __syncthreads();
    }

    // ---- 5. back-transformation ------------------------------------------
    {
        // Each wave owns the rows i = wave (mod 8) of Z, so the only exchange is
        // the partial dot products (double-buffered).  The reflectors of the applied steps k_0 > k_1 > ... (tau != 0) are staged from the scratch
        // into three LDS buffers two steps ahead: step t issues the loads of
        // v_{k_{t+2}} right after its barrier and stores them after its update
        // (so their latency overlaps the update and the next step's dot products;
        // a barrier waits for every load in flight), the barrier of step t + 1
        // orders the stores before their use, and the buffer they overwrite was
        // last read in step t - 1, which every wave finished before the barrier
        // of step t.
        {
            double *const s_vb = s_v;   // 3 n doubles (the vectors of step 1 are dead)
            auto next_k = [&](int k) {
                while (k >= 0 && s_tau[k] == 0.0) --k;
                return k;
            };
            const int nper = (n + TE_T - 1) / TE_T;   // staged entries per thread (n <= 4 * TE_T)
            for (int rc = 0; rc < R; rc += 64) {
                const int r = rc + lane;
                const bool rv = r < R;
                int kc = next_k(n - 3);
                int kn = kc >= 0 ? next_k(kc - 1) : -1;
                int kf = kn >= 0 ? next_k(kn - 1) : -1;   // staged two steps ahead
                if (kc >= 0)
                    for (int i = kc + 1 + tid; i < n; i += TE_T) s_vb[i] = Vr[i + (int64_t)n * kc];
                if (kn >= 0)
                    for (int i = kn + 1 + tid; i < n; i += TE_T) s_vb[n + i] = Vr[i + (int64_t)n * kn];
                __syncthreads();
                int buf = 0, par = 0;
                while (kc >= 0) {
                    const double *v = s_vb + buf * n;
                    const double tau = s_tau[kc];
                    const int i0 = kc + 1 + (((wave - kc - 1) % TE_W) + TE_W) % TE_W;
                    // rows i0, i0 + 8, ... in batches of 4 whose loads are issued
                    // together (indices clamped; the extra terms are multiplied by 0)
                    double sacc = 0.0;
                    if (rv)
                        for (int i = i0; i < n; i += 4 * TE_W) {
                            double vv[4], zz[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const int ii = i + u * TE_W, ic = ii < n ? ii : n - 1;
                                vv[u] = ii < n ? v[ic] : 0.0;
                                zz[u] = Z[(int64_t)ic * R + r];
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u) sacc += vv[u] * zz[u];
                        }
                    double *pb = part + par * (TE_W * 64);
                    pb[wave * 64 + lane] = sacc;
                    __syncthreads();
                    double pre[4];
                    if (kf >= 0) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int i = tid + q * TE_T;
                            pre[q] = (q < nper && i > kf && i < n) ? Vr[i + (int64_t)n * kf] : 0.0;
                        }
                    }
                    double c = 0.0;
#pragma unroll
                    for (int w = 0; w < TE_W; ++w) c += pb[w * 64 + lane];
                    c *= tau;
                    if (rv)
                        for (int i = i0; i < n; i += 4 * TE_W) {
                            double vv[4], zz[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const int ii = i + u * TE_W, ic = ii < n ? ii : n - 1;
                                vv[u] = v[ic];
                                zz[u] = Z[(int64_t)ic * R + r];
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                if (i + u * TE_W < n) Z[(int64_t)(i + u * TE_W) * R + r] = zz[u] - c * vv[u];
                        }
                    if (kf >= 0) {
                        double *vf = s_vb + ((buf + 2) % 3) * n;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int i = tid + q * TE_T;
                            if (q < nper && i > kf && i < n) vf[i] = pre[q];
                        }
                    }
                    kc = kn;
                    kn = kf;
                    kf = kf >= 0 ? next_k(kf - 1) : -1;
                    buf = (buf + 1) % 3;
                    par ^= 1;
                }
                __syncthreads();
            }
        }
    }

    // ---- 6. sign rule and output -----------------------------------------
    double *const s_sgn = part;
    for (int r = tid; r < R; r += TE_T) {
        double best = -1.0;
        int arg = 0;   // in range even when every entry is NaN
        for (int i = 0; i < n; ++i) {
            const double v = fabs(Z[(int64_t)i * R + r]);
            if (v > best) {
                best = v;
                arg = i;
            }
        }
        s_sgn[r] = (sign_rule && Z[(int64_t)arg * R + r] < 0.0) ? -1.0 : 1.0;
        if (lam) lam[r] = s_lam[r] * sc_out;
    }
    __syncthreads();
    for (int64_t e = tid; e < (int64_t)n * R; e += TE_T) {
        const int i = (int)(e % n), r = (int)(e / n);
        U[i + ldu * r] = s_sgn[r] * Z[(int64_t)i * R + r];
    }
}

}  // namespace sth
