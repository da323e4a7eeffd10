// Device bodies of the Gram / TTT kernels (one workgroup each), shared by the
// single-tensor kernels and the batched ones.
#pragma once
#include "common.h"
#include <type_traits>

namespace sth {

constexpr int GRAM_FLUSH = 4;  // chunks of 32 rows accumulated in FP32 before an FP64 flush

// Position of an octet of rows p0 .. p0 + 7 of a (L, I, M) tensor: p0 = a + L b.
struct GramPos {
    int64_t a, b;
};

// Loads the 8 consecutive rows p0..p0+7 of column i (clamped) of a (L, I, M)
// tensor, pos the place of p0; rows from pend on repeat an earlier one.  The
// values are masked when they are stored (gram_mask): a select or a branch here
// would wait for its loads before the chunk in hand is multiplied.  VEC: the
// octet is one contiguous run (L a multiple of 8, as p0 is, or a chunk within a
// fibre) or lies wholly past pend.
template <typename T, bool VEC>
__device__ __forceinline__ void gram_load_octet(const T *__restrict__ X, int64_t L, int64_t I,
                                                int64_t i, GramPos pos, int64_t p0, int64_t pend, T (&x)[8]) {
    const int64_t ic = min(i, I - 1);
    if constexpr (VEC) {
        __builtin_memcpy(x, X + (p0 < pend ? pos.a + L * (ic + I * pos.b) : L * ic), sizeof(x));
    } else {
        const T *src = X + (p0 < pend ? pos.a + L * (ic + I * pos.b) : L * ic);
        int64_t a = pos.a;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = *src;
            const bool wrap = a + 1 == L;
            const int64_t d = wrap ? L * (I - 1) + 1 : 1;   // the next row of the same column
            a = wrap ? 0 : a + 1;
            src += p0 + j + 1 < pend ? d : 0;
        }
    }
}

// Zeroes the rows of an octet from pend on.
template <typename T>
__device__ __forceinline__ void gram_mask(int64_t p0, int64_t pend, T (&x)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (p0 + j >= pend) x[j] = (T)0;
}

// Unit u of a TB x 32 slab (TB columns i, 4 octets of rows).  Lanes run along
// i when L = 1 (contiguous in memory), along the octets otherwise.
__device__ __forceinline__ void gram_unit(int u, int TB, bool lfast, int &il, int &oct) {
    if (lfast) {
        il = u % TB;
        oct = u / TB;
    } else {
        oct = u & 3;
        il = u >> 2;
    }
}

// XCD-aware mapping of a launch of total_wg workgroups: consecutive logical
// ids (same row range, all blocks) land on the same XCD.
__device__ __forceinline__ int64_t xcd_logical_id(int64_t total_wg) {
    const int64_t per_xcd = (total_wg + 7) / 8;
    return (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
}

// One workgroup of the Gram/TTT: logical id lid = row range * nblocks + block.
// The next chunk's loads are in flight while one is multiplied; they are taken
// unmasked and their place in the tensor is carried along (no division per
// chunk).  512^3's later modes in bf16x6: 96 us each (108 with a branch and a
// division at each octet's load, which waited for the loads at once).
//
// FIBRES (L no multiple of 8): the octets of a chunk that lies within one fibre
// are loaded whole, the others value by value.
template <typename T, int PREC, int WT, bool SYM, bool FIBRES = false>
__device__ __forceinline__ void gram_body(const T *__restrict__ A, const T *__restrict__ B,
                                          int64_t L, int64_t IA, int64_t IB, int64_t P,
                                          int64_t kper, int nkc, int nbi, int nbj, int nblocks,
                                          int64_t total_wg, int64_t lid,
                                          double *__restrict__ partials) {
    constexpr int TB = 32 * WT;                 // block edge
    constexpr int NQ = Frag<PREC>::NQ;
    constexpr int UNITS = TB * 4;               // octets per slab
    constexpr int UPT = (UNITS + 255) / 256;    // octets per thread per slab
    typedef typename Acc<PREC>::type AccT;
    constexpr bool F64ACC = (PREC == P_FP64);

    // LDS: slab A then slab B, each [q][il][oct] quads
    extern __shared__ uint4 s_g[];
    uint4 *sA = s_g;
    uint4 *sB = s_g + NQ * TB * 4;

    if (lid >= total_wg) return;
    const int kc = (int)(lid / nblocks);
    const int q = (int)(lid - (int64_t)kc * nblocks);
    int bi, bj;
    if (SYM) {
        // lower-triangle enumeration: q -> (bi >= bj)
        bi = 0;
        while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
        bj = q - bi * (bi + 1) / 2;
    } else {
        bi = q % nbi;
        bj = q / nbi;
    }
    const bool diag = SYM && (bi == bj);
    const int64_t i0 = (int64_t)bi * TB, j0 = (int64_t)bj * TB;
    const int64_t pbeg = (int64_t)kc * kper;
    const int64_t pend = min(P, pbeg + kper);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = wave >> 1, wj = wave & 1;
    const bool active = !(diag && wi < wj);
    const bool lfast = (L == 1);

    AccT acc[WT][WT];
    f64x4 acc64[WT][WT];
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
        for (int y = 0; y < WT; ++y) {
            acc[x][y] = AccT{0, 0, 0, 0};
            acc64[x][y] = f64x4{0, 0, 0, 0};
        }

    T ra[UPT][8], rb[UPT][8];
    // units past the slab (one-tile blocks) repeat its last octet
    int il[UPT], oct[UPT];
    GramPos pos[UPT];
    const int64_t q32 = KC / L, r32 = KC - q32 * L;   // a chunk further: a += r32, b += q32
#pragma unroll
    for (int s = 0; s < UPT; ++s) {
        gram_unit(min((int)threadIdx.x + 256 * s, UNITS - 1), TB, lfast, il[s], oct[s]);
        const int64_t p = pbeg + 8 * oct[s];
        pos[s].b = p / L;
        pos[s].a = p - pos[s].b * L;
    }
    auto step = [&](GramPos &p) {   // a chunk further
        p.a += r32;
        p.b += q32;
        if (p.a >= L) {
            p.a -= L;
            ++p.b;
        }
    };
    int64_t ca = FIBRES ? pbeg - pbeg / L * L : 0;   // the chunk's place in its fibre
    auto load_octets = [&](int64_t pc, auto vec) {
        constexpr bool VEC = decltype(vec)::value;
#pragma unroll
        for (int s = 0; s < UPT; ++s) {
            gram_load_octet<T, VEC>(A, L, IA, i0 + il[s], pos[s], pc + 8 * oct[s], pend, ra[s]);
            if (!diag) gram_load_octet<T, VEC>(B, L, IB, j0 + il[s], pos[s], pc + 8 * oct[s], pend, rb[s]);
            if constexpr (!FIBRES) step(pos[s]);
        }
    };
    auto load_slab = [&](int64_t pc, auto vec) {
        if constexpr (FIBRES) {
            if (ca + KC <= L && pc + KC <= pend) load_octets(pc, std::true_type());   // the same for the whole workgroup
            else load_octets(pc, std::false_type());
            ca += r32;
            if (ca >= L) ca -= L;
#pragma unroll
            for (int s = 0; s < UPT; ++s) step(pos[s]);
        } else {
            load_octets(pc, vec);
        }
    };
    auto store_slab = [&](int64_t pc) {
        const bool ragged = pc + KC > pend;
#pragma unroll
        for (int s = 0; s < UPT; ++s) {
            if (threadIdx.x + 256 * s < UNITS) {
                if (ragged) {
                    gram_mask(pc + 8 * oct[s], pend, ra[s]);
                    if (!diag) gram_mask(pc + 8 * oct[s], pend, rb[s]);
                }
                FragQ<PREC> f;
                make_frag(ra[s], f.f);
#pragma unroll
                for (int qq = 0; qq < NQ; ++qq) sA[(qq * TB + il[s]) * 4 + oct[s]] = f.q[qq];
                if (!diag) {
                    make_frag(rb[s], f.f);
#pragma unroll
                    for (int qq = 0; qq < NQ; ++qq) sB[(qq * TB + il[s]) * 4 + oct[s]] = f.q[qq];
                }
            }
        }
    };

    const int nch = (int)((pend - pbeg + KC - 1) / KC);
    const uint4 *sBr = diag ? sA : sB;
    auto run = [&](auto vec) {
    if (nch > 0) load_slab(pbeg, vec);
    for (int c = 0; c < nch; ++c) {
        __syncthreads();  // previous chunk's reads are done
        store_slab(pbeg + (int64_t)c * KC);
        __syncthreads();
        if (c + 1 < nch) load_slab(pbeg + (int64_t)(c + 1) * KC, vec);
        if (active) {
            Frag<PREC> fa[WT], fb[WT];
#pragma unroll
            for (int x = 0; x < WT; ++x) {
                FragQ<PREC> t;
                const int il = wi * (16 * WT) + 16 * x + (lane & 15);
#pragma unroll
                for (int qq = 0; qq < NQ; ++qq) t.q[qq] = sA[(qq * TB + il) * 4 + (lane >> 4)];
                fa[x] = t.f;
            }
#pragma unroll
            for (int y = 0; y < WT; ++y) {
                FragQ<PREC> t;
                const int jl = wj * (16 * WT) + 16 * y + (lane & 15);
#pragma unroll
                for (int qq = 0; qq < NQ; ++qq) t.q[qq] = sBr[(qq * TB + jl) * 4 + (lane >> 4)];
                fb[y] = t.f;
            }
#pragma unroll
            for (int x = 0; x < WT; ++x)
#pragma unroll
                for (int y = 0; y < WT; ++y) mma_frag(fa[x], fb[y], acc[x][y]);
            if (!F64ACC && ((c + 1) % GRAM_FLUSH == 0 || c + 1 == nch)) {
#pragma unroll
                for (int x = 0; x < WT; ++x)
#pragma unroll
                    for (int y = 0; y < WT; ++y) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc64[x][y][v] += (double)acc[x][y][v];
                        acc[x][y] = AccT{0, 0, 0, 0};
                    }
            }
        }
    }
    };
    if (!FIBRES && L % 8 == 0) run(std::true_type());
    else run(std::false_type());
    if (!active) return;
    // partial block (TB x TB, column-major) for (kc, q)
    double *dst = partials + ((int64_t)kc * nblocks + q) * (int64_t)TB * TB;
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
        for (int y = 0; y < WT; ++y) {
            const int jl = wj * (16 * WT) + 16 * y + (lane & 15);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int il = wi * (16 * WT) + 16 * x + drow<PREC>(lane >> 4, v);
                double val = F64ACC ? (double)acc[x][y][v] : acc64[x][y][v];
                dst[il + TB * jl] = val;
            }
        }
}

// ---------------------------------------------------------------------------
// First-mode (L = 1) variant for FP32 data.  Each row p of the contraction
// is a contiguous run of I floats, so a slab of TB columns x 32 rows is read
// with 16-byte loads along i (lanes 0..TB/4-1 cover one row).  A thread
// holds 4 columns x LPT rows; the rows it holds are mapped to LPT
// consecutive fragment slots of one lane group:
//   row pc + ph + PH*s  ->  group g = ph % 4, slot j = LPT*(ph / 4) + s,
// the same bijection for A and B, which is all the matrix cores need.
// LDS holds two slabs per operand (double buffering, one barrier per chunk)
// and the loads run two chunks ahead of the matrix cores.
template <int PREC>
__device__ __forceinline__ void l1_store(uint8_t *slab, int TB, int g, int row, int slot0,
                                         const float *v, int nv) {
    // slab: base of one operand buffer, quads [qq][g][row]
    if constexpr (PREC == P_BF16X3 || PREC == P_BF16X6) {
        constexpr int NP = (PREC == P_BF16X3) ? 2 : 3;
        __bf16 part[NP][4];
        for (int k = 0; k < nv; ++k) {
            float x = v[k];
            __bf16 h = to_bf16(x);
            float r1 = x - from_bf16(h);
            __bf16 m = to_bf16(r1);
            part[0][k] = h;
            part[1][k] = m;
            if constexpr (NP == 3) part[2][k] = to_bf16(r1 - from_bf16(m));
        }
#pragma unroll
        for (int qq = 0; qq < NP; ++qq) {
            uint8_t *q = slab + ((size_t)((qq * 4 + g) * TB + row)) * 16 + 2 * slot0;
            if (nv == 4) {
                uint2 w;
                __builtin_memcpy(&w, part[qq], 8);
                *reinterpret_cast<uint2 *>(q) = w;
            } else {
                uint32_t w;
                __builtin_memcpy(&w, part[qq], 4);
                *reinterpret_cast<uint32_t *>(q) = w;
            }
        }
    } else if constexpr (PREC == P_FP32) {
        // slot j -> quad j / 4, element j % 4
        const int qq = slot0 / 4, e = slot0 % 4;
        float *q = reinterpret_cast<float *>(slab + ((size_t)((qq * 4 + g) * TB + row)) * 16) + e;
        for (int k = 0; k < nv; ++k) q[k] = v[k];
    } else {
        // FP64: slot j -> quad j / 2, element j % 2
        for (int k = 0; k < nv; ++k) {
            const int j = slot0 + k;
            double *q = reinterpret_cast<double *>(slab + ((size_t)(((j / 2) * 4 + g) * TB + row)) * 16) + (j % 2);
            *q = (double)v[k];
        }
    }
}

// place of a row in a stage plane (16-byte entries): rows 16 apart differ in their
// low bits, so that the stores (rows four apart in consecutive lanes) and the
// fragment reads (16 consecutive rows) are both free of bank conflicts
__device__ __forceinline__ int l1_row(int r) { return r ^ ((r >> 4) & 3); }

// Waves form a WI x WJ grid over the TB x TB output block, each owning
// WTI x WTJ tiles of 16 x 16 (TB = 16 WTI WI = 16 WTJ WJ).
// Every load is issued unconditionally (rows and columns past the range are
// clamped, chunks past the end repeat the last one, a diagonal block loads its
// one operand twice, from cache) and taken as it is: rows from pend on become
// zero when they are stored.  A branch or a select at the load makes the compiler
// wait for the chunks in flight before the one in hand is multiplied.
// I >= 4: 16-byte loads of four columns (any alignment).
// FULLI: I is a multiple of TB; see below.
// V4LD (batched mode-1 launches, any I >= 4): thread (parity, operand, row quad
// iq, group g) owns rows 4 iq .. 4 iq + 3 of one operand and the 8 columns g of
// every chunk of its parity (threads [0, 2 TB) the even chunks, the rest the odd
// ones): eight 16-byte loads per chunk give four rows' fragments; the same 32
// values per thread as two chunks of two operands in flight.  Where the matrix
// cores bound the Gram (bf16x6 at I = 512) the FULLI loads are faster, so the
// single-tensor path keeps those.
// With the selects at the loads (and, V4LD, 4-way bank conflicts of its stores)
// the Grams of the later modes of 256 mixed tensors took 2.80 ms, now 2.12 ms.
template <int PREC, int WTI, int WTJ, int WI, int WJ, bool FULLI = false, bool V4LD = false>
__device__ __forceinline__ void gram_l1_body(const float *__restrict__ Y, int64_t I, int64_t P,
                                             int64_t kper, int nkc, int nblocks, int64_t total_wg,
                                             int64_t lid, double *__restrict__ partials) {
    constexpr int TB = 16 * WTI * WI;
    static_assert(TB == 16 * WTJ * WJ, "square output block");
    constexpr int NTH = 64 * WI * WJ;
    constexpr int NQ = Frag<PREC>::NQ;
    constexpr int IQ = TB / 4;          // 16-byte column quads per row
    constexpr int PH = NTH / IQ;        // rows covered by one pass of the workgroup
    constexpr int LPT = KC / PH;        // rows (loads) per thread per chunk
    constexpr int SLAB = NQ * 4 * TB * 16;  // bytes of one operand buffer
    typedef typename Acc<PREC>::type AccT;
    constexpr bool F64ACC = (PREC == P_FP64);
    extern __shared__ uint4 s_g[];
    uint8_t *lds = reinterpret_cast<uint8_t *>(s_g);  // [buf][operand][SLAB]

    if (lid >= total_wg) return;
    const int kc = (int)(lid / nblocks);
    const int q = (int)(lid - (int64_t)kc * nblocks);
    int bi = 0;
    while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
    const int bj = q - bi * (bi + 1) / 2;
    const bool diag = (bi == bj);
    const int64_t i0 = (int64_t)bi * TB, j0 = (int64_t)bj * TB;
    const int64_t pbeg = (int64_t)kc * kper;
    const int64_t pend = min(P, pbeg + kper);
    const int nch = (int)((pend - pbeg + KC - 1) / KC);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = wave / WJ, wj = wave % WJ;
    // a wave whose tiles lie wholly above the diagonal of a diagonal block idles
    const bool active = !(diag && (wi + 1) * 16 * WTI <= wj * 16 * WTJ);
    const int iq = tid % IQ, ph = tid / IQ;
    const int g_st = ph % 4, slot0 = LPT * (ph / 4);

    // FULLI: thread (il, kq) owns column il of the block and the KPT
    // consecutive rows kq * KPT .. of each chunk (lanes along the column, so
    // every load instruction reads 256 contiguous bytes); it splits them into
    // whole fragment quads and writes 16 bytes per quad, consecutive lanes to
    // consecutive rows of the slab (no LDS bank conflicts).
    constexpr int KG = NTH / TB;      // row groups per chunk
    constexpr int KPT = KC / KG;      // rows per thread per chunk (4 * LPT floats)
    static_assert(!FULLI || (KPT == 4 * LPT && KPT % 8 == 0), "thread tiling of the full path");
    const int il = tid % TB, kq = tid / TB;
    auto load = [&](int64_t pc, int64_t c0, float4 (&r)[LPT]) {
        if constexpr (FULLI) {
            float *rf = &r[0].x;
            const float *src = Y + c0 + il;
#pragma unroll
            for (int s = 0; s < KPT; ++s) {
                const int64_t p = pc + kq * KPT + s;
                rf[s] = src[I * (p < pend ? p : pend - 1)];
            }
            return;
        }
        const int64_t col = c0 + 4 * iq;
#pragma unroll
        for (int s = 0; s < LPT; ++s) {
            const int64_t p = pc + ph + PH * s;
            const float *src = Y + I * (p < pend ? p : pend - 1);
            // the quad across column I - 1 is read from I - 4 on
            const f32x4u v = *reinterpret_cast<const f32x4u *>(src + min(col, I - 4));
            r[s] = make_float4(v.x, v.y, v.z, v.w);
        }
    };
    // pc: the chunk's first row; its rows from pend on become zero here
    auto store = [&](int buf, int op, int64_t pc, float4 (&r)[LPT]) {
        if (pc + KC > pend) {
#pragma unroll
            for (int s = 0; s < 4 * LPT; ++s) {
                const int64_t p = FULLI ? pc + kq * KPT + s : pc + ph + PH * (s / 4);
                if (p >= pend) (&r[0].x)[s] = 0.f;
            }
        }
        if constexpr (!FULLI) {
            // and moved into place here (columns from I on hold anything: they
            // reach no output that is read)
            const int64_t sh = (op ? j0 : i0) + 4 * iq - (I - 4);
            if (sh > 0) {
#pragma unroll
                for (int s = 0; s < LPT; ++s) {
                    // values first: a select between the array's elements is one between
                    // addresses and keeps the whole array in scratch memory (200 x 10485
                    // in bf16x3 67 us)
                    const float y = r[s].y, z = r[s].z, w = r[s].w;
                    r[s].x = sh == 1 ? y : (sh == 2 ? z : w);
                    r[s].y = sh == 1 ? z : w;
                    r[s].z = w;
                }
            }
        }
        uint8_t *slab = lds + (size_t)(buf * 2 + op) * SLAB;
        if constexpr (FULLI) {
            const float *rf = &r[0].x;
            uint4 *sq = reinterpret_cast<uint4 *>(slab);
#pragma unroll
            for (int o = 0; o < KPT / 8; ++o) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = rf[8 * o + e];
                FragQ<PREC> t;
                make_frag(v, t.f);
                const int g = kq * (KPT / 8) + o;
#pragma unroll
                for (int qq = 0; qq < NQ; ++qq) sq[(qq * 4 + g) * TB + il] = t.q[qq];
            }
            return;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float v[LPT];
#pragma unroll
            for (int s = 0; s < LPT; ++s) v[s] = (&r[s].x)[c];
            l1_store<PREC>(slab, TB, g_st, 4 * iq + c, slot0, v, LPT);
        }
    };

    AccT acc[WTI][WTJ];
    f64x4 acc64[WTI][WTJ];
#pragma unroll
    for (int x = 0; x < WTI; ++x)
#pragma unroll
        for (int y = 0; y < WTJ; ++y) {
            acc[x][y] = AccT{0, 0, 0, 0};
            acc64[x][y] = f64x4{0, 0, 0, 0};
        }

    auto compute = [&](int buf, int c) {
        if (!active) return;
        const uint4 *sA = reinterpret_cast<const uint4 *>(lds + (size_t)(buf * 2 + 0) * SLAB);
        const uint4 *sB = reinterpret_cast<const uint4 *>(lds + (size_t)(buf * 2 + (diag ? 0 : 1)) * SLAB);
        const int g = lane >> 4;
        Frag<PREC> fa[WTI], fb[WTJ];
#pragma unroll
        for (int x = 0; x < WTI; ++x) {
            FragQ<PREC> t;
            const int row = wi * (16 * WTI) + 16 * x + (lane & 15);
#pragma unroll
            for (int qq = 0; qq < NQ; ++qq) t.q[qq] = sA[(qq * 4 + g) * TB + (V4LD ? l1_row(row) : row)];
            fa[x] = t.f;
        }
#pragma unroll
        for (int y = 0; y < WTJ; ++y) {
            FragQ<PREC> t;
            const int row = wj * (16 * WTJ) + 16 * y + (lane & 15);
#pragma unroll
            for (int qq = 0; qq < NQ; ++qq) t.q[qq] = sB[(qq * 4 + g) * TB + (V4LD ? l1_row(row) : row)];
            fb[y] = t.f;
        }
#pragma unroll
        for (int x = 0; x < WTI; ++x)
#pragma unroll
            for (int y = 0; y < WTJ; ++y) mma_frag(fa[x], fb[y], acc[x][y]);
        if (!F64ACC && ((c + 1) % GRAM_FLUSH == 0 || c + 1 == nch)) {
#pragma unroll
            for (int x = 0; x < WTI; ++x)
#pragma unroll
                for (int y = 0; y < WTJ; ++y) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc64[x][y][v] += (double)acc[x][y][v];
                    acc[x][y] = AccT{0, 0, 0, 0};
                }
        }
    };

    if constexpr (V4LD) {
        static_assert(NTH == 4 * TB, "one task per thread");
        constexpr int TQ4 = TB / 4;
        const int par4 = tid / (2 * TB), op4 = (tid / TB) & 1, iq4 = (tid % TB) % TQ4, g4 = (tid % TB) / TQ4;
        // 16-byte loads (4-byte aligned when I % 4 != 0); the quad that runs past
        // row I - 1 and those after it are read from row I - 4 on
        const int64_t rq = (op4 ? j0 : i0) + 4 * iq4;
        const int64_t rs = min(rq, I - 4);
        const int r0 = (int)(rs - (op4 ? j0 : i0));   // its first row within the block
        const float *src4 = Y + rs;
        float rv[4][8];
        auto load4 = [&](int cn) {
            const int64_t pc = pbeg + (int64_t)(cn < nch ? cn : nch - 1) * KC;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t pp = pc + 8 * g4 + j;
                const f32x4u v = *reinterpret_cast<const f32x4u *>(src4 + I * (pp < pend ? pp : pend - 1));
                rv[0][j] = v.x;
                rv[1][j] = v.y;
                rv[2][j] = v.z;
                rv[3][j] = v.w;
            }
        };
        auto store4 = [&](int buf, int cn) {
            const int64_t pc = pbeg + (int64_t)(cn < nch ? cn : nch - 1) * KC;
            if (pc + KC > pend) {
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) gram_mask(pc + 8 * g4, pend, rv[rr]);
            }
            if (rq >= I) return;   // those rows of the slab reach no output that is read
            uint4 *sq = reinterpret_cast<uint4 *>(lds + (size_t)(buf * 2 + op4) * SLAB);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                if (r0 + rr < 0) continue;   // a row of the block before
                FragQ<PREC> t;
                make_frag(rv[rr], t.f);
#pragma unroll
                for (int qq = 0; qq < NQ; ++qq) sq[(qq * 4 + g4) * TB + l1_row(r0 + rr)] = t.q[qq];
            }
        };
        if (nch > 0) {
            load4(par4);
            if (par4 == 0) store4(0, 0);
        }
        __syncthreads();
        // chunk c in buffer 0 and chunk c + 1 in flight on the odd threads;
        // every load and LDS store is issued unconditionally (clamped chunks
        // past the end are stored and never multiplied)
        for (int c = 0; c < nch; c += 2) {
            if (par4 == 0) load4(c + 2);
            compute(0, c);
            if (par4 == 1) store4(1, c + 1);
            __syncthreads();
            if (par4 == 1) load4(c + 3);
            if (c + 1 < nch) compute(1, c + 1);
            if (par4 == 0) store4(0, c + 2);
            __syncthreads();
        }
    } else {
    float4 ra0[LPT], rb0[LPT], ra1[LPT], rb1[LPT];
    auto prefetch = [&](int cn, float4 (&ra)[LPT], float4 (&rb)[LPT]) {
        const int64_t pc = pbeg + (int64_t)(cn < nch ? cn : nch - 1) * KC;
        load(pc, i0, ra);
        load(pc, j0, rb);
    };
    auto store2 = [&](int buf, int cn, float4 (&ra)[LPT], float4 (&rb)[LPT]) {
        const int64_t pc = pbeg + (int64_t)(cn < nch ? cn : nch - 1) * KC;
        store(buf, 0, pc, ra);
        if (!diag) store(buf, 1, pc, rb);
    };
    if (nch > 0) {
        prefetch(0, ra0, rb0);
        prefetch(1, ra1, rb1);
        store2(0, 0, ra0, rb0);
    }
    __syncthreads();
    // chunk c in buffer 0, chunk c + 1 in flight in ra1 / rb1; every load is issued
    // unconditionally (chunks past the end repeat the last one and are not multiplied)
    for (int c = 0; c < nch; c += 2) {
        prefetch(c + 2, ra0, rb0);
        compute(0, c);
        store2(1, c + 1, ra1, rb1);
        __syncthreads();
        prefetch(c + 3, ra1, rb1);
        if (c + 1 < nch) compute(1, c + 1);
        store2(0, c + 2, ra0, rb0);
        __syncthreads();
    }
    }
    if (!active) return;
    double *dst = partials + ((int64_t)kc * nblocks + q) * (int64_t)TB * TB;
#pragma unroll
    for (int x = 0; x < WTI; ++x)
#pragma unroll
        for (int y = 0; y < WTJ; ++y) {
            const int jl = wj * (16 * WTJ) + 16 * y + (lane & 15);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int il = wi * (16 * WTI) + 16 * x + drow<PREC>(lane >> 4, v);
                dst[il + TB * jl] = F64ACC ? (double)acc[x][y][v] : acc64[x][y][v];
            }
        }
}

// ---- skinny Gram: L = 1 and I <= 160 (a short first mode, J_1 = M huge) --
// Y (I x P, column-major) is read once, in blocks of 32 CH columns (each one
// contiguous run of 128 I CH bytes) dealt round-robin to the workgroups:
// workgroup k takes blocks k, k + nkc, ..., so that at any moment the chip
// streams one contiguous region (independent far-apart streams per
// workgroup camp on a few HBM channels).
// The whole lower triangle of its partial Gram is held in registers as 32 x 32
// super tiles (2 x 2 tiles of 16 x 16), at most SK_MS per wave.  Per stage CH
// chunks of 32 columns go through LDS as matrix-core fragments: thread task
// (row i, group g, chunk c) loads the 8 values Y(i, p0 + 32 c + 8 g + j),
// consecutive lanes on consecutive rows (256-byte loads), splits them into
// the precision's fragment and stores it; the next stage's loads are in flight
// while the current one is multiplied.  FP32 accumulators are flushed into
// FP64 every GRAM_FLUSH chunks; partial super tiles go to the workspace and
// gram_reduce_kernel<32, true> sums them in a fixed order.
constexpr int SK_MAXI = 160;
constexpr int SK_W = 8, SK_T = 64 * SK_W;
constexpr int SK_MS = 2;      // super tiles per wave: 15 lower 32 x 32 tiles at I = 160
constexpr int SK_MS1_MAXI = 96;   // one super tile per wave is enough: 6 lower tiles

__host__ __device__ inline int sk_ns(int64_t I) { return (int)(((I + 15) / 16 + 1) / 2); }

// QUAD: I >= 4, any alignment of the rows.  MS: super tiles per wave (1 where
// I <= SK_MS1_MAXI).
//
// What bounds it: the reading of Y against the splitting of its values into bf16
// parts with bf16x6 (I = 48); the matrix cores with FP32 products and with FP64 ones
// (these in the batch only, gram_tri64_kernel takes them elsewhere).  48^5 in bf16x6
// 351 us (579): with the selects beside the loads every stage waited out its own
// loads before it was multiplied; with the loader's tasks on the waves that
// multiply, the one came after the other; and rows stored four apart met 4-way bank
// conflicts.
template <int PREC, int CH, bool QUAD, int MS>
__device__ __forceinline__ void gram_skinny_body(const float *__restrict__ Y, int I, int64_t P, int nkc, int kc,
                                                 double *__restrict__ partials) {
    constexpr int NQ = Frag<PREC>::NQ;
    typedef typename Acc<PREC>::type AccT;
    constexpr bool F64ACC = (PREC == P_FP64);
    extern __shared__ uint4 s_sk[];
    const int NS = sk_ns(I), NSS = NS * (NS + 1) / 2, TBp = 32 * NS;
    const int64_t nblk = (P + 32 * CH - 1) / (32 * CH);
    const int nst = kc < nblk ? (int)((nblk - 1 - kc) / nkc + 1) : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4;
    const int stage_q = CH * NQ * 4 * TBp;   // uint4 per stage buffer

    int sbi[MS], sbj[MS];
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        const int q = wave + SK_W * m;
        int bi = -1, bj = 0;
        if (q < NSS) {
            bi = 0;
            while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
            bj = q - bi * (bi + 1) / 2;
        }
        sbi[m] = bi;
        sbj[m] = bj;
    }
    AccT acc[MS][2][2];
    f64x4 acc64[MS][2][2];
#pragma unroll
    for (int m = 0; m < MS; ++m)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                acc[m][x][y] = AccT{0, 0, 0, 0};
                acc64[m][x][y] = f64x4{0, 0, 0, 0};
            }

    // QUAD: task (row quad iq, group g, chunk c) loads the 4 x 8 block
    // Y(4 iq .. 4 iq + 3, p0 + 32 c + 8 g + j) with eight 16-byte loads (consecutive
    // lanes on consecutive row quads; the last quad of I % 4 != 0 rows is read from
    // row I - 4 on) and builds the four rows' fragments.  Otherwise task
    // (row i, group g, chunk c) loads the 8 values of one row with 4-byte loads.
    constexpr int RPT = QUAD ? 4 : 1;               // rows per task
    const int TQ = (I + RPT - 1) / RPT;             // row groups
    const int ntask = TQ * 4 * CH;
    // loader tasks start at the last wave, super tiles at the first: where there
    // are fewer of both than waves, different waves load and multiply.  Rows from
    // I on of a stage hold anything: they reach only outputs that are not read.
    const int tk = SK_T - 64 - 64 * wave + lane;
    const bool has_task = tk < ntask;   // one task per thread at most
    const int iq = min(tk, ntask - 1) % TQ, rest = min(tk, ntask - 1) / TQ, gg = rest & 3, tc = rest >> 2;
    const int row0 = QUAD ? min(4 * iq, I - 4) : iq;
    const int col0 = 32 * tc + 8 * gg;
    float raw[RPT][8];
    // The loads alone, unmasked (columns from P on read column p0): a select here
    // would wait for its load before the stage is multiplied.
    auto load = [&](int st) {
        const int64_t p0 = ((int64_t)st * nkc + kc) * 32 * CH;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t pp = p0 + col0 + j;
            const int64_t a = row0 + (int64_t)I * (pp < P ? pp : p0);
            if constexpr (QUAD) {
                const f32x4u v = *reinterpret_cast<const f32x4u *>(Y + a);   // 4-byte alignment suffices
                raw[0][j] = v.x;
                raw[1][j] = v.y;
                raw[2][j] = v.z;
                raw[3][j] = v.w;
            } else {
                raw[0][j] = Y[a];
            }
        }
    };
    auto store = [&](int st) {
        if (!has_task) return;
        uint4 *sb = s_sk + (size_t)(st & 1) * stage_q;
        const int64_t left = P - ((int64_t)st * nkc + kc) * 32 * CH;   // columns of the stage within Y
        if (left < 32 * CH) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int rr = 0; rr < RPT; ++rr)
                    if (col0 + j >= left) raw[rr][j] = 0.f;
        }
#pragma unroll
        for (int rr = 0; rr < RPT; ++rr) {   // rows shared by the last two quads are stored twice, alike
            FragQ<PREC> f;
            make_frag(raw[rr], f.f);
#pragma unroll
            for (int qq = 0; qq < NQ; ++qq) sb[((tc * NQ + qq) * 4 + gg) * TBp + l1_row(row0 + rr)] = f.q[qq];
        }
    };
    auto frag = [&](const uint4 *sb, int c, int row, Frag<PREC> &f) {
        FragQ<PREC> t;
#pragma unroll
        for (int qq = 0; qq < NQ; ++qq) t.q[qq] = sb[((c * NQ + qq) * 4 + g) * TBp + l1_row(row)];
        f = t.f;
    };

    int chunk = 0;
    if (nst > 0) {
        load(0);
        store(0);
    }
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        if (st + 1 < nst) load(st + 1);
        const uint4 *sb = s_sk + (size_t)(st & 1) * stage_q;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
#pragma unroll
            for (int m = 0; m < MS; ++m) {
                if (sbi[m] < 0) continue;   // uniform within the wave
                Frag<PREC> fa[2], fb[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) frag(sb, c, 32 * sbi[m] + 16 * x + (lane & 15), fa[x]);
                if (sbi[m] != sbj[m]) {
#pragma unroll
                    for (int y = 0; y < 2; ++y) frag(sb, c, 32 * sbj[m] + 16 * y + (lane & 15), fb[y]);
                } else {
                    fb[0] = fa[0];
                    fb[1] = fa[1];
                }
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y) mma_frag(fa[x], fb[y], acc[m][x][y]);
            }
            ++chunk;
            if (!F64ACC && chunk % GRAM_FLUSH == 0) {
#pragma unroll
                for (int m = 0; m < MS; ++m)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
#pragma unroll
                        for (int y = 0; y < 2; ++y) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc64[m][x][y][v] += (double)acc[m][x][y][v];
                            acc[m][x][y] = AccT{0, 0, 0, 0};
                        }
            }
        }
        if (st + 1 < nst) store(st + 1);
        __syncthreads();
    }
    // partial super tiles: element (il, jl) of super tile q at [(kc NSS + q) 1024 + il + 32 jl]
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        if (sbi[m] < 0) continue;
        const int q = wave + SK_W * m;
        double *dst = partials + ((int64_t)kc * NSS + q) * 1024;
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double val = F64ACC ? (double)acc[m][x][y][v] : acc64[m][x][y][v] + (double)acc[m][x][y][v];
                    dst[(16 * x + drow<PREC>(g, v)) + 32 * (16 * y + (lane & 15))] = val;
                }
    }
}

}  // namespace sth
