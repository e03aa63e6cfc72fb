// The matrix-core product behind every blocked solve and factorization.
//
//   C = beta * C + alpha * A * B        (column-major, real-view units)
//
// One template serves the FP64 product (v_mfma_f64_16x16x4_f64), the FP32
// product (v_mfma_f32_16x16x4_f32) and the mixed one (FP64 operands rounded
// to FP32 as they are staged, FP32 accumulators flushed into FP64 ones every
// KCHUNK values of K, so that rounding grows with the chunk and not with K).
//
// Tiling: a 256-thread workgroup (4 wavefronts) owns a BM x BN tile of C,
// each wavefront a (BM/WM) x (BN/WN) sub-tile held as 16x16 accumulator
// blocks.  K advances BK at a time through a ring of two LDS stages, filled by
// direct global-to-LDS loads (16 bytes a lane) a slice ahead, one barrier per
// slice.
//
// What bounds it: the matrix cores.  On the DTRSM 16384 top update (M = K =
// 8192, N = 16384) staging through registers, with a bounds test around each
// load, ran at 58 TF/s; without the tests at 65.2 (the loop then spends 9.4 k
// cycles where its products take 8.2 k: the LDS stores and the waits before
// them stall both workgroups of a CU at once); with direct loads at 71.7, and
// with 8-deep slices, whose smaller ring lets a third workgroup in, at 72.4
// (95 % of what the FP64 matrix cores sustain).  Deeper rings change nothing
// there (72.4 with three stages, 69.9 with four and one workgroup fewer).
//
// Loads without guards.  A tile that would hang over the last row is moved up
// to end there (its first rows repeat the previous tile's and are not
// stored), and columns of B beyond N read column N-1 (not stored either), so
// every slice but a ragged last one is plain 16-byte loads from pointers that
// only advance.  Only the last slice of a K that BK does not divide, and
// products with fewer rows than the tile, take guarded loads and LDS stores, and
// the slices on the diagonal of a triangular A go to LDS four bytes a lane, so
// that each element has an address of its own and none above the diagonal is
// read (a solve of 128 x 128 with a refinement step: 68 us, by guarded loads 74).
//
// LDS layout.  A direct load writes a wavefront's 1 KB contiguously, so there
// is no padding; bank conflicts are kept away by permuting, within a column,
// which 16-byte piece each lane fetches.  B (BK consecutive k per column):
// piece p of column j lies at p ^ swz(j), so the 16 columns a fragment reads
// fall on distinct banks.  A in FP32: the 16-row
// blocks of column k lie at block ^ (k % 4), so the four columns a fragment
// reads do.  (A in FP64 needs none: 16 rows fill the 128 bytes of a clock.)
//
// MFMA operand layout (16x16x4): lane l holds A[l%16][k0 + l/16] and
// B[k0 + l/16][l%16].  Result element v of lane l is, in FP32, row 4(l/16) + v
// of column l%16 and, in FP64, row 4v + l/16; there the A fragment is fed with
// its rows in the transposed 4x4 order (slot s carries row 4(s%4) + s/4),
// which makes it row 4(l/16) + v as well.  So each lane ends up with four
// consecutive rows of one column: C moves in 16-byte accesses and the (re, im)
// rows of a complex element stay in one lane.
//
// Complex data: a complex M x K matrix A is the real 2M x 2K matrix whose
// 2x2 blocks are [[re, -im], [im, re]]; complex B and C are real matrices of
// twice the rows.  A is staged as it is stored (a slice of BK real columns is
// BK/2 complex ones) and expanded when a fragment is read: row r of real column
// 2c + q is component (r ^ q) & 1 of the complex element, negated where q = 1
// and r is even.  That halves A's global and LDS traffic against staging the
// expanded form, for one exclusive-or per fragment.
//
// Workgroup -> tile mapping: consecutive workgroup ids land on different
// XCDs, so ids are remapped to give each XCD a contiguous run of tiles, walked
// in groups of 8 tile-rows whose A and B panels share that XCD's L2.

#pragma once

#include <type_traits>

#include "internal.h"
#include "tile_choice.h"

namespace hsma {
namespace gemmk {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double fma_rn(double a, double b, double c) { return __fma_rn(a, b, c); }
__device__ __forceinline__ float fma_rn(float a, float b, float c) { return __fmaf_rn(a, b, c); }
__device__ __forceinline__ double mul_rn(double a, double b) { return __dmul_rn(a, b); }
__device__ __forceinline__ float mul_rn(float a, float b) { return __fmul_rn(a, b); }

template <typename T>
struct Mma;
template <>
struct Mma<double> {
    typedef dbl4 Acc;
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // Row of the A fragment that slot s of the instruction carries.
    static __device__ __forceinline__ int a_row(int s) { return 4 * (s & 3) + (s >> 2); }
    static __device__ __forceinline__ double flip(double v, unsigned mask) {
        return __hiloint2double(__double2hiint(v) ^ (int)mask, __double2loint(v));
    }
};
template <>
struct Mma<float> {
    typedef flt4 Acc;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int a_row(int s) { return s; }
    static __device__ __forceinline__ float flip(float v, unsigned mask) {
        return __uint_as_float(__float_as_uint(v) ^ mask);
    }
};

template <typename TG, bool CX>
constexpr int ring_bytes(int bm, int bn, int bk) {
    return 2 * ((CX ? bk / 2 : bk) * bm + bn * bk) * (int)sizeof(TG);
}
// Workgroups per CU the ring allows (160 KB of LDS per CU, at most `most`);
// the launch bound then caps registers so that many stay resident.
constexpr int occupancy(int bytes, int most) {
    const int n = 160 * 1024 / bytes;
    return n >= most ? most : (n >= 1 ? n : 1);
}

typedef __attribute__((address_space(3))) void lds_void;

// One BM x BN tile (tm, tn).  TG is the data type in memory and LDS, TM the
// type on the matrix cores; GD is TG, or HSMA_GLOBAL TG where pointers come
// from a descriptor table.  TRI: A is lower triangular (p.tri_a, p.k_lower).
template <typename TG, typename TM, bool CX, bool TRI, int BM, int BN, int BK, int WM, int WN,
          int KCHUNK, typename P, typename GD>
__device__ __forceinline__ void gemm_tile(const P &p, const GD *__restrict__ Ag,
                                          const GD *__restrict__ Bg, GD *__restrict__ Cg, int tm,
                                          int tn) {
    constexpr bool MIXED = !std::is_same<TG, TM>::value;
    constexpr int ES = CX ? 2 : 1;
    constexpr int TMR = BM / WM, TNC = BN / WN;
    constexpr int FM = TMR / 16, FN = TNC / 16;
    constexpr int V = 16 / (int)sizeof(TG);  // elements per 16-byte piece
    constexpr int KA = CX ? BK / 2 : BK;     // stored columns of A per slice
    constexpr int PA = BM / V, PB = BK / V;  // pieces per column of A, of B
    constexpr bool SWZ_A = sizeof(TG) == 4 && !CX && BM >= 64;
    // Where in a slice the next fill is issued: before the first read of LDS (-1)
    // or at k-step FILL_AT.  Every read of LDS after it waits for it.  With 128 x
    // 128 tiles two workgroups share a CU and fall into turns, one filling while
    // the other multiplies, and a fill before the first read is best where the
    // products are plain (72.3 against 67.8 TF/s in FP64 at 8192^3, FP32 140
    // against 132), in mid-slice where fragments need work (complex 71.4 against
    // 69.0, mixed 106 against 101) and for smaller tiles.
    constexpr int FILL_AT = (CX || MIXED || BM * BN < 128 * 128) ? BK / 8 - 1 : -1;
    static_assert(!TRI || !SWZ_A, "the triangle is masked by LDS position");
    static_assert(WM * WN == 4, "four wavefronts");
    static_assert(TMR % 16 == 0 && TNC % 16 == 0, "16x16 blocks");
    static_assert(BK % 4 == 0 && BK % V == 0 && BM % V == 0, "whole pieces and k-steps");
    static_assert((PB & (PB - 1)) == 0 && PB <= 32 && (PA & (PA - 1)) == 0, "powers of two");
    typedef TG VG __attribute__((ext_vector_type(V), aligned(sizeof(TG))));
    typedef TG VL __attribute__((ext_vector_type(V)));
    typedef typename Mma<TM>::Acc Acc;
    typedef typename Mma<TG>::Acc AccG;

    __shared__ __attribute__((aligned(16))) TG As[2][KA * BM];
    __shared__ __attribute__((aligned(16))) TG Bs[2][BN * BK];

    const int m0 = tm * BM, n0 = tn * BN;
    const int M = p.M, N = p.N;
    // Lower-triangular C (c_lower): a tile whose first column lies right of
    // its last row (in elements) is empty.
    if constexpr (!MIXED && !TRI) {
        if (p.c_lower && n0 > (m0 + BM - 1) / ES) return;
    }
    // A lower-triangular A has nothing right of column m0 + BM - 1 here.
    const int K = (TRI && p.k_lower && m0 + BM < p.K) ? m0 + BM : p.K;
    const int ms = first_row(M, BM, m0);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % WM) * TMR, wn0 = (wave / WM) * TNC;

    // Piece e = tid + 256 it of a slice: A's stored column e / PA and the
    // piece of it that the LDS position e % PA holds; B's column e / PB.
    constexpr int A_VEC = KA * PA, B_VEC = BN * PB;
    constexpr int A_IT = (A_VEC + 255) / 256, B_IT = (B_VEC + 255) / 256;
    static_assert((A_VEC % 256 == 0 || A_IT == 1) && (B_VEC % 256 == 0 || B_IT == 1), "whole passes");
    static_assert(A_VEC % 64 == 0 && B_VEC % 64 == 0, "whole wavefronts");
    // Wavefronts that take part in the (single) pass of a small operand.
    const bool a_on = A_VEC % 256 == 0 || wave * 64 < A_VEC, b_on = B_VEC % 256 == 0 || wave * 64 < B_VEC;
    constexpr int JD = 16 / PB > 0 ? 16 / PB : 1;
    // (of 16 consecutive columns, so that the column block drops out)
    auto swz_b = [](int j) { return (j & 15) / JD % PB; };
    auto a_k = [&](int it) { return (tid + it * 256) / PA; };
    auto a_i = [&](int it) { return V * (((tid + it * 256) % PA) ^ (SWZ_A ? 4 * (a_k(it) & 3) : 0)); };
    auto b_j = [&](int it) { return (tid + it * 256) / PB; };
    auto b_k = [&](int it) { return V * (((tid + it * 256) % PB) ^ swz_b(b_j(it))); };
    const int64_t a_col = (int64_t)ES * p.lda;  // one stored column of A
    const GD *pa[A_IT], *pb[B_IT];
#pragma unroll
    for (int it = 0; it < A_IT; ++it) pa[it] = Ag + (a_k(it) * a_col + ms + a_i(it));
#pragma unroll
    for (int it = 0; it < B_IT; ++it) {
        const int c = n0 + b_j(it);
        pb[it] = Bg + ((int64_t)(c < N ? c : N - 1) * p.ldb + b_k(it));
    }

    // Slice at k0 into stage `buf`.
    auto fill = [&](int k0, int buf) {
        const bool direct = direct_slice(M, BM, K, BK, TRI, ms, k0);
        if (direct || (TRI && k0 + BK <= K)) {
            if (direct) {
#pragma unroll
                for (int it = 0; it < A_IT; ++it)
                    if (a_on) __builtin_amdgcn_global_load_lds((const void *)pa[it],
                                                         (lds_void *)&As[buf][V * (wave * 64 + it * 256)], 16, 0, 0);
            } else if constexpr (TRI) {
                // On the diagonal, four bytes a lane: what lies above it (and
                // rows beyond M) takes an element of its column that may be read.
                static_assert(sizeof(TG) == 8 && KA * BM * 2 % 256 == 0, "two lanes an element, whole passes");
#pragma unroll
                for (int it = 0; it < KA * BM * 2 / 256; ++it) {
                    const int e = (tid + it * 256) / 2, c = k0 / ES + e / BM;
                    const GD *src = Ag + (c * a_col + tri_row(ES, M, ms + e % BM, c));
                    __builtin_amdgcn_global_load_lds((const void *)((const char *)src + 4 * (tid & 1)),
                                                     (lds_void *)((char *)&As[buf][0] + 4 * (wave * 64 + it * 256)), 4, 0, 0);
                }
            }
#pragma unroll
            for (int it = 0; it < B_IT; ++it)
                if (b_on) __builtin_amdgcn_global_load_lds((const void *)pb[it],
                                                     (lds_void *)&Bs[buf][V * (wave * 64 + it * 256)], 16, 0, 0);
        } else {
            // Element by element: rows kept below M, nothing read at or
            // beyond K, where both operands are zero.
#pragma unroll
            for (int it = 0; it < A_IT; ++it) {
                if (!a_on) break;
                VL v = {};
                if (k0 / ES + a_k(it) < K / ES) {
                    const GD *col = pa[it] - (ms + a_i(it));
#pragma unroll
                    for (int t = 0; t < V; ++t) {
                        const int r = ms + a_i(it) + t;
                        v[t] = col[TRI ? tri_row(ES, M, r, k0 / ES + a_k(it)) : below(ES, M, r)];
                    }
                }
                *reinterpret_cast<VL *>(&As[buf][V * (tid + it * 256)]) = v;
            }
#pragma unroll
            for (int it = 0; it < B_IT; ++it) {
                if (!b_on) break;
                VL v = {};
#pragma unroll
                for (int t = 0; t < V; ++t)
                    if (k0 + b_k(it) + t < K) v[t] = pb[it][t];
                *reinterpret_cast<VL *>(&Bs[buf][V * (tid + it * 256)]) = v;
            }
        }
#pragma unroll
        for (int it = 0; it < A_IT; ++it) pa[it] += KA * a_col;
#pragma unroll
        for (int it = 0; it < B_IT; ++it) pb[it] += BK;
    };
    // Every wavefront's fill has landed (LDS stores too), and every wavefront is
    // done reading the stage that the next fill overwrites.
    auto arrive = [&] { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    Acc acc[FM][FN];
    AccG accg[MIXED ? FM : 1][MIXED ? FN : 1];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            acc[i][j] = Acc{0, 0, 0, 0};
            if constexpr (MIXED) accg[i][j] = AccG{0, 0, 0, 0};
        }

    const int nk = (K + BK - 1) / BK;
    if (nk > 0) fill(0, 0);
    arrive();
    const int lr = lane & 15, lk = lane >> 4;
    const int row_a = Mma<TM>::a_row(lr);
    // This lane's A element within a 16-row block (the component swap of a
    // complex odd column), and the sign of the swapped real row.
    const int off_a = CX ? (row_a ^ (lk & 1)) : row_a;
    const unsigned neg = (CX && (lk & 1) && !(row_a & 1)) ? 0x80000000u : 0u;
    int ai[FM], bk[BK / 4];
#pragma unroll
    for (int i = 0; i < FM; ++i) ai[i] = 16 * (SWZ_A ? (wm0 / 16 + i) ^ lk : wm0 / 16 + i) + off_a;
#pragma unroll
    for (int s = 0; s < BK / 4; ++s)
        bk[s] = (wn0 + lr) * BK + V * (((4 * s + lk) / V) ^ swz_b(lr)) + (4 * s + lk) % V;
    int buf = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const bool ahead = kt + 1 < nk;
        if (FILL_AT < 0 && ahead) fill((kt + 1) * BK, buf ^ 1);
        const TG *as = As[buf];
        const TG *bs = Bs[buf];
        if constexpr (TRI) {
            // Slices that reach the tile's first row hold places on or above the
            // diagonal: nothing above it, a unit diagonal as 1.
            if (kt * BK + BK > ms) {
                for (int e = tid; e < KA * BM; e += 256) {
                    const int c = kt * KA + e / BM, r = ms + e % BM;
                    if (r / ES < c) As[buf][e] = 0;
                    else if (p.tri_a == 2 && r / ES == c) As[buf][e] = (CX && (r & 1)) ? 0 : 1;
                }
                __syncthreads();
            }
        }
#pragma unroll
        for (int s = 0; s < BK / 4; ++s) {
            const int ka = CX ? 2 * s + (lk >> 1) : 4 * s + lk;
            TM fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                fa[i] = (TM)as[ka * BM + ai[i]];
                if constexpr (CX) fa[i] = Mma<TM>::flip(fa[i], neg);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = (TM)bs[bk[s] + 16 * j * BK];
            if (FILL_AT == s && ahead) fill((kt + 1) * BK, buf ^ 1);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = Mma<TM>::mma(fa[i], fb[j], acc[i][j]);
        }
        if constexpr (MIXED) {
            if ((kt + 1) % (KCHUNK / BK) == 0 || kt + 1 == nk) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) accg[i][j][v] += (TG)acc[i][j][v];
                        acc[i][j] = Acc{0, 0, 0, 0};
                    }
            }
        }
        arrive();
        buf ^= 1;
    }

    // ---- epilogue: C = beta*C + alpha*acc, four rows of a column at a time ----
    const TG alr = (TG)p.alpha_re, ali = (TG)p.alpha_im, ber = (TG)p.beta_re, bei = (TG)p.beta_im;
    const bool beta_zero = ber == 0 && bei == 0;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int row = ms + wm0 + 16 * i + 4 * lk;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = n0 + wn0 + 16 * j + lr;
            if (col >= N) continue;
            GD *dst = Cg + (int64_t)col * p.ldc + row;
            TG v[4], c[4] = {0, 0, 0, 0};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                if constexpr (MIXED) v[h] = accg[i][j][h];
                else v[h] = acc[i][j][h];
            }
            bool lower = false;
            if constexpr (!MIXED && !TRI) lower = p.c_lower;
            auto keep = [&](int h) { return row + h >= m0 && row + h < M && !(lower && col > (row + h) / ES); };
            const bool all = row >= m0 && row + 3 < M && !(lower && col > row / ES);
            typedef typename std::conditional<std::is_same<GD, TG>::value, VG, HSMA_GLOBAL VG>::type VGW;
            if (!beta_zero) {
                if (all) {
#pragma unroll
                    for (int h = 0; h < 4; h += V) {
                        const VG t = *reinterpret_cast<VGW *>(dst + h);
#pragma unroll
                        for (int e = 0; e < V; ++e) c[h + e] = t[e];
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 4; ++h)
                        if (keep(h)) c[h] = dst[h];
                }
            }
            TG r[4];
            // Every rounding spelled out: all tile shapes give the same bits.
            if constexpr (CX) {
#pragma unroll
                for (int h = 0; h < 4; h += 2) {
                    r[h] = fma_rn(alr, v[h], -mul_rn(ali, v[h + 1]));
                    r[h + 1] = fma_rn(alr, v[h + 1], mul_rn(ali, v[h]));
                    if (!beta_zero) {
                        r[h] = fma_rn(ber, c[h], fma_rn(-bei, c[h + 1], r[h]));
                        r[h + 1] = fma_rn(ber, c[h + 1], fma_rn(bei, c[h], r[h + 1]));
                    }
                }
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    r[h] = mul_rn(alr, v[h]);
                    if (!beta_zero) r[h] = fma_rn(ber, c[h], r[h]);
                }
            }
            if (all) {
#pragma unroll
                for (int h = 0; h < 4; h += V) {
                    VG t;
#pragma unroll
                    for (int e = 0; e < V; ++e) t[e] = r[h + e];
                    *reinterpret_cast<VGW *>(dst + h) = t;
                }
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    if (keep(h)) dst[h] = r[h];
            }
        }
    }
}

// Tile of workgroup `bid` (of `nb`, a multiple of 8); false if it has none.
__device__ __forceinline__ bool tile_of(int bid, int nb, int tiles_m, int tiles_n, bool rows_first, int &tm,
                                        int &tn) {
    const int T = tiles_m * tiles_n;
    if (rows_first) {
        // A triangular operand (K bounded by the tile row) or a triangular C
        // (tiles above the diagonal skipped): a tile row's work grows with
        // its index, so contiguous runs of rows per XCD would leave the XCD
        // holding the bottom rows with about twice the average.  Bottom rows
        // come first instead, and consecutive workgroups (which the hardware
        // deals out to the XCDs in turn) walk a row, so every XCD gets an
        // eighth of every row.
        if (bid >= T) return false;
        tm = tiles_m - 1 - bid / tiles_n;
        tn = bid % tiles_n;
        return true;
    }
    const int t = (bid % 8) * (nb / 8) + bid / 8;
    if (t >= T) return false;
    constexpr int GROUP = 8;
    const int full = GROUP * tiles_n;
    const int first = t / full * GROUP;
    const int size = (tiles_m - first) < GROUP ? (tiles_m - first) : GROUP;
    tm = first + (t % full) % size;
    tn = (t % full) / size;
    return true;
}

template <typename TG, typename TM, bool CX, bool TRI, int BM, int BN, int BK, int WM, int WN,
          int KCHUNK, int OCC, typename P>
__global__ __launch_bounds__(256, OCC) void hsma_gemm(const P p) {
    int tm, tn;
    if (!tile_of(blockIdx.x, gridDim.x, p.tiles_m, p.tiles_n, p.k_lower || p.c_lower, tm, tn)) return;
    gemm_tile<TG, TM, CX, TRI, BM, BN, BK, WM, WN, KCHUNK>(p, p.A, p.B, p.C, tm, tn);
}

// Launch of one product with tiles of BM x BN.
template <typename TG, typename TM, bool CX, bool TRI, int BM, int BN, int BK, int WM, int WN, int MOST = 3,
          int KCHUNK = BK, typename P>
hsma_status launch_tiles(P p, int phase, hipStream_t s) {
    constexpr int OCC = occupancy(ring_bytes<TG, CX>(BM, BN, BK), MOST);
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    const int64_t T = (int64_t)p.tiles_m * p.tiles_n;
    const int64_t grid = (T + 7) / 8 * 8;
    if (grid > 0x7fffffff) return HSMA_INVALID_SIZE;
    // A lower-triangular C computes about half of the product.
    ProfScope prof(phase, (p.c_lower ? 1.0 : 2.0) * p.M * (double)p.N * p.K, s);
    hipLaunchKernelGGL((hsma_gemm<TG, TM, CX, TRI, BM, BN, BK, WM, WN, KCHUNK, OCC, P>),
                       dim3((unsigned)grid), dim3(256), 0, s, p);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

}  // namespace gemmk
}  // namespace hsma
