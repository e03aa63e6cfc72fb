// Cholesky factorization and solve on the library's TRSM (the first consumer
// the paper names for TRSM, Sec. 1: the forward and backward substitutions of
// LU and Cholesky).
//
// A = L L^H (real symmetric or complex Hermitian positive definite, lower
// triangle) by recursion on halves:
//     L11 = chol(A11)
//     L21 = A21 inv(L11)^H            the right-side, conjugate-transpose TRSM
//     A22 <- A22 - L21 L21^H          lower triangle only, FP64 matrix cores
//     L22 = chol(A22)
// with diagonal blocks of at most 256 rows (128 complex) factored by one
// workgroup in registers.  The solve L L^H X = B is two TRSMs: L Y = B, then L^H X = Y.
//
// No definiteness check is made: a non-positive pivot gives NaN (the square
// root of a negative number), which propagates, as the TRSM propagates a zero
// diagonal.  The strict upper triangle of A is neither read nor written.

#include <algorithm>
#include <type_traits>

#include "dpp_fma.h"
#include "gemm_core.h"

namespace hsma {

hsma_status trsm_impl(hsma_diag diag, int64_t m, int64_t n, const void *alpha, const void *A,
                      int64_t lda, void *B, int64_t ldb, hsma_dtype dtype, int ib_override,
                      int path, hipStream_t s, int *path_used, int *ib_used,
                      const hsma_trsm_options *opt, hsma_trsm_report *rep);

namespace {

using gemmk::Mma;

// Rows of the base kernel in the real view: 16 blocks of 16 rows.
constexpr int kBaseRows = 256;
constexpr int kBaseWaves = 8;
constexpr int kBaseSlots = 17;  // 136 blocks on or below the diagonal, over 8 wavefronts

int base_order(bool cx) { return kBaseRows / (cx ? 2 : 1); }

template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Lane N of each 16-lane row, to the 16 lanes of that row.
template <int N>
__device__ __forceinline__ double bcast(double v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xf, 0xf, false);  // row_newbcast:N
}

// The square root d of a pivot p and its reciprocal: a third-order step from
// the hardware's estimate of 1/sqrt(p) (about 2^-23), a correction of d against
// p, and one of the reciprocal against d; both end within an ulp where nothing
// on the way over- or underflows.
__device__ __forceinline__ void root(double p, double &d, double &inv) {
    double y = __builtin_amdgcn_rsq(p);
    const double r = __fma_rn(-(p * y), y, 1.0);
    y = __fma_rn(__fma_rn(r, 0.375, 0.5), r * y, y);
    const double q = p * y;
    d = __fma_rn(__fma_rn(-q, q, p), 0.5 * y, q);
    inv = __fma_rn(__fma_rn(-d, y, 1.0), y, y);
}

// What lane l ^ 1 holds, to lane l.
__device__ __forceinline__ double swap_pair(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0xb1, 0xf, 0xf, false);  // quad_perm:[1,0,3,2]
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xb1, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// The sixteen steps of a block column: each the root of the pivot, the scaled
// column, and its product off the columns behind it, in the 16 rows of the
// diagonal block (e, a copy per 16-lane row, so pivots and columns move by row
// broadcasts) and in this lane's own row (x; `diag`: a row of the diagonal
// block).  Complex: eight steps; the second real column of an element is the
// first with its components exchanged and one negated, exactly, so that what is
// subtracted is the product of the factor that is stored, and the pivot's
// imaginary part is zero.  FAST: by `root`; false comes back if a pivot was
// outside 2^-900 .. 2^900 (zero, negative, NaN), and the values are not to be
// used.  Otherwise by the library's root and division, for any pivots.
template <bool CX, bool FAST>
__device__ __forceinline__ bool eliminate(double (&e)[16], double (&x)[16], int lr, bool diag) {
    constexpr unsigned kLow = (1023u - 900u) << 20, kSpan = 1800u << 20;
    unsigned most = 0;  // over the pivots' high words, from that of 2^-900
    static_for<0, CX ? 8 : 16>([&](auto K) {
        constexpr int c = (CX ? 2 : 1) * decltype(K)::value;
        const double p = bcast<c>(e[c]);
        double d, inv, unused[16];
        if constexpr (FAST) {
            const unsigned above = (unsigned)__double2hiint(p) - kLow;
            most = above > most ? above : most;
            root(p, d, inv);
        } else {
            d = sqrt(p);
            inv = 1.0 / d;
        }
        double l = e[c] * inv, xl = x[c] * inv;
        if constexpr (CX) {
            if (lr == c + 1) l = 0;
            if (diag && lr == c + 1) xl = 0;
            const double l2 = Mma<double>::flip(swap_pair(l), lr & 1 ? 0 : 0x80000000u);
            const double xl2 = Mma<double>::flip(swap_pair(xl), lr & 1 ? 0 : 0x80000000u);
            if constexpr (c < 14) {
                smallk::fnma_rows<false, c + 2>(e, unused, l, 0, l, 0);
                smallk::fnma_rows<false, c + 2>(e, unused, l2, 0, l2, 0);
                smallk::fnma_rows<false, c + 2>(x, unused, l, 0, xl, 0);
                smallk::fnma_rows<false, c + 2>(x, unused, l2, 0, xl2, 0);
            }
            x[c] = diag && lr == c ? d : xl;
            x[c + 1] = diag && lr == c + 1 ? d : xl2;
        } else {
            if constexpr (c < 15) {
                smallk::fnma_rows<false, c + 1>(e, unused, l, 0, l, 0);
                smallk::fnma_rows<false, c + 1>(x, unused, l, 0, xl, 0);
            }
            x[c] = diag && lr == c ? d : xl;
        }
    });
    return most < kSpan;
}

// One diagonal block of at most 256 rows in the real view (256 real, 128
// complex), right-looking over 16-column blocks, by one workgroup of eight
// wavefronts.  A complex factor is the real view's factor: a Hermitian A's real
// view is symmetric, and that of L has a positive diagonal and zeros above it.
//
// The whole lower triangle is in registers as 16 x 16 accumulators: lane (g,
// lr) holds row lr, columns 4g .. 4g + 3 of its blocks, negated, and blocks are
// dealt to the wavefronts in the order of their columns, so whatever is still to
// be updated is spread evenly at every step.  Step j: block column j is in LDS.
// Four wavefronts eliminate its sixteen columns, a row per lane and a block row
// per 16 lanes, each 16 lanes with a copy of the diagonal block's rows, so a
// pivot, its root and its column reach every row by row broadcasts and the
// sixteen steps need no barrier.  The factored column goes to LDS (and from
// there to memory, by the other four while the next column is eliminated), every
// wavefront subtracts its blocks' products on the matrix cores (a row of L as it
// lies is both operands), and column j + 1 goes to LDS.
//
// What bounds it: the sixteen dependent pivots of a step (about 4100 cycles, two
// thirds of them the two rows' multiply-adds) and the products (64 cycles a
// block of those left, 4300 on average).  Letting four wavefronts eliminate
// while the others subtract the step before is slower (70 us against 64): both
// use the FP64 units.  256 rows: 62 us, 64 rows 10; the 64-row kernel
// with a barrier, a root and a division per column took 22.
//
// A block's products are summed from zero and meet it once per block column: one
// by one, 256 of them would each be rounded at the size of A.  Relative error of
// the factor of order 1000 in the norm, added one by one / so / with the 64-row
// kernel: real 2.9e-16, 1.1e-16, 1.6e-16; complex 2.9e-16, 1.1e-16, 2.1e-16 (60 us
// a base without).
template <bool CX>
__global__ __launch_bounds__(64 * kBaseWaves, 2) void hsma_potrf_base(double *__restrict__ A_, int64_t lda, int n) {
    constexpr int ES = CX ? 2 : 1;
    typedef double V2 __attribute__((ext_vector_type(2), aligned(8)));
    typedef typename Mma<double>::Acc Acc;
    __shared__ double col[kBaseRows * 16];   // block column j as it stands
    __shared__ double both[2][kBaseRows * 16];   // ... and factored, j even and odd
    HSMA_GLOBAL double *A = (HSMA_GLOBAL double *)A_;
    const int lane = threadIdx.x & 63, g = lane >> 4, lr = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mr = ES * n, nb = (mr + 15) / 16;
    // Column c of a block in LDS: columns 4 apart on different banks.
    auto at = [](int c) { return 16 * (c ^ ((c >> 2) & 1)); };
    auto put = [&](const Acc &v, int i) {
#pragma unroll
        for (int h = 0; h < 4; ++h) col[256 * i + at(4 * g + h) + lr] = -v[h];
    };

    // Block (bi, bm) of each slot (bm < 0: none).
    int bi[kBaseSlots], bm[kBaseSlots];
    Acc acc[kBaseSlots];
    int m = 0, rem = w;
#pragma unroll
    for (int u = 0; u < kBaseSlots; ++u) {
        while (m < nb && rem >= nb - m) {
            rem -= nb - m;
            ++m;
        }
        bm[u] = m < nb ? m : -1;
        bi[u] = m + rem;
        rem += kBaseWaves;
        acc[u] = Acc{0, 0, 0, 0};
        if (bm[u] >= 0) {
            // (Every block on its way before the first is looked at; places beyond
            // the matrix or above its diagonal read a value below.)
            const int R = 16 * bi[u] + lr, C0 = 16 * bm[u] + 4 * g;
            if constexpr (CX) {
                const int r = R / 2 < n ? R / 2 : n - 1;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = C0 / 2 + h < r ? C0 / 2 + h : r;
                    const V2 z = *reinterpret_cast<const HSMA_GLOBAL V2 *>(A + 2 * (r + c * lda));
                    acc[u][2 * h] = z.x;
                    acc[u][2 * h + 1] = z.y;
                }
            } else {
                const int r = R < n ? R : n - 1;
#pragma unroll
                for (int h = 0; h < 4; ++h) acc[u][h] = A[r + (C0 + h < r ? C0 + h : r) * lda];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < kBaseSlots; ++u) {
        if (bm[u] >= 0) {
            const int R = 16 * bi[u] + lr, C0 = 16 * bm[u] + 4 * g;
#pragma unroll
            for (int h = 0; h < 4; h += ES) {
                const int C = C0 + h;
                if constexpr (CX) {
                    // Component (R ^ C) & 1 of element (R / 2, C / 2), the
                    // diagonal's second taken as zero.
                    const double re = acc[u][h], im = C / 2 == R / 2 ? 0.0 : acc[u][h + 1];
                    acc[u][h] = R & 1 ? -im : -re;
                    acc[u][h + 1] = R & 1 ? -re : im;
                    if (R >= mr || C / 2 > R / 2) acc[u][h] = acc[u][h + 1] = 0;
                } else {
                    acc[u][h] = R >= mr || C > R ? 0 : -acc[u][h];
                }
            }
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (R >= mr && C0 + h == R) acc[u][h] = -1.0;  // beyond the matrix: the identity
        }
    }
#pragma unroll
    for (int u = 0; u < kBaseSlots; ++u)
        if (bm[u] == 0) put(acc[u], bi[u]);
    __syncthreads();

    // Block column j of the factor to memory, by wavefronts 4..7 while the others
    // work on the next.
    auto store = [&](int j) {
        const int i = 4 * (w - 4) + g, R = 16 * i + lr;
        if (i < j || R >= mr) return;
#pragma unroll
        for (int c = 0; c < 16; c += ES) {
            const int C = 16 * j + c;
            const double x = both[j & 1][256 * i + at(c) + lr];
            // (Complex: component R & 1 of element (R / 2, C / 2).)
            if (C / ES <= R / ES) A[R + C * lda] = CX && (R & 1) && C / 2 == R / 2 ? 0.0 : x;
        }
    };

    for (int j = 0; j < nb; ++j) {
        double *fac = both[j & 1];
        if (w < 4 && 4 * w + 3 >= j && 4 * w < nb) {
            const int i = 4 * w + g;
            const bool in = i >= j && i < nb;
            const double *own = col + 256 * (in ? i : j);
            double e[16], x[16];
            auto load = [&] {
#pragma unroll
                for (int c = 0; c < 16; ++c) e[c] = col[256 * j + at(c) + lr];
#pragma unroll
                for (int c = 0; c < 16; ++c) x[c] = own[at(c) + lr];
            };
            load();
            if (__builtin_expect(!__all(eliminate<CX, true>(e, x, lr, i == j)), 0)) {
                load();
                eliminate<CX, false>(e, x, lr, i == j);
            }
            if (in) {
#pragma unroll
                for (int c = 0; c < 16; ++c) fac[256 * i + at(c) + lr] = x[c];
            }
        } else if (w >= 4 && j > 0) {
            store(j - 1);
        }
        __syncthreads();
        if (j + 1 == nb) break;
        // (The columns 4g .. 4g + 3 in the order they lie in, the same for both
        // operands.  The places are formed anew at each step: 34 of them do not
        // fit beside the blocks.)
        int fa0 = 64 * g + Mma<double>::a_row(lr), fb0 = 64 * g + lr;
        asm volatile("" : "+v"(fa0), "+v"(fb0));
#pragma unroll
        for (int u = 0; u < kBaseSlots; ++u) {
            if (bm[u] > j) {
                double fa[4], fb[4];
                Acc t = {0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    fa[s] = fac[256 * bm[u] + fa0 + 16 * s];
                    fb[s] = fac[256 * bi[u] + fb0 + 16 * s];
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) t = Mma<double>::mma(fa[s], fb[s], t);
#pragma unroll
                for (int h = 0; h < 4; ++h) acc[u][h] += t[h];
                if (bm[u] == j + 1) put(acc[u], bi[u]);
            }
        }
        __syncthreads();
    }
    if (w >= 4) store(nb - 1);
}

hsma_status potrf_base(bool cx, int n, double *A, int64_t lda, hipStream_t s) {
    ProfScope prof(HSMA_PHASE_FACTOR, (cx ? 4.0 : 1.0) * n * (double)n * n / 3.0, s);
    const dim3 block(64 * kBaseWaves);
    if (cx) hipLaunchKernelGGL(hsma_potrf_base<true>, dim3(1), block, 0, s, A, lda, n);
    else hipLaunchKernelGGL(hsma_potrf_base<false>, dim3(1), block, 0, s, A, lda, n);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

// The split of an order-n step: n1 is n/2 rounded up to a multiple of 64.
int64_t split(int64_t n) { return (n / 2 + 63) / 64 * 64; }

// Largest n1 * n2 over every step of the recursion (the first half can be
// larger than n/2, so a step inside it can need more than the top one).
int64_t max_split_product(bool cx, int64_t n) {
    if (n <= base_order(cx)) return 0;
    const int64_t n1 = split(n), n2 = n - n1;
    return std::max(n1 * n2, std::max(max_split_product(cx, n1), max_split_product(cx, n2)));
}

// `work` holds at least es * n1 * n2 doubles for every split of the
// recursion (the copy of L21^H that the trailing update reads as its right
// operand).
hsma_status potrf_rec(bool cx, int64_t n, double *A, int64_t lda, double *work, hipStream_t s) {
    if (n <= base_order(cx)) return potrf_base(cx, (int)n, A, lda, s);
    const int es = cx ? 2 : 1;
    const int64_t n1 = split(n), n2 = n - n1;
    double *A11 = A, *A21 = A + es * n1, *A22 = A + es * (n1 + n1 * lda);
    HSMA_TRY(potrf_rec(cx, n1, A11, lda, work, s));
    // L21 = A21 inv(L11)^H: X L11^H = A21, the right-side conjugate-transpose
    // TRSM (transpose for real data), which also leaves L21^H (n1 x n2) in
    // work: the right operand of the update.
    HSMA_TRY(trsm_right_lower_keep(cx, n2, n1, A11, lda, A21, lda, work, s));
    // A22 <- A22 - L21 L21^H on the lower triangle: one product with the
    // lower-triangular store.
    HSMA_TRY(launch_gemm(cx, GemmRole::Herk, (int)(es * n2), (int)n2, (int)(es * n1), cplx{-1.0, 0.0},
                         A21, lda, work, es * n1, cplx{1.0, 0.0}, A22, es * lda, 0, s, 0, 1));
    return potrf_rec(cx, n2, A22, lda, work, s);
}

}  // namespace
}  // namespace hsma

extern "C" hsma_status hsma_potrf(int64_t n, void *A, int64_t lda, hsma_dtype dtype,
                                  hsma_stream_t stream) {
    using namespace hsma;
    if (dtype != HSMA_R64F && dtype != HSMA_C64F && !is_single(dtype)) return HSMA_INVALID_VALUE;
    if (is_single(dtype)) return HSMA_NOT_SUPPORTED;
    if (n < 0) return HSMA_INVALID_SIZE;
    if (lda < std::max<int64_t>(1, n)) return HSMA_INVALID_SIZE;
    if (n == 0) return HSMA_SUCCESS;
    if (!A) return HSMA_INVALID_POINTER;
    if (n > (int64_t)1 << 30) return HSMA_INVALID_SIZE;
    DeviceInfo dev;
    HSMA_TRY(device_info(&dev));
    if (!dev.arch_ok) return HSMA_NOT_SUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool cx = dtype == HSMA_C64F;
    const int es = cx ? 2 : 1;
    double *Ad = static_cast<double *>(A);
    if (n <= base_order(cx)) return potrf_base(cx, (int)n, Ad, lda, s);
    void *ws = nullptr;
    HSMA_TRY(ws_alloc(&ws, (size_t)es * max_split_product(cx, n) * sizeof(double), s));
    hsma_status st = potrf_rec(cx, n, Ad, lda, static_cast<double *>(ws), s);
    hsma_status st2 = ws_free(ws, s);
    return st != HSMA_SUCCESS ? st : st2;
}

extern "C" hsma_status hsma_potrs(int64_t n, int64_t nrhs, const void *L, int64_t lda, void *B,
                                  int64_t ldb, hsma_dtype dtype, hsma_stream_t stream) {
    using namespace hsma;
    if (dtype != HSMA_R64F && dtype != HSMA_C64F && !is_single(dtype)) return HSMA_INVALID_VALUE;
    if (is_single(dtype)) return HSMA_NOT_SUPPORTED;
    if (n < 0 || nrhs < 0) return HSMA_INVALID_SIZE;
    if (lda < std::max<int64_t>(1, n) || ldb < std::max<int64_t>(1, n)) return HSMA_INVALID_SIZE;
    if (n == 0 || nrhs == 0) return HSMA_SUCCESS;
    if (!L || !B) return HSMA_INVALID_POINTER;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const double one[2] = {1.0, 0.0};
    // L Y = B, then L^H X = Y
    HSMA_TRY(trsm_impl(HSMA_NON_UNIT, n, nrhs, one, L, lda, B, ldb, dtype, 0, 0, s, nullptr,
                       nullptr, nullptr, nullptr));
    return hsma_trsm_general(HSMA_LEFT, HSMA_LOWER, dtype == HSMA_C64F ? HSMA_OP_C : HSMA_OP_T,
                             HSMA_NON_UNIT, n, nrhs, one, L, lda, B, ldb, dtype, stream);
}
