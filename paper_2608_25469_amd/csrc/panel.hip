// Panel solve: X = alpha inv(L) B for up to 512 real-view rows (512 real, 256
// complex) in one launch, in place.  The blocked path (m > 64) walks L in such
// panels and runs matrix products between them.
//
// Paper, Sec. 4.3: diagonal blocks are inverted, and the solve becomes matrix
// products.  Here the inverted blocks are 16 x 16 (real view): just large
// enough for the matrix cores, and small enough that every workgroup inverts
// them for itself, in registers, instead of reading them from a workspace
// that other launches fill.
//
// One workgroup of eight wavefronts solves 16 columns.  The rows are cut into
// 16-row blocks, dealt to the wavefronts in turn (wavefront w holds blocks w,
// w + 8, ...), each block of the right-hand side one 16 x 16 accumulator.
// Step i: the owner of block i multiplies it by the block's inverse (X_i),
// publishes -X_i in LDS and stores X_i; after one barrier every wavefront
// adds L_ji (-X_i) to its blocks j > i, the owner of block i + 1 to that block
// first, so that X_{i+1} is under way while the others still update (the
// barrier of step i + 1 then finds it done).
//
// No operand changes layout.  With the rows of an A fragment in the order that
// makes a lane's results four consecutive rows 4g + v of column l%16 (g =
// l/16, see gemm_core.h), a result is the next product's B fragment as it
// stands, if k-step s takes k = 4g + s instead of 4s + g; the A fragments are
// loaded in that order, straight from L (16 consecutive rows of four columns
// per load), D steps ahead.
//
// What bounds it: for few columns the chain of a step (four products for the
// block, four for its update, LDS and the barrier: about 700 cycles per 16
// rows), otherwise the matrix cores.

#include <type_traits>

#include "dpp_fma.h"
#include "gemm_core.h"

namespace hsma {
namespace {

using gemmk::Mma;
using gemmk::fma_rn;
using gemmk::mul_rn;

constexpr int kWaves = 8;

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
template <int N>
__device__ __forceinline__ float bcast(float v) {
    return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x150 + N, 0xf, 0xf, false));
}

template <typename T>
__device__ __forceinline__ T div_rn(T a, T b) {
    if constexpr (sizeof(T) == 8) return __ddiv_rn(a, b);
    else return __fdiv_rn(a, b);
}

// NQ: blocks per wavefront (rows <= 128 NQ in the real view).
template <typename T, bool CX, int NQ>
struct Solve {
    static constexpr int ES = CX ? 2 : 1;
    static constexpr int NB = kWaves * NQ;          // blocks
    static constexpr int D = NQ == 4 ? 3 : 4;       // steps an A fragment is loaded ahead
    static constexpr int V = 16 / (int)sizeof(T);
    typedef HSMA_GLOBAL T GT;
    typedef typename Mma<T>::Acc Acc;
    typedef T VG __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    typedef T V2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));

    struct Shared {
        T inv[NB][256];    // inverse of block j: element (r, k) at 16 k + (r ^ k)
        T x[2][4 * 64];    // -X_i: element v of lane l at 64 v + l
    };

    const GT *A;       // the panel's diagonal block of L
    int64_t lda;
    int mr, nb;        // real-view rows, blocks
    int w, lane, g, lr, arow;
    GT *col;           // this lane's column of B
    bool col_ok;
    Shared &sh;
    Acc acc[NQ];
    T a[D][NQ][4];     // L_ji of steps i, i + 1, ..: slot i % D

    __device__ __forceinline__ explicit Solve(Shared &s) : sh(s) {}

    // Four values of column `col` at rows r..r+3 (0 at or beyond mr).
    __device__ __forceinline__ Acc load4(int r) const {
        Acc v = {0, 0, 0, 0};
        if (r + 4 <= mr) {
#pragma unroll
            for (int h = 0; h < 4; h += V) {
                const VG t = *reinterpret_cast<const HSMA_GLOBAL VG *>(col + r + h);
#pragma unroll
                for (int e = 0; e < V; ++e) v[h + e] = t[e];
            }
        } else {
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (r + h < mr) v[h] = col[r + h];
        }
        return v;
    }
    __device__ __forceinline__ void store4(int r, Acc v) const {
        if (!col_ok) return;
        if (r + 4 <= mr) {
#pragma unroll
            for (int h = 0; h < 4; h += V) {
                VG t;
#pragma unroll
                for (int e = 0; e < V; ++e) t[e] = v[h + e];
                *reinterpret_cast<HSMA_GLOBAL VG *>(col + r + h) = t;
            }
        } else {
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (r + h < mr) col[r + h] = v[h];
        }
    }

    // This lane's part of L_ji for step I and its blocks w + 8 q, q >= Q0:
    // row 16 j + arow (kept below mr), columns 16 I + 4 g .. + 3.  Complex:
    // the two complex elements that hold them, expanded at use.
    template <int I>
    __device__ __forceinline__ void load_l() {
        constexpr int Q0 = (I + 1) / kWaves;
        // (Past the last step: columns 0..15, which a panel of two blocks has.)
        const int i = I < nb - 1 ? I : 0;
        static_for<Q0, NQ>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            const int r = 16 * (w + kWaves * q) + arow;
            if constexpr (CX) {
                const int cr = r / 2 < mr / 2 ? r / 2 : mr / 2 - 1;
                const GT *p = A + 2 * (cr + (int64_t)(8 * i + 2 * g) * lda);
                const V2 e0 = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p);
                const V2 e1 = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p + 2 * lda);
                a[I % D][q][0] = e0.x;
                a[I % D][q][1] = e0.y;
                a[I % D][q][2] = e1.x;
                a[I % D][q][3] = e1.y;
            } else {
                const GT *p = A + (r < mr ? r : mr - 1) + (int64_t)(16 * i + 4 * g) * lda;
#pragma unroll
                for (int s = 0; s < 4; ++s) a[I % D][q][s] = p[s * lda];
            }
        });
    }

    // acc_q += L_ji (-X_i).
    template <int I, int Q>
    __device__ __forceinline__ void update(const T (&xb)[4]) {
        T f[4];
        const T(&e)[4] = a[I % D][Q];
        if constexpr (CX) {
            // Real row r, real column 2c + q of the expansion: component
            // (r ^ q) & 1, negated where q = 1 and r is even.
            const bool odd = arow & 1;
            f[0] = odd ? e[1] : e[0];
            f[1] = odd ? e[0] : -e[1];
            f[2] = odd ? e[3] : e[2];
            f[3] = odd ? e[2] : -e[3];
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) f[s] = e[s];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[Q] = Mma<T>::mma(f[s], xb[s], acc[Q]);
    }

    // X_J = inv(L_JJ) acc, published and stored (by its owner).
    template <int J>
    __device__ __forceinline__ void finish() {
        constexpr int q = J / kWaves;
        T f[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) f[s] = sh.inv[J][16 * (4 * g + s) + (arow ^ (4 * g + s))];
        if (16 * J + 16 > mr) {  // rows beyond the panel hold no numbers
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (16 * J + 4 * g + v >= mr) acc[q][v] = 0;
        }
        Acc x = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 4; ++s) x = Mma<T>::mma(f[s], acc[q][s], x);
#pragma unroll
        for (int v = 0; v < 4; ++v) sh.x[J & 1][64 * v + lane] = -x[v];
        store4(16 * J + 4 * g, x);
    }

    // Step I: X_I is in LDS once the barrier is passed.
    template <int I>
    __device__ __forceinline__ void step() {
        if constexpr (I + 1 < NB) {
            if (I + 1 < nb) {
                constexpr int W1 = (I + 1) % kWaves, Q1 = (I + 1) / kWaves;
                __syncthreads();
                T xb[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) xb[s] = sh.x[I & 1][64 * s + lane];
                if (w == W1) {
                    update<I, Q1>(xb);
                    finish<I + 1>();
                } else if (w > W1) {
                    update<I, Q1>(xb);
                }
                static_for<Q1 + 1, NQ>([&](auto Q) { update<I, decltype(Q)::value>(xb); });
                if constexpr (I + D + 1 < NB) load_l<I + D>();
                step<I + 1>();
            }
        }
    }

    // Inverses of this wavefront's diagonal blocks, one per 16-lane row: lane
    // c holds row c of the block and solves for column c of the inverse, the
    // coefficients reaching the lanes by row broadcasts.
    __device__ __forceinline__ void invert(bool unit) {
        constexpr int N = 16 / ES;  // order of a block
        const int q = g < NQ ? g : NQ - 1;
        const int j = w + kWaves * q;
        const int rows = mr / ES;
        const int c = lane & (N - 1);
        const int d0 = N * j < rows ? N * j : 0;  // (a block beyond the panel is not used)
        const int row = d0 + c < rows ? d0 + c : rows - 1;
        const bool in = d0 + c < rows;
        const GT *p = A + (int64_t)ES * row;
        T lre[N], lim[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            // Only the strict lower triangle and the diagonal are read.
            const int cc = d0 + k < row ? d0 + k : row;
            if constexpr (CX) {
                const V2 e = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p + 2 * (int64_t)cc * lda);
                lre[k] = e.x;
                lim[k] = e.y;
            } else {
                lre[k] = p[(int64_t)cc * lda];
                lim[k] = 0;
            }
        }
        T dr = 1, di = 0;
        if (!unit && in) {
            // Column c holds the diagonal (row - d0 == c here).
            T er = 0, ei = 0;
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (k == c) {
                    er = lre[k];
                    ei = lim[k];
                }
            if constexpr (CX) {
                const T den = fma_rn(er, er, mul_rn(ei, ei));
                dr = div_rn(er, den);
                di = -div_rn(ei, den);
            } else {
                dr = div_rn((T)1, er);
            }
        }
        T yr[N], yi[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if (!(in && k < c)) lre[k] = lim[k] = 0;
            yr[k] = k == c ? 1 : 0;
            yi[k] = 0;
        }
        static_for<0, N>([&](auto K) {
            constexpr int k = decltype(K)::value;
            const T er = bcast<k>(dr), ei = CX ? bcast<k>(di) : 0;
            if constexpr (CX) {
                const T xr = fma_rn(yr[k], er, -mul_rn(yi[k], ei));
                const T xi = fma_rn(yr[k], ei, mul_rn(yi[k], er));
                yr[k] = xr;
                yi[k] = xi;
            } else {
                yr[k] = mul_rn(yr[k], er);
            }
            // (One column at a time: otherwise every broadcast coefficient of
            // the unrolled walk is formed first and spills.)
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (sizeof(T) == 8 && !CX) {
                if constexpr (k + 1 < N) smallk::fnma_rows<false, k + 1>(yr, yi, lre[k], 0, yr[k], 0);
            } else static_for<k + 1, N>([&](auto R) {
                constexpr int r = decltype(R)::value;
                const T cr = bcast<r>(lre[k]);
                if constexpr (CX) {
                    const T ci = bcast<r>(lim[k]);
                    yr[r] = fma_rn(ci, yi[k], fma_rn(-cr, yr[k], yr[r]));
                    yi[r] = fma_rn(-ci, yr[k], fma_rn(-cr, yi[k], yi[r]));
                } else {
                    yr[r] = fma_rn(-cr, yr[k], yr[r]);
                }
            });
        });
        if (g >= NQ || (CX && (lane & 8))) return;
        T *dst = sh.inv[j];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (CX) {
                const int k0 = 2 * c, k1 = 2 * c + 1;
                dst[16 * k0 + ((2 * i) ^ k0)] = yr[i];
                dst[16 * k0 + ((2 * i + 1) ^ k0)] = yi[i];
                dst[16 * k1 + ((2 * i) ^ k1)] = -yi[i];
                dst[16 * k1 + ((2 * i + 1) ^ k1)] = yr[i];
            } else {
                dst[16 * c + (i ^ c)] = yr[i];
            }
        }
    }

    __device__ __forceinline__ void run(const PanelParams<T> &p, int tile) {
        A = (const GT *)p.A;
        lda = p.lda;
        mr = ES * p.rows;
        nb = (mr + 15) / 16;
        lane = threadIdx.x & 63;
        w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        g = lane >> 4;
        lr = lane & 15;
        arow = Mma<T>::a_row(lr);
        const int64_t c = 16 * (int64_t)tile + lr;
        col_ok = c < p.n;
        col = (GT *)p.B + (int64_t)ES * (col_ok ? c : p.n - 1) * p.ldb;

        invert(p.unit);
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, NQ>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            acc[q] = load4(16 * (w + kWaves * q) + 4 * g);
        });
        // (A panel of one block has nothing below it: its L may end before
        // column 15.)
        if (nb > 1) {
            static_for<0, D>([&](auto I) {
                if constexpr (decltype(I)::value + 1 < NB) load_l<decltype(I)::value>();
            });
        }
        if (p.alpha_re != 1 || p.alpha_im != 0) {
            static_for<0, NQ>([&](auto Q) {
                Acc &v = acc[decltype(Q)::value];
                if constexpr (CX) {
#pragma unroll
                    for (int h = 0; h < 4; h += 2) {
                        const T re = v[h], im = v[h + 1];
                        v[h] = fma_rn(p.alpha_re, re, -mul_rn(p.alpha_im, im));
                        v[h + 1] = fma_rn(p.alpha_re, im, mul_rn(p.alpha_im, re));
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 4; ++h) v[h] = mul_rn(p.alpha_re, v[h]);
                }
            });
        }
        if (w == 0) finish<0>();
        step<0>();
    }
};

// One panel (descs == nullptr), or many: descriptor d owns workgroups
// [tile0, tile0 + ceil(n / 16)), found by binary search.
template <typename T, bool CX, int NQ>
__global__ __launch_bounds__(64 * kWaves, 2) void hsma_panel(const PanelParams<T> one,
                                                             const PanelParams<T> *__restrict__ descs, int nd) {
    typedef Solve<T, CX, NQ> S;
    __shared__ typename S::Shared sh;
    PanelParams<T> p = one;
    int tile = blockIdx.x;
    if (descs) {
        int lo = 0, hi = nd - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (descs[mid].tile0 <= tile) lo = mid;
            else hi = mid - 1;
        }
        p = descs[lo];
        tile -= p.tile0;
    }
    S s(sh);
    s.run(p, tile);
}

template <typename T, bool CX>
hsma_status launch(const PanelParams<T> &one, const PanelParams<T> *descs, int nd, int max_rows, int64_t tiles,
                   hipStream_t s) {
    const int mr = max_rows * (CX ? 2 : 1);
    if (mr > kPanelRows || tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
    const dim3 grid((unsigned)tiles), block(64 * kWaves);
    if (mr <= 128) hipLaunchKernelGGL((hsma_panel<T, CX, 1>), grid, block, 0, s, one, descs, nd);
    else if (mr <= 256) hipLaunchKernelGGL((hsma_panel<T, CX, 2>), grid, block, 0, s, one, descs, nd);
    else hipLaunchKernelGGL((hsma_panel<T, CX, 4>), grid, block, 0, s, one, descs, nd);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

}  // namespace

template <typename T>
hsma_status launch_panel(bool cx, const PanelParams<T> &p, hipStream_t s) {
    if (p.rows <= 0 || p.n <= 0) return HSMA_SUCCESS;
    ProfScope prof(HSMA_PHASE_LEAF, (cx ? 4.0 : 1.0) * p.rows * (double)p.rows * (double)p.n, s);
    const int64_t tiles = (p.n + 15) / 16;
    return cx ? launch<T, true>(p, nullptr, 0, p.rows, tiles, s) : launch<T, false>(p, nullptr, 0, p.rows, tiles, s);
}
template hsma_status launch_panel<double>(bool, const PanelParams<double> &, hipStream_t);
template hsma_status launch_panel<float>(bool, const PanelParams<float> &, hipStream_t);

hsma_status launch_panel_grouped(bool cx, const PanelParams<double> *descs, int nd, int max_rows, int64_t tiles,
                                 double flops, hipStream_t s) {
    if (nd <= 0 || tiles <= 0) return HSMA_SUCCESS;
    ProfScope prof(HSMA_PHASE_LEAF, flops, s);
    const PanelParams<double> none{};
    return cx ? launch<double, true>(none, descs, nd, max_rows, tiles, s)
              : launch<double, false>(none, descs, nd, max_rows, tiles, s);
}

}  // namespace hsma
