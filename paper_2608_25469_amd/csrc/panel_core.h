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
// w + 8, ...), each block's products one 16 x 16 accumulator.
// Step i: X_i is in LDS; every wavefront adds L_ji (-X_i) to its blocks j > i +
// 1 (the owner of block i + 2 then multiplies that block by its inverse: y),
// while the owner of block i + 1 forms X_{i+1} = y - P X_i with P =
// inv(L_{i+1,i+1}) L_{i+1,i}, prepared at the start, and publishes it in LDS.
// There is no barrier: X_i has a place of its own, a count in LDS says how many
// are there, and a wavefront waits for nothing but the X it needs, so only four
// products lie on the chain from one X to the next.
//
// No operand changes layout.  With the rows of an A fragment in the order that
// makes a lane's results four consecutive rows 4g + v of column l%16 (g =
// l/16, see gemm_core.h), a result is the next product's B fragment as it
// stands, if k-step s takes k = 4g + s instead of 4s + g; the A fragments are
// loaded in that order, straight from L (16 consecutive rows of four columns
// per load), D steps ahead.
//
// What bounds it: for few columns the chain of a step (four products for the
// block, four for its update, LDS: 750 cycles per 16 rows in panels of 128 rows,
// 1030 of 256, 1700 of 512, where the products of the other blocks and their 8
// bytes per lane of L stand in the way) after a start of 10 000 to 23 000
// cycles (loads, inversions).  For many columns the same chains, of which a CU runs
// two at once where registers and LDS allow (WIDE: panels of 128 rows, 256 in
// FP32, several strips of 16 columns a workgroup, so that the start is paid once):
// DTRSM 128 x 300000 292 us, one strip a workgroup and one workgroup a CU 396;
// STRSM 65 x 300000 146 us and 316; the products with inverted blocks before
// panels 329 and 142.

#pragma once

#include <type_traits>

#include "dpp_fma.h"
#include "gemm_core.h"
#include "panel_index.h"

namespace hsma {
namespace panelk {

using gemmk::Mma;
using gemmk::fma_rn;
using gemmk::mul_rn;

constexpr int kWaves = kPanelWaves;

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

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ const void *uniform(const void *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const void *)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ bool finite(double v) { return __builtin_amdgcn_class(v, 0x1f8); }
__device__ __forceinline__ bool finite(float v) { return __builtin_amdgcn_classf(v, 0x1f8); }

template <typename T>
__device__ __forceinline__ T div_rn(T a, T b) {
    if constexpr (sizeof(T) == 8) return __ddiv_rn(a, b);
    else return __fdiv_rn(a, b);
}

// The words that carry X between workgroups: written and read past the caches
// of an XCD (relaxed atomics at agent scope), each its own message.  An empty
// place holds a signalling NaN, which no arithmetic returns, so a word that is
// anything else has arrived and no flag or order between words is needed.
template <typename T>
struct Word;
template <>
struct Word<double> {
    typedef unsigned long long U;
    static constexpr U kEmpty = 0x7ff05a5a5a5a5a5aull;
};
template <>
struct Word<float> {
    typedef unsigned U;
    static constexpr U kEmpty = 0x7f805a5au;
};
template <typename T>
__device__ __forceinline__ void mail_store(T *p, T v) {
    typedef typename Word<T>::U U;
    __hip_atomic_store(reinterpret_cast<U *>(p), __builtin_bit_cast(U, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T mail_load(const T *p) {
    typedef typename Word<T>::U U;
    return __builtin_bit_cast(T, __hip_atomic_load(reinterpret_cast<const U *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
template <typename T>
__device__ __forceinline__ bool is_empty(T v) {
    return __builtin_bit_cast(typename Word<T>::U, v) == Word<T>::kEmpty;
}

// Every wait ends, whatever went wrong elsewhere: after PanelParams::looks looks a
// wavefront goes on, every X that it forms is NaN, and it looks once and no more at
// whatever it needs later.  2^20 looks are 1.7 s at the mail (1.6 us each) and
// about 50 ms in LDS (some 100 cycles); what they wait for takes microseconds.

// NQ: blocks per wavefront (rows <= 128 NQ in the real view).  CHAIN: the panel
// is one of a chain.  AT: the right-hand side lies at strides.  WIDE: many more
// strips than the chip takes at once, so registers for two workgroups a CU and
// not for the latency of one, and several strips a workgroup.
template <typename T, bool CX, int NQ, bool CHAIN, bool AT = false, bool WIDE = false>
struct Solve {
    static constexpr int ES = CX ? 2 : 1;
    static constexpr int NB = kWaves * NQ;          // blocks
    static constexpr int D = WIDE ? 2 : NQ == 1 && sizeof(T) == 8 && !CX ? 3 : NQ == 4 ? 3 : 4;       // steps an A fragment is loaded ahead
    static constexpr int V = 16 / (int)sizeof(T);
    typedef HSMA_GLOBAL T GT;
    typedef typename Mma<T>::Acc Acc;
    typedef T VG __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    typedef T V2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));

    struct Shared {
        // Block j: P_j (element (r, k) at 16 k + (r ^ k)), then -X_j (element v of
        // lane l at 64 v + l).
        T blk[NB][256];
        T inv[NB][256];    // inv(L_jj), laid out as P_j; both are read by j's owner alone
        T diag[NB][16];    // reciprocals of L_jj's diagonal (complex: (re, im) of the 8 elements)
        T pivot[NB][16];   // L_jj's diagonal, likewise
        T left[CHAIN ? 2 : 1][CHAIN ? 2 * 256 : 1];  // two blocks of -X from before the panel
        int ticket;
        int done;          // blocks of X formed, of this strip and those before it
    };

    const GT *A;       // the panel's diagonal block of L
    int64_t lda;
    const HSMA_GLOBAL char *at[NQ];  // this lane's row of block w + 8 q, column 4 g of the panel
    int mr, nb;        // real-view rows, blocks
    int before;        // blocks of the strips before this one
    int w, lane, g, lr, arow;
    GT *col;           // this lane's column of B
    bool col_ok;
    int64_t rs;        // AT: from one row to the next, in components
    bool conj;
    GT *keep;          // AT: this lane's column of the copy of X
    Shared &sh;
    Acc acc[NQ];       // L X of the blocks solved so far, negated, from zero
    // The right-hand side of blocks w + 8 q, before alpha: place q % 2 (WIDE: one place).
    static constexpr int RP = NQ > 1 && !WIDE ? 2 : 1;
    Acc rhs[RP];
    T are, aim;        // alpha
    T a[D][NQ][4];     // L_ji of steps i, i + 1, ..: slot i % D
    T *mail;           // CHAIN: this strip's blocks of -X, from block 0 of the solve
    int left;          // blocks before the panel
    int spare;         // panel_spare(left)
    int looks;         // of a wait; 0: one has given up
    bool unit;
    // Of this wavefront's next block, read from LDS a step before their use (a
    // set for each of its blocks does not fit beside them):
    T fi[4];           // inv(L_jj) without its diagonal, as A fragments
    T fp[4];           // P_j = inv(L_jj) L_{j,j-1}, as A fragments
    Acc y;             // the sums of inv(L_jj) beside its diagonal, and of P; then X_j
    Acc main;          // the diagonal's part

    __device__ __forceinline__ explicit Solve(Shared &s) : sh(s) {}

    // Four values of column `col` at rows r..r+3, r = r0 + dr (0 at or beyond mr).
    __device__ __forceinline__ Acc load4(int r0, int dr) const {
        Acc v = {0, 0, 0, 0};
        const int r = r0 + dr;
        if constexpr (AT) {
#pragma unroll
            for (int h = 0; h < 4; h += ES) {
                if (r + h < mr) {
                    const GT *e = col + (r + h) / ES * rs;
                    if constexpr (CX) {
                        const V2 z = *reinterpret_cast<const HSMA_GLOBAL V2 *>(e);
                        v[h] = z.x;
                        v[h + 1] = conj ? -z.y : z.y;
                    } else {
                        v[h] = *e;
                    }
                }
            }
        } else if (r0 + 16 <= mr) {
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
        if constexpr (AT) {
#pragma unroll
            for (int h = 0; h < 4; h += ES) {
                if (r + h < mr) {
                    GT *e = col + (r + h) / ES * rs;
                    if constexpr (CX) {
                        *reinterpret_cast<HSMA_GLOBAL V2 *>(e) = V2{v[h], conj ? -v[h + 1] : v[h + 1]};
                        if (keep) *reinterpret_cast<HSMA_GLOBAL V2 *>(keep + r + h) = V2{v[h], v[h + 1]};
                    } else {
                        *e = v[h];
                        if (keep) keep[r + h] = v[h];
                    }
                }
            }
        } else if (r + 4 <= mr) {
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

    // This lane's part of L for block row w + 8 q and columns 16 i + 4 g .. + 3
    // (i counts from the panel's first column, negative before it): a scalar
    // number of bytes from the lane's place.
    __device__ __forceinline__ void load_a(int q, int i, T (&f)[4]) const {
        const HSMA_GLOBAL char *p = at[q] + (int64_t)i * (16 * lda * (int64_t)sizeof(T));
        if constexpr (CX) {
            const V2 e0 = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p);
            const V2 e1 = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p + 2 * lda * (int64_t)sizeof(T));
            f[0] = e0.x;
            f[1] = e0.y;
            f[2] = e1.x;
            f[3] = e1.y;
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) f[s] = *reinterpret_cast<const GT *>(p + s * lda * (int64_t)sizeof(T));
        }
    }

    // This lane's part of L_ji for step I and its blocks w + 8 q, q >= Q0:
    // row 16 j + arow (kept below mr), columns 16 I + 4 g .. + 3; where the step
    // has no use for them, columns it may read (panel_index.h).  Complex: the two
    // complex elements that hold them, expanded at use.
    template <int I>
    __device__ __forceinline__ void load_l() {
        constexpr int Q0 = (I + 2) / kWaves;
        static_for<Q0, NQ>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            load_a(q, panel_column(I, q, w, nb, spare), a[I % D][q]);
        });
    }

    // This lane's part of L_{j,j-1} as a B fragment: rows 16 j + 4g .. + 3 (0
    // beyond the panel) of column 16 (j - 1) + lr.
    __device__ __forceinline__ void load_b(int j, T (&f)[4]) const {
        const int r = 16 * j + 4 * g;
        if constexpr (CX) {
            const GT *p = A + 2 * (int64_t)(8 * (j - 1) + lr / 2) * lda;
            const bool odd = lr & 1;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (r + 2 * h < mr) {
                    const V2 e = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p + r + 2 * h);
                    f[2 * h] = odd ? -e.y : e.x;
                    f[2 * h + 1] = odd ? e.x : e.y;
                }
            }
        } else {
            const GT *p = A + (int64_t)(16 * (j - 1) + lr) * lda;
            if (16 * j + 16 <= mr) {
#pragma unroll
                for (int s = 0; s < 4; s += V) {
                    const VG t = *reinterpret_cast<const HSMA_GLOBAL VG *>(p + r + s);
#pragma unroll
                    for (int e = 0; e < V; ++e) f[s + e] = t[e];
                }
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (r + s < mr) f[s] = p[r + s];
            }
        }
    }

    // The A fragments of a 16 x 16 block in LDS.
    __device__ __forceinline__ void read_a(const T *blk, T (&f)[4]) const {
#pragma unroll
        for (int s = 0; s < 4; ++s) f[s] = blk[16 * (4 * g + s) + (arow ^ (4 * g + s))];
    }

    __device__ __forceinline__ void read_inverse(int j) {
        read_a(sh.inv[j], fi);
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (arow / ES == (4 * g + s) / ES) fi[s] = 0;
    }

    // acc_q += L_ji (-X_i).
    template <int I, int Q>
    __device__ __forceinline__ void update(const T (&xb)[4]) {
        multiply<Q>(a[I % D][Q], xb);
    }
    template <int Q>
    __device__ __forceinline__ void multiply(const T (&e)[4], const T (&xb)[4]) {
        T f[4];
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

    // CHAIN: the products with every X before the panel, two blocks (a group)
    // at a time: a wavefront fetches a quarter of a block from the mail and LDS
    // hands it round.  Four groups are on their way at once, and one that came
    // back empty is asked for again two rounds before it is needed: a look costs
    // 1.6 us, so with one group on its way the panel falls ever further behind
    // the one before it.  L is loaded four blocks ahead (WIDE: two).
    __device__ __forceinline__ void apply_left() {
        const int groups = left / 2;  // a multiple of 8: panels have 16 blocks
        constexpr int LA = WIDE ? 2 : 4;  // blocks that L is loaded ahead
        T l[LA][NQ][4], nx[4], again = 0;
        bool behind = false;  // the last group had to be waited for
        const T *src = mail + 256 * (w >> 2) + 64 * (w & 3) + lane;
        static_for<0, 4>([&](auto K) {
            constexpr int k = decltype(K)::value;
            nx[k] = mail_load(src + 512 * k);
            if constexpr (k < LA) static_for<0, NQ>([&](auto Q) { load_a(decltype(Q)::value, k - left, l[k][decltype(Q)::value]); });
        });
        for (int t4 = 0; t4 < groups; t4 += 4) {
            static_for<0, 4>([&](auto H) {
                constexpr int h = decltype(H)::value;
                const int t = t4 + h;
                const bool late = __any(is_empty(nx[h]));
                if (late && behind) nx[h] = again;
                int polls = 0;
                for (; __any(is_empty(nx[h])) && polls < looks; ++polls) nx[h] = mail_load(src + 512 * (int64_t)t);
                if (polls == looks) looks = 0;
                behind = late;
                if (late && t + 1 < groups) again = mail_load(src + 512 * (int64_t)(t + 1));
                T *buf = sh.left[h & 1];
                buf[256 * (w >> 2) + 64 * (w & 3) + lane] = nx[h];
                constexpr int s2 = (h + 2) % 4;
                if (t + 2 < groups && __any(is_empty(nx[s2]))) nx[s2] = mail_load(src + 512 * (int64_t)(t + 2));
                if (t + 4 < groups) nx[h] = mail_load(src + 512 * (int64_t)(t + 4));
                __syncthreads();
                static_for<0, 2>([&](auto K) {
                    constexpr int k = decltype(K)::value, slot = (2 * h + k) % LA;
                    T xb[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) xb[s] = buf[256 * k + 64 * s + lane];
                    static_for<0, NQ>([&](auto Q) {
                        constexpr int q = decltype(Q)::value;
                        multiply<q>(l[slot][q], xb);
                        // (Beyond the last: the first columns again.)
                        load_a(q, (t + LA / 2 < groups ? 2 * t + LA : 0) + k - left, l[slot][q]);
                    });
                });
            });
        }
    }

    // CHAIN: block J of the panel into the mail (by its owner).
    __device__ __forceinline__ void mail_send(int J, const Acc &x) {
        T *dst = mail + 256 * (int64_t)(left + J) + lane;
#pragma unroll
        for (int v = 0; v < 4; ++v) mail_store(dst + 64 * v, -x[v]);
    }

    // y + main = inv(L_JJ) (alpha B_J + acc) (by the owner of block J, X_0 ..
    // X_{J-2} applied).  The products meet the right-hand side here and not at
    // their start, and the diagonal's part stays apart from the sums: added to
    // them one by one, each of the small terms would be rounded at its size.
    // What the reciprocal and its product round off the diagonal's part is its
    // residual over the diagonal and joins the sums, so that an X is rounded about
    // as often as in a division: 500 x 300 is 6.7e-17 off the exact result in the
    // norm (1.06e-16 without; inverted blocks of 64 rows 8.5e-17; rounding the
    // exact one 4.7e-17), in the same 36.3 us.
    template <int J>
    __device__ __forceinline__ void prepare() {
        constexpr int q = J / kWaves;
        const Acc r = rhs[q % RP];
        if constexpr (WIDE && q + 1 < NQ) rhs[0] = load4(16 * (J + kWaves), 4 * g);
        Acc b;
        if (CX && aim != 0) {
#pragma unroll
            for (int h = 0; h < 4; h += 2) {
                b[h] = fma_rn(are, r[h], fma_rn(-aim, r[h + 1], acc[q][h]));
                b[h + 1] = fma_rn(are, r[h + 1], fma_rn(aim, r[h], acc[q][h + 1]));
            }
        } else {
#pragma unroll
            for (int h = 0; h < 4; ++h) b[h] = fma_rn(are, r[h], acc[q][h]);
        }
        if (16 * J + 16 > mr) {  // rows beyond the panel hold no numbers
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (16 * J + 4 * g + v >= mr) b[v] = 0;
        }
        // (A unit diagonal's reciprocals and pivots are 1 and nothing is rounded;
        // real data takes the same way, in the shadow of the products.)
        if (CX && unit) {
            y = Acc{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 4; ++s) y = Mma<T>::mma(fi[s], b[s], y);
            main = b;
            // (As below: alone where it is not finite.)
            if (__builtin_expect(__ballot(!finite((b[0] - b[0]) + (b[1] - b[1]) + (b[2] - b[2]) + (b[3] - b[3]))) != 0, 0)) {
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    if (!finite(b[h])) y[h] = 0;
            }
            return;
        }
        const T *d = sh.diag[J] + 4 * g, *l = sh.pivot[J] + 4 * g;
        T dv[4], lv[4], rest[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            dv[h] = d[h];
            lv[h] = l[h];
        }
        y = Acc{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 4; ++s) y = Mma<T>::mma(fi[s], b[s], y);
        if constexpr (CX) {
#pragma unroll
            for (int h = 0; h < 4; h += 2) {
                main[h] = fma_rn(b[h], dv[h], -mul_rn(b[h + 1], dv[h + 1]));
                main[h + 1] = fma_rn(b[h], dv[h + 1], mul_rn(b[h + 1], dv[h]));
                const T e0 = fma_rn(lv[h + 1], main[h + 1], fma_rn(-lv[h], main[h], b[h]));
                const T e1 = fma_rn(-lv[h + 1], main[h], fma_rn(-lv[h], main[h + 1], b[h + 1]));
                rest[h] = fma_rn(e0, dv[h], -mul_rn(e1, dv[h + 1]));
                rest[h + 1] = fma_rn(e0, dv[h + 1], mul_rn(e1, dv[h]));
            }
        } else {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                main[h] = mul_rn(dv[h], b[h]);
                rest[h] = mul_rn(fma_rn(-lv[h], main[h], b[h]), dv[h]);
            }
        }
        const T all = (rest[0] + rest[1]) + (rest[2] + rest[3]);
        // (The diagonal's part in the shadow of the products.)
        static_for<0, 4>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, CX ? 8 : 4, 0);
        });
        // An infinity or a NaN in B, an overflow or an infinite pivot leaves no
        // number as the residual.  The diagonal's part then stands as it is, and
        // alone where it is not finite (the sums hold 0 times infinity there).
        if (__builtin_expect(__ballot(!finite(all)) != 0, 0)) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                if (!finite(rest[h])) rest[h] = 0;
                if (!finite(main[h])) y[h] = 0;
            }
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) y[h] += rest[h];
    }

    // X_J to the other wavefronts (by its owner): LDS takes a wavefront's
    // writes in order.
    template <int J>
    __device__ __forceinline__ void publish() {
#pragma unroll
        for (int v = 0; v < 4; ++v) y[v] += main[v];
        if (__builtin_expect(looks == 0, 0)) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                y[v] = (T)__builtin_nan("");
                asm volatile("" : "+v"(y[v]));  // (a branch, not a selection on the chain)
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) sh.blk[J][64 * v + lane] = -y[v];
        asm volatile("" ::: "memory");
        __hip_atomic_store(&sh.done, before + J + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if constexpr (WIDE) {  // (at once, not kept until it is off the others' way)
            if constexpr (CHAIN) mail_send(J, y);
            store4(16 * J + 4 * g, y);
        }
    }
    // X_i is in its place, or this wavefront's further X are NaN (publish).
    __device__ __forceinline__ void await_block(int i) {
        int polls = looks;
        while (__builtin_amdgcn_readfirstlane(
                   __hip_atomic_load(&sh.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) <= before + i) {
            if (--polls < 0) {
                looks = 0;
                break;
            }
        }
        asm volatile("" ::: "memory");
    }

    // Step I: everything X_I is for.
    template <int I>
    __device__ __forceinline__ void step() {
        if constexpr (I + 1 < NB) {
            if (I + 1 < nb) {
                constexpr int W1 = (I + 1) % kWaves, Q1 = (I + 1) / kWaves;
                constexpr int W2 = (I + 2) % kWaves, Q2 = (I + 2) / kWaves;
                const bool chain = w == W1;
                if constexpr (I + 2 < NB)
                    if (w == W2) read_inverse(I + 2);
                if (chain) __builtin_amdgcn_s_setprio(3);
                await_block(I);
                T xb[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) xb[s] = sh.blk[I][64 * s + lane];
                Acc mine = y;  // X_I at its owner
                if (chain) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) y = Mma<T>::mma(fp[s], xb[s], y);
                    publish<I + 1>();
                    __builtin_amdgcn_s_setprio(0);
                }
                if constexpr (I + 2 < NB) {
                    // Blocks I + 2 and up; the owner of I + 2 readies it, and
                    // leaves its later blocks until it has formed X_{I+2}.
                    if (w == W2) {
                        __builtin_amdgcn_s_setprio(2);
                        update<I, Q2>(xb);
                        if (I + 2 < nb) prepare<I + 2>();
                        read_a(sh.blk[I + 2], fp);
                        __builtin_amdgcn_s_setprio(0);
                    } else {
                        if constexpr (I > 0) {
                            if (chain) {
                                T xp[4];
#pragma unroll
                                for (int s = 0; s < 4; ++s) xp[s] = sh.blk[I - 1][64 * s + lane];
                                static_for<Q1 + 1, NQ>([&](auto Q) { update<I - 1, decltype(Q)::value>(xp); });
                            }
                        }
                        if (w > W2) update<I, Q2>(xb);
                        static_for<Q2 + 1, NQ>([&](auto Q) { update<I, decltype(Q)::value>(xb); });
                    }
                }
                // X_I leaves from its owner.
                if (!WIDE && w == I % kWaves) {
                    if constexpr (CHAIN) mail_send(I, mine);
                    store4(16 * I + 4 * g, mine);
                }
                if constexpr (I + D + 1 < NB) load_l<I + D - 1>();
                // The next row of blocks, six steps before the first of them is
                // readied; all wavefronts at once, so that the counts of loads
                // on their way agree and none waits for more than it needs.
                if constexpr (!WIDE && I % kWaves == 0 && I / kWaves + 1 < NQ)
                    rhs[(I / kWaves + 1) % RP] = load4(16 * (w + I + kWaves), 4 * g);
                step<I + 1>();
            }
        }
    }

    // What the steps have left: the last block (nothing waits for it here).
    __device__ __forceinline__ void drain() {
        const int J = nb - 1;
        if (!WIDE && w == J % kWaves) {
            if constexpr (CHAIN) mail_send(J, y);
            store4(16 * J + 4 * g, y);
        }
    }

    // Inverses of this wavefront's diagonal blocks, one per 16-lane row: lane
    // c holds row c of the block and solves for column c of the inverse, the
    // coefficients reaching the lanes by row broadcasts.
    static constexpr int N = 16 / ES;  // order of a block in elements
    __device__ __forceinline__ int inv_block() const { return w + kWaves * (g < NQ ? g : NQ - 1); }
    __device__ __forceinline__ void load_diag(T (&lre)[N], T (&lim)[N]) const {
        const int rows = mr / ES, c = lane & (N - 1);
        const int d0 = N * inv_block() < rows ? N * inv_block() : 0;  // (a block beyond the panel is not used)
        const int row = d0 + c < rows ? d0 + c : rows - 1;
        // Only the strict lower triangle and the diagonal are read.
        const HSMA_GLOBAL char *p = (const HSMA_GLOBAL char *)(A + (int64_t)ES * (row + d0 * lda));
        const int64_t step = ES * lda * (int64_t)sizeof(T), last = (row - d0) * step;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int64_t to = d0 + k < row ? k * step : last;
            if constexpr (CX) {
                const V2 e = *reinterpret_cast<const HSMA_GLOBAL V2 *>(p + to);
                lre[k] = e.x;
                lim[k] = e.y;
            } else {
                lre[k] = *reinterpret_cast<const GT *>(p + to);
                lim[k] = 0;
            }
        }
    }
    __device__ __forceinline__ void invert(T (&lre)[N], T (&lim)[N]) {
        const int j = inv_block(), c = lane & (N - 1);
        const int d0 = N * j < mr / ES ? N * j : 0;
        const bool in = d0 + c < mr / ES;
        T dr = 1, di = 0, er = 1, ei = 0;
        if (!unit && in) {
            // Column c holds the diagonal (row - d0 == c here).
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
        if (g < NQ && !(CX && (lane & 8))) {
            sh.diag[j][ES * c] = dr;
            sh.pivot[j][ES * c] = er;
            if constexpr (CX) {
                sh.diag[j][2 * c + 1] = di;
                sh.pivot[j][2 * c + 1] = ei;
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
                if constexpr (WIDE && CX) __builtin_amdgcn_sched_barrier(0);
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

    __device__ __forceinline__ void run(const PanelParams<T> &p, int group) {
        A = (const GT *)uniform(p.A);
        lda = (int64_t)uniform((const void *)p.lda);
        mr = ES * p.rows;
        nb = (mr + 15) / 16;
        w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        left = CHAIN ? p.left : 0;
        spare = panel_spare(left);
        places(threadIdx.x & 63);
        are = p.alpha_re;
        aim = p.alpha_im;
        looks = __builtin_amdgcn_readfirstlane(p.looks);
        unit = __builtin_amdgcn_readfirstlane(p.unit);
        const int strips = (int)((p.n + 15) / 16), per = !WIDE || CHAIN || p.per < 1 ? 1 : p.per;
        const int last = (group + 1) * per < strips ? (group + 1) * per - 1 : strips - 1;
        int strip = group * per;
        before = 0;
        // The right-hand side, the diagonal blocks and the blocks before them are
        // all on their way before the first is waited for.
        T lb[NQ][4];
        {
            T lre[N], lim[N];
            start_strip(p, strip);
            load_diag(lre, lim);
            if constexpr (!WIDE) load_before(lb);
            invert(lre, lim);
            if constexpr (WIDE) {
                __builtin_amdgcn_sched_barrier(0);
                load_before(lb);
            }
        }
        for (;;) {
            // (Places and offsets are formed anew for each strip: kept, they and
            // not the solve would take the registers.)
            if constexpr (WIDE && !CHAIN) {
                int id = lane;
                asm volatile("" : "+v"(id), "+s"(lda), "+s"(A));
                places(id);
            }
            static_for<0, NQ>([&](auto Q) { acc[decltype(Q)::value] = Acc{0, 0, 0, 0}; });
            static_for<0, NQ>([&](auto Q) {
                constexpr int q = decltype(Q)::value;
                const int j = w + kWaves * q;
                T f[4];
                read_a(sh.inv[j], f);
                Acc t = {0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < 4; ++s) t = Mma<T>::mma(f[s], lb[q][s], t);
                // Row 4g + v, column lr, to the A fragments' order through LDS.
#pragma unroll
                for (int v = 0; v < 4; ++v) sh.blk[j][16 * lr + ((4 * g + v) ^ lr)] = t[v];
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (WIDE && !CHAIN) {
                // (Nothing is carried from one strip to the next.)
                static_for<0, D>([&](auto I) {
                    static_for<0, NQ>([&](auto Q) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) a[decltype(I)::value][decltype(Q)::value][s] = 0;
                    });
                });
#pragma unroll
                for (int s = 0; s < 4; ++s) fi[s] = fp[s] = 0;
                y = main = Acc{0, 0, 0, 0};
                if constexpr (RP > 1) rhs[RP - 1] = y;
            }
            // (A panel of one block has nothing below it: its L may end before
            // column 15.)
            if (nb > 1) {
                static_for<0, D - 1>([&](auto I) {
                    if constexpr (decltype(I)::value + 2 < NB) load_l<decltype(I)::value>();
                });
            }
            if constexpr (CHAIN) {
                if (left > 0) apply_left();
            }
            if (w == 0) {
                read_inverse(0);
                prepare<0>();
                publish<0>();
            } else if (w == 1 && nb > 1) {
                read_inverse(1);
                prepare<1>();
                read_a(sh.blk[1], fp);
            }
            step<0>();
            drain();
            if (!WIDE || CHAIN || strip == last) break;
            // The next strip: the inverses stand, P has to be formed anew where
            // X has taken its place, once every wavefront has read that.
            start_strip(p, ++strip);
            load_before(lb);
            before += nb;
            __syncthreads();
        }
    }

    // What follows from a lane's number.
    __device__ __forceinline__ void places(int id) {
        lane = id;
        g = lane >> 4;
        lr = lane & 15;
        arow = Mma<T>::a_row(lr);
        static_for<0, NQ>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            const int r = panel_row(q, w, arow, mr, spare);
            at[q] = (const HSMA_GLOBAL char *)(A + (CX ? r & ~1 : r) + 4 * g * lda);
        });
    }

    // This lane's column of strip t of 16, and its first right-hand side.
    __device__ __forceinline__ void start_strip(const PanelParams<T> &p, int t) {
        const int64_t c = 16 * (int64_t)t + lr;
        col_ok = c < p.n;
        col = (GT *)p.B + (int64_t)ES * (col_ok ? c : p.n - 1) * (AT ? p.cs : p.ldb);
        if constexpr (AT) {
            rs = ES * p.rs;
            conj = p.conj;
            keep = p.keep ? (GT *)p.keep + (int64_t)ES * (col_ok ? c : p.n - 1) * p.ldkeep : nullptr;
        }
        if constexpr (CHAIN) mail = p.mail + 256 * (int64_t)p.nblk * t;
        rhs[0] = load4(16 * w, 4 * g);
    }

    // The blocks before this wavefront's diagonal blocks (0 where there is none).
    __device__ __forceinline__ void load_before(T (&lb)[NQ][4]) const {
        static_for<0, NQ>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            const int j = w + kWaves * q;
#pragma unroll
            for (int s = 0; s < 4; ++s) lb[q][s] = 0;
            if (j > 0 && j < nb) load_b(j, lb[q]);
        });
    }
};

// One panel (descs == nullptr), or many: descriptor d owns workgroups from tile0,
// one for every `per` strips of 16 columns, found by binary search.
template <typename T>
__device__ __forceinline__ int find(const PanelParams<T> *__restrict__ descs, int nd, int tile) {
    int lo = 0, hi = nd - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (descs[mid].tile0 <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <typename T, bool CX, int NQ, bool AT, bool WIDE>
__global__ __launch_bounds__(64 * kWaves, WIDE || (NQ == 1 && sizeof(T) == 8 && !CX) ? 4 : 2) void hsma_panel(const PanelParams<T> one,
                                                                        const PanelParams<T> *__restrict__ descs,
                                                                        int nd) {
    typedef Solve<T, CX, NQ, false, AT, WIDE> S;
    __shared__ typename S::Shared sh;
    PanelParams<T> p = one;
    int tile = blockIdx.x;
    if (descs) {
        p = descs[find(descs, nd, tile)];
        tile -= p.tile0;
    }
    if (threadIdx.x == 0) sh.done = 0;
    __syncthreads();
    S s(sh);
    s.run(p, tile);
}

// A chain: workgroups take tickets, and ticket t of one solve is panel t /
// strips, strip t % strips, so a workgroup waits only for workgroups that
// started before it.  `one` describes panel 0 with the solve's row count in
// `rows`; with descs each descriptor is one panel, listed so that a solve's
// panels come in order.
template <typename T, bool CX, bool AT, bool WIDE>
__global__ __launch_bounds__(64 * kWaves, WIDE ? 4 : 2) void hsma_chain(const PanelParams<T> one,
                                                                        const PanelParams<T> *__restrict__ descs,
                                                                        int nd, unsigned *__restrict__ tickets) {
    typedef Solve<T, CX, kChainRows / (16 * kWaves), true, AT, WIDE> S;
    __shared__ typename S::Shared sh;
    if (threadIdx.x == 0) {
        sh.done = 0;
        sh.ticket = (int)atomicAdd(tickets, 1u);
    }
    __syncthreads();
    int tile = __builtin_amdgcn_readfirstlane(sh.ticket);
    PanelParams<T> p = one;
    if (descs) {
        p = descs[find(descs, nd, tile)];
        tile -= p.tile0;
    } else {
        constexpr int ES = CX ? 2 : 1, H = kChainRows / ES;
        const int strips = (int)((p.n + 15) / 16);
        const int r = tile / strips;
        tile -= r * strips;
        p.left = r * (kChainRows / 16);
        p.A = one.A + ES * ((int64_t)r * H) * (1 + one.lda);
        p.B = one.B + ES * (int64_t)r * H * (AT ? one.rs : 1);
        if constexpr (AT)
            if (p.keep) p.keep += ES * (int64_t)r * H;
        p.rows = one.rows - r * H < H ? one.rows - r * H : H;
    }
    S s(sh);
    s.run(p, tile);
}

}  // namespace panelk
}  // namespace hsma
