// Shared by the small-regime kernels (strip.hip, tiny.hip): the DPP broadcast,
// complex products and reciprocals with every rounding fixed, and the strip
// descriptor.
//
// Paper, Sec. 4.2.1: columns of B are independent, so each column is a
// separate forward substitution; the triangular operand is shared.  A lane
// keeps a column in VGPRs and each coefficient of L reaches the lanes by a
// 64-bit DPP row_newbcast, with no memory traffic.

#pragma once

#include <type_traits>

#include "internal.h"
#include "dpp_fma.h"

namespace hsma {
namespace smallk {


// Complex product and reciprocal with every rounding fixed (no contraction
// left to the compiler): the small-solve kernels share them, so the same
// problem gives the same bits in every kernel that solves it.
__device__ __forceinline__ void cmul_rn(double ar, double ai, double br, double bi, double &r,
                                        double &i) {
    r = __fma_rn(ar, br, -__dmul_rn(ai, bi));
    i = __fma_rn(ar, bi, __dmul_rn(ai, br));
}
// 1/d (real) or conj(d)/|d|^2 (complex).
__device__ __forceinline__ void recip_rn(bool cx, double dr, double di, double &rr, double &ri) {
    if (cx) {
        const double den = __fma_rn(dr, dr, __dmul_rn(di, di));
        rr = __ddiv_rn(dr, den);
        ri = -__ddiv_rn(di, den);
    } else {
        rr = __ddiv_rn(1.0, dr);
        ri = 0.0;
    }
}

// Every row and bank is enabled, so no lane keeps an old value: mov_dpp
// (old value undefined) needs no copy of the destination first, unlike
// update_dpp with a tied old operand.
template <int N>
__device__ __forceinline__ double bcast16(double v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xf, 0xf, false);  // row_newbcast:N
}

// Work item of the small-solve kernel (strip.hip): one strip of at most 16
// columns of one problem.
struct SmallItem {
    const double *A;
    double *B;        // first column of the strip
    int64_t lda, ldb; // element units
    int32_t m, ncols;
    double ar, ai;    // alpha
};

}  // namespace smallk
}  // namespace hsma
