// FP64 and mixed-precision matrix-core products of the blocked path (the
// kernel is gemm_core.h): tile shapes per role, single and grouped launches.
//
// Paper, Sec. 4.3: the large solve is a sequence of matrix products, the
// trailing updates B_r <- B_r - A_{r,:} X between the panel solves (panel.hip);
// Cholesky's lower-triangular update and the residual of refinement run on
// the same kernel.

#include <algorithm>

#include "gemm_core.h"
#include "tile_choice.h"

namespace hsma {
namespace {

using gemmk::gemm_tile;
using gemmk::launch_tiles;

int phase_of(GemmRole role) {
    return role == GemmRole::Update || role == GemmRole::UpdateMixed ? HSMA_PHASE_UPDATE
           : role == GemmRole::Herk                                  ? HSMA_PHASE_FACTOR
                                                                     : HSMA_PHASE_OTHER;
}

// Workgroups per CU that a tile's accumulators leave registers for: a 64 x 64
// sub-tile per wavefront takes 128 of the 256 that two per SIMD have (a third
// would spill).
constexpr int most_wg(int bm, int bn) { return bm * bn >= 128 * 128 ? 2 : 3; }

template <bool CX, int BM, int BN, int BK, int WM, int WN, bool TRI = false>
hsma_status tiles64(const GemmParams &p, GemmRole role, hipStream_t s) {
    return launch_tiles<double, double, CX, TRI, BM, BN, BK, WM, WN, most_wg(BM, BN)>(p, phase_of(role), s);
}

template <bool CX>
hsma_status launch_role(GemmRole role, const GemmParams &p, hipStream_t s) {
    DeviceInfo dev;
    const int64_t cus = (device_info(&dev) == HSMA_SUCCESS && dev.num_cus > 0) ? dev.num_cus : 256;
    if (role == GemmRole::Residual) {
        // Where 128 x 128 tiles leave CUs idle, a slice's latency counts and not
        // its products: half as many slices, of smaller tiles.  A solve and a
        // refinement step with smaller / larger tiles, us: 64 x 17 51 / 62, 128 x
        // 128 43 / 68, 2000 x 300 416 / 617, complex 64 x 64 83 / 104; 2000 x 1900
        // (240 tiles) 762 / 922.
        if ((int64_t)((p.M + 127) / 128) * ((p.N + 127) / 128) < cus) return tiles64<CX, 64, 64, 32, 2, 2, true>(p, role, s);
        return tiles64<CX, 128, 128, 16, 2, 2, true>(p, role, s);
    }
    if (role == GemmRole::Herk) {
        // Lower-triangular C: the shape with the fewest rounds of non-empty
        // tiles (tile_choice.h).
        const int best = lower_tile_shape(p.M, p.N, CX, 1, cus);
        if (best == 0) return tiles64<CX, 128, 128, 16, 2, 2>(p, role, s);
        if (best == 1) return tiles64<CX, 128, 64, 16, 2, 2>(p, role, s);
        if (best == 2) return tiles64<CX, 64, 64, 32, 2, 2>(p, role, s);
        if (best == 3) return tiles64<CX, 64, 32, 32, 2, 2>(p, role, s);
        return tiles64<CX, 32, 32, 64, 2, 2>(p, role, s);
    }
    // Trailing updates.  Each element's K order is the same in every shape.
    switch (update_tile_shape(p.M, p.N, cus)) {
        case 0: return tiles64<CX, 128, 128, 16, 2, 2>(p, role, s);
        case 1: return tiles64<CX, 128, 64, 16, 2, 2>(p, role, s);
        case 2: return tiles64<CX, 64, 64, 32, 2, 2>(p, role, s);
        case 3: return tiles64<CX, 64, 32, 32, 2, 2>(p, role, s);
        default: return tiles64<CX, 32, 32, 64, 2, 2>(p, role, s);
    }
}

// Mixed precision (real data): operands rounded to FP32 (round to nearest
// even) as fragments are read, FP32 accumulators flushed into FP64 every 256
// values of K.  At 8192^3: 106 TF/s with this tile, 102 with 128 x 64, 94 with
// 64 x 64 (the FP64 operands make the LDS ring as large as the FP64 product's).
hsma_status launch_mixed(const GemmParams &p, hipStream_t s) {
    DeviceInfo dev;
    const int64_t cus = (device_info(&dev) == HSMA_SUCCESS && dev.num_cus > 0) ? dev.num_cus : 256;
    auto tiles = [&](int bm, int bn) { return (int64_t)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn); };
    if (p.M >= 128 && tiles(128, 128) >= 2 * cus)
        return launch_tiles<double, float, false, false, 128, 128, 16, 2, 2, 2, 256>(p, HSMA_PHASE_UPDATE, s);
    if (p.M >= 64 && tiles(64, 64) >= cus)
        return launch_tiles<double, float, false, false, 64, 64, 16, 2, 2, 3, 256>(p, HSMA_PHASE_UPDATE, s);
    return launch_tiles<double, float, false, false, 32, 32, 64, 2, 2, 3, 256>(p, HSMA_PHASE_UPDATE, s);
}

// Grouped launch: descriptor d owns tiles [d.tile0, d.tile0 + tiles_m
// tiles_n) of the grid; each workgroup finds its descriptor by binary search
// over the ascending tile0 values and computes one tile of that product.
template <bool CX, int BM, int BN, int BK, int WM, int WN, int OCC>
__global__ __launch_bounds__(256, OCC) void hsma_gemm_grouped(const GemmParams *__restrict__ descs, int nd) {
    const int t = blockIdx.x;
    int lo = 0, hi = nd - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (descs[mid].tile0 <= t) lo = mid;
        else hi = mid - 1;
    }
    const GemmParams p = descs[lo];
    const int local = t - p.tile0;
    if (local < 0 || local >= p.tiles_m * p.tiles_n) return;
    gemm_tile<double, double, CX, false, BM, BN, BK, WM, WN, BK>(
        p, (const HSMA_GLOBAL double *)p.A, (const HSMA_GLOBAL double *)p.B, (HSMA_GLOBAL double *)p.C,
        local % p.tiles_m, local / p.tiles_m);
}

template <bool CX, int BM, int BN, int BK, int WM, int WN>
hsma_status grouped_t(const GemmParams *descs, int nd, int64_t tiles, int phase, double flops,
                      hipStream_t s) {
    constexpr int OCC = gemmk::occupancy(gemmk::ring_bytes<double, CX>(BM, BN, BK), most_wg(BM, BN));
    ProfScope prof(phase, flops, s);
    hipLaunchKernelGGL((hsma_gemm_grouped<CX, BM, BN, BK, WM, WN, OCC>), dim3((unsigned)tiles), dim3(256), 0,
                       s, descs, nd);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

template <bool CX>
hsma_status grouped_shape(int bm, int bn, const GemmParams *descs, int nd, int64_t tiles, double flops,
                          hipStream_t s) {
    const int phase = HSMA_PHASE_UPDATE;
    if (bm == 32 && bn == 32) return grouped_t<CX, 32, 32, 64, 2, 2>(descs, nd, tiles, phase, flops, s);
    if (bm == 64 && bn == 64) return grouped_t<CX, 64, 64, 32, 2, 2>(descs, nd, tiles, phase, flops, s);
    if (bm == 128 && bn == 128) return grouped_t<CX, 128, 128, 16, 2, 2>(descs, nd, tiles, phase, flops, s);
    return HSMA_NOT_SUPPORTED;
}

}  // namespace

void gemm_grouped_tile(int max_n, int *bm, int *bn) { *bm = *bn = max_n <= 32 ? 32 : max_n <= 256 ? 64 : 128; }

hsma_status launch_gemm_grouped(bool cplx_, int bm, int bn, const GemmParams *descs,
                                int nd, int64_t total_tiles, double flops, hipStream_t s) {
    if (nd <= 0 || total_tiles <= 0) return HSMA_SUCCESS;
    if (total_tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
    return cplx_ ? grouped_shape<true>(bm, bn, descs, nd, total_tiles, flops, s)
                 : grouped_shape<false>(bm, bn, descs, nd, total_tiles, flops, s);
}

hsma_status launch_gemm(bool cplx_, GemmRole role, int M, int N, int K, cplx alpha,
                        const double *A, int64_t lda, const double *B, int64_t ldb, cplx beta,
                        double *C, int64_t ldc, int tri_a, hipStream_t s, int k_lower,
                        int c_lower) {
    if (M <= 0 || N <= 0) return HSMA_SUCCESS;
    GemmParams p{};
    p.M = M;
    p.N = N;
    p.K = K;
    p.A = A;
    p.lda = lda;
    p.B = B;
    p.ldb = ldb;
    p.C = C;
    p.ldc = ldc;
    p.alpha_re = alpha.re;
    p.alpha_im = alpha.im;
    p.beta_re = beta.re;
    p.beta_im = beta.im;
    p.tri_a = tri_a;
    p.k_lower = (k_lower && tri_a) ? 1 : 0;
    p.c_lower = c_lower ? 1 : 0;
    if (cplx_ && ((M | K) & 1)) return HSMA_INVALID_SIZE;
    if (role == GemmRole::UpdateMixed) {
        if (cplx_) return HSMA_NOT_SUPPORTED;
        return launch_mixed(p, s);
    }
    return cplx_ ? launch_role<true>(role, p, s) : launch_role<false>(role, p, s);
}

}  // namespace hsma
