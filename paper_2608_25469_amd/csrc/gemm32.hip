// FP32 matrix-core product for the single-precision solves (STRSM, CTRSM): the
// trailing updates of the blocked path on FP32 data with FP32 accumulation, on
// the FP32 matrix cores (twice the FP64 matrix rate on gfx950).  The kernel is
// gemm_core.h.

#include "gemm_core.h"

namespace hsma {
namespace {

template <bool CX, int BM, int BN, int BK>
hsma_status tiles32(const GemmParamsT<float> &p, hipStream_t s) {
    return gemmk::launch_tiles<float, float, CX, false, BM, BN, BK, 2, 2, (BM * BN >= 128 * 128 ? 2 : 3)>(
        p, HSMA_PHASE_UPDATE, s);
}

// Thin updates of the deepest levels: narrower tiles when a 128 x 128 grid
// would leave CUs idle.  A real operand's larger tile (140 against 133 TF/s at
// 8192^3) where it still gives four rounds.
template <bool CX>
hsma_status update32(const GemmParamsT<float> &p, hipStream_t s) {
    DeviceInfo dev;
    const int64_t cus = (device_info(&dev) == HSMA_SUCCESS && dev.num_cus > 0) ? dev.num_cus : 256;
    auto tiles = [&](int bm, int bn) { return (int64_t)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn); };
    // (A tile taller than the product would load it element by element: an update of
    // 44 x 300000 of K = 256 154 us with 32 x 32 tiles, 545 with 256 x 128.)
    if constexpr (!CX) {
        if (p.M >= 256 && tiles(256, 128) >= 4 * cus) return tiles32<CX, 256, 128, 16>(p, s);
    }
    if (p.M >= 128 && tiles(128, 128) >= 2 * cus) return tiles32<CX, 128, 128, 16>(p, s);
    if (p.M >= 128 && tiles(128, 64) >= 2 * cus) return tiles32<CX, 128, 64, 32>(p, s);
    if (p.M >= 64 && tiles(64, 64) >= 2 * cus) return tiles32<CX, 64, 64, 32>(p, s);
    if (p.M < 64) return tiles32<CX, 32, 32, 64>(p, s);
    return tiles32<CX, 64, 32, 64>(p, s);
}

}  // namespace

hsma_status launch_gemm(bool cplx_, GemmRole role, int M, int N, int K, cplx alpha,
                        const float *A, int64_t lda, const float *B, int64_t ldb, cplx beta,
                        float *C, int64_t ldc, int tri_a, hipStream_t s) {
    if (M <= 0 || N <= 0) return HSMA_SUCCESS;
    if (role != GemmRole::Update || tri_a) return HSMA_NOT_SUPPORTED;
    if (cplx_ && ((M | K) & 1)) return HSMA_INVALID_SIZE;
    GemmParamsT<float> p{};
    p.M = M;
    p.N = N;
    p.K = K;
    p.A = A;
    p.lda = lda;
    p.B = B;
    p.ldb = ldb;
    p.C = C;
    p.ldc = ldc;
    p.alpha_re = (float)alpha.re;
    p.alpha_im = (float)alpha.im;
    p.beta_re = (float)beta.re;
    p.beta_im = (float)beta.im;
    return cplx_ ? update32<true>(p, s) : update32<false>(p, s);
}

}  // namespace hsma
