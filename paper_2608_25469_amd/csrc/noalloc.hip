// hsma_trsm_noalloc: the operation of hsma_trsm for callers that cannot
// allocate device memory (code under HIP graph capture, tight serving loops,
// harnesses that forbid hipMalloc).
//
// hsma_trsm takes no device memory beyond its inputs and outputs: the small
// kernels work in registers and LDS, and so do the blocked path's panels.  So
// this is the same schedule without the entry point's options.  The sizes it
// takes are those whose I_B-block workspace would fit the scratch size that
// hsma_noalloc_scratch_bytes states.

#include "internal.h"

namespace hsma {

size_t blocked_workspace_bytes(bool cx, int64_t m, int ib);
int panel_span(bool cx, int block_size);
hsma_status blocked_trsm(bool cx, bool unit, int64_t m, int64_t n, cplx alpha, const double *A,
                         int64_t lda, double *B, int64_t ldb, int span, hipStream_t s, bool mixed);
int lookup_block_size(bool cx, int64_t m, int64_t n);

namespace {

constexpr size_t kScratchBytes = (size_t)HSMA_NOALLOC_SCRATCH_BYTES;

}  // namespace
}  // namespace hsma

extern "C" hsma_status hsma_trsm_noalloc(hsma_diag diag, int64_t m, int64_t n, const void *alpha,
                                         const void *A, int64_t lda, void *B, int64_t ldb,
                                         hsma_dtype dtype, hsma_stream_t stream) {
    using namespace hsma;
    bool quick = false;
    HSMA_TRY(validate(diag, dtype, m, n, alpha, A, lda, B, ldb, &quick));
    if (quick) return HSMA_SUCCESS;
    const bool cx = dtype == HSMA_C64F;
    const double *a = static_cast<const double *>(alpha);
    const cplx al{a[0], cx ? a[1] : 0.0};
    const bool azero = al.re == 0.0 && al.im == 0.0;
    const int ib = (m > 64 && !azero) ? lookup_block_size(cx, m, n) : 0;
    // Size check before any device call.
    if (ib && blocked_workspace_bytes(cx, m, ib) > kScratchBytes) return HSMA_WORKSPACE_TOO_SMALL;
    DeviceInfo dev;
    HSMA_TRY(device_info(&dev));
    if (!dev.arch_ok) return HSMA_NOT_SUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    double *Bd = static_cast<double *>(B);
    const double *Ad = static_cast<const double *>(A);
    if (azero) return launch_zero(m, n, cx ? 2 : 1, Bd, ldb, s);
    if (m <= 64) return launch_small_solve(cx, diag == HSMA_UNIT, (int)m, n, al, Ad, lda, Bd, ldb, s);
    return blocked_trsm(cx, diag == HSMA_UNIT, m, n, al, Ad, lda, Bd, ldb, panel_span(cx, 0), s, false);
}

extern "C" uint64_t hsma_noalloc_scratch_bytes(void) { return (uint64_t)hsma::kScratchBytes; }
