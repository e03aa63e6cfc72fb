// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "../../include/hsma.h"

// Problems with m, n <= HSMA_TINY_MAX take the fused four-per-wavefront
// kernel (tiny.hip), alone and in batches.
#ifndef HSMA_TINY_MAX
#define HSMA_TINY_MAX 16
#endif

// Size of the allocation-free entry point's per-device scratch array.
#define HSMA_NOALLOC_SCRATCH_BYTES (64ull << 20)

namespace hsma {

// Record a failing HIP call for hsma_last_hip_error() and turn it into a status.
hsma_status hip_fail(hipError_t e);

#define HSMA_HIP(call)                                   \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) return ::hsma::hip_fail(e_); \
    } while (0)

#define HSMA_TRY(call)                                   \
    do {                                                 \
        hsma_status s_ = (call);                         \
        if (s_ != HSMA_SUCCESS) return s_;               \
    } while (0)

// Global-memory address space.  Pointers that kernels read out of descriptor
// tables are generic; loads and stores through a generic pointer become FLAT
// instructions, which count against the LDS wait counter as well, so every
// wait for an LDS read would also wait for the global loads in flight.
// Kernels convert such pointers with a cast to HSMA_GLOBAL before use.
#define HSMA_GLOBAL __attribute__((address_space(1)))

// Two doubles moved as one 16-byte access (a complex value, or two
// consecutive real entries); it assumes only 8-byte alignment.
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

// Complex scalar as two doubles (interleaved storage).
struct cplx {
    double re, im;
};

// Per-device facts read once.
struct DeviceInfo {
    int device = -1;
    int num_cus = 0;
    int arch_ok = 0;   // gfx950
};
hsma_status device_info(DeviceInfo *out);

// While profiling is enabled, records an event pair around the enclosed
// kernel launch on stream s (see hsma_profile_begin).
class ProfScope {
  public:
    ProfScope(int phase, double flops, hipStream_t s);
    ~ProfScope();
    ProfScope(const ProfScope &) = delete;
    ProfScope &operator=(const ProfScope &) = delete;

  private:
    hipStream_t s_;
    int idx_;
};

// Workspace from the library's per-device block cache (alloc.cpp): usable
// in stream order on s; ws_free hands the block back after the work already
// enqueued on s.
hsma_status ws_alloc(void **p, size_t bytes, hipStream_t s);
hsma_status ws_free(void *p, hipStream_t s);
// Return a block whose last use has completed on the device: reusable on any
// stream at once (no event).
hsma_status ws_free_idle(void *p);
size_t ws_cached_bytes();

// ---------------------------------------------------------------------------
// Kernel launchers (each enqueues on `s`; arguments already validated).
// ---------------------------------------------------------------------------

// B <- alpha * inv(tril(A)) * B for m <= 64; panels of 64 columns.
hsma_status launch_small_solve(bool cplx_, bool unit, int m, int64_t n, cplx alpha,
                               const double *A, int64_t lda, double *B, int64_t ldb,
                               hipStream_t s);

// Fused very small solves (m, n <= HSMA_TINY_MAX): one problem, or a device
// table of items in the batched layout, four per workgroup.
bool tiny_fits(int64_t m, int64_t n);
size_t tiny_item_bytes();
hsma_status launch_tiny_one(bool cx, bool unit, int m, int n, cplx alpha, const double *A,
                            int64_t lda, double *B, int64_t ldb, hipStream_t s);
hsma_status launch_tiny_group(bool cx, bool unit, const void *items, int count, hipStream_t s);

// The same on FP32 data (m <= 64).
hsma_status launch_small_solve(bool cplx_, bool unit, int m, int64_t n, cplx alpha,
                               const float *A, int64_t lda, float *B, int64_t ldb,
                               hipStream_t s);

// Argument checks of one problem (the documented order); FP32 data types
// pass only with allow32, else HSMA_NOT_SUPPORTED.
hsma_status validate(int diag, int dtype, int64_t m, int64_t n, const void *alpha, const void *A,
                     int64_t lda, const void *B, int64_t ldb, bool *quick, bool allow32 = false);
bool is_single(int dtype);
bool is_complex(int dtype);
cplx read_alpha(int dtype, const void *alpha);

// B <- 0 on FP32 data (m x n, leading dimension ldb, `es` floats per element).
hsma_status launch_zero32(int64_t m, int64_t n, int es, float *B, int64_t ldb, hipStream_t s);

// B <- 0 (m x n, leading dimension ldb, `es` doubles per element).
hsma_status launch_zero(int64_t m, int64_t n, int es, double *B, int64_t ldb, hipStream_t s);

// General matrix product used by the blocked path, in real-view units:
//   C = beta * C + alpha * op(A) * B,
// C is M x N (ldc), B is K x N (ldb).  Real: A is M x K (lda).  Complex: A is
// (M/2) x (K/2) complex (lda in complex elements) and is expanded on the fly
// to its M x K real representation; B and C are complex matrices viewed as
// real with twice the rows (ldb, ldc in doubles).
// tri_a: A is the m x m diagonal block of a lower-triangular matrix, read only
// on and below its diagonal (0: plain, 1: lower non-unit, 2: lower unit).
enum class GemmRole { Update, Residual, UpdateMixed, Herk };

// Parameters of one product (also the descriptor of a grouped launch, read
// by the kernel from device memory); T is the data type in memory.
template <typename T>
struct GemmParamsT {
    int M, N, K;          // real-view sizes
    const T *A;
    int64_t lda;          // real: components of T; complex: complex elements
    const T *B;
    int64_t ldb;          // components of T
    T *C;
    int64_t ldc;          // components of T
    T alpha_re, alpha_im, beta_re, beta_im;
    int tri_a;            // 0 plain, 1 lower non-unit, 2 lower unit (diagonal block of L)
    int tiles_m, tiles_n;
    int tile0;            // grouped launch: first tile of this product in the grid
    int k_lower;          // 1: A is lower triangular as a whole (with tri_a), so a
                          // tile of rows [m0, m0 + BM) stops its K loop at m0 + BM
    int c_lower;          // 1: only the lower triangle of C (column <= row, in
                          // elements) is computed and stored
};
typedef GemmParamsT<double> GemmParams;

// Tile shape of a grouped launch of updates whose widest product has max_n columns
// (not tuned: the widest product's columns, up to four tiles of the next smaller
// shape).
void gemm_grouped_tile(int max_n, int *bm, int *bn);
// Launch over nd descriptors already in device memory (tile0 / tiles_m /
// tiles_n filled for the shape gemm_grouped_tile returned); total_tiles is
// the grid size.  flops is for the phase profiler.
hsma_status launch_gemm_grouped(bool cplx_, int bm, int bn, const GemmParams *descs,
                                int nd, int64_t total_tiles, double flops, hipStream_t s);

// k_lower = 1: A (with tri_a != 0) is a whole lower-triangular matrix, so
// each row tile reads only the columns left of its last row.
// c_lower = 1: only C's lower triangle (element column <= element row) is
// written; tiles wholly above the diagonal do nothing.
hsma_status launch_gemm(bool cplx_, GemmRole role, int M, int N, int K,
                        cplx alpha, const double *A, int64_t lda, const double *B,
                        int64_t ldb, cplx beta, double *C, int64_t ldc, int tri_a, hipStream_t s,
                        int k_lower = 0, int c_lower = 0);
// An update on FP32 data (FP32 matrix cores, FP32 accumulation).
hsma_status launch_gemm(bool cplx_, GemmRole role, int M, int N, int K, cplx alpha, const float *A,
                        int64_t lda, const float *B, int64_t ldb, cplx beta, float *C, int64_t ldc,
                        int tri_a, hipStream_t s);

// One panel solve (panel.hip): X = alpha inv(L) B in place for `rows` rows, L
// at A, unit or not; at most kPanelRows real-view rows.
constexpr int kPanelRows = 512;
constexpr int kMaxLooks = 1 << 20;
template <typename T>
struct PanelParams {
    const T *A;
    int64_t lda;         // elements
    T *B;
    int64_t ldb, n;      // elements, columns
    T alpha_re, alpha_im;
    int rows, unit;
    int tile0;           // grouped launch: first workgroup of this panel
    // A panel of a chain (launch_chain): `left` 16-row blocks lie before it, and
    // X moves through `mail`, 256 values per block, `nblk` blocks per strip of 16
    // columns.
    int left, nblk;
    T *mail;
    // `at` != 0: element (r, c) of the right-hand side lies at B + r rs + c cs
    // (elements; rs and cs may be negative), conjugated if `conj`, and keep, if
    // given, receives X as well (leading dimension ldkeep).
    int at, conj;
    int64_t rs, cs;
    T *keep;
    int64_t ldkeep;
    int per;             // strips of 16 columns a workgroup solves one after another (0: one; chains: one)
    int looks = kMaxLooks;  // of a wavefront at what it waits for, before it takes NaN instead
};
template <typename T>
hsma_status launch_panel(bool cx, const PanelParams<T> &p, hipStream_t s);
// Panels of up to wide_rows real-view rows whose strips are many times what the
// chip takes at once run on a kernel of their own, several strips a workgroup:
// `per` for a launch whose panels have these numbers of strips and at most max_rows
// rows (1: the other kernel).
constexpr int wide_rows(int elem) { return elem == 8 ? 128 : 256; }
int panel_per(bool cx, int elem, int max_rows, const int64_t *strips, size_t count);
// The workgroups of a panel with at most *per strips each, and *per with them
// shared out evenly.
int64_t panel_share(int64_t strips, int *per);
template <typename T>
hsma_status launch_panel_wide(bool cx, const PanelParams<T> &one, const PanelParams<T> *descs, int nd, int max_rows,
                              int64_t groups, hipStream_t s);
hsma_status launch_chain_wide(bool cx, const PanelParams<double> *descs, int nd, int64_t tiles, unsigned *tickets,
                              hipStream_t s);
// Workgroups of 512 that one launch can have (2^32 threads).
constexpr int64_t kMaxGroups = ((int64_t)1 << 32) / 512 - 1;
// Rows of a panel of a solve with n columns, unless the caller says (blocked.cpp).
int panel_span(bool cx, int elem, int64_t n);
// A whole solve as one launch: panels of kChainRows real-view rows in order, a
// workgroup per panel and strip of 16 columns, X handed on through `ws`
// (chain_bytes).  Rows any number.
constexpr int kChainRows = 256;
template <typename T>
size_t chain_bytes(bool cx, int64_t m, int64_t n);
// Device memory a blocked solve in panels of `span` rows needs (0: none).
template <typename T>
size_t blocked_bytes(bool cx, int64_t m, int64_t n, int span, bool mixed);
// A right-hand side at strides (PanelParams::at) solved where it lies, in one
// launch; allowed where solves_in_one says so.
bool solves_in_one(bool cx, int64_t m, int64_t n);
hsma_status blocked_in_one(bool cx, int64_t m, PanelParams<double> p, hipStream_t s);
// Whether such a solve runs as a chain (blocked.cpp); elem: bytes of a component.
bool chain_rule(bool cx, int elem, int64_t m, int64_t n);
template <typename T>
hsma_status launch_chain(bool cx, const PanelParams<T> &p, int64_t m, void *ws, hipStream_t s);
// nd descriptors in device memory, ascending tile0; `tiles` workgroups in all.
// Chains: every descriptor one panel of a solve, a solve's panels in order; the
// mail they point into is `words` values at `mail`, with 256 bytes more.
hsma_status launch_chain_grouped(bool cx, const PanelParams<double> *descs, int nd, int64_t tiles, double *mail,
                                 int64_t words, double flops, hipStream_t s);
hsma_status launch_panel_grouped(bool cx, const PanelParams<double> *descs, int nd, int max_rows, int64_t groups,
                                 bool wide, double flops, hipStream_t s);

// dst (R x C, ldd) = src^H for src C x R (ldsrc); the transpose for real data.
// X L^H = B for a lower, non-unit L (m x n X and B, n x n L; FP64 real or
// complex), the solve of a Cholesky step: X overwrites B, and xh (n x m,
// leading dimension n) receives X^H as well.
hsma_status trsm_right_lower_keep(bool cx, int64_t m, int64_t n, const double *A, int64_t lda, double *B,
                                  int64_t ldb, double *xh, hipStream_t s);
hsma_status launch_conj_transpose(bool cx, const double *src, int64_t ldsrc, double *dst,
                                  int64_t ldd, int64_t R, int64_t C, hipStream_t s);

// Synthetic serving inputs (Philox4x32-10, see hsma_generate_inputs).
struct GenRequest {
    double *L, *B;   // lda = ldb = m
    int64_t m, n;
    uint64_t key;
    bool cx;
};
hsma_status launch_gen_inputs(bool cx, int64_t m, int64_t n, uint64_t key, double *L, double *B,
                              hipStream_t s);
hsma_status gen_inputs_grouped(const GenRequest *reqs, int count, hipStream_t s);

}  // namespace hsma
