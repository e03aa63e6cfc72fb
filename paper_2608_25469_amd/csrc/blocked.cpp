// Blocked path for m > 64 (paper Sec. 4.3).
//
// The paper inverts the diagonal blocks of L and walks them left-looking (B_r
// -= A_{r,0:r} X_{0:r}, a product whose K grows with r, then X_r = inv(D_r)
// B_r).  Here the rows are cut into panels of `span` rows and the same algebra
// is walked recursively: solve the top half of the panels, apply one update
//      B_bot <- beta B_bot - L_{bot,top} X_top
// and solve the bottom half.  Half of all flops land in a single (m/2) x n x
// (m/2) product, so the matrix cores see large, square-ish products instead of
// slivers.  One panel is one launch (panel.hip), which inverts the panel's 16 x
// 16 diagonal blocks in registers and runs its own products; it needs no
// workspace.  alpha is folded into the first write of each row block (beta =
// alpha on the first update a panel receives, or alpha in its solve if none).
//
// The panel height.  A panel costs one launch and a chain of steps, one per 16
// rows, an update one launch and a K loop, so the tallest panel the kernel
// takes is the default.  A caller's block_size sets the height instead.
//
// Against inverted I_B blocks (a zero fill, a chunk inversion of 22 us, two
// products per merge level, then an in-place product per block): DTRSM 500 x
// 300 148 -> 36 us, 16384 78.2 -> 64.8 ms, STRSM 4096 1510 -> 801 us.

#include <algorithm>

#include "internal.h"

namespace hsma {

// Whether a solve runs as one chain launch (panel.hip) instead of the recursion:
// where few columns leave the recursion's launches mostly empty.  Measured, us,
// chain / recursion in panels of 512 real-view rows: DTRSM 513 x 256 48 / 64, 1000
// x 256 73 / 83, 1000 x 1024 77 / 88, 2000 x 256 140 / 189, 2000 x 1024 189 / 220,
// 4000 x 256 275 / 427, 4000 x 1024 567 / 585, 8000 x 256 774 / 1068, 1500 x 1024
// 158 / 151; ZTRSM 300 x 256 49 / 57, 1000 x 300 130 / 200, 2000 x 1024 508 / 605,
// 4000 x 256 624 / 1038, 8000 x 256 1983 / 2804; STRSM 1000 x 256 51 / 61, 4000 x
// 256 174 / 326, 8000 x 256 437 / 742.  Beyond the rule an earlier chain was behind
// or level: DTRSM 1024 x 4096 180 (130), 8192 x 1024 1992 (1747), ZTRSM 4096 x 1024
// 1800 (1751).  Up to 512 real-view rows one panel is as fast (37 against 41) and
// needs no mail.
bool chain_rule(bool cx, int elem, int64_t m, int64_t n) {
    const int64_t mr = m * (cx ? 2 : 1), mail = mr * ((n + 15) / 16 * 16) * elem;
    if (mr <= kPanelRows || n > 1024 || mail > (int64_t)HSMA_NOALLOC_SCRATCH_BYTES / 2) return false;
    return n <= 256 || (double)mr * (double)mr * (double)n <= (double)((int64_t)1 << 35);
}

// Panels of 512 real-view rows are the shortest way through the rows.  Through many
// columns it is panels of 128 rows (FP32: 256), which have a kernel that takes them
// two workgroups a CU and shares its start, with products between them.  Tall /
// short panels, us: DTRSM 300 x 24576 161 / 129, 512 x 24576 212 / 229, 512 x 32768
// 279 / 286, 700 x 32768 497 / 512, 300 x 49152 318 / 219, 512 x 49152 415 / 389;
// ZTRSM 65 x 32768 92 / 85, 256 x 32768 311 / 314, 150 x 49152 335 / 234; STRSM 512 x
// 32768 194 / 170; CTRSM 256 x 32768 203 / 165.
constexpr int64_t kWideColumns = 32768;
int panel_span(bool cx, int elem, int64_t n) {
    return (n >= kWideColumns ? wide_rows(elem) : kPanelRows) / (cx ? 2 : 1);
}

namespace {

// T is double (DTRSM, ZTRSM) or float (STRSM, CTRSM); complex data is
// interleaved (re, im) of T, and every offset below counts components of T.
template <typename T>
struct Ctx {
    bool cx;
    bool unit;
    bool mixed = false;  // trailing updates on the FP32 matrix cores (double only)
    int64_t m, n;
    cplx alpha;
    const T *A;
    int64_t lda;
    T *B;
    int64_t ldb;
    int span;
    hipStream_t s;
    int es() const { return cx ? 2 : 1; }
};

template <typename T>
hsma_status panel(const Ctx<T> &c, int64_t b, bool touched) {
    const int64_t r0 = b * c.span;
    const cplx al = touched ? cplx{1.0, 0.0} : c.alpha;
    PanelParams<T> p{};
    p.A = c.A + c.es() * (r0 + r0 * c.lda);
    p.lda = c.lda;
    p.B = c.B + c.es() * r0;
    p.ldb = c.ldb;
    p.n = c.n;
    p.alpha_re = (T)al.re;
    p.alpha_im = (T)al.im;
    p.rows = (int)std::min<int64_t>(c.span, c.m - r0);
    p.unit = c.unit;
    return launch_panel<T>(c.cx, p, c.s);
}

template <typename T>
hsma_status update(const Ctx<T> &c, int64_t r1, int64_t r2, int64_t k0, bool touched) {
    // B[r1:r2] = beta B[r1:r2] - L[r1:r2, k0:r1] B[k0:r1]
    const int es = c.es();
    const cplx beta = touched ? cplx{1.0, 0.0} : c.alpha;
    return launch_gemm(c.cx, c.mixed ? GemmRole::UpdateMixed : GemmRole::Update,
                       (int)(es * (r2 - r1)), (int)c.n, (int)(es * (r1 - k0)),
                       cplx{-1.0, 0.0}, c.A + es * (r1 + k0 * c.lda), c.lda, c.B + es * k0,
                       es * c.ldb, beta, c.B + es * r1, es * c.ldb, 0, c.s);
}

template <typename T>
hsma_status recurse(const Ctx<T> &c, int64_t b0, int64_t nb, bool touched) {
    if (nb == 1) return panel(c, b0, touched);
    const int64_t h = nb / 2;
    HSMA_TRY(recurse(c, b0, h, touched));
    const int64_t r1 = (b0 + h) * c.span;
    const int64_t r2 = std::min<int64_t>((b0 + nb) * c.span, c.m);
    HSMA_TRY(update(c, r1, r2, b0 * c.span, touched));
    return recurse(c, b0 + h, nb - h, true);
}

// One chain launch, or recursion (span 0 stands for both: the rule decides).
template <typename T>
bool use_chain(bool cx, int64_t m, int64_t n, int span, bool mixed) {
    return span == 0 && !mixed && chain_rule(cx, sizeof(T), m, n);
}

template <typename T>
hsma_status blocked_t(bool cx, bool unit, int64_t m, int64_t n, cplx alpha, const T *A,
                      int64_t lda, T *B, int64_t ldb, int span, void *ws, hipStream_t s, bool mixed) {
    if (use_chain<T>(cx, m, n, span, mixed)) {
        PanelParams<T> p{};
        p.A = A;
        p.lda = lda;
        p.B = B;
        p.ldb = ldb;
        p.n = n;
        p.alpha_re = (T)alpha.re;
        p.alpha_im = (T)alpha.im;
        p.unit = unit;
        return launch_chain<T>(cx, p, m, ws, s);
    }
    Ctx<T> c;
    c.mixed = mixed;
    c.cx = cx;
    c.unit = unit;
    c.m = m;
    c.n = n;
    c.alpha = alpha;
    c.A = A;
    c.lda = lda;
    c.B = B;
    c.ldb = ldb;
    c.span = span > 0 ? span : panel_span(cx, sizeof(T), n);
    c.s = s;
    return recurse(c, 0, (m + c.span - 1) / c.span, false);
}

}  // namespace

template <typename T>
size_t blocked_bytes(bool cx, int64_t m, int64_t n, int span, bool mixed) {
    return use_chain<T>(cx, m, n, span, mixed) ? chain_bytes<T>(cx, m, n) : 0;
}
template size_t blocked_bytes<double>(bool, int64_t, int64_t, int, bool);
template size_t blocked_bytes<float>(bool, int64_t, int64_t, int, bool);

// Enqueue the blocked solve: in panels of `span` rows, or as the rules say (0).
// `ws` holds blocked_bytes.
hsma_status blocked_trsm(bool cx, bool unit, int64_t m, int64_t n, cplx alpha, const double *A,
                         int64_t lda, double *B, int64_t ldb, int span, void *ws, hipStream_t s,
                         bool mixed) {
    return blocked_t<double>(cx, unit, m, n, alpha, A, lda, B, ldb, span, ws, s, mixed);
}

// The FP32 solve (STRSM, CTRSM).
hsma_status blocked_trsm32(bool cx, bool unit, int64_t m, int64_t n, cplx alpha, const float *A,
                           int64_t lda, float *B, int64_t ldb, int span, void *ws, hipStream_t s) {
    return blocked_t<float>(cx, unit, m, n, alpha, A, lda, B, ldb, span, ws, s, false);
}

// A right-hand side that is read and written through strides: a transposed or
// reversed B, where the recursion's products would need a copy.  One panel, or a
// chain, touches each element once on the way in and once on the way out, so
// the strides cost nothing and the two copies (two launches, four passes over
// B) go.
bool solves_in_one(bool cx, int64_t m, int64_t n) {
    return m > 64 && (m <= panel_span(cx, sizeof(double), n) || chain_rule(cx, sizeof(double), m, n));
}

hsma_status blocked_in_one(bool cx, int64_t m, PanelParams<double> p, hipStream_t s) {
    p.at = 1;
    if (m <= panel_span(cx, sizeof(double), p.n)) {
        p.rows = (int)m;
        return launch_panel<double>(cx, p, s);
    }
    void *ws = nullptr;
    HSMA_TRY(ws_alloc(&ws, chain_bytes<double>(cx, m, p.n), s));
    const hsma_status st = launch_chain<double>(cx, p, m, ws, s);
    const hsma_status st2 = ws_free(ws, s);
    return st != HSMA_SUCCESS ? st : st2;
}

// B <- inv(L) B by one panel or chain whose wavefronts look at most `looks` + 1
// times (looks >= 1) at what they wait for.  Not in the public header: this is how
// the end of a wait that gives up is tested.
extern "C" hsma_status hsma_internal_short_waits(int cx, int64_t m, int64_t n, const double *A, int64_t lda,
                                                 double *B, int64_t ldb, int looks, hsma_stream_t stream) {
    if (!solves_in_one(cx, m, n) || looks < 1) return HSMA_NOT_SUPPORTED;
    PanelParams<double> p{};
    p.A = A;
    p.lda = lda;
    p.B = B;
    p.n = n;
    p.alpha_re = 1;
    p.rs = 1;
    p.cs = ldb;
    p.looks = looks;
    return blocked_in_one(cx, m, p, static_cast<hipStream_t>(stream));
}

// R <- R - tril(L) X, the residual of refinement and of the backward-error
// report (FP64 products).  One product over the whole triangle: each row
// tile accumulates its full row of L times X in one FP64 accumulator chain
// (K up to the tile's last row, the part above the diagonal masked to zero,
// a unit diagonal taken as 1) and subtracts it from R once.  This order has
// nothing in common with the solve's recursion, so the rounding of the solve's
// updates does not cancel out of the residual and the reported backward error
// measures the solve, not its panels alone.
hsma_status triangular_residual(bool cx, bool unit, int64_t m, int64_t n, const double *A,
                                int64_t lda, const double *X, int64_t ldx, double *R, int64_t ldr,
                                hipStream_t s) {
    const int es = cx ? 2 : 1;
    return launch_gemm(cx, GemmRole::Residual, (int)(es * m), (int)n, (int)(es * m),
                       cplx{-1.0, 0.0}, A, lda, X, es * ldx, cplx{1.0, 0.0}, R, es * ldr,
                       unit ? 2 : 1, s, /*k_lower=*/1);
}

}  // namespace hsma
