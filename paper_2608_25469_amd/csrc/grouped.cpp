// Grouped blocked path: many problems with m > 64 advanced together.
//
// Each problem follows exactly the schedule the single-problem blocked path
// gives it (a chain, or the same panels and the same recursive sequence of
// panel solves and trailing updates), so every result is bit-for-bit the one
// the problem gets alone.  What changes is how the work is launched: all chains
// of a data type are one launch (or a few, where their mail is large), and of the recursions the k-th operation of
// every problem goes into one grouped launch, so a batch of hundreds of
// mid-sized solves costs a few launches instead of a few per problem.  The
// in-order walk of the recursion alternates panel, update, panel, ..., so step
// k is a panel for every problem when k is even and an update when k is odd;
// each step is one launch per data type.  All descriptors of the call go to
// the device in one copy.

#include <algorithm>
#include <cstring>
#include <vector>

#include "internal.h"

namespace hsma {

hsma_status upload_async(const void *host, size_t bytes, void *dev, hipStream_t s);

namespace {

struct Prob {
    bool cx, unit;
    int64_t m, n;
    cplx alpha;
    const double *A;
    int64_t lda;
    double *B;
    int64_t ldb;
    int span;
    int64_t nb;
    int es() const { return cx ? 2 : 1; }
};

struct Op {
    bool panel;
    int64_t blk;           // panel
    int64_t r1, r2, k0;    // update
    bool touched;
};

void walk(const Prob &p, int64_t b0, int64_t nb, bool touched, std::vector<Op> &out) {
    if (nb == 1) {
        out.push_back(Op{true, b0, 0, 0, 0, touched});
        return;
    }
    const int64_t h = nb / 2;
    walk(p, b0, h, touched, out);
    out.push_back(Op{false, 0, (b0 + h) * p.span, std::min<int64_t>((b0 + nb) * p.span, p.m), b0 * p.span,
                     touched});
    walk(p, b0 + h, nb - h, true, out);
}

GemmParams make(int M, int N, int K, cplx alpha, const double *A, int64_t lda, const double *B,
                int64_t ldb, cplx beta, double *C, int64_t ldc) {
    GemmParams g{};
    g.M = M;
    g.N = N;
    g.K = K;
    g.A = A;
    g.lda = lda;
    g.B = B;
    g.ldb = ldb;
    g.C = C;
    g.ldc = ldc;
    g.alpha_re = alpha.re;
    g.alpha_im = alpha.im;
    g.beta_re = beta.re;
    g.beta_im = beta.im;
    return g;
}

struct Launch {
    bool panel = false, chain = false;
    bool cx = false;
    size_t img_off = 0;
    int64_t tiles = 0;
    size_t words = 0;  // of mail
    int max_rows = 0, per = 1, bm = 0, bn = 0;
    double flops = 0;
    std::vector<GemmParams> gemms;
    std::vector<PanelParams<double>> panels;
};

PanelParams<double> op_panel(const Prob &p, const Op &o) {
    const int es = p.es();
    const int64_t r0 = o.blk * p.span;
    const cplx al = o.touched ? cplx{1.0, 0.0} : p.alpha;
    PanelParams<double> q{};
    q.A = p.A + es * (r0 + r0 * p.lda);
    q.lda = p.lda;
    q.B = p.B + es * r0;
    q.ldb = p.ldb;
    q.n = p.n;
    q.alpha_re = al.re;
    q.alpha_im = al.im;
    q.rows = (int)std::min<int64_t>(p.span, p.m - r0);
    q.unit = p.unit;
    return q;
}

// The mail of the chains of one launch, which every launch of a call uses in
// turn.  It holds 32768 workgroups' blocks, many times what the chip runs at
// once, so that nothing is lost between two launches; without a bound a batch
// of large chains takes as much again as its B matrices.
constexpr size_t kMailWords = ((size_t)1 << 30) / sizeof(double);

// Strips of chains that are listed side by side.
constexpr int64_t kSideBySide = 768;

// The panels of chains [first, end) of ps as one launch, where end is as far as
// their mail fits (one chain always does).  Panels are listed by their place in
// their chain (all first panels, all second ones, ...), the longest chains
// first: a panel waits only for the one before it, so each round of the list
// is work that can start once the round before it is under way, and no solve
// holds the chip with panels that wait while another has not begun.  Of a batch
// that is many times the chip, as many solves at a time as fill it: what a panel
// mails is then read again while it is in the caches.  A descriptor's mail is an
// offset until the mail has a place.
size_t chain_launch(const std::vector<Prob> &ps, size_t first, Launch *l) {
    l->chain = l->panel = true;
    std::vector<size_t> mail;
    size_t end = first;
    for (; end < ps.size(); ++end) {
        const Prob &p = ps[end];
        const size_t words = chain_bytes<double>(p.cx, p.m, p.n) / sizeof(double);
        if (end > first && l->words + words > kMailWords) break;
        mail.push_back(l->words);
        l->words += words;
        l->flops += (p.cx ? 4.0 : 1.0) * p.m * (double)p.m * (double)p.n;
    }
    for (size_t from = 0; from < mail.size();) {
        size_t to = from;
        for (int64_t strips = 0; to < mail.size() && strips < kSideBySide; ++to) strips += (ps[first + to].n + 15) / 16;
        for (int64_t r = 0, more = 1; more; ++r) {
            more = 0;
            for (size_t i = from; i < to; ++i) {
                const Prob &p = ps[first + i];
                const int64_t h = kChainRows / p.es(), r0 = r * h;
                if (r0 >= p.m) continue;
                more = 1;
                PanelParams<double> q{};
                q.A = p.A + p.es() * (r0 + r0 * p.lda);
                q.lda = p.lda;
                q.B = p.B + p.es() * r0;
                q.ldb = p.ldb;
                q.n = p.n;
                q.alpha_re = p.alpha.re;
                q.alpha_im = p.alpha.im;
                q.rows = (int)std::min(h, p.m - r0);
                q.unit = p.unit;
                q.left = (int)(r * (kChainRows / 16));
                q.nblk = (int)((p.m * p.es() + 15) / 16);
                q.mail = reinterpret_cast<double *>(mail[i] * sizeof(double));
                q.tile0 = (int)std::min<int64_t>(l->tiles, 0x7fffffff);
                l->tiles += (p.n + 15) / 16;
                l->panels.push_back(q);
            }
        }
        from = to;
    }
    return end;
}

GemmParams op_update(const Prob &p, const Op &o) {
    const int es = p.es();
    return make((int)(es * (o.r2 - o.r1)), (int)p.n, (int)(es * (o.r1 - o.k0)), cplx{-1.0, 0.0},
                p.A + es * (o.r1 + o.k0 * p.lda), p.lda, p.B + es * o.k0, es * p.ldb,
                o.touched ? cplx{1.0, 0.0} : p.alpha, p.B + es * o.r1, es * p.ldb);
}

// A launch's descriptors start at a multiple of 256 bytes.
size_t padded(size_t bytes) { return (bytes + 255) / 256 * 256; }

}  // namespace

// What one problem (m > 64) adds at most to the device memory of a grouped
// call: its mail, and its descriptors as if no launch took another's.
size_t grouped_bytes(bool cx, int64_t m, int64_t n) {
    const int64_t mr = m * (cx ? 2 : 1);
    if (chain_rule(cx, sizeof(double), m, n))
        return chain_bytes<double>(cx, m, n) + 512 + padded((mr + kChainRows - 1) / kChainRows * sizeof(PanelParams<double>));
    const int64_t span = panel_span(cx, sizeof(double), n);
    const size_t panels = (m + span - 1) / span;
    return panels * padded(sizeof(PanelParams<double>)) + (panels - 1) * padded(sizeof(GemmParams)) + 512;
}

// Enqueue every problem (validated; m > 64; alpha != 0) on stream s.
hsma_status grouped_blocked(const hsma_problem *probs, int64_t count, hipStream_t s) {
    if (count <= 0) return HSMA_SUCCESS;
    std::vector<Prob> ps, chains[2];
    ps.reserve(count);
    std::vector<Op> ops;  // of problem i of ps from first[i] on
    std::vector<size_t> first;
    size_t steps = 0;
    for (int64_t i = 0; i < count; ++i) {
        const hsma_problem &q = probs[i];
        Prob p;
        p.cx = q.dtype == HSMA_C64F;
        p.unit = q.diag == HSMA_UNIT;
        p.m = q.m;
        p.n = q.n;
        p.alpha = cplx{q.alpha_re, p.cx ? q.alpha_im : 0.0};
        p.A = static_cast<const double *>(q.A);
        p.lda = q.lda;
        p.B = static_cast<double *>(q.B);
        p.ldb = q.ldb;
        p.span = panel_span(p.cx, sizeof(double), p.n);
        p.nb = (p.m + p.span - 1) / p.span;
        if (chain_rule(p.cx, sizeof(double), p.m, p.n)) {
            chains[p.cx].push_back(p);
            continue;
        }
        first.push_back(ops.size());
        walk(p, 0, p.nb, false, ops);
        steps = std::max(steps, ops.size() - first.back());
        ps.push_back(p);
    }
    first.push_back(ops.size());

    // Each step's products share one launch whatever their widths: the tile
    // shape follows the widest.  Separate launches for narrow right-hand
    // sides would add kernel boundaries to the dependent chain, and on a
    // served mix (n log-uniform in [1, 512]) cost more than the columns the
    // wide tiles leave idle.
    std::vector<Launch> launches;
    size_t img_bytes = 0, mail_words = 0;
    for (int cxi = 0; cxi < 2; ++cxi) {
        std::vector<Prob> &cs = chains[cxi];
        std::stable_sort(cs.begin(), cs.end(), [](const Prob &a, const Prob &b) { return a.m > b.m; });
        for (size_t at = 0; at < cs.size();) {
            Launch l;
            at = chain_launch(cs, at, &l);
            if (l.tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
            l.cx = cxi;
            l.img_off = img_bytes;
            img_bytes += padded(l.panels.size() * sizeof(PanelParams<double>));
            mail_words = std::max(mail_words, l.words);
            launches.push_back(std::move(l));
        }
    }
    for (size_t k = 0; k < steps; ++k) {
        for (int cxi = 0; cxi < 2; ++cxi) {
            Launch l;
            l.cx = cxi;
            l.panel = k % 2 == 0;
            int max_n = 0;
            std::vector<int64_t> strips;
            for (size_t pi = 0; pi < ps.size(); ++pi) {
                const Prob &p = ps[pi];
                if (p.cx != (bool)cxi || k >= first[pi + 1] - first[pi]) continue;
                const Op &o = ops[first[pi] + k];
                if (l.panel) {
                    PanelParams<double> q = op_panel(p, o);
                    strips.push_back((q.n + 15) / 16);
                    l.max_rows = std::max(l.max_rows, q.rows);
                    l.flops += (p.cx ? 4.0 : 1.0) * q.rows * (double)q.rows * (double)q.n;
                    l.panels.push_back(q);
                } else {
                    l.gemms.push_back(op_update(p, o));
                    max_n = std::max(max_n, l.gemms.back().N);
                }
            }
            if (l.panels.empty() && l.gemms.empty()) continue;
            if (l.panel) {
                l.per = panel_per(cxi, sizeof(double), l.max_rows, strips.data(), strips.size());
                for (PanelParams<double> &q : l.panels) {
                    if (l.tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
                    q.per = l.per;
                    q.tile0 = (int)l.tiles;
                    l.tiles += panel_share((q.n + 15) / 16, &q.per);
                }
            } else {
                gemm_grouped_tile(max_n, &l.bm, &l.bn);
                for (GemmParams &g : l.gemms) {
                    g.tiles_m = (g.M + l.bm - 1) / l.bm;
                    g.tiles_n = (g.N + l.bn - 1) / l.bn;
                    if (l.tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
                    g.tile0 = (int)l.tiles;
                    l.tiles += (int64_t)g.tiles_m * g.tiles_n;
                    l.flops += 2.0 * g.M * (double)g.N * g.K;
                }
            }
            if (l.tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
            l.img_off = img_bytes;
            img_bytes += padded(l.panels.size() * sizeof(PanelParams<double>) + l.gemms.size() * sizeof(GemmParams));
            launches.push_back(std::move(l));
        }
    }

    std::vector<unsigned char> img(img_bytes, 0);
    for (const Launch &l : launches) {
        if (l.panel) std::memcpy(img.data() + l.img_off, l.panels.data(), l.panels.size() * sizeof(PanelParams<double>));
        else std::memcpy(img.data() + l.img_off, l.gemms.data(), l.gemms.size() * sizeof(GemmParams));
    }
    void *dev = nullptr;
    // (The tickets of a launch of chains follow its mail.)
    HSMA_TRY(ws_alloc(&dev, img_bytes + (mail_words ? mail_words * sizeof(double) + 256 : 0), s));
    unsigned char *base = static_cast<unsigned char *>(dev);
    double *mail = reinterpret_cast<double *>(base + img_bytes);
    for (const Launch &l : launches) {
        if (!l.chain) continue;
        unsigned char *img_l = img.data() + l.img_off;
        for (size_t i = 0; i < l.panels.size(); ++i) {
            PanelParams<double> q = l.panels[i];
            q.mail = mail + reinterpret_cast<uintptr_t>(q.mail) / sizeof(double);
            std::memcpy(img_l + i * sizeof(q), &q, sizeof(q));
        }
    }
    hsma_status st = upload_async(img.data(), img.size(), dev, s);
    for (const Launch &l : launches) {
        if (st != HSMA_SUCCESS) break;
        const void *d = base + l.img_off;
        if (l.chain)
            st = launch_chain_grouped(l.cx, static_cast<const PanelParams<double> *>(d), (int)l.panels.size(), l.tiles,
                                      mail, (int64_t)l.words, l.flops, s);
        else if (l.panel)
            st = launch_panel_grouped(l.cx, static_cast<const PanelParams<double> *>(d), (int)l.panels.size(),
                                      l.max_rows, l.tiles, l.per > 1, l.flops, s);
        else
            st = launch_gemm_grouped(l.cx, l.bm, l.bn, static_cast<const GemmParams *>(d), (int)l.gemms.size(),
                                     l.tiles, l.flops, s);
    }
    const hsma_status st2 = ws_free(dev, s);
    return st != HSMA_SUCCESS ? st : st2;
}

}  // namespace hsma
