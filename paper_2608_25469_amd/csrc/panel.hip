// Launches of the panel and chain kernels (panel_core.h); those for very many
// columns are in panel_wide.hip.

#include <algorithm>

#include "panel_core.h"

namespace hsma {

using namespace panelk;

namespace {

// Empties the mail (n words) and clears the ticket counter.
template <typename T>
__global__ __launch_bounds__(256) void hsma_mail_empty(T *mail, int64_t n, unsigned *tickets) {
    typedef typename Word<T>::U U;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        reinterpret_cast<U *>(mail)[i] = Word<T>::kEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) *tickets = 0;
}

template <typename T, bool CX>
hsma_status launch(const PanelParams<T> &one, const PanelParams<T> *descs, int nd, int max_rows, int64_t groups, bool wide,
                   hipStream_t s) {
    const int mr = max_rows * (CX ? 2 : 1);
    if (mr > kPanelRows || groups > kMaxGroups) return HSMA_INVALID_SIZE;
    if (wide) return launch_panel_wide<T>(CX, one, descs, nd, max_rows, groups, s);
    const dim3 grid((unsigned)groups), block(64 * kWaves);
    auto go = [&](auto AT) {
        constexpr bool at = decltype(AT)::value;
        // (Strides are for m > 64: complex ones have more than 128 real-view rows.)
        constexpr int least = CX && at ? 2 : 1;
        if (mr <= 128) hipLaunchKernelGGL((hsma_panel<T, CX, least, at, false>), grid, block, 0, s, one, descs, nd);
        else if (mr <= 256) hipLaunchKernelGGL((hsma_panel<T, CX, 2, at, false>), grid, block, 0, s, one, descs, nd);
        else hipLaunchKernelGGL((hsma_panel<T, CX, 4, at, false>), grid, block, 0, s, one, descs, nd);
    };
    if constexpr (sizeof(T) == 8) {
        if (one.at) go(std::true_type{});
        else go(std::false_type{});
    } else {
        if (one.at) return HSMA_NOT_SUPPORTED;
        go(std::false_type{});
    }
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

}  // namespace

// Mail of every strip, then a ticket counter.
template <typename T>
size_t chain_bytes(bool cx, int64_t m, int64_t n) {
    const int64_t blocks = (m * (cx ? 2 : 1) + 15) / 16, strips = (n + 15) / 16;
    return (size_t)(blocks * strips) * 256 * sizeof(T) + 256;
}
template size_t chain_bytes<double>(bool, int64_t, int64_t);
template size_t chain_bytes<float>(bool, int64_t, int64_t);

template <typename T>
hsma_status empty_mail(T *mail, int64_t words, unsigned *tickets, hipStream_t s) {
    const int64_t blocks = std::min<int64_t>((words + 1023) / 1024, 4096);
    ProfScope prof(HSMA_PHASE_OTHER, 0.0, s);
    hipLaunchKernelGGL(hsma_mail_empty<T>, dim3((unsigned)blocks), dim3(256), 0, s, mail, words, tickets);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

template <typename T>
hsma_status launch_chain(bool cx, const PanelParams<T> &q, int64_t m, void *ws, hipStream_t s) {
    const int es = cx ? 2 : 1;
    const int64_t blocks = (m * es + 15) / 16, strips = (q.n + 15) / 16;
    const int64_t panels = (m * es + kChainRows - 1) / kChainRows;
    if (panels * strips > 0x7fffffff || blocks * strips > 0x7fffffff) return HSMA_INVALID_SIZE;
    PanelParams<T> p = q;
    p.rows = (int)m;
    p.nblk = (int)blocks;
    p.mail = static_cast<T *>(ws);
    const int64_t words = 256 * blocks * strips;
    unsigned *tickets = reinterpret_cast<unsigned *>(p.mail + words);
    HSMA_TRY(empty_mail<T>(p.mail, words, tickets, s));
    ProfScope prof(HSMA_PHASE_LEAF, (cx ? 4.0 : 1.0) * m * (double)m * (double)p.n, s);
    const dim3 grid((unsigned)(panels * strips)), block(64 * kWaves);
    auto go = [&](auto AT) {
        constexpr bool at = decltype(AT)::value;
        if (cx) hipLaunchKernelGGL((hsma_chain<T, true, at, false>), grid, block, 0, s, p, nullptr, 0, tickets);
        else hipLaunchKernelGGL((hsma_chain<T, false, at, false>), grid, block, 0, s, p, nullptr, 0, tickets);
    };
    if constexpr (sizeof(T) == 8) {
        if (p.at) go(std::true_type{});
        else go(std::false_type{});
    } else {
        if (p.at) return HSMA_NOT_SUPPORTED;
        go(std::false_type{});
    }
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}
template hsma_status launch_chain<double>(bool, const PanelParams<double> &, int64_t, void *, hipStream_t);
template hsma_status launch_chain<float>(bool, const PanelParams<float> &, int64_t, void *, hipStream_t);

// A workgroup's strips share its start (loads and inversions of L, worth a strip
// or two).  Of the numbers that make whole rounds of the workgroups the chip holds
// (two a CU) the most rounds, unless fewer save a twentieth.  Below four strips a CU
// one strip each is as fast (128 x 9000 19 us against 22; 16384 24.5 and 23.0).
int panel_per(bool cx, int elem, int max_rows, const int64_t *strips, size_t count) {
    int64_t total = 0;
    for (size_t i = 0; i < count; ++i) total += strips[i];
    DeviceInfo dev;
    const int64_t cus = (device_info(&dev) == HSMA_SUCCESS && dev.num_cus > 0) ? dev.num_cus : 256;
    if (max_rows * (cx ? 2 : 1) > wide_rows(elem) || total < 4 * cus) return 1;
    int64_t best = 0;
    double best_cost = 0;
    for (int rounds = 8; rounds >= 1; rounds /= 2) {
        const int64_t per = std::max<int64_t>(2, (total + 2 * cus * rounds - 1) / (2 * cus * rounds));
        int64_t groups = 0;
        for (size_t i = 0; i < count; ++i) groups += (strips[i] + per - 1) / per;
        const double cost = (double)((groups + 2 * cus - 1) / (2 * cus)) * ((double)total / groups + 2);
        if (best == 0 || cost < 0.95 * best_cost) {
            best = per;
            best_cost = cost;
        }
    }
    return (int)best;
}

int64_t panel_share(int64_t strips, int *per) {
    const int64_t groups = (strips + *per - 1) / *per;
    *per = (int)((strips + groups - 1) / groups);
    return groups;
}

template <typename T>
hsma_status launch_panel(bool cx, const PanelParams<T> &p, hipStream_t s) {
    if (p.rows <= 0 || p.n <= 0) return HSMA_SUCCESS;
    ProfScope prof(HSMA_PHASE_LEAF, (cx ? 4.0 : 1.0) * p.rows * (double)p.rows * (double)p.n, s);
    const int64_t strips = (p.n + 15) / 16;
    PanelParams<T> q = p;
    q.per = panel_per(cx, sizeof(T), p.rows, &strips, 1);
    const bool wide = q.per > 1;
    const int64_t groups = panel_share(strips, &q.per);
    return cx ? launch<T, true>(q, nullptr, 0, p.rows, groups, wide, s)
              : launch<T, false>(q, nullptr, 0, p.rows, groups, wide, s);
}
template hsma_status launch_panel<double>(bool, const PanelParams<double> &, hipStream_t);
template hsma_status launch_panel<float>(bool, const PanelParams<float> &, hipStream_t);

hsma_status launch_chain_grouped(bool cx, const PanelParams<double> *descs, int nd, int64_t tiles, double *mail,
                                 int64_t words, double flops, hipStream_t s) {
    if (nd <= 0 || tiles <= 0) return HSMA_SUCCESS;
    if (tiles > 0x7fffffff) return HSMA_INVALID_SIZE;
    unsigned *tickets = reinterpret_cast<unsigned *>(mail + words);
    HSMA_TRY(empty_mail<double>(mail, words, tickets, s));
    ProfScope prof(HSMA_PHASE_LEAF, flops, s);
    const PanelParams<double> none{};
    DeviceInfo dev;
    const int64_t cus = (device_info(&dev) == HSMA_SUCCESS && dev.num_cus > 0) ? dev.num_cus : 256;
    // Two workgroups a CU (panel_core.h, WIDE) where there are rounds of them: 200 of
    // DTRSM 513..1024 x 513..1024 5.51 -> 4.06 ms, of ZTRSM 13.8 -> 12.3; a lone chain is
    // shorter with a CU and all its registers to each workgroup.
    if (tiles >= 4 * cus) return launch_chain_wide(cx, descs, nd, tiles, tickets, s);
    const dim3 grid((unsigned)tiles), block(64 * kWaves);
    if (cx) hipLaunchKernelGGL((hsma_chain<double, true, false, false>), grid, block, 0, s, none, descs, nd, tickets);
    else hipLaunchKernelGGL((hsma_chain<double, false, false, false>), grid, block, 0, s, none, descs, nd, tickets);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

hsma_status launch_panel_grouped(bool cx, const PanelParams<double> *descs, int nd, int max_rows, int64_t groups,
                                 bool wide, double flops, hipStream_t s) {
    if (nd <= 0 || groups <= 0) return HSMA_SUCCESS;
    ProfScope prof(HSMA_PHASE_LEAF, flops, s);
    const PanelParams<double> none{};
    return cx ? launch<double, true>(none, descs, nd, max_rows, groups, wide, s)
              : launch<double, false>(none, descs, nd, max_rows, groups, wide, s);
}

}  // namespace hsma
