// The panel kernel for many more strips than the chip takes at once
// (panel_core.h, WIDE), in panels of up to 128 real-view rows (FP32: 256), and
// that of chains for batches of many: a unit of its own, so that it compiles beside
// the others.

#include "panel_core.h"

namespace hsma {

using namespace panelk;

template <typename T>
hsma_status launch_panel_wide(bool cx, const PanelParams<T> &one, const PanelParams<T> *descs, int nd, int max_rows,
                              int64_t groups, hipStream_t s) {
    const int mr = max_rows * (cx ? 2 : 1);
    // (Strides are for m > 64, so complex ones never have 128 real-view rows.)
    if (mr > wide_rows(sizeof(T)) || (one.at && (cx || sizeof(T) == 4))) return HSMA_NOT_SUPPORTED;
    const dim3 grid((unsigned)groups), block(64 * kWaves);
    auto go = [&](auto CX, auto AT) {
        constexpr bool z = decltype(CX)::value, at = decltype(AT)::value;
        if (mr <= 128) hipLaunchKernelGGL((hsma_panel<T, z, 1, at, true>), grid, block, 0, s, one, descs, nd);
        else if constexpr (sizeof(T) == 4) hipLaunchKernelGGL((hsma_panel<T, z, 2, at, true>), grid, block, 0, s, one, descs, nd);
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if constexpr (sizeof(T) == 8) {
        if (one.at) go(no, yes);
        else cx ? go(yes, no) : go(no, no);
    } else {
        cx ? go(yes, no) : go(no, no);
    }
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}
template hsma_status launch_panel_wide<double>(bool, const PanelParams<double> &, const PanelParams<double> *, int, int,
                                               int64_t, hipStream_t);
template hsma_status launch_panel_wide<float>(bool, const PanelParams<float> &, const PanelParams<float> *, int, int,
                                              int64_t, hipStream_t);

hsma_status launch_chain_wide(bool cx, const PanelParams<double> *descs, int nd, int64_t tiles, unsigned *tickets,
                              hipStream_t s) {
    const PanelParams<double> none{};
    const dim3 grid((unsigned)tiles), block(64 * kWaves);
    if (cx) hipLaunchKernelGGL((hsma_chain<double, true, false, true>), grid, block, 0, s, none, descs, nd, tickets);
    else hipLaunchKernelGGL((hsma_chain<double, false, false, true>), grid, block, 0, s, none, descs, nd, tickets);
    HSMA_HIP(hipGetLastError());
    return HSMA_SUCCESS;
}

}  // namespace hsma
