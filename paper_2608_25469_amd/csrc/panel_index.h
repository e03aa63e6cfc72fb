// Which elements of L the panel kernel's loads of a step read (host and device
// code).  L's strict upper triangle is never read, also not by the loads whose
// values nobody uses: every wavefront issues the same number of loads at a step,
// so that none waits for more than it needs, and those it has no use for go to
// columns left of its row.
//
// Row block j = w + 8 q belongs to wavefront w; step I multiplies column block I
// with row blocks I + 2 and up.  `spare` is a column block that every row block
// may read: 0, or, where blocks lie left of the panel, -1.  Row block 0 has
// nothing left of it in a lone panel; its place is then the panel's last row.

#pragma once

#ifdef __HIPCC__
#define HSMA_HD __host__ __device__ __forceinline__
#else
#define HSMA_HD inline
#endif

namespace hsma {

constexpr int kPanelWaves = 8;

HSMA_HD int panel_spare(int left) { return left > 0 ? -1 : 0; }

// Row (real view) that a lane reads in row block w + 8 q of a panel of mr rows;
// arow: its row in the block.
HSMA_HD int panel_row(int q, int w, int arow, int mr, int spare) {
    const int r = 16 * (w + kPanelWaves * q) + arow;
    return r < mr && !(w == 0 && q == 0 && spare == 0) ? r : mr - 1;
}

// Column block that wavefront w reads in its row block w + 8 q at step I of a
// panel of nb blocks (q at least (I + 2) / 8, nb at least 2).
HSMA_HD int panel_column(int I, int q, int w, int nb, int spare) {
    if (q == (I + 2) / kPanelWaves && w < (I + 2) % kPanelWaves) return spare;
    return I < nb - 1 ? I : spare;
}

}  // namespace hsma
