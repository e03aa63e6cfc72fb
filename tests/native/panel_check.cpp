// Host check of what the panel kernel's loads of a step read
// (csrc/panel_index.h): for every panel height and kernel size, real and
// complex, alone and with blocks before it, every element lies in the panel's
// rows, in L's columns and not above the diagonal, and the loads that a step
// uses are the step's.
#include <cstdio>
#include <initializer_list>

#include "panel_index.h"

using namespace hsma;

int main() {
    long long bad = 0, seen = 0;
    for (int es = 1; es <= 2; ++es)
        for (int nq : {1, 2, 4})
            for (int left : {0, 16}) {
                const int spare = panel_spare(left), NB = kPanelWaves * nq;
                for (int mr = 17; mr <= 16 * NB; mr += es) {
                    if (mr % es) continue;
                    const int nb = (mr + 15) / 16;
                    for (int I = 0; I + 2 < NB; ++I)
                        for (int q = (I + 2) / kPanelWaves; q < nq; ++q)
                            for (int w = 0; w < kPanelWaves; ++w) {
                                const int col = panel_column(I, q, w, nb, spare), j = w + kPanelWaves * q;
                                const bool used = j >= I + 2 && j < nb && I < nb - 1;
                                bad += used && col != I;
                                for (int arow = 0; arow < 16; ++arow) {
                                    const int r = panel_row(q, w, arow, mr, spare);
                                    bad += used && 16 * j + arow < mr && r != 16 * j + arow;
                                    for (int c = 16 * col; c < 16 * col + 16; ++c, ++seen)
                                        bad += !(r >= 0 && r < mr && c >= -16 * left && c / es <= r / es);
                                }
                            }
                }
            }
    if (bad || seen < 1000000) {
        std::printf("%lld of %lld elements wrong\n", bad, seen);
        return 1;
    }
    std::printf("panel loads ok\n");
    return 0;
}
