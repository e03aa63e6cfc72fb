// Host check of the slices that a product's tile loads as they lie
// (csrc/tile_choice.h): no element outside A, and none above the diagonal of a
// triangular A, real and complex, for every tile of sizes around the tile's
// multiples; and of the rows read in the place of those above it or beyond A.
#include <cstdio>
#include <initializer_list>

#include "tile_choice.h"

using namespace hsma;

int main() {
    long long bad = 0, direct = 0;
    for (int es : {1, 2})
        for (int bm : {64, 128})
            for (int bk : {16, 32})
                for (bool tri : {false, true})
                    for (int M : {2, 16, 62, 64, 66, 126, 128, 130, 190, 256, 300, 514}) {
                        if (M % es) continue;
                        for (int m0 = 0; m0 < M; m0 += bm) {
                            const int ms = first_row(M, bm, m0);
                            bad += ms < 0 || ms > m0 || (ms < m0 && ms + bm != M);
                            const int K = tri && m0 + bm < M ? m0 + bm : M;
                            for (int k0 = 0; k0 < K; k0 += bk) {
                                for (int r = ms; tri && r < ms + bm; ++r)
                                    for (int c = k0 / es; c < (k0 + bk) / es && c < K / es; ++c) {
                                        const int t = tri_row(es, M, r, c);
                                        bad += t < 0 || t >= M || t / es < c || t % es != r % es;
                                        bad += r < M && r / es >= c && t != r;
                                    }
                                if (!direct_slice(M, bm, K, bk, tri, ms, k0)) continue;
                                ++direct;
                                for (int r = ms; r < ms + bm; ++r)
                                    for (int c = k0; c < k0 + bk; ++c) bad += r >= M || c >= K || (tri && c / es > r / es);
                            }
                        }
                    }
    // No update tile taller than its product, but the smallest.
    for (int M = 1; M <= 300; ++M)
        for (long long N : {1, 33, 300, 4097, 300000}) bad += kUpdateShapes[update_tile_shape(M, N, 256)].bm > (M > 32 ? M : 32);
    if (bad || direct < 100) {
        std::printf("%lld wrong in %lld slices\n", bad, direct);
        return 1;
    }
    std::printf("slices ok\n");
    return 0;
}
