// Tile shapes of the FP64 product, and which slices a tile loads without a look at
// each element (no HIP dependency).
//
// A workgroup stages its A and B tiles through an LDS ring of two slices; the
// ring's size sets how many workgroups a CU holds (160 KB of LDS, at most
// three).  For a lower-triangular C only the tiles on or below the diagonal run, and
// each runs the whole K, so a launch takes about ceil(non-empty tiles / resident
// slots) rounds of one tile's time (slots counted as for 16-deep slices, three a CU
// for the small shapes; their 32- and 64-deep ones hold two);
// lower_tile_shape picks the shape with the fewest rounds times tile area,
// weighted by the shape's relative throughput (narrower tiles reuse less of
// what they stage).

#pragma once

#include <algorithm>
#include <cstdint>

namespace hsma {

// First row in memory of the tile that begins at row m0 of M: moved up where it
// would hang over.
constexpr int first_row(int M, int bm, int m0) { return m0 + bm > M && M >= bm ? M - bm : m0; }

// Whether the slice of columns [k0, k0 + bk) of a tile (first row ms) is loaded
// as it lies: all of it in A, and left of the diagonal of a triangular A (of all
// rows, since rows further down have more of it).
constexpr bool direct_slice(int M, int bm, int K, int bk, bool tri, int ms, int k0) {
    return ms + bm <= M && k0 + bk <= K && !(tri && k0 + bk > ms);
}

// Row that is read in the place of row r (real view, es of them an element): kept
// below M; of a triangle, and at element column c, also kept at or below the
// diagonal.
constexpr int below(int es, int M, int r) { return r < M ? r : M - es + r % es; }
constexpr int tri_row(int es, int M, int r, int c) { return below(es, M, r / es < c ? c * es + r % es : r); }

constexpr int kTileBK = 16;

constexpr int tile_lds_bytes(int bm, int bn) { return 2 * (kTileBK * (bm + 4) + bn * (kTileBK + 1)) * 8; }

constexpr int tile_occupancy(int bm, int bn) {
    return (160 * 1024 / tile_lds_bytes(bm, bn)) >= 3 ? 3 : ((160 * 1024 / tile_lds_bytes(bm, bn)) >= 2 ? 2 : 1);
}

struct TileShape {
    int bm, bn;
    double eff;  // throughput relative to 128 x 128
};
// The weights of the two smallest shapes are extrapolated from the others by
// operand reuse (bm bn / (bm + bn) per staged element: 64, 43, 32, 21, 16).
constexpr int kNumLowerShapes = 5;
constexpr TileShape kLowerShapes[kNumLowerShapes] = {
    {128, 128, 1.0}, {128, 64, 0.85}, {64, 64, 0.7}, {64, 32, 0.5}, {32, 32, 0.35}};

// Tiles of an M x N (real-view) lower-triangular C that hold an element on
// or below the diagonal; complex C has two real-view rows per row.
inline int64_t lower_tiles(int64_t M, int64_t N, bool cx, int bm, int bn) {
    const int64_t tm_n = (M + bm - 1) / bm, tn_n = (N + bn - 1) / bn;
    int64_t tiles = 0;
    for (int64_t tm = 0; tm < tm_n; ++tm) {
        const int64_t last = cx ? (tm * bm + bm - 1) / 2 : tm * bm + bm - 1;
        tiles += std::min<int64_t>(tn_n, last / bn + 1);
    }
    return tiles;
}

// Index into kLowerShapes for `count` products of that size on `cus` CUs.
inline int lower_tile_shape(int64_t M, int64_t N, bool cx, int count, int64_t cus) {
    int best = 0;
    double best_cost = 0.0;
    for (int k = 0; k < kNumLowerShapes; ++k) {
        const TileShape &t = kLowerShapes[k];
        const int64_t tiles = lower_tiles(M, N, cx, t.bm, t.bn) * count;
        const int64_t slots = (int64_t)tile_occupancy(t.bm, t.bn) * cus;
        const double cost = (double)((tiles + slots - 1) / slots) * t.bm * t.bn / t.eff;
        if (k == 0 || cost < best_cost) {
            best = k;
            best_cost = cost;
        }
    }
    return best;
}

// Tile of a plain product.  A tile alone on its CU cannot hide its own
// latencies and runs at `solo` of the matrix rate; with `wg` of them resident
// the CU reaches `full` of it.  Measured on MI355X in FP64 at K = 1024, TF/s
// with one tile per CU and with many (the units give 76): 128 x 128 56 and 67,
// 128 x 64 47 and 67, 64 x 64 38 and 60, 64 x 32 32 and 57, 32 x 32 29 and 48.  A
// launch takes its full rounds of cus * wg tiles and then what the rest needs.
// Against "at least four tiles per CU or the next smaller shape": 2500 x 1777
// from the right 333 us to 310.
struct UpdateShape {
    int bm, bn, wg;
    double solo, full;
};
constexpr int kNumUpdateShapes = 5;
constexpr UpdateShape kUpdateShapes[kNumUpdateShapes] = {{128, 128, 2, 0.74, 0.89},
                                                         {128, 64, 3, 0.62, 0.88},
                                                         {64, 64, 2, 0.50, 0.79},
                                                         {64, 32, 3, 0.42, 0.75},
                                                         {32, 32, 2, 0.38, 0.63}};

// Index into kUpdateShapes for an M x N product on `cus` CUs (M in real-view
// rows); ties go to the larger tile, and a tile taller than the product, which
// loads it element by element, is out (updates of 44 and 128 rows, n = 300000: 637
// us against 689).
inline int update_tile_shape(int64_t M, int64_t N, int64_t cus) {
    int best = -1;
    double best_cost = 0.0;
    for (int k = 0; k < kNumUpdateShapes; ++k) {
        const UpdateShape &t = kUpdateShapes[k];
        if (t.bm > M && k + 1 < kNumUpdateShapes) continue;
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        const int64_t rounds = tiles / (cus * t.wg), rest = tiles - rounds * cus * t.wg;
        const double area = (double)t.bm * t.bn;
        double cost = (double)rounds * t.wg * area / t.full;
        if (rest > 0) cost += std::max(area / t.solo, (double)((rest + cus - 1) / cus) * area / t.full);
        if (best < 0 || cost < best_cost) {
            best = k;
            best_cost = cost;
        }
    }
    return best;
}

}  // namespace hsma
