// Which pipeline counts a single graph: rules on its sizes and options alone
// (plain C++, so that they are tested on the host).
#pragma once

#include <algorithm>

#include <stdint.h>

namespace bbc {

// One side's walk of all wedges (wedge.hip), the count from both sides
// (top.h), the products of the whole sign matrix (dense.hip).
enum class Route { kOneSided, kTwoSided, kMatrix };

struct RouteInput {
    int64_t n_u, n_v, m;
    bool anchors_u;   // the anchor side is U
    bool per_vertex;  // per-vertex output
    bool blocks;      // dense blocks are named
    bool knobs;       // an option that shapes the walk is set
    bool dup_check;   // repeated pairs are an error
    int n_cu;
};

// Padded sign matrix (rpad rows of anchors, kpad columns) and output tile of
// its products.
struct MatrixShape {
    int32_t tile, rpad, kpad;
};

// Ranks of a side that the count from both sides can take: the keys of its
// hashed slots have at most 28 bits.  Wide sides gain most, since the one-sided
// walk's wave regime ends at 2^20 ranks: 598 and 7.9 ms (5M x 5M, 40M uniform
// edges), 509 and 35 (the same, power law), 4502 and 330 (18M x 18M, 120M power
// law).
constexpr int64_t kTopMaxSide = 1ll << 28;

// Whether a graph fits the count from both sides: positions of both sides'
// lists (2 m) must fit 30 bits, the ranks of a side the hashed slots' keys,
// and neither side may be more than kTopRatio times the other (a small side of
// hubs over a large side of low degrees leaves nothing for the order to save,
// and its hubs' middles are all short lists: 102 ms against 16 ms for the
// one-sided walk on 2.5M x 100K vertices and 100M edges, 25 : 1; at 8 : 1 the
// count from both sides takes 1.9 and 3.4 ms on 800K x 100K and 5M power-law
// edges, 3.1 and 3.4 on 12M skewed ones, 641 and 607 us on 10K x 80K and 1M).
constexpr int64_t kTopRatio = 8;
inline bool two_sided_fits(const RouteInput& r) {
    return r.m > 0 && r.m <= (1ll << 29) && r.n_u >= 1 && r.n_v >= 1 && r.n_u <= kTopRatio * r.n_v &&
           r.n_v <= kTopRatio * r.n_u && std::max(r.n_u, r.n_v) <= kTopMaxSide;
}

// Whether a total gains from both sides: up to a mean degree of kTopDegree over
// both sides.  Denser lists give long slices, which the one-sided walk reads
// without flattening, and their equal degrees leave the order little to save.
// us, one-sided and two-sided: 897 and 605 (20000 x 20000, 1M uniform edges,
// mean 50), 949 and 863 (40000 x 20000, 1.5M power-law, 53), 3410 and 3796
// (200000 x 100000, 10M skewed, 71), 915 and 1203 (20000 x 20000, 2M uniform,
// 100), 1371 and 3023 (the same, 4M).
constexpr double kTopDegree = 64;
inline bool mean_degree_at_most(const RouteInput& r, double d) {
    return (double)r.m * (double)r.m <= d * d * (double)r.n_u * (double)r.n_v;
}

// Whether a per-vertex count gains from both sides: its launches and second
// readings pay from 60K edges, and on a smaller side of 5000 to 32767 vertices
// (at most two of the one-sided walk's wide bands) only up to a mean degree of
// 70 over both sides.  us, one-sided and two-sided: 313 and 372 (5000 x 2500,
// 75K edges), 459 and 407 (8000 x 5000, 60K), 835 and 593 (23117 x 9041,
// 301K), 2900 and 2181 (66000 x 13000, 2M: mean 68), 1188 and 1420 (30000 x
// 6000, 1M: mean 75), 5296 and 11000 (20000 x 20000, 4M, uniform), 10176 and
// 5411 (80000 x 40000, 8M, uniform), 46266 and 12959 (the same, power law),
// 15280 and 2046 (100003 x 50021, 2M); a wider smaller side keeps its gain at
// any density: 14781 and 12074 (40000 x 40000, 8M uniform), 91881 and 53441
// (16M), 65313 and 36622 (34000 x 34000, 12M).
inline bool two_sided_full_pays(const RouteInput& r) {
    const int64_t side = std::min(r.n_u, r.n_v);
    return r.m >= 60000 && (side >= 32768 || (side >= 5000 && mean_degree_at_most(r, 70)));
}

// Whether a total is counted by matrix products: the signed adjacency matrix S of
// the whole graph as bytes, and the pair terms of S S^T and |S| |S|^T on the
// matrix cores: no ranks, lists or schedule, and five launches instead of
// about forty.  Its time in us is close to the sum of 40 for the launches and
// the status copy, the clearing (3 MB per us), the products (1.2 to 2.3 Gops
// per us with 64- and 128-row tiles) and an atomic per edge (25K per us); the
// walks take at least 120, growing to 300 at 30K edges, and 0.1 per 1000
// edges, whatever the degrees (more the more wedges they have).  Measured,
// matrix against walk: 32 and 156 us (30 x 20, 100 edges), 65 and 246 (2000 x
// 1000, 20K), 178 and 337 (5000 x 5000, 75K), 289 and 341 (10000 x 5000,
// 150K), 913 and 348 (10000 x 10000, 200K), 151 and 1491 (3000 x 3000, 2M),
// 322 and 354 (40000 x 2000, 400K).  The line lies 15% below the walk's.  The
// output tiles have 64 rows where the larger ones would number less than one
// per CU (103 and 114 us at 2500 rows, 101 and 92 us at 3000).
constexpr int64_t kMatMaxBytes = 64ll << 20;  // a graph of few edges should not grow the arena beyond that
inline bool matrix_pays(const RouteInput& r, MatrixShape* shape) {
    const int64_t n_s = r.anchors_u ? r.n_u : r.n_v, n_c = r.anchors_u ? r.n_v : r.n_u;
    // one pair's counts fit 16 bits; a repeated edge is not counted twice here
    if (r.m <= 0 || n_s < 2 || n_c < 1 || n_c > 65535 || !r.dup_check) return false;
    const int64_t t = (n_s + 127) / 128;
    const int32_t tile = t * (t + 1) / 2 < r.n_cu ? 64 : 128;
    const int64_t rpad = (n_s + tile - 1) / tile * tile, kpad = (n_c + 63) / 64 * 64;
    const double bytes = (double)rpad * kpad, ops = 2.0 * rpad * bytes, m = (double)r.m;
    const double matrix = 40 + bytes / 3e6 + ops / (tile == 64 ? 1.2e9 : 2.2e9) + m / 25e3;
    const double walk = 0.85 * (120 + 180 * std::min(1.0, m / 30e3) + m / 10e3);
    if (bytes > kMatMaxBytes || matrix > walk) return false;
    *shape = MatrixShape{tile, (int32_t)rpad, (int32_t)kpad};
    return true;
}

// log2 of the counter words per band of the count from both sides, at most
// `words`: narrower bands where a side holds few, so that the bands of the
// heaviest vertices spread over the chip.
inline int band_log(int words, int64_t widest_side) {
    int lw = 0;
    while ((2 << lw) <= words) ++lw;
    while (lw > 9 && ((int64_t)16 << lw) > widest_side) --lw;
    return lw;
}

// Most entries that the band index of one side's lists (n_a lists, m entries in
// all) can have, over the bands of the other side's n_b ranks: bands of
// 2^(lw - 1) to 2^(lw + 2) ranks.  Up to kTopFewBands bands every list that is
// not empty has an entry per band and one more, beyond that only lists of as
// many entries as there are bands.
constexpr int64_t kTopFewBands = 16;
inline int64_t index_words(int64_t n_a, int64_t n_b, int64_t m, int lw) {
    const auto bands = [&](int log) { return (n_b + (1ll << log) - 1) >> log; };
    const int64_t most = bands(lw - 1), least = bands(lw + 2);
    if (most <= 1) return 0;
    const int64_t few = least <= kTopFewBands ? (std::min(most, kTopFewBands) + 1) * std::min(n_a, m) : 0;
    const int64_t many = most > kTopFewBands ? m + m / std::max(kTopFewBands + 1, least) : 0;
    return std::max(few, many);
}

// The route of a graph (with kMatrix, its matrix).
inline Route choose_route(const RouteInput& r, MatrixShape* shape) {
    if (r.blocks) return Route::kOneSided;
    if (!r.knobs && !r.per_vertex && matrix_pays(r, shape)) return Route::kMatrix;
    const bool pays = r.per_vertex ? !r.knobs && two_sided_full_pays(r) : mean_degree_at_most(r, kTopDegree);
    return pays && two_sided_fits(r) ? Route::kTwoSided : Route::kOneSided;
}

}  // namespace bbc
