// Work units of a request: how its pairs are cut into row tiles and column
// chunks.  Plain C++ for the host and the kernels.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

#ifdef __HIPCC__
#define TPCF_HD __host__ __device__ inline
#else
#define TPCF_HD inline
#endif

namespace tpcf {

// Threads per block and the i-points each lane keeps in registers.
constexpr int kWaves = 4;
constexpr int kWaveSize = 64;
constexpr int kBlock = kWaves * kWaveSize;

// Pairs of a request.
inline uint64_t pairs_of(bool auto_pairs, int64_t na, int64_t nb, int64_t rb, int64_t re) {
    if (!auto_pairs)
        return (uint64_t)(re - rb) * (uint64_t)nb;
    // sum over i in [rb, re) of (na - 1 - i)
    const int64_t cnt = re - rb;
    return (uint64_t)cnt * (uint64_t)(na - 1) - (uint64_t)((rb + re - 1) * cnt / 2);
}

// Rows that a tile of at most T holds on average.
inline int64_t tile_rows(int64_t rows, int64_t T) {
    const int64_t tiles = (rows + T - 1) / T;
    return tiles > 0 ? (rows + tiles - 1) / tiles : T;
}

// Columns that the row tiles of a request meet, all tiles together: its units
// at chunks of bj columns are about this over bj, however few rows a tile has.
inline int64_t tile_columns(bool auto_pairs, int64_t na, int64_t nb, int64_t rb, int64_t re, int64_t T) {
    const int64_t tiles = (re - rb + T - 1) / T;
    return auto_pairs ? tiles * (na - rb) - T * (tiles * (tiles - 1) / 2) : tiles * nb;
}

// Column chunk width of a plan for a launch over `load` pairs, whose tiles are
// taken to hold T rows: 64 columns up to `busy`, as many as still leave 4096
// units (16 items a wavefront slot's worth of wavefronts), and from there on
// as many as leave 65536, at most max_cols (multiples of 256 above 256); but
// wide enough that a list of `columns` columns of tiles stays below max_units
// (kMaxUnits: about 0.8 GB of units; catalogs of 1e8 points would otherwise
// need tens of GB of them).  A launch ends when its last item does, so items
// are kept short against it, but a narrow item prepares its rows for few
// columns.  Measured, default before (4096 units from the start) against 512
// columns: DD+DR+RR of 1e5 x 1e5 3.83 -> 2.83 ms, FP64 of 1.5e5 x 3e5 28.6 ->
// 25.9, 24 fields in a batch 8.03 -> 7.25; at 256 columns the first takes
// 3.79.  With jackknife regions, whose boundaries cut the chunks again, 1024
// columns are better than 512 (7.2 against 7.65 ms).
constexpr double kMaxUnits = 16777216.0;

inline int64_t chunk_width(double columns, uint64_t load, int64_t T, int64_t max_cols, int64_t busy,
                    double max_units = kMaxUnits) {
    int64_t bj = std::min(busy, (int64_t)((double)load / 4096.0 / (double)T));
    bj = std::max(bj, (int64_t)((double)load / 65536.0 / (double)T));
    bj = bj > 256 ? (bj + 255) / 256 * 256 : (bj + 63) / 64 * 64;
    if (bj > max_cols)
        bj = max_cols;
    if (bj < 64)
        bj = 64;
    const double need = columns / max_units;    // columns per unit for max_units units
    if ((double)bj < need)
        bj = ((int64_t)need + 256) / 256 * 256;
    return bj;
}

// Places of keys in ascending order, equal ones in the order that they come:
// 11 bits at a time, those that differ anywhere.  Unit lists of batches and
// region counts are ordered by it on their first call (30000 units of an RR
// list 3.1 -> 1.3 ms with their making; sorting the units themselves took 100
// ns each).
inline std::vector<uint32_t> order_of(const std::vector<uint64_t> &key) {
    const size_t n = key.size();
    std::vector<uint32_t> at(n), to(n);
    uint64_t differ = 0;
    for (size_t i = 0; i < n; ++i) {
        at[i] = (uint32_t)i;
        differ |= key[i] ^ key[0];
    }
    if (n < 512) {
        std::stable_sort(at.begin(), at.end(), [&key](uint32_t x, uint32_t y) { return key[x] < key[y]; });
        return at;
    }
    for (int shift = 0; shift < 64; shift += 11) {
        if (!(differ >> shift & 2047))
            continue;
        uint32_t count[2049] = {};
        for (uint32_t i : at)
            ++count[(key[i] >> shift & 2047) + 1];
        for (int v = 0; v < 2048; ++v)
            count[v + 1] += count[v];
        for (uint32_t i : at)
            to[count[key[i] >> shift & 2047]++] = i;
        at.swap(to);
    }
    return at;
}

// Units of a single request that are computed from their number instead of
// read from a list: row tiles of T rows from row rb to re, column chunks of
// bj columns (both powers of two).
//   kind 1 (DR): unit = chunk * tiles + tile, chunks from column 0;
//   kind 2 (auto-pairs with rows to the catalog's end): chunks from column
//     rb, a triangle of S rows (row s: the s + 1 blocks of max(T, bj) that
//     reach its columns, `sub` units each) folded into a rectangle: row p of
//     it holds triangle rows p and S - 1 - p;
//   kind 3 (auto-pairs of a row range): as kind 1 from column rb; units below
//     the diagonal are empty.
// Some units at the edges are empty.
struct UnitGrid {
    int32_t kind;                // 0: no grid (PairArgs::units)
    int32_t rb, re, T, bj;
    int32_t tiles;               // kinds 1, 3: row tiles
    int32_t cols;                // end of the columns
    int32_t S, sub;              // kind 2
};

// End of the part of columns [j, j1) that a pass of at most `step` columns
// takes (j + step itself may lie beyond 32 bits).
TPCF_HD int32_t part_end(int32_t j, int32_t j1, int32_t step) { return j1 - j > step ? j + step : j1; }

// The aligned 64-column blocks that [j, j1) meets, 64 of them at most: bit b is
// set for block (j >> 6) + b.
TPCF_HD uint64_t blocks_met(int32_t j, int32_t j1) {
    const int32_t n = ((j1 - 1) >> 6) - (j >> 6) + 1;
    return n < 64 ? ((uint64_t)1 << n) - 1 : ~(uint64_t)0;
}

// Unit u of a grid; false when it is empty.
TPCF_HD bool grid_unit(const UnitGrid &g, uint32_t u, int32_t *i0, int32_t *i1, int32_t *j0,
                                          int32_t *j1) {
    uint32_t c, t;
    if (g.kind == 2) {
        const uint32_t S = (uint32_t)g.S, sub = (uint32_t)g.sub, w = (S + 1) * sub;
        const uint32_t p = u / w, first = (p + 1) * sub;
        uint32_t x = u - p * w, s = p;
        if (x >= first) {
            x -= first;
            s = S - 1 - p;
        }
        if (g.bj >= g.T) {
            c = s;
            t = x;
        } else {
            t = x / sub;
            c = s * sub + (x - t * sub);
        }
    } else {
        c = u / (uint32_t)g.tiles;
        t = u - c * (uint32_t)g.tiles;
    }
    const int64_t a = (int64_t)g.rb + (int64_t)t * g.T, b = (g.kind == 1 ? 0 : (int64_t)g.rb) + (int64_t)c * g.bj;
    if (a >= g.re || b >= g.cols)
        return false;
    *i0 = (int32_t)a;
    *i1 = (int32_t)(a + g.T < g.re ? a + g.T : g.re);
    *j0 = (int32_t)b;
    *j1 = (int32_t)(b + g.bj < g.cols ? b + g.bj : g.cols);
    return g.kind == 1 || *j1 > *i0 + 1;
}

// Units of a single request (see UnitGrid): tile and chunk are powers of two,
// the chunk at most chunk_width's.  No list is built, uploaded or kept.
// `full`: cut as if every tile were full, else by the rows that each has.
inline UnitGrid make_grid(bool auto_pairs, int64_t na, int64_t nb, int64_t rb, int64_t re, int rows, int64_t max_cols,
                   int32_t *n_units, bool full = true) {
    UnitGrid g{};
    *n_units = 0;
    const uint64_t pairs = pairs_of(auto_pairs, na, nb, rb, re);
    if (pairs == 0)
        return g;
    const int64_t T = (int64_t)kWaves * kWaveSize * rows;
    const int64_t want = chunk_width((double)tile_columns(auto_pairs, na, nb, rb, re, T), pairs,
                                     full ? T : tile_rows(re - rb, T), max_cols, 512);
    int64_t bj = 64;
    while (2 * bj <= want && bj < ((int64_t)1 << 22))
        bj *= 2;
    g.rb = (int32_t)rb;
    g.re = (int32_t)re;
    g.T = (int32_t)T;
    g.cols = (int32_t)nb;
    const int64_t tiles = (re - rb + T - 1) / T;
    g.tiles = (int32_t)tiles;
    for (;; bj *= 2) {
        const int64_t first = auto_pairs ? rb : 0, chunks = (nb - first + bj - 1) / bj;
        int64_t n;
        g.bj = (int32_t)bj;
        if (auto_pairs && re == na) {
            const int64_t q = bj < T ? T / bj : 1;
            const int64_t S = (chunks + q - 1) / q;
            g.kind = 2;
            g.S = (int32_t)S;
            g.sub = (int32_t)(bj < T ? q : bj / T);
            n = g.sub * (S * (S + 1) / 2);
        } else {
            g.kind = auto_pairs ? 3 : 1;
            n = chunks * tiles;
        }
        // chunks widen until the list would be short enough, but no further
        // than the number of items (kWaves a unit) needs to stay below 2^32;
        // a wavefront's item is then at most 2^30 pairs, of which its LDS
        // counts hold four
        if (n <= (int64_t)kMaxUnits || (bj >= ((int64_t)1 << 21) && n < ((int64_t)1 << 30))) {
            *n_units = (int32_t)n;
            return g;
        }
    }
}

}  // namespace tpcf
