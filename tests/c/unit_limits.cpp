// How many units a request is cut into, and how large they are, at catalogs
// of up to 2^31 - 1024 points (nothing is counted).  Prints the number of
// requests checked.
#include <stdio.h>

#include "units.h"

using namespace tpcf;

static const int64_t kQueueSlack = 8;    // the queues round the items up to their number

// Units of a list (DR, or one tile's columns of auto-pairs at a time) at chunks of bj columns.
static double list_units(bool auto_pairs, int64_t na, int64_t nb, int64_t rb, int64_t re, int64_t T, int64_t bj) {
    double n = 0;
    const int64_t tiles = (re - rb + T - 1) / T;
    if (!auto_pairs)
        return (double)tiles * (double)((nb + bj - 1) / bj);
    for (int64_t t = 0; t < tiles; ++t)
        n += (double)((na - (rb + t * T) + bj - 1) / bj);
    return n;
}

int main() {
    int done = 0;
    // a fixed room for the list: whatever the rows are, the chunks are wide enough for it
    const double room = 170000.0;
    for (int64_t nb : {(int64_t)1000, (int64_t)1000000, (int64_t)30000000, (int64_t)500000000, (int64_t)2147482623})
        for (int64_t cnt : {1, 2, 7, 63, 64, 300, 1023, 1024, 1025, 5000, 20000})
            for (int rows : {1, 2, 4})
                for (int full = 0; full < 2; ++full)
                    for (int aut = 0; aut < 2; ++aut) {
                        const int64_t T = 256 * rows, rb = nb / 3, re = rb + cnt;
                        if (re > nb || (aut && nb < 1000000 && cnt > 500))
                            continue;
                        const uint64_t pairs = pairs_of(aut, nb, nb, rb, re);
                        const int64_t bj = chunk_width((double)tile_columns(aut, nb, nb, rb, re, T), pairs,
                                                       full ? T : tile_rows(cnt, T), 2048, 512, room);
                        const double n = list_units(aut, nb, nb, rb, re, T, bj);
                        if (bj < 64 || n > 1.1 * room + (double)((cnt + T - 1) / T)) {
                            printf("%s %lld rows x %lld, %d rows a lane: %.0f units of %lld columns\n",
                                   aut ? "auto" : "cross", (long long)cnt, (long long)nb, rows, n, (long long)bj);
                            return 1;
                        }
                        ++done;
                    }
    // cut by the rows that they have, requests of any few rows have chunks of the same width as a full tile's
    for (int64_t cnt : {1, 64, 300, 600}) {
        int32_t few = 0, all = 0;
        const UnitGrid g = make_grid(false, 2000, 1000000, 0, cnt, 4, 2048, &few, false);
        const UnitGrid f = make_grid(false, 2000, 1000000, 0, 1024, 4, 2048, &all, false);
        if (g.bj != f.bj || few != all) {
            printf("%lld rows: %d units of %d columns, 1024 rows %d of %d\n", (long long)cnt, few, g.bj, all, f.bj);
            return 1;
        }
        ++done;
    }
    // items are numbered with 32 bits, and one's pairs leave room in the counts that a wavefront keeps over several
    for (int64_t n : {(int64_t)1000000, (int64_t)100000000, (int64_t)1500000000, (int64_t)2147482623})
        for (int rows : {2, 4})
            for (int64_t max_cols : {256, 2048, 65536})
                for (int kind = 1; kind <= 3; ++kind)
                    for (int full = 0; full < 2; ++full) {
                        int32_t units = 0;
                        const UnitGrid g = make_grid(kind != 1, n, n, kind == 3 ? 5 : 0, kind == 3 ? n - 7 : n, rows,
                                                     max_cols, &units, full);
                        const int64_t item = (int64_t)(g.T / kWaves) * g.bj;
                        if (g.kind != kind || units <= 0 || (int64_t)units * kWaves > ((int64_t)1 << 32) - kQueueSlack ||
                            item > ((int64_t)1 << 30)) {
                            printf("kind %d of %lld, %d rows a lane: %d units, items of %lld pairs\n", kind,
                                   (long long)n, rows, units, (long long)item);
                            return 1;
                        }
                        // the last units lie inside
                        for (uint32_t u = (uint32_t)units - 1; u + 1000 > (uint32_t)units; --u) {
                            int32_t i0, i1, j0, j1;
                            if (grid_unit(g, u, &i0, &i1, &j0, &j1) &&
                                (i0 < g.rb || i0 >= i1 || i1 > g.re || j0 < 0 || j0 >= j1 || j1 > n))
                                return 1;
                        }
                        ++done;
                    }
    printf("%d\n", done);
    return 0;
}
