// Every pair of a request lies in exactly one unit of its grid, and no unit
// leaves the request: checked pair by pair over ragged sizes, row ranges,
// rows per lane and chunk limits.  Prints the number of requests checked.
#include <stdio.h>

#include <vector>

#include "units.h"

using namespace tpcf;

static int check(bool auto_pairs, int64_t na, int64_t nb, int64_t rb, int64_t re, int rows, int64_t max_cols) {
    int32_t n = 0;
    const UnitGrid g = make_grid(auto_pairs, na, nb, rb, re, rows, max_cols, &n);
    std::vector<unsigned char> seen((size_t)(na * nb), 0);
    for (int32_t u = 0; u < n; ++u) {
        int32_t i0, i1, j0, j1;
        if (!grid_unit(g, (uint32_t)u, &i0, &i1, &j0, &j1))
            continue;
        if (i0 < rb || i1 > re || i0 >= i1 || j0 < 0 || j1 > nb || j0 >= j1 || i1 - i0 > 256 * rows)
            return 1;
        for (int32_t i = i0; i < i1; ++i)
            for (int32_t j = j0; j < j1; ++j)
                if (!auto_pairs || j > i)
                    ++seen[(size_t)i * nb + j];
    }
    for (int64_t i = 0; i < na; ++i)
        for (int64_t j = 0; j < nb; ++j)
            if (seen[(size_t)i * nb + j] != (i >= rb && i < re && (!auto_pairs || j > i)))
                return 1;
    return 0;
}

int main() {
    const int64_t sizes[] = {0, 1, 2, 63, 64, 65, 500, 512, 513, 1023, 1025, 2047, 2304, 3001};
    const int64_t caps[] = {256, 768, 2048, 65536};
    int done = 0;
    for (int64_t na : sizes)
        for (int64_t max_cols : caps)
            for (int rows = 1; rows <= 4; rows *= 2) {
                const int64_t ranges[][2] = {{0, na}, {na / 3, na}, {na / 7, na - na / 5}, {na / 2, na / 2}};
                for (auto &r : ranges) {
                    if (check(true, na, na, r[0], r[1], rows, max_cols)) {
                        printf("auto %lld [%lld, %lld) rows %d cols %lld\n", (long long)na, (long long)r[0],
                               (long long)r[1], rows, (long long)max_cols);
                        return 1;
                    }
                    const int64_t nb = (na * 5 + 77) % 1900;
                    if (check(false, na, nb, r[0], r[1], rows, max_cols)) {
                        printf("cross %lld %lld [%lld, %lld) rows %d cols %lld\n", (long long)na, (long long)nb,
                               (long long)r[0], (long long)r[1], rows, (long long)max_cols);
                        return 1;
                    }
                    done += 2;
                }
            }
    // large requests: as many units as 32-bit items allow, none too large
    for (int64_t n : {(int64_t)1000000, (int64_t)100000000, (int64_t)2147482623}) {
        int32_t units = 0;
        const UnitGrid g = make_grid(true, n, n, 0, n, 4, 2048, &units);
        if (units <= 0 || units >= (1 << 30) || (int64_t)g.bj * g.T > ((int64_t)1 << 32))
            return 1;
        ++done;
    }
    printf("%d\n", done);
    return 0;
}
