// order_of() against std::stable_sort, with keys of every kind.  Prints the
// number of lists checked.
#include <stdio.h>

#include <numeric>
#include <random>

#include "units.h"

using namespace tpcf;

int main() {
    std::mt19937_64 g(5);
    int done = 0;
    for (size_t n : {0, 1, 2, 100, 511, 512, 513, 5000, 70001})
        for (int kind = 0; kind < 6; ++kind) {
            std::vector<uint64_t> key(n);
            for (size_t i = 0; i < n; ++i) {
                const uint64_t r = g();
                key[i] = kind == 0 ? 7 : kind == 1 ? r : kind == 2 ? r % 3 : kind == 3 ? (r % 50) << 40 :
                         kind == 4 ? ~(r % 100000) : (r & 1) << 63 | r % 2048;
            }
            std::vector<uint32_t> want(n);
            std::iota(want.begin(), want.end(), 0u);
            std::stable_sort(want.begin(), want.end(), [&](uint32_t x, uint32_t y) { return key[x] < key[y]; });
            if (order_of(key) != want) {
                printf("%zu keys of kind %d\n", n, kind);
                return 1;
            }
            ++done;
        }
    printf("%d\n", done);
    return 0;
}
