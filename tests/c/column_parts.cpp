// Walks over a request's columns as the kernels do, up to the last column that
// a catalog can have: parts of a fixed length, and the aligned 64-column blocks
// of parts of 64 blocks.  Every column once, no position beyond 32 bits.
// Prints the number of walks.
#include <stdio.h>

#include "units.h"

using namespace tpcf;

int main() {
    const int32_t last = 2147482623;        // 2^31 - 1025
    int done = 0;
    for (int32_t end : {1, 63, 64, 65, 4096, 70001, 200000, last - 64, last - 1, last})
        for (int32_t len : {1, 2, 63, 64, 65, 4095, 4096, 4097, 65536, 65537, 131073, 199999}) {
            if (len > end)
                continue;
            const int32_t begin = end - len;
            // parts of 65536 columns
            int64_t n = 0;
            for (int32_t j = begin, e; j < end; j = e) {
                e = part_end(j, end, 65536);
                if (e <= j || e > end || e - j > 65536)
                    return 1;
                n += e - j;
            }
            if (n != len)
                return 1;
            // parts of up to 64 blocks, and the columns of each block that is met
            n = 0;
            for (int32_t j = begin, e; j < end; j = e) {
                e = part_end(j, end, 4096 - (j & 63));
                const int32_t b0 = j >> 6;
                for (uint64_t left = blocks_met(j, e); left; left &= left - 1) {
                    const int64_t b = (int64_t)(b0 + __builtin_ctzll(left)) << 6;
                    const int64_t lo = b > j ? b : j, hi = b + 64 < e ? b + 64 : e;
                    if (b > last || lo >= hi) {
                        printf("columns %d to %d: block at %lld\n", j, e, (long long)b);
                        return 1;
                    }
                    n += hi - lo;
                }
            }
            if (n != len)
                return 1;
            ++done;
        }
    printf("%d\n", done);
    return 0;
}
