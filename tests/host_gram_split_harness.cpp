// For every pair of widths and a range of row counts, one line:
// n bx by scratch-entries; then for every tile count and type (1 complex64)
// "t n tiles type few blocks"; last "c entries" of the call that allocates nothing.
#include <cstdio>

#include "gram_split.h"

int main() {
    const int64_t rows[] = {1, 500, 1024, 1025, 2048, 2049, 20000, 100000, 131071, 131072,
                            140000, 200000, 262143, 262144, 600000, 1048575, 1048576, 4096000};
    for (int64_t n : rows) {
        for (int bx = 1; bx <= 64; ++bx)
            for (int by = 1; by <= 64; ++by)
                std::printf("s %lld %d %d %zu\n", (long long)n, bx, by, gplhr::gram_part_entries(n, bx, by));
        for (int t = 1; t <= 72; ++t)
            for (int c64 = 0; c64 < 2; ++c64)
                std::printf("t %lld %d %d %d %lld\n", (long long)n, t, c64, (int)gplhr::gram_few_rows(n, t),
                            (long long)gplhr::gram_row_blocks(n, t, c64));
    }
    std::printf("c %zu\n", gplhr::GRAM_NOALLOC_ENTRIES);
    return 0;
}
