// For every pair of widths and a range of row counts, one line:
// n bx by scratch-entries; then for every tile count "t n tiles few blocks".
#include <cstdio>

#include "gram_split.h"

int main() {
    const int64_t rows[] = {1, 500, 1024, 1025, 2048, 2049, 20000, 100000, 262144, 600000, 4096000};
    for (int64_t n : rows) {
        for (int bx = 1; bx <= 64; ++bx)
            for (int by = 1; by <= 64; ++by)
                std::printf("s %lld %d %d %zu\n", (long long)n, bx, by, gplhr::gram_part_entries(n, bx, by));
        for (int t = 1; t <= 72; ++t)
            std::printf("t %lld %d %d %lld\n", (long long)n, t, (int)gplhr::gram_few_rows(n, t),
                        (long long)gplhr::gram_row_blocks(n, t > 8));
    }
    return 0;
}
