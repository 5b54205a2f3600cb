// Prints upd_slab_column for every lane group, entry, slab width and way of
// loading, one line each: lim lk h pairs column.
#include <cstdio>

#include "update_cols.h"

int main() {
    for (int pairs = 0; pairs < 2; ++pairs)
        for (int lim = 1; lim <= 8; ++lim)
            for (int lk = 0; lk < 4; ++lk)
                for (int h = 0; h < 2; ++h)
                    std::printf("%d %d %d %d %d\n", lim, lk, h, pairs, gplhr::upd_slab_column(lim, lk, h, pairs != 0));
    return 0;
}
