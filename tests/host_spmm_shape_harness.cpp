// Reads "x n b cols most plane row_len stage cut list" per line and prints the shape the
// sparse product runs with and, if asked to list them, each workgroup's rows in the
// orders it may take:
//   shape grid lpr rpw rpb sp order
//   rows even  row0:nr row0:nr ...
// or, for "eighths most total" (entries), whether they are even.
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "spmm_shape.h"

int main() {
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string kind;
        in >> kind;
        if (kind == "eighths") {
            int32_t most, total;
            in >> most >> total;
            std::printf("%d\n", (int)gplhr::spmm_even(most, total));
            continue;
        }
        long long n, row_len;
        int b, cols, most, plane, stage, cut, list;
        in >> n >> b >> cols >> most >> plane >> row_len >> stage >> cut >> list;
        int64_t grid = 0;
        const gplhr::SpmmShape s = gplhr::spmm_launch_shape(n, b, cols, most, plane, row_len, stage, cut != 0, grid);
        std::printf("shape %lld %d %d %d %d %d\n", (long long)grid, s.lpr, s.rpw, s.rpb, s.sp, s.order);
        if (list)
            for (int even = 0; even < 2; ++even) {
                std::printf("rows %d", even);
                for (int64_t k = 0; k < grid; ++k) {
                    const gplhr::SpmmRows r = s.sp > 0 ? gplhr::spmm_plane_rows(s, (uint32_t)k)
                                                       : gplhr::spmm_natural_rows(s, n, (uint32_t)k, even != 0);
                    std::printf(" %lld:%d", (long long)r.row0, r.nr);
                }
                std::printf("\n");
            }
    }
    return 0;
}
