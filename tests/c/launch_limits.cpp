// Grids of the kernels that take 256 / R rows per workgroup, for row counts up to
// the largest a plan takes: fewer than 2^32 threads, and no workgroup too many.
#include <cstdio>

#include "mpk_internal.h"

int main() {
    for (int64_t n : {(int64_t)1, (int64_t)255, (int64_t)256, (int64_t)257, (int64_t)1 << 26,
                      ((int64_t)1 << 26) + 1, (int64_t)1 << 28, (int64_t)INT32_MAX - 1})
        for (int R = 1; R <= 16; ++R) {
            const int64_t rows = 256 / R, grid = mpk::row_grid(n, rows);
            if (grid < 1 || grid * 256 >= (int64_t)1 << 32 || (grid - 1) * rows >= n ||
                (grid * rows < n && grid < (int64_t)1 << 22)) {
                std::printf("n = %lld, R = %d: %lld workgroups\n", (long long)n, R, (long long)grid);
                return 1;
            }
        }
    return 0;
}
