// Check the plans that the multi-step kernels are launched with
// (paper_2002_02503_amd/csrc/host.cpp), which the kernels rely on unchecked, for
// tests/test_host_plans.py: column tiles over all row lengths.  A failed
// expectation exits 2.
#include <cstdint>
#include <cstdio>

#include "host.hpp"

using namespace lbm;

static int g_fail = 0;
#define EXPECT(cond, ...)                                                         \
    do {                                                                          \
        if (!(cond) && g_fail < 20) {                                             \
            std::fprintf(stderr, "%s:%d: expectation failed: %s (", __FILE__, __LINE__, #cond); \
            std::fprintf(stderr, __VA_ARGS__);                                    \
            std::fprintf(stderr, ")\n");                                          \
            ++g_fail;                                                             \
        }                                                                         \
    } while (0)

// A column tile: within the box, its ring in the block's threads (one LDS slot
// each), and no single row where the box has more.
static void check_tile(size_t elem, int threads, int64_t nx, int64_t ny, int tx, int ty)
{
    EXPECT(tx >= 1 && ty >= 1 && tx <= nx && ty <= ny, "%zu bytes, %ld x %ld: %d x %d", elem, long(nx), long(ny), tx, ty);
    EXPECT((tx + 2) * (ty + 2) <= threads, "%zu bytes, %ld x %ld: %d x %d", elem, long(nx), long(ny), tx, ty);
    EXPECT(ty >= 2 || ny == 1, "%zu bytes, %ld x %ld: %d x %d", elem, long(nx), long(ny), tx, ty);
}

static void test_column_tiles()
{
    for (size_t elem : {size_t(2), size_t(4), size_t(8)}) {
        for (int64_t nx = 1; nx <= 1100; ++nx) {
            for (int64_t ny : {1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 63, 64, 65, 100, 129, 255, 1000, 65535}) {
                int tx = 0, ty = 0;
                column_tile(elem, nx, ny, &tx, &ty);
                check_tile(elem, two_step_threads(elem), nx, ny, tx, ty);
                tx = ty = 0;
                batch_column_tile(elem, nx, ny, &tx, &ty);
                check_tile(elem, batch_columns_threads(elem), nx, ny, tx, ty);
            }
        }
        for (int64_t nx : {int64_t(65537), int64_t(100001), int64_t(1) << 21, (int64_t(1) << 27) + 1}) {
            int tx = 0, ty = 0;
            column_tile(elem, nx, 50, &tx, &ty);
            check_tile(elem, two_step_threads(elem), nx, 50, tx, ty);
            batch_column_tile(elem, nx, 50, &tx, &ty);
            check_tile(elem, batch_columns_threads(elem), nx, 50, tx, ty);
        }
    }
}

int main()
{
    test_column_tiles();
    if (g_fail) return 2;
    std::printf("host plan driver: ok\n");
    return 0;
}
