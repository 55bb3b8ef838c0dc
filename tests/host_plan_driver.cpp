// Check the plans that the multi-step kernels are launched with
// (paper_2002_02503_amd/csrc/host.cpp), which the kernels rely on unchecked, for
// tests/test_host_plans.py: column tiles over all row lengths, tile plans over box
// sizes, lattices, types and compute units, with the limits that bound the
// kernels' threads, LDS, offsets and wrapped coordinates; the shapes for which a
// default is taken; and the division by a constant that set-up and
// readers use.  A failed expectation exits 2.
#include <cstdint>
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <limits>
#include <random>
#include <vector>

#include "collide.hpp"
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
    // the ring of a last column, and its neighbours, are within a period of the box
    const int64_t x_end = (nx + tx - 1) / tx * tx, y_end = (ny + ty - 1) / ty * ty;
    EXPECT((nx < 3 || x_end < 2 * nx) && (ny < 3 || y_end < 2 * ny), "%ld x %ld: %d x %d", long(nx), long(ny), tx, ty);
}

// A tile plan, whichever box it is for.
static void check_plan(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, const TilePlan& p)
{
    const int64_t elem = int64_t(storage_bytes(dtype)), n[3] = {nx, ny, nz}, t[3] = {p.tx, p.ty, p.tz};
    bool ok = p.steps >= 2 && p.steps <= kTileMaxSteps && p.block >= 64 && p.block <= 1024 && p.block % 64 == 0;
    // the regions of a full tile: the stored one in LDS, the later ones with one thread per site
    int64_t region = 1, second = 1;
    for (int a = 0; a < L.D; ++a) {
        const bool wraps = a == 0 && p.tx == nx;  // inside the tile
        const int64_t ring = wraps ? 0 : p.steps - 1;
        ok = ok && t[a] >= 1 && t[a] <= n[a];
        region *= t[a] + 2 * ring;
        second *= t[a] + 2 * std::max<int64_t>(ring - 1, 0);
        // ring sites within a period of the box, for three sites and more
        ok = ok && (n[a] < 3 || (ring <= n[a] && n[a] - 1 + ring < 2 * n[a]));
    }
    ok = ok && region * L.Q * elem <= 160 * 1024 && region < (1 << 15) && second <= p.block;
    ok = ok && tile_region(L, p, nx, p.steps) == region && (L.D == 3 || nz == 1);
    // offsets in 32 bits
    ok = ok && double(nx) * double(ny) * double(nz) * L.Q * double(elem) <= 4294967296.0;
    // a launch of fewer steps is a smaller region
    for (int k = 2; k < p.steps; ++k) ok = ok && tile_region(L, p, nx, k) < region;
    EXPECT(ok, "D%dQ%d dtype %d %ld x %ld x %ld: %d x %d x %d, %d steps, %d threads", L.D, L.Q, dtype, long(nx), long(ny),
           long(nz), p.tx, p.ty, p.tz, p.steps, p.block);
}

static void test_tile_plans()
{
    const int64_t sides[] = {1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 129, 200, 511, 1000, 4097, 65535};
    const int64_t wide[] = {100001, 1 << 21, (int64_t(1) << 27) + 1, (int64_t(1) << 29), INT32_MAX};
    int plans = 0;
    for (int lat = 0; lat < 4; ++lat) {
        LatticeInfo L;
        lattice_info(lat, &L);
        for (int dtype = 0; dtype < 4; ++dtype) {
            for (int cus : {1, 64, 256, 304}) {
                auto one = [&](int64_t nx, int64_t ny, int64_t nz) {
                    TilePlan p{};
                    if (!tile_plan(L, dtype, nx, ny, nz, cus, &p)) return;
                    EXPECT(L.R == 1, "a ring of one site");
                    check_plan(L, dtype, nx, ny, nz, p);
                    ++plans;
                };
                for (int64_t nx : sides)
                    for (int64_t ny : sides)
                        for (int64_t nz : sides)
                            if (L.D == 3 || nz == 1) one(nx, ny, nz);
                for (int64_t nx : wide)
                    for (int64_t ny : {int64_t(1), int64_t(2), int64_t(65535)}) one(nx, ny, 1);
            }
        }
    }
    EXPECT(plans > 10000, "%d plans", plans);
    // D2Q9 on both sides of 4 GiB (36 bytes a site in FP32)
    LatticeInfo L;
    lattice_info(0, &L);
    TilePlan p{};
    EXPECT(tile_plan(L, 1, 10922, 10922, 1, 256, &p) && !tile_plan(L, 1, 10923, 10923, 1, 256, &p), "4 GiB");
}

static void test_column_limits()
{
    // the two-step kernel's offsets inside a z-plane, 19 * 4 bytes a site
    LatticeInfo L;
    lattice_info(1, &L);
    const int64_t most = ((int64_t(1) << 31) - 1) / (19 * 4);
    EXPECT(columns_fit(L, 1, most, 1, 9) && !columns_fit(L, 1, most + 1, 1, 9), "one row");
    EXPECT(columns_fit(L, 1, 5315, 5316, 2) && !columns_fit(L, 1, 5316, 5316, 2), "a plane");
    EXPECT(!columns_fit(L, 1, 0, 8, 8) && !columns_fit(L, 1, 8, -1, 8) && !columns_fit(L, 4, 8, 8, 8), "no box, no type");
    EXPECT(!columns_fit(L, 1, INT64_MAX, INT64_MAX, INT64_MAX), "beyond 2^31");
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
        if (elem == 8) {
            int tx = 0, ty = 0;
            column_tile(elem, 224, 224, &tx, &ty);
            EXPECT(tx == 56 && ty == 5, "%d x %d", tx, ty);
            column_tile(elem, 240, 240, &tx, &ty);
            EXPECT(tx == 80 && ty == 3, "%d x %d", tx, ty);
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

// n equal boxes
static bool batch_pays(int lat, int dtype, int n, int64_t nx, int64_t ny, int64_t nz, std::vector<int64_t> more = {})
{
    LatticeInfo L;
    lattice_info(lat, &L);
    for (int k = 0; k < n; ++k) more.insert(more.end(), {nx, ny, nz});
    return batch_columns_pay(L, dtype, int(more.size() / 3), more.data());
}

static void test_batch_rule()
{
    // lattice codes: 0 D2Q9, 1 D3Q19, 2 D3Q39, 3 D3Q15; dtype codes: 0 FP64 .. 3 BF16
    for (int lat : {1, 3}) {
        for (int dtype : {0, 1}) {
            for (int64_t a : {24, 32, 40, 48, 64, 96}) EXPECT(batch_pays(lat, dtype, 64, a, a, a), "%ld", long(a));
            EXPECT(!batch_pays(lat, dtype, 8, 20, 20, 20), "few sites");
            EXPECT(!batch_pays(lat, dtype, 200, 20, 20, 20), "small boxes");
            // one layer, few rows, narrow: mostly ring, or few lanes
            EXPECT(!batch_pays(lat, dtype, 8, 1000, 1000, 1), "a layer");
            EXPECT(!batch_pays(lat, dtype, 8, 1000, 1000, 2), "two layers");
            EXPECT(!batch_pays(lat, dtype, 8, 1000, 1, 1000), "one row");
            EXPECT(!batch_pays(lat, dtype, 40, 20000, 2, 2), "few rows");
            EXPECT(!batch_pays(lat, dtype, 60, 4, 4, 5000), "narrow");
            EXPECT(!batch_pays(lat, dtype, 60, 8, 8, 2000), "narrow");
            EXPECT(!batch_pays(lat, dtype, 8, 40, 40, 40, {2000, 2000, 1}), "one layer among boxes");
            EXPECT(batch_pays(lat, dtype, 64, 40, 40, 40, {40, 40, 1, 5, 5, 400}), "a small share of thin boxes");
        }
        EXPECT(!batch_pays(lat, 2, 64, 40, 40, 40) && !batch_pays(lat, 3, 64, 40, 40, 40), "16-bit");
    }
    EXPECT(!batch_pays(0, 1, 64, 1000, 1000, 1) && !batch_pays(2, 1, 64, 40, 40, 40), "no column kernel");
    const int64_t wide = (int64_t(1) << 21);
    EXPECT(!batch_pays(1, 1, 2, wide, 2, 2), "rows at the limit");
}

static bool single_pays(int lat, int dtype, int64_t nx, int64_t ny, int64_t nz)
{
    LatticeInfo L;
    lattice_info(lat, &L);
    return columns_pay(L, dtype, nx, ny, nz);
}

static void test_single_rule()
{
    EXPECT(!single_pays(1, 1, 640, 500, 3) && !single_pays(1, 1, 1024, 300, 2), "few planes on whole lines");
    EXPECT(single_pays(1, 1, 640, 500, 4) && !single_pays(1, 0, 1000, 1000, 3), "few planes");
    for (int dtype : {0, 1}) {
        for (int lat : {1, 3}) {
            for (int64_t a : {64, 80, 100, 127, 128, 160, 201, 255, 256}) EXPECT(single_pays(lat, dtype, a, a, a), "%ld", long(a));
            EXPECT(!single_pays(lat, dtype, 48, 48, 48) && !single_pays(lat, dtype, 65, 65, 65), "few sites");
            EXPECT(!single_pays(lat, dtype, 1024, 1024, 1) && !single_pays(lat, dtype, 1000, 1, 1000), "a layer");
            EXPECT(!single_pays(lat, dtype, 100000, 2, 2), "few rows");
        }
        for (int lat : {1, 3}) {
            EXPECT(!single_pays(lat, dtype, 3, 3, 60000), "narrow");
            EXPECT(single_pays(lat, dtype, 16, 16, 4000) && single_pays(lat, dtype, 5, 30, 3000), "short rows");
            EXPECT(single_pays(lat, dtype, 4, 4, 30000) == (dtype == 0), "narrow");
            EXPECT(single_pays(lat, dtype, 30, 3, 5000) == (dtype == 0), "narrow");
            EXPECT(single_pays(lat, dtype, 64, 3, 2400) == (dtype == 0), "narrow");
        }
        EXPECT(!single_pays(1, dtype, 1000, 1000, 2) && single_pays(1, dtype, 1000, 1000, 4), "few planes");
        EXPECT(single_pays(1, dtype, 512, 512, 2) && single_pays(1, dtype, 700, 700, 3), "few planes");
        EXPECT(!single_pays(0, dtype, 2000, 2000, 1) && !single_pays(2, dtype, 128, 128, 128), "no column kernel");
    }
    for (int dtype : {2, 3}) {
        // rows of whole lines, whatever ny is
        for (int64_t ny : {96, 100, 101, 130, 250, 256}) {
            EXPECT(!single_pays(1, dtype, 256, ny, 256) && !single_pays(1, dtype, 128, ny, 200), "%ld rows", long(ny));
            EXPECT(!single_pays(1, dtype, 64, 2 * ny, 250), "%ld rows", long(ny));
        }
        EXPECT(single_pays(1, dtype, 130, 130, 130) && single_pays(1, dtype, 255, 255, 255), "ragged");
        EXPECT(!single_pays(1, dtype, 12, 12, 20000) && !single_pays(1, dtype, 200, 2, 6000), "narrow");
        EXPECT(single_pays(1, dtype, 20, 20, 6000) && single_pays(1, dtype, 10, 20, 12000), "short rows");
        EXPECT(!single_pays(1, dtype, 1000, 1000, 4) && !single_pays(1, dtype, 700, 700, 5), "few planes");
        EXPECT(!single_pays(1, dtype, 160, 160, 160) && !single_pays(1, dtype, 240, 240, 240), "rows of whole sectors");
        EXPECT(single_pays(1, dtype, 208, 120, 120) && single_pays(1, dtype, 400, 200, 100), "in the caches, idle lanes");
        EXPECT(!single_pays(3, dtype, 130, 130, 130) && !single_pays(1, dtype, 101, 101, 101), "D3Q15, few sites");
    }
}

// Whether the box has a tile plan and takes it by default.
static bool tile_taken(int lat, int dtype, int64_t nx, int64_t ny, int64_t nz)
{
    LatticeInfo L;
    lattice_info(lat, &L);
    TilePlan p;
    const bool has = tile_plan(L, dtype, nx, ny, nz, 256, &p);
    EXPECT(has, "%ld x %ld x %ld", long(nx), long(ny), long(nz));
    return has && tile_default(L, dtype, nx, ny, nz, p);
}

static void test_tile_rule()
{
    EXPECT(tile_taken(0, 0, 64, 64, 1) && tile_taken(0, 0, 1024, 1024, 1), "D2Q9");
    EXPECT(tile_taken(1, 0, 16, 16, 16) && tile_taken(1, 0, 32, 32, 32) && tile_taken(1, 0, 17, 17, 20), "FP64");
    for (int lat : {1, 3}) EXPECT(!tile_taken(lat, 0, 64, 10, 24) && !tile_taken(lat, 0, 64, 3, 72), "mostly ring");
    EXPECT(!tile_taken(1, 0, 41, 115, 4), "mostly ring");
    for (int dtype : {1, 2, 3}) EXPECT(tile_taken(1, dtype, 64, 10, 24) && tile_taken(1, dtype, 41, 115, 4), "half the bytes");
}

// over<N> gives the bits of the division, signed zeros included; a subnormal
// quotient is the correction rounded to the subnormal numbers' spacing, so where
// x / N lies half-way between two of them it may be the other one.
template <int N>
static void test_over()
{
    auto same = [](double x) {
        const double a = over<N>(x), b = x / double(N);
        const double least = std::numeric_limits<double>::min();
        const bool subnormal = b != 0.0 && b > -least && b < least;
        EXPECT(std::memcmp(&a, &b, sizeof(a)) == 0 || (a != a && b != b) ||
                   (subnormal && a - b <= std::numeric_limits<double>::denorm_min() &&
                    b - a <= std::numeric_limits<double>::denorm_min()),
               "%a / %d: %a, not %a", x, N, a, b);
    };
    const double inf = std::numeric_limits<double>::infinity(), big = std::numeric_limits<double>::max();
    const double tiny = std::numeric_limits<double>::denorm_min(), least = std::numeric_limits<double>::min();
    for (double x : {0.0, inf, big, tiny, 3 * tiny, double(N) * tiny, least, least * N, 1.0, double(N), std::numeric_limits<double>::quiet_NaN()}) {
        same(x);
        same(-x);
    }
    std::mt19937_64 rng(N);
    for (int k = 0; k < 200000; ++k) {
        uint64_t bits = rng();
        double x;
        std::memcpy(&x, &bits, sizeof(x));
        same(x);                              // any exponent
        same(double(int64_t(bits >> 8)) / 1e18);  // ordinary values
    }
}

int main()
{
    test_column_tiles();
    test_column_limits();
    test_tile_plans();
    test_batch_rule();
    test_single_rule();
    test_tile_rule();
    test_over<2>();
    test_over<6>();
    test_over<24>();
    test_over<120>();
    test_over<36>();
    test_over<72>();
    test_over<6480>();
    if (g_fail) return 2;
    std::printf("host plan driver: ok\n");
    return 0;
}
