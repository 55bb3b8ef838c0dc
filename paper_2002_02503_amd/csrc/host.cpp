// Host-only parts of the library (host.hpp): no HIP call, so the file also
// builds and runs under the host sanitizers.
#include "host.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <sstream>

#include "lattice.hpp"

namespace lbm {

template <class L>
static void fill_info(LatticeInfo* out)
{
    out->D = L::D;
    out->Q = L::Q;
    out->two_n = L::TWO_N;
    out->k_default = L::K_DEFAULT;
    out->k_max = L::K_MAX;
    out->R = L::R;
    out->T0 = L::T0;
    out->c.resize(L::Q * 3);
    out->w.resize(L::Q);
    out->mrow.resize(L::Q);
    for (int i = 0; i < L::Q; ++i) {
        for (int a = 0; a < 3; ++a) out->c[i * 3 + a] = L::c[i][a];
        out->w[i] = L::w[i];
        out->mrow[i] = mem_row<L>(i);
    }
}

bool lattice_info(int lat, LatticeInfo* out)
{
    switch (lat) {
    case kD2Q9: fill_info<D2Q9>(out); return true;
    case kD3Q15: fill_info<D3Q15>(out); return true;
    case kD3Q19: fill_info<D3Q19>(out); return true;
    case kD3Q39: fill_info<D3Q39>(out); return true;
    default: return false;
    }
}

size_t storage_bytes(int dtype)
{
    switch (dtype) {
    case 0: return 8;
    case 1: return 4;
    case 2: return 2;
    case 3: return 2;
    default: return 0;
    }
}

// *why := "box <box>: <what>"
static bool reject(std::string* why, int box, const char* what)
{
    *why = "box " + std::to_string(box) + ": " + what;
    return false;
}

bool check_boxes(const LatticeInfo& L, int dtype, int nbox, const int64_t* dims, const double* tau, std::string* why)
{
    const size_t elem = storage_bytes(dtype);
    int64_t total = 0;
    for (int b = 0; b < nbox; ++b) {
        const int64_t* d = dims + 3 * b;
        for (int a = 0; a < 3; ++a)
            if (d[a] < 1 || d[a] > INT32_MAX) {
                char buf[128];
                snprintf(buf, sizeof(buf), "box %d: dims[%d] = %lld outside [1, 2^31)", b, a, (long long)d[a]);
                *why = buf;
                return false;
            }
        const int64_t nx = d[0], ny = d[1], nz = d[2];
        // the step kernels index x-rows r = z ny + y in 32 bits
        if (ny * nz > INT32_MAX) return reject(why, b, "ny * nz must be below 2^31");
        if (L.D == 2 && nz != 1) return reject(why, b, "a 2-D lattice needs nz == 1");
        if (!std::isfinite(tau[b]) || !(tau[b] > 0.5)) return reject(why, b, "tau must be finite and > 1/2");
        total += nx * ny * nz;
        if (total > kMaxSites) return reject(why, b, "the total site count must be at most 2^36");
        // lane offsets inside one population row are formed in 32 bits
        if (nx * int64_t(elem) > INT32_MAX)
            return reject(why, b, "a population row (nx * storage bytes) must be below 2 GiB");
        // y and z are grid coordinates of the single-box kernels
        if (ny > 65535 || nz > 65535) return reject(why, b, "ny and nz must be at most 65535");
        if (nbox > 1) {
            // a batch box is addressed with 32-bit element offsets
            const uint64_t padded = (uint64_t(nx * ny * nz) + kBlockSites - 1) / kBlockSites * kBlockSites;
            if (padded * uint64_t(L.Q) * elem >= (uint64_t(1) << 31))
                return reject(why, b, "a box of a batch must hold less than 2 GiB of populations");
            // the batched step splits a lane's site with a float reciprocal,
            // exact while x0 + 64 stays below 2^22
            if (nx > (int64_t(1) << 21)) return reject(why, b, "a box of a batch needs nx at most 2^21");
        }
    }
    return true;
}

bool columns_fit(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz)
{
    const size_t elem = storage_bytes(dtype);
    if (L.D != 3 || L.R != 1 || elem == 0) return false;
    if (nx < 1 || ny < 1 || nz < 1 || nx > INT32_MAX || ny > INT32_MAX || nz > INT32_MAX) return false;
    const uint64_t plane_sites = uint64_t(nx) * uint64_t(ny);  // below 2^62
    return plane_sites <= ((uint64_t(1) << 31) - 1) / (uint64_t(L.Q) * elem);
}

bool two_step_fits(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz)
{
    return columns_fit(L, dtype, nx, ny, nz) && nx % kTwoStepTileX == 0 &&
           ny % two_step_tile_y(storage_bytes(dtype)) == 0;
}

// n cut into pieces of at most `most`, of nearly equal size.
static int even_piece(int64_t n, int64_t most)
{
    const int64_t pieces = (n + most - 1) / most;
    return int((n + pieces - 1) / pieces);
}

// Widest x-piece of a column: at most 128 sites, and at least two rows with
// their ring in the block's threads.
static int widest_piece(int threads) { return std::min(128, threads / 4 - 2); }

void column_tile(size_t elem, int64_t nx, int64_t ny, int* tx, int* ty)
{
    const int widest = widest_piece(two_step_threads(elem));
    *tx = (nx % kTwoStepTileX == 0) ? kTwoStepTileX : even_piece(nx, widest);
    if (elem == 8 && nx % 16 == 0 && *tx % 8 != 0) {
        // one piece more, if those start on half a line
        const int64_t more = (nx + *tx - 1) / *tx + 1;
        const int finer = int((nx + more - 1) / more);
        if (finer % 8 == 0) *tx = finer;
    }
    *ty = even_piece(ny, two_step_threads(elem) / (*tx + 2) - 2);
}

void batch_column_tile(size_t elem, int64_t nx, int64_t ny, int* tx, int* ty)
{
    *tx = even_piece(nx, widest_piece(batch_columns_threads(elem)));
    const int64_t most = std::min<int64_t>(ny, batch_columns_threads(elem) / (*tx + 2) - 2);
    int64_t best = 0;
    for (int64_t t = most; t >= 1; --t) {
        const int piece = even_piece(ny, t);
        const int64_t cost = (ny + piece - 1) / piece * column_rounds(*tx, piece);
        if (t == most || cost < best) {
            best = cost;
            *ty = piece;
        }
    }
}

bool columns_pay(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz)
{
    const int64_t elem = int64_t(storage_bytes(dtype));
    if (!columns_fit(L, dtype, nx, ny, nz) || nx > kMaxSites / ny / nz) return false;
    if (ny < 2 || nz < 2 || ny * nz < kColumnsRows) return false;
    const int64_t sites = nx * ny * nz;
    int tx = 0, ty = 0;
    column_tile(size_t(elem), nx, ny, &tx, &ty);
    if (elem == 8 ? tx * ty < kColumnsLeast64 : tx * ty < kColumnsLeast && (nx > 64 || ty < 16)) return false;
    if (!two_step_fits(L, dtype, nx, ny, nz)) {
        const bool lines = nx * elem % 128 == 0;
        if (nz < (elem == 8 ? (sites < kColumnsThin64 ? 2 : 4) : elem == 4 ? (lines ? 4 : 3) : 12)) return false;
    }
    if (elem == 2) {
        if (L.Q != 19 || nx % kTwoStepTileX == 0 || sites < kColumnsSites16) return false;
        const int64_t block = std::min<int64_t>(256, (nx + 63) / 64 * 64);
        const int64_t lanes = (nx + block - 1) / block * block;  // of the one-site step on a row
        return !(nx * elem % 32 == 0 && 5 * nx >= 4 * lanes && sites * L.Q * elem >= kColumnsState16);
    }
    return sites >= (two_step_fits(L, dtype, nx, ny, nz) ? kTwoStepSites : kColumnsSites);
}

bool batch_columns_pay(const LatticeInfo& L, int dtype, int nbox, const int64_t* dims)
{
    const int64_t elem = int64_t(storage_bytes(dtype));
    if (elem < 4) return false;
    int64_t sites = 0;
    for (int b = 0; b < nbox; ++b) {
        const int64_t* d = dims + 3 * b;
        if (!columns_fit(L, dtype, d[0], d[1], d[2])) return false;
        sites += d[0] * d[1] * d[2];
    }
    if (sites < kBatchColumnsSites || sites < kBatchColumnsMean * nbox) return false;
    int64_t rounds = 0;
    for (int b = 0; b < nbox; ++b) {
        const int64_t nx = dims[3 * b], ny = dims[3 * b + 1], nz = dims[3 * b + 2];
        int tx = 0, ty = 0;
        batch_column_tile(size_t(elem), nx, ny, &tx, &ty);
        const int64_t r = elem == 4 ? column_plane_cost(tx, ty) : column_rounds(tx, ty);
        rounds += ((nx + tx - 1) / tx) * ((ny + ty - 1) / ty) * (nz * r + 2 * column_rounds1(tx, ty));
    }
    // 256 sites a round against two steps of every site
    return 10 * 256 * rounds <= (elem == 4 ? 18 : 20) * 2 * sites;
}

int64_t tile_region(const LatticeInfo& L, const TilePlan& p, int64_t nx, int steps)
{
    const int64_t g = 2 * (steps - 1);
    return (p.tx + (p.tx == nx ? 0 : g)) * (p.ty + g) * (L.D == 3 ? p.tz + g : 1);
}

bool tile_plan_fits(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, const TilePlan& p)
{
    const int64_t elem = int64_t(storage_bytes(dtype));
    if (L.R != 1 || elem == 0 || nx < 1 || ny < 1 || nz < 1) return false;
    if (p.tx < 1 || p.ty < 1 || p.tz < 1 || p.tx > nx || p.ty > ny || p.tz > nz) return false;
    if (p.steps < 2 || p.steps > kTileMaxSteps || p.block < 64 || p.block > 1024 || p.block % 64 != 0) return false;
    if (L.D == 2 && nz != 1) return false;
    const int64_t n[3] = {nx, ny, nz};
    for (int a = 0; a < L.D; ++a)
        if (n[a] > 2 && p.steps - 1 > n[a]) return false;
    if (p.tx > 1024 || p.ty > 1024 || p.tz > 1024) return false;
    if (tile_region(L, p, nx, p.steps) * L.Q * elem > kTileMaxLds) return false;
    if (tile_region(L, p, nx, p.steps - 1) > p.block) return false;
    const int64_t limit = int64_t(1) << 32;
    if (nx > limit / (L.Q * elem) / ny / nz) return false;
    return true;
}

// Whether a fitting plan is expected to be faster than the one-site step
// (host.hpp, tile_plan).
static bool tile_pays(const LatticeInfo& L, int64_t nx, int64_t ny, int64_t nz, int64_t cus, const TilePlan& p)
{
    const int64_t tiles = ((nx + p.tx - 1) / p.tx) * ((ny + p.ty - 1) / p.ty) * ((nz + p.tz - 1) / p.tz);
    int64_t rounds = 0;  // of a tile over all its steps
    for (int s = p.steps; s >= 1; --s) rounds += (tile_region(L, p, nx, s) + 255) / 256;
    if (L.D == 3) return p.tx == nx && (tiles + cus - 1) / cus * rounds <= kTileRounds3d;
    return tiles <= cus || ny > 1;
}

bool tile_plan(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, int cus, TilePlan* out)
{
    if (L.R != 1 || nx < 1 || ny < 1 || nz < 1 || cus < 1) return false;
    if (nx > kMaxSites / ny / nz) return false;
    const int64_t share = nx * ny * nz / cus;  // sites of a compute unit
    TilePlan p{1, 1, 1, 0, 0};
    if (L.D == 2) {
        if (storage_bytes(dtype) == 2 && share > kTileShare16) return false;
        // a tile per compute unit while the box is small, then 32 x 16
        p.tx = even_piece(nx, share <= 32 ? 8 : share <= 128 ? 16 : 32);
        p.ty = even_piece(ny, share <= 32 ? 4 : share <= 256 ? 8 : 16);
        p.steps = share <= 256 ? 8 : 5;
    } else {
        if (share > kTileShare3d) return false;
        p.tx = even_piece(nx, 64);
        while (int64_t(p.tx) * p.ty * p.tz < share) {
            int& side = p.ty <= p.tz ? p.ty : p.tz;
            if (2 * side > (p.ty <= p.tz ? ny : nz)) break;
            side *= 2;
        }
        p.steps = share <= 32 ? 3 : 2;
    }
    // fewer steps where the box is narrower than the ring, LDS too small or the
    // rings cost too much
    for (; p.steps >= 2; --p.steps) {
        const int64_t n = tile_region(L, p, nx, p.steps);
        const int64_t rounds = (n + 1023) / 1024;
        const int64_t least = tile_region(L, p, nx, p.steps - 1);
        const int64_t threads = std::max(least, (n + rounds - 1) / rounds);
        p.block = int(std::min<int64_t>(1024, (threads + 63) / 64 * 64));
        if (tile_plan_fits(L, dtype, nx, ny, nz, p) && tile_pays(L, nx, ny, nz, cus, p)) {
            *out = p;
            return true;
        }
    }
    return false;
}

bool tile_default(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, const TilePlan& p)
{
    if (L.D == 2 || dtype != 0 || p.steps > 2) return true;
    const int64_t region = tile_region(L, p, nx, p.steps);
    if (region <= 4 * p.tx * p.ty * p.tz) return true;
    const int64_t tiles = ((nx + p.tx - 1) / p.tx) * ((ny + p.ty - 1) / p.ty) * ((nz + p.tz - 1) / p.tz);
    return tiles * region * L.Q * 8 <= kTileRingLoads;
}

uint64_t geometry_hash(const std::vector<int64_t>& dims)
{
    uint64_t x = 1469598103934665603ULL;  // FNV-1a over the dims
    for (int64_t d : dims) {
        for (int k = 0; k < 8; ++k) {
            x ^= uint64_t((d >> (8 * k)) & 0xff);
            x *= 1099511628211ULL;
        }
    }
    return x;
}

bool check_checkpoint(const void* buf, size_t bytes, const CkptHeader& expect, std::string* why)
{
    if (!buf || bytes < sizeof(CkptHeader) + expect.payload_bytes) {
        char msg[128];
        snprintf(msg, sizeof(msg), "checkpoint buffer needs %zu bytes", size_t(sizeof(CkptHeader) + expect.payload_bytes));
        *why = msg;
        return false;
    }
    CkptHeader hd;
    std::memcpy(&hd, buf, sizeof(hd));
    if (hd.magic != kCkptMagic) {
        *why = "not a checkpoint written by lbm_get_state";
        return false;
    }
    if (hd.lattice != expect.lattice || hd.dtype != expect.dtype || hd.K != expect.K || hd.nbox != expect.nbox ||
        hd.nsites != expect.nsites || hd.geometry_hash != expect.geometry_hash ||
        hd.payload_bytes != expect.payload_bytes) {
        *why = "checkpoint does not match this handle (lattice, dtype, K or geometry)";
        return false;
    }
    if (hd.t < 0) {
        *why = "checkpoint has a negative time";
        return false;
    }
    return true;
}

void relayout_host(const LatticeInfo& L, int64_t nx, int64_t ny, int64_t nz, size_t elem, int layout,
                   bool to_natural, const char* src, char* dst)
{
    const int64_t tile = int64_t(L.Q) * nx;
    auto wrap = [](int64_t v, int64_t n) { return ((v % n) + n) % n; };
    for (int j = 0; j < L.Q; ++j) {
        const int jo = (j == 0) ? 0 : ((j & 1) ? j + 1 : j - 1);
        int64_t o[3];
        for (int a = 0; a < 3; ++a) {
            const int c = L.c[j * 3 + a];
            o[a] = (layout == kSwapped) ? c : (layout == kNatural ? 0 : (c > 0 ? c : 0));
        }
        const int64_t r = (layout == kNatural || layout == kTwistEven) ? L.mrow[j] : L.mrow[jo];
        for (int64_t z = 0; z < nz; ++z)
            for (int64_t y = 0; y < ny; ++y) {
                const int64_t zs = wrap(z + o[2], nz), ys = wrap(y + o[1], ny);
                const int64_t lay_row = (zs * ny + ys) * tile + r * nx;
                const int64_t nat_row = (z * ny + y) * tile + int64_t(L.mrow[j]) * nx;
                for (int64_t x = 0; x < nx; ++x) {
                    const int64_t xs = wrap(x + o[0], nx);
                    if (to_natural) std::memcpy(dst + (nat_row + x) * elem, src + (lay_row + xs) * elem, elem);
                    else std::memcpy(dst + (lay_row + xs) * elem, src + (nat_row + x) * elem, elem);
                }
            }
    }
}

bool tune_cache_lookup(const char* path, const std::string& key, LaunchChoice* out)
{
    if (!path || !*path) return false;
    std::ifstream in(path);
    std::string line;
    bool found = false;
    while (std::getline(in, line)) {
        const size_t bar = line.find(" | ");
        if (bar == std::string::npos || line.compare(0, bar, key) != 0 || bar != key.size()) continue;
        std::istringstream rest(line.substr(bar + 3));
        LaunchChoice c;
        if (rest >> c.kernel >> c.block >> c.grid) {
            *out = c;  // the last entry for a key wins
            found = true;
        }
    }
    return found;
}

void tune_cache_store(const char* path, const std::string& key, const LaunchChoice& c)
{
    if (!path || !*path) return;
    // a last line without its newline (a write cut short, an edit) must not
    // swallow the new entry
    bool newline = false;
    {
        std::ifstream in(path, std::ios::binary | std::ios::ate);
        if (in && in.tellg() > 0) {
            in.seekg(-1, std::ios::end);
            char last = '\n';
            newline = in.get(last) && last != '\n';
        }
    }
    std::ofstream out(path, std::ios::app);
    if (newline) out << "\n";
    out << key << " | " << c.kernel << " " << c.block << " " << c.grid << "\n";
}

}  // namespace lbm
