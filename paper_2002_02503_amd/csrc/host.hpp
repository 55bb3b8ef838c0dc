// Host-only parts of the library, free of any HIP call or type: lattice
// tables, argument checks, the checkpoint header, rearrangement of a state
// between its layouts, and the tune cache.  Used by the C-ABI implementation
// (api.hip); plain C++, so it also builds with the host compiler alone (the
// sanitizer test builds it with AddressSanitizer and UBSan on the CPU).
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace lbm {

// Where a single box's populations are, as the step kernels leave them.
//   kNatural:   population i of site x in its own row tile, tile row m(i)
//               (every batch, and the two-buffer single-box steps);
//   kSwapped:   at site x + c_i, tile row m(opp(i)) (k_step_ip after an odd
//               number of its steps);
//   kTwistEven: at site x + b_i, b_i the positive part of c_i, tile row m(i)
//               (k_step_tw after an even number of its steps);
//   kTwistOdd:  at site x + b_i, tile row m(opp(i)) (k_step_tw, odd).
enum StateLayout : int { kNatural = 0, kSwapped = 1, kTwistEven = 2, kTwistOdd = 3 };

// Host copy of a lattice's tables (from the compile-time descriptors).
struct LatticeInfo {
    int D, Q, two_n, k_default, k_max, R;
    double T0;
    std::vector<int> c;     // Q * 3
    std::vector<double> w;  // Q
    std::vector<int> mrow;  // Q: tile row m(i) of population i
};
bool lattice_info(int lat, LatticeInfo* out);

// Bytes per stored population of a dtype code (8, 4, 2, 2), 0 if unknown.
size_t storage_bytes(int dtype);

// Limits of the addressing, checked before anything else happens.
constexpr int64_t kMaxSites = int64_t(1) << 36;  // total sites: keeps chunk and tile counts in int
constexpr int kBlockSites = 64;                  // sites per block of a batched box's layout (one wave)

// Output tile of the two-step kernel (step2.hpp): kTwoStepTileX x
// two_step_tile_y(elem) sites of a z-plane per block, which also computes the
// one-site ring around them in its first step.  8-byte storage takes half the
// rows, so that the kernel's two LDS planes (2 Q (TX + 2)(TY + 2) values)
// stay within a compute unit's 160 KiB.  (Measured on D3Q19 256^3: 64 x 8
// tiles ran 8.5% faster than 32 x 16 in FP32, and 64 x 4 9% faster than 32 x 8
// in FP64: the ring costs more arithmetic, but each population row's ring
// cache lines are shared by twice as many sites.)
constexpr int kTwoStepTileX = 64;
constexpr int two_step_tile_y(size_t elem) { return elem == 8 ? 4 : 8; }

// Threads of its blocks: whole waves for the tile and its ring.
constexpr int two_step_threads(size_t elem)
{
    return ((kTwoStepTileX + 2) * (two_step_tile_y(elem) + 2) + 63) / 64 * 64;
}

// Threads of a block of the batched two-step kernel (step2_batch.hpp).  FP64:
// what its two LDS planes leave room for (448 threads: 756 against 720 us per
// step of 256 boxes of sides 16-64, 17.6 million sites, 4 rounds).  Else 704:
// 1024 would fit too, but ran at 360 us against 351 (8 rounds).
constexpr int batch_columns_threads(size_t elem) { return elem == 8 ? 512 : 704; }

// Whether the two-step kernel applies to a single nx x ny x nz box: a 3-D
// lattice whose velocity components are at most 1 in magnitude (a one-site
// ring), nx and ny multiples of the tile, and one z-plane of populations
// (Q nx ny values) below 2 GiB, since offsets inside a plane are formed in
// 32 bits.
bool two_step_fits(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz);

// The same kernel on columns of any size ("columns"): the lattice and the plane
// limit alone.
bool columns_fit(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz);

// Column tile of the two-step kernel for a box: 64 x two_step_tile_y where nx
// is a multiple of 64; else x in even pieces of at most 128, since rows that
// do not start on a cache line pay for partly used lines at both ends of a
// piece, and as many rows as the block's threads hold.  A piece leaves room for
// two rows at least (110 sites at most in FP64, where 111 to 128 left one):
// step 1 takes three sites for each site of a single row, two for two.
// Measured, us per step (tile): D3Q19 FP32 201 x 150 x 77 54 (101 x 4), 62 (67 x
// 8), 71 (51 x 11); 100^3 21 (100 x 4), 29 (50 x 10), 33 (34 x 17); 255^3 363 (128 x 3), 411 (64 x
// 8); 160^3 83 (80 x 6 and 160 x 2), 93 (32 x 18); FP64 100^3 38 (100 x 2), 44
// (50 x 6), 120^3 69 (60 x 5), 84 (120 x 1), 240^3 589 (80 x 3), 912 (120 x 1;
// one-site step 706), 255^3 542 (85 x 3), 689 (128 x 1).  FP64 rows of whole lines
// whose pieces would start elsewhere are cut once more where that mends it: 224^3
// 490 (56 x 5), 594 (75 x 3; one-site step 573), 400 x 200 x 100 350 (80 x 3), 442
// (100 x 2).
void column_tile(size_t elem, int64_t nx, int64_t ny, int* tx, int* ty);

// Rounds of a compute unit's four SIMDs that a plane of a column tile takes:
// waves of step 1 and of step 2, four at a time.
constexpr int column_rounds1(int tx, int ty) { return ((tx + 2) * (ty + 2) + 255) / 256; }
constexpr int column_rounds(int tx, int ty) { return column_rounds1(tx, ty) + (tx * ty + 255) / 256; }

// What a plane costs a block of the batched two-step kernel, in rounds: four at
// least, since the latency of a plane's loads and collisions shows when its
// lanes are fewer.  With the bare rounds the blocks that got the small boxes of a
// mixed batch ended last, after one-site steps were done (us per step, one-site,
// bare rounds and these: 47 D3Q19 FP32 boxes of sides 12-56 47, 55 and 44, 159
// D3Q15 of 11-39 47, 59 and 45; in FP64 the latter 93, 85 and 70).
constexpr int column_plane_cost(int tx, int ty)
{
    return column_rounds(tx, ty) < 4 ? 4 : column_rounds(tx, ty);
}

// Column tile of the batched two-step kernel: x in even pieces of at most 128
// (126 in FP64, for two rows: 30 boxes of 128 x 128 x 8 173 us per step, 227 with
// one), and the rows that take the fewest rounds over the box, since the busiest
// SIMD sets the time of a plane.
void batch_column_tile(size_t elem, int64_t nx, int64_t ny, int* tx, int* ty);

// Whether the default for a single box is the two-step kernel, rather than the
// one-site step: large boxes, in 16-bit storage only where rows are not whole
// cache lines.
// Two-step against one-site, us per step of D3Q19 FP32: tiles of 64 columns 64^3
// 7.3 / 8.5, 128^3 36 / 53, 256^3 248 / 422; other tiles 65^3 12.0 / 12.0,
// 80^3 13 / 17, 100^3 17.4 / 35, 201 x 150 x 77 54 / 76, 255^3 363 / 646, FP64 100^3
// 38 / 59.  In 16-bit storage on rows of whole lines both are bound by instruction
// issue and nothing is gained (FP16 128^3 26.4 / 26, 256^3 209 / 206; also where ny
// is no multiple of the tile: BF16 128 x 130 x 130 36 / 30); on others D3Q19 needs
// more sites (BF16 101^3 26 / 24, 130^3 43 / 50, FP16 201 x 150 x 77 41 / 48) and D3Q15
// does not gain (BF16 130^3 39 / 35); nor do large states with rows of whole 32-byte
// sectors that fill four fifths of the one-site step's lanes (BF16 160^3 74 / 64,
// 240^3 285 / 244, but 208 x 120 x 120 50 / 54 and 400 x 200 x 100 163 / 180).  A box
// of one layer or of few rows computes the ring for nothing: 1024 x 1024 x 1 37 / 28, 1000 x 1 x 1000 36 / 32, 100000 x 2 x 2
// 18 / 13, but 512 x 512 x 2 13.9 / 15.6 and 1000 x 2 x 500 24 / 32.
// Few planes: a column adds two planes of step 1, and a cut between blocks two
// more.  Other tiles than the whole 64-column ones gain from three planes on in
// FP32 (1000 x 1000 x 2 69 / 65, x 3 90 / 98), from four on rows of whole lines (1024 x
// 300 x 3 26.7 / 25.2, x 4 31.5 / 32.9), in FP64 from four on where the state is past
// the caches (1000 x 1000 x 3 187 / 168, x 4 222 / 224, 700 x 700 x 3 85 / 95), in 16-bit
// storage from about twelve (BF16 1000 x 1000 x 4 98 / 81, 700 x 700 x 5 58 / 54, 500 x
// 500 x 10 49 / 52).
// A column of few sites leaves the latency of its planes open: below 256 sites
// only boxes of short rows gain, which leave most lanes of the one-site step idle;
// in FP64 columns of 16 sites do (two-step / one-site: FP32 4 x 4 x 30000 105 / 61, 8 x
// 8 x 10000 54 / 44, 64 x 3 x 2188 14.4 / 13.2, 64 x 5 x 1313 12.1 / 13.2, 16 x 8 x 3282
// 21.6 / 17.8, 16 x 16 x 1641 15.0 / 17.5, 10 x 20 x 2101 22 / 26; BF16 30 x 3 x 22778 122 /
// 48, 7 x 20 x 14643 104 / 141; FP64 3 x 3 x 60000 207 / 205, 4 x 4 x 30000 109 / 138).
constexpr int64_t kTwoStepSites = 64 * 64 * 64;
constexpr int64_t kColumnsSites = 400000;
constexpr int64_t kColumnsSites16 = 2000000;  // D3Q19 in 16-bit storage
constexpr int64_t kColumnsState16 = int64_t(128) << 20;  // bytes: both buffers past the Infinity Cache
constexpr int64_t kColumnsRows = 64;          // x-rows
constexpr int kColumnsLeast = 256;            // sites of a column
constexpr int kColumnsLeast64 = 16;           // in FP64
constexpr int64_t kColumnsThin64 = 1500000;   // sites of an FP64 state in the caches
bool columns_pay(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz);

// Whether the default for a batch is the two-step kernel: FP32 and FP64 batches
// large enough in all and box by box, whose planes fill the blocks and whose
// columns are not all ring.  D3Q19, us per step, one-step against two-step: 256
// boxes of sides 16-64 FP32 437 / 347 (17.2 million sites) and FP64 778 / 581
// (15.4), 24-40 FP32 215 / 181, 16-32 93 / 89, 8-24 31 / 43; 16 boxes of 16-64
// (820,000 sites) 24 / 20; 16-bit storage is bound by instruction issue (256
// boxes of 32-64 BF16 369 / 496).
// The shapes go by the rounds that the columns take over two steps, ring and the
// two extra step-1 planes of a column included, against the two rounds of 256
// sites: up to 1.8 times as many in FP32, where a plane counts four rounds at
// least (fewer lanes leave its latency open), up to 2 in FP64.  One-step against
// two-step, (times as many): FP32 boxes of 48^3 177 / 119 (1.36), 100 x 100 x 10
// 101 / 92 (1.79), 300 x 300 x 8 147 / 153 (1.84), 16 x 16 x 400 153 / 161 (2.0),
// 1000 x 1000 x 1 201 / 433 (3.8), 4 x 4 x 5000 120 / 1136 (32); FP64 24^3 180 / 121
// (1.85), 200 x 200 x 6 196 / 182 (2.0), 20000 x 4 x 4 665 / 897 (2.05), 4 x 4 x 5000
// 251 / 1206 (16).
constexpr int64_t kBatchColumnsSites = 700000;
constexpr int64_t kBatchColumnsMean = 24 * 24 * 24;
bool batch_columns_pay(const LatticeInfo& L, int dtype, int nbox, const int64_t* dims);

constexpr int kTileMaxSteps = 16;
constexpr int64_t kTileMaxLds = 160 * 1024;  // a compute unit's LDS

// Plan of the tile kernel (step_tile.hpp): tile tx x ty x tz, `steps` steps a
// launch, blocks of `block` threads.
struct TilePlan {
    int tx, ty, tz, steps, block;
};

// Sites of step 1's region of a full tile, for `steps` steps (no ring in x when
// the tile holds whole x-rows).
int64_t tile_region(const LatticeInfo& L, const TilePlan& p, int64_t nx, int steps);

// Whether the plan runs on an nx x ny x nz box: a one-site ring per step, the
// region of step 1 in LDS, that of step 2 with one thread per site, ring
// coordinates within one period of the box (any for one and two sites) and
// the state below 4 GiB (offsets are formed in 32 bits).
bool tile_plan_fits(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, const TilePlan& p);

// The plan for a box on a device of `cus` compute units; false: none, because
// none fits or the one-site step is faster.
//   - D2Q9: every size, but in 16-bit storage, whose steps are bound by
//     instruction issue, only up to kTileShare16 sites per compute unit, and
//     with more tiles than units not for a single row (100000 sites: 2.9 us per
//     step one-site, 3.6 tiled; two rows of them 5.9 and 4.9).  Measured, us per
//     step, one-site against the plan (tile, steps): 64^2 FP64 2.52 / 0.96 (8 x 4, 8), 256^2 FP32 3.29 / 1.65 (32 x 8,
//     8), 601 x 400 FP32 5.9 / 3.2 (32 x 16, 5), 1024^2 FP32 14.4 / 8.0 and
//     FP64 26.5 / 10.4 (32 x 16, 5), 4096^2 FP32 190 / 121; BF16 1024^2 9.1 / 9.9.
//   - D3Q15 and D3Q19: up to kTileShare3d sites per compute unit.  The ring
//     costs more in three dimensions, so two steps (three up to 32 sites per
//     unit) and whole x-rows, whose loads use full lines: 16^3 FP32 3.09 / 1.91
//     (16 x 2 x 1, 3), 32^3 FP32 3.64 / 2.85 (32 x 2 x 2, 2), FP64 4.48 / 3.86,
//     8 x 64 x 64 6.3 / 2.9; at 64^3 (8.5 / 8.4) and above nothing is gained.  A
//     compute unit's SIMDs take at most kTileRounds3d rounds of four waves over
//     the steps, and rows are whole: 200 x 200 x 1 (8 rounds) 3.8 / 5.2, 40000 x 1 x
//     1 (12) 3.1 / 5.4, 33^3 (6) 4.3 / 4.1, 300 x 10 x 10 (4, rows in pieces) 3.9 / 4.2.
// Block: step 1's region in as few rounds as 1024 threads allow (32^3 with the
// threads that step 2 needs, 128, took 4.0 us per step).
constexpr int64_t kTileShare3d = 160;
constexpr int64_t kTileRounds3d = 4;
constexpr int64_t kTileShare16 = 1024;
bool tile_plan(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, int cus, TilePlan* out);

// Whether a box with a plan takes it by default.  In FP64, where a site's values
// are twice as long, a two-step launch whose first step reads more than four
// times the tile loses once those loads pass 8 MB: us per step, one-site against the
// plan, D3Q19 64 x 10 x 24 (64 x 1 x 1 tiles, 21 MB) 3.82 / 4.37, 41 x 115 x 4 (41 x 2 x 1,
// 17 MB) 4.30 / 4.67, 64 x 4 x 23 (8.1 MB) 3.28 / 3.34, 64 x 7 x 8 (4.9 MB) 3.18 / 3.15, 42 x
// 10 x 10 (5.7 MB) 3.42 / 3.03; with at most four times, 32^3 (20 MB) 4.48 / 3.86;
// three-step launches gain (17 x 17 x 20 3.46 / 2.36).
constexpr int64_t kTileRingLoads = int64_t(8) << 20;
bool tile_default(const LatticeInfo& L, int dtype, int64_t nx, int64_t ny, int64_t nz, const TilePlan& p);

// The argument checks of lbm_create / lbm_create_batch for nbox boxes
// (dims: nbox * 3, tau: nbox).  True when every box is valid; otherwise false
// with the reason in *why.
bool check_boxes(const LatticeInfo& L, int dtype, int nbox, const int64_t* dims, const double* tau, std::string* why);

// FNV-1a hash of the box dimensions (checkpoint header, tune-cache key).
uint64_t geometry_hash(const std::vector<int64_t>& dims);

// The 64-byte header in front of a checkpoint's raw populations.
constexpr uint64_t kCkptMagic = 0x314b4350434d424cULL;  // "LBMCPCK1"
struct CkptHeader {
    uint64_t magic;
    int32_t lattice, dtype, K, nbox;
    int64_t nsites, t;
    uint64_t geometry_hash;
    uint64_t payload_bytes;
    uint64_t reserved;  // keeps the header 64 bytes, so the payload is 64-byte aligned
};
static_assert(sizeof(CkptHeader) == 64, "checkpoint header layout");

// Check a checkpoint of `bytes` bytes at `buf` against the header a handle
// would write (`expect`, t ignored).  True when it matches; otherwise false
// with the reason in *why.  Reads at most sizeof(CkptHeader) bytes of buf.
bool check_checkpoint(const void* buf, size_t bytes, const CkptHeader& expect, std::string* why);

// Rearrange a single box's state (row tiles, nx * ny * nz sites, elem bytes
// per value) between `layout` and the natural layout: to_natural reads src in
// `layout` and writes dst natural; otherwise the reverse.  src and dst hold
// Q * nx * ny * nz values each and do not overlap.
void relayout_host(const LatticeInfo& L, int64_t nx, int64_t ny, int64_t nz, size_t elem, int layout,
                   bool to_natural, const char* src, char* dst);

// Tune cache: a text file of lines "<key> | <kernel> <block> <grid>".
struct LaunchChoice {
    int kernel, block, grid;
};
// The last entry for `key` in the file at `path` (NULL or "" : none).
bool tune_cache_lookup(const char* path, const std::string& key, LaunchChoice* out);
void tune_cache_store(const char* path, const std::string& key, const LaunchChoice& c);

}  // namespace lbm
