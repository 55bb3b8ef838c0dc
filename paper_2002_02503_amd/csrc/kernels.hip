// HIP kernels for gfx950 (MI355X) around the step: initialisation, moments,
// FP64 reductions and a copy kernel used to calibrate bandwidth measurements.
// The step kernels are in step.hpp (single box) and step_batch.hpp (batch).
//
// Data layout: blocked structure of arrays, row tiles for a single box and
// 64-site blocks for a batch (see internal.hpp, BoxDesc).  Two buffers
// alternate: a step reads one and writes the other, so a step never reads what
// it writes.  The stored value is G_i = S (f_i - w_i), the deviation from the
// rest weights in units of the lattice's weight quantum 1/S.
//
// The step is bandwidth bound (about 400 single-precision operations against
// 2 Q S bytes per site, far below the FP32 ridge of the chip), so it uses no
// matrix cores: every population is read once (pull form of eq. lbe, periodic
// wrap) and written once, and the collision runs entirely in registers.
#include <algorithm>

#include "device.hpp"
#include "step_launch.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// Set-up, moments and reductions work on chunks: runs of consecutive sites
// of one box.  The reductions take one block per chunk; set-up and moments one
// thread per site, `slices` blocks per chunk.
// ---------------------------------------------------------------------------

// Blocks run through the slices of a chunk before the next chunk, so those at
// work at a time are neighbours in memory: cut into chunks first, D3Q19 moments
// took, us a call within a run of steps, 333 against 281 (256^3 FP32), 221 against
// 185 (FP16) and, in a batch of 500 boxes of 40^3, whose boxes share the lines of
// their fields, 430 against 353 (FP16).  A row of the grid holds kGridChunks
// chunks, so that no dimension comes near 2^32 threads.
constexpr int kGridChunks = 32768;

static dim3 chunk_grid(int nchunks, unsigned slices)
{
    return dim3(slices * unsigned(std::min(nchunks, kGridChunks)),
                unsigned((nchunks + kGridChunks - 1) / kGridChunks));
}

__device__ __forceinline__ int block_chunk(unsigned slices)
{
    return int(blockIdx.y) * kGridChunks + int(blockIdx.x / slices);
}

__device__ __forceinline__ int block_site(unsigned slices)
{
    return int(blockIdx.x % slices) * int(blockDim.x) + int(threadIdx.x);
}

// Place of site k of a chunk: its block (for a single box its x-row) and its
// position there, and for a single box y and z.  The chunk carries its first
// site's place, so 32-bit divisions of x0 + k suffice (a 64-bit division of
// the site index took some 100 instructions).
struct SitePos {
    long long row;
    int x, y, z;
};

template <bool COORDS>
__device__ __forceinline__ SitePos locate(const ChunkDesc& ch, int k, const BoxDesc& b)
{
    const unsigned xx = unsigned(ch.x0) + unsigned(k);
    const unsigned q = xx / unsigned(b.w);
    SitePos p;
    p.row = ch.row0 + q;
    p.x = int(xx - q * unsigned(b.w));
    p.y = p.z = 0;
    if constexpr (COORDS) {
        const unsigned yy = unsigned(ch.y0) + q;
        const unsigned dz = yy / unsigned(b.ny);
        p.y = int(yy - dz * unsigned(b.ny));
        p.z = ch.z0 + int(dz);
    }
    return p;
}

// Element of population 0 of a site in the natural layout (blocks of w sites,
// BoxDesc); population i is m(i) * w further on.
template <int Q>
__device__ __forceinline__ long long site_elem(const SitePos& p, int w)
{
    return p.row * Q * w + p.x;
}

// A site's wrapped neighbour coordinates, x + k - R at [k].
template <class L>
struct Around {
    int x[2 * L::R + 1], y[2 * L::R + 1], z[2 * L::R + 1];

    __device__ __forceinline__ Around(const SitePos& p, const BoxDesc& b)
    {
#pragma unroll
        for (int k = 0; k <= 2 * L::R; ++k) {
            x[k] = wrap_coord(p.x + k - L::R, b.nx);
            y[k] = wrap_coord(p.y + k - L::R, b.ny);
            z[k] = wrap_coord(p.z + k - L::R, b.nz);
        }
    }
};

// Element of population I of a site of a single box (row tiles, w = nx) when
// the state is in layout LAYOUT (StateLayout, internal.hpp): swapped: cell
// x + c_i, tile row m(opp(i)); twisted: cell x + b_i (b_i the positive part of
// c_i), tile row m(i) at even times and m(opp(i)) at odd times.
template <class L, int LAYOUT, int I>
__device__ __forceinline__ long long layout_elem(const Around<L>& at, const BoxDesc& b)
{
    const long long tile = (long long)L::Q * b.nx;
    constexpr bool SW = (LAYOUT == kSwapped);
    constexpr int ox = L::R + (SW ? L::c[I][0] : twist_offset<L>(I, 0));
    constexpr int oy = L::R + (SW ? L::c[I][1] : twist_offset<L>(I, 1));
    constexpr int oz = L::R + (SW ? L::c[I][2] : twist_offset<L>(I, 2));
    constexpr int m = (LAYOUT == kTwistEven) ? mem_row<L>(I) : mem_row<L>(opp(I));
    return ((long long)at.z[oz] * b.ny + at.y[oy]) * tile + (long long)m * b.nx + at.x[ox];
}

// Initialisation: f := f^eq_K(rho, u) (eq. hermite), evaluated in double and
// rounded once to the storage type (set-up, not part of the step), written in
// the natural layout or (single box) the twisted layout of an even time.
template <class L, class S, int K, int LAYOUT>
__global__ __launch_bounds__(256) void k_init(const double* __restrict__ rho, const double* __restrict__ u,
                                              S* __restrict__ dst, const ChunkDesc* __restrict__ chunks,
                                              const BoxDesc* __restrict__ boxes, long long nsites, int nchunks,
                                              unsigned slices)
{
    using ST = Store<S>;
    static_assert(LAYOUT == kNatural || LAYOUT == kTwistEven, "init writes a layout of time 0");
    const int c = block_chunk(slices);
    if (c >= nchunks) return;
    const ChunkDesc ch = chunks[c];
    const BoxDesc b = boxes[ch.box];
    S* base = dst + b.mem;
    const int k = block_site(slices);
    if (k >= ch.count) return;
    const long long s = ch.start + k;
    const SitePos pos = locate<LAYOUT != kNatural>(ch, k, b);
    const double ux = u[s];
    const double uy = u[nsites + s];
    const double uz = (L::D == 3) ? u[2 * nsites + s] : 0.0;
    double g[L::Q];
    equilibrium_scaled<L, K>(rho[s] - 1.0, ux, uy, uz, g);
    if constexpr (LAYOUT == kNatural) {
        S* q = base + site_elem<L::Q>(pos, b.w);
        unroll<L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            ST::put_d(q + (long long)mem_row<L>(i) * b.w, g[i]);
        });
    } else {
        const Around<L> at(pos, b);
        unroll<L::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            ST::put_d(base + layout_elem<L, LAYOUT, i>(at, b), g[i]);
        });
    }
}

// rho - 1 and rho u (eq. mme) of one stored site, in double (outside the
// step, for output and reductions).  `p` points at population 0 of the site,
// w is the block width of the box's layout.
template <class L, class S, int READ>
__device__ __forceinline__ void site_moments(const S* __restrict__ p, int w, double& dsum, double (&j)[3])
{
    using ST = Store<S>;
    dsum = 0.0;
    j[0] = j[1] = j[2] = 0.0;
    unroll<L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
        constexpr int m = mem_row<L>(i);
        const S* q = p + (long long)m * w;
        const double gi = double(READ == kStreamAll ? ST::get_nt(q) : ST::get(q));
        dsum += gi;
        if constexpr (cx != 0) j[0] += double(cx) * gi;
        if constexpr (cy != 0) j[1] += double(cy) * gi;
        if constexpr (cz != 0) j[2] += double(cz) * gi;
    });
    // stored units are 1/S of a population
    dsum = over<L::S>(dsum);
    j[0] = over<L::S>(j[0]);
    j[1] = over<L::S>(j[1]);
    if constexpr (L::D == 3) j[2] = over<L::S>(j[2]);
}

// The same for a single box whose state is in one of the in-place steps'
// layouts (layout_elem).
template <class L, class S, int LAYOUT>
__device__ __forceinline__ void relaid_site_moments(const S* __restrict__ base, const SitePos& pos, const BoxDesc& b,
                                                    double& dsum, double (&j)[3])
{
    using ST = Store<S>;
    const Around<L> at(pos, b);
    dsum = 0.0;
    j[0] = j[1] = j[2] = 0.0;
    unroll<L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
        const double gi = double(ST::get(base + layout_elem<L, LAYOUT, i>(at, b)));
        dsum += gi;
        if constexpr (cx != 0) j[0] += double(cx) * gi;
        if constexpr (cy != 0) j[1] += double(cy) * gi;
        if constexpr (cz != 0) j[2] += double(cz) * gi;
    });
    dsum = over<L::S>(dsum);
    j[0] = over<L::S>(j[0]);
    j[1] = over<L::S>(j[1]);
    if constexpr (L::D == 3) j[2] = over<L::S>(j[2]);
}

template <class L, class S, int LAYOUT, int READ>
__device__ __forceinline__ void stored_site_moments(const S* __restrict__ base, const ChunkDesc& ch, int k,
                                                    const BoxDesc& b, double& dsum, double (&j)[3])
{
    const SitePos pos = locate<LAYOUT != kNatural>(ch, k, b);
    if constexpr (LAYOUT != kNatural) relaid_site_moments<L, S, LAYOUT>(base, pos, b, dsum, j);
    else site_moments<L, S, READ>(base + site_elem<L::Q>(pos, b.w), b.w, dsum, j);
}

// Bound by HBM.  D3Q19 256^3 from the natural layout, us a call within a run of
// steps, FP32 / FP16 / FP64: 290 / 188 / 490 with the state and the fields touched
// non-temporally, 331 / 216 / 577 with the default policy.  The in-place layouts,
// whose cells are shared between sites, keep the default policy.
template <class L, class S, int LAYOUT, int READ>
__global__ __launch_bounds__(256) void k_moments(const S* __restrict__ src, double* __restrict__ rho,
                                                 double* __restrict__ u, const ChunkDesc* __restrict__ chunks,
                                                 const BoxDesc* __restrict__ boxes, long long nsites, int nchunks,
                                                 unsigned slices)
{
    const int c = block_chunk(slices);
    if (c >= nchunks) return;
    const ChunkDesc ch = chunks[c];
    const BoxDesc b = boxes[ch.box];
    const S* base = src + b.mem;
    const int k = block_site(slices);
    if (k >= ch.count) return;
    const long long s = ch.start + k;
    double d, j[3];
    stored_site_moments<L, S, LAYOUT, READ>(base, ch, k, b, d, j);
    const double r = 1.0 + d;
    auto put = [](double* q, double v) {
        if constexpr (READ != kReadCached) __builtin_nontemporal_store(v, q);
        else *q = v;
    };
    put(rho + s, r);
#pragma unroll
    for (int a = 0; a < L::D; ++a) put(u + a * nsites + s, j[a] / r);
}

// ---------------------------------------------------------------------------
// FP64 reductions with a fixed order: per-chunk partials (one block per
// chunk, LDS tree), then per-box (or global) sums over chunks in order.  Bound
// by HBM (api.hip, read_policy, on the loads).
// ---------------------------------------------------------------------------

constexpr int kRedBlock = 256;

template <int NV>
__device__ __forceinline__ void block_tree(double (&acc)[NV], const bool (&is_max)[NV])
{
    __shared__ double sh[NV][kRedBlock];
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 0; k < NV; ++k) sh[k][tid] = acc[k];
    __syncthreads();
    for (int off = kRedBlock / 2; off > 0; off >>= 1) {
        if (tid < off) {
#pragma unroll
            for (int k = 0; k < NV; ++k)
                sh[k][tid] = is_max[k] ? fmax(sh[k][tid], sh[k][tid + off]) : sh[k][tid] + sh[k][tid + off];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = sh[k][0];
}

template <class L, class S, int LAYOUT, int READ>
__global__ __launch_bounds__(kRedBlock) void k_totals_partial(const S* __restrict__ src,
                                                              const ChunkDesc* __restrict__ chunks,
                                                              const BoxDesc* __restrict__ boxes,
                                                              double* __restrict__ partial)
{
    const ChunkDesc ch = chunks[blockIdx.x];
    const BoxDesc b = boxes[ch.box];
    const S* base = src + b.mem;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = threadIdx.x; k < ch.count; k += kRedBlock) {
        double d, j[3];
        stored_site_moments<L, S, LAYOUT, READ>(base, ch, k, b, d, j);
        acc[0] += d;
        acc[1] += j[0];
        acc[2] += j[1];
        acc[3] += j[2];
    }
    const bool is_max[4] = {false, false, false, false};
    block_tree<4>(acc, is_max);
    if (threadIdx.x == 0) {
        partial[blockIdx.x * 4 + 0] = double(ch.count) + acc[0];  // sum rho = sites + sum (rho - 1)
        partial[blockIdx.x * 4 + 1] = acc[1];
        partial[blockIdx.x * 4 + 2] = acc[2];
        partial[blockIdx.x * 4 + 3] = acc[3];
    }
}

__global__ __launch_bounds__(kRedBlock) void k_totals_final(const double* __restrict__ partial,
                                                            const int* __restrict__ box_chunk_begin,
                                                            double* __restrict__ out)
{
    const int b = blockIdx.x;
    const int c0 = box_chunk_begin[b], c1 = box_chunk_begin[b + 1];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c = c0 + int(threadIdx.x); c < c1; c += kRedBlock)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += partial[c * 4 + k];
    const bool is_max[4] = {false, false, false, false};
    block_tree<4>(acc, is_max);
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) out[b * 4 + k] = acc[k];
}

template <class L, class S, int LAYOUT, int READ>
__global__ __launch_bounds__(kRedBlock) void k_residual_partial(const S* __restrict__ src,
                                                                const double* __restrict__ rho_ref,
                                                                const double* __restrict__ u_ref,
                                                                const ChunkDesc* __restrict__ chunks,
                                                                const BoxDesc* __restrict__ boxes,
                                                                long long nsites, double* __restrict__ partial)
{
    const ChunkDesc ch = chunks[blockIdx.x];
    const BoxDesc b = boxes[ch.box];
    const S* base = src + b.mem;
    auto ref = [](const double* q) { return READ != kReadCached ? __builtin_nontemporal_load(q) : *q; };
    double acc[4] = {0.0, 0.0, 0.0, 0.0};  // max |du|, sum du^2, max |drho|, sum drho^2
    for (int k = threadIdx.x; k < ch.count; k += kRedBlock) {
        const long long s = ch.start + k;
        double d, j[3];
        stored_site_moments<L, S, LAYOUT, READ>(base, ch, k, b, d, j);
        const double r = 1.0 + d;
#pragma unroll
        for (int a = 0; a < L::D; ++a) {
            const double du = j[a] / r - ref(u_ref + a * nsites + s);
            acc[0] = fmax(acc[0], fabs(du));
            acc[1] += du * du;
        }
        const double dr = r - ref(rho_ref + s);
        acc[2] = fmax(acc[2], fabs(dr));
        acc[3] += dr * dr;
    }
    const bool is_max[4] = {true, false, true, false};
    block_tree<4>(acc, is_max);
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) partial[blockIdx.x * 4 + k] = acc[k];
}

// sqrt_l2: write the square roots of the two sums (the L2 norms) instead of
// the sums themselves.
__global__ __launch_bounds__(kRedBlock) void k_residual_final(const double* __restrict__ partial, int nchunks,
                                                              double* __restrict__ out, int sqrt_l2)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c = threadIdx.x; c < nchunks; c += kRedBlock) {
        acc[0] = fmax(acc[0], partial[c * 4 + 0]);
        acc[1] += partial[c * 4 + 1];
        acc[2] = fmax(acc[2], partial[c * 4 + 2]);
        acc[3] += partial[c * 4 + 3];
    }
    const bool is_max[4] = {true, false, true, false};
    block_tree<4>(acc, is_max);
    if (threadIdx.x == 0) {
        out[0] = acc[0];
        out[1] = sqrt_l2 ? sqrt(acc[1]) : acc[1];
        out[2] = acc[2];
        out[3] = sqrt_l2 ? sqrt(acc[3]) : acc[3];
    }
}

// ---------------------------------------------------------------------------
// Plain 16-byte-vector copy with non-temporal accesses, one vector per thread.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_copy(const u32x4* __restrict__ src, u32x4* __restrict__ dst, size_t n)
{
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

// Calls f(integral_constant layout, integral_constant policy) for a runtime
// StateLayout and ReadPolicy; the in-place layouts, whose cells are shared
// between sites, keep the default policy.
template <class F>
static hipError_t by_layout(int layout, int read, F&& f)
{
    switch (layout) {
    case kNatural:
        return read == kStreamAll      ? f(ic<kNatural>{}, ic<kStreamAll>{})
               : read == kStreamFields ? f(ic<kNatural>{}, ic<kStreamFields>{})
                                       : f(ic<kNatural>{}, ic<kReadCached>{});
    case kSwapped: return f(ic<kSwapped>{}, ic<kReadCached>{});
    case kTwistEven: return f(ic<kTwistEven>{}, ic<kReadCached>{});
    case kTwistOdd: return f(ic<kTwistOdd>{}, ic<kReadCached>{});
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_init(int lat, int dtype, int K, int layout, const double* rho, const double* u, void* dst,
                       const ChunkDesc* chunks, int nchunks, int chunk_sites, const BoxDesc* boxes,
                       long long nsites, hipStream_t s)
{
    if (layout != kNatural && layout != kTwistEven) return hipErrorInvalidValue;
    return dispatch(lat, dtype, K, [&](auto Lt, auto* Sp, auto Kc) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        constexpr int KK = decltype(Kc)::value;
        const unsigned slices = unsigned((chunk_sites + 255) / 256);
        const dim3 grid = chunk_grid(nchunks, slices);
        if (layout == kTwistEven)
            k_init<L, S, KK, kTwistEven><<<grid, 256, 0, s>>>(rho, u, static_cast<S*>(dst), chunks, boxes, nsites,
                                                              nchunks, slices);
        else
            k_init<L, S, KK, kNatural><<<grid, 256, 0, s>>>(rho, u, static_cast<S*>(dst), chunks, boxes, nsites,
                                                            nchunks, slices);
        return hipGetLastError();
    });
}

hipError_t launch_moments(int lat, int dtype, const void* src, int layout, int read, double* rho, double* u,
                          const ChunkDesc* chunks, int nchunks, int chunk_sites, const BoxDesc* boxes,
                          long long nsites, hipStream_t s)
{
    const unsigned slices = unsigned((chunk_sites + 255) / 256);
    const dim3 grid = chunk_grid(nchunks, slices);
    return dispatch_ld(lat, dtype, [&](auto Lt, auto* Sp, auto) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return by_layout(layout, read, [&](auto Lay, auto Read) -> hipError_t {
            constexpr int LAY = decltype(Lay)::value;
            constexpr int READ = decltype(Read)::value;
            k_moments<L, S, LAY, READ><<<grid, 256, 0, s>>>(static_cast<const S*>(src), rho, u, chunks, boxes, nsites,
                                                      nchunks, slices);
            return hipGetLastError();
        });
    });
}

hipError_t launch_totals(int lat, int dtype, const void* src, int layout, int read, const ChunkDesc* chunks, int nchunks,
                         const int* box_chunk_begin, int nbox, const BoxDesc* boxes, double* partial, double* out,
                         hipStream_t s)
{
    return dispatch_ld(lat, dtype, [&](auto Lt, auto* Sp, auto) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        hipError_t e = by_layout(layout, read, [&](auto Lay, auto Read) -> hipError_t {
            constexpr int LAY = decltype(Lay)::value;
            constexpr int READ = decltype(Read)::value;
            k_totals_partial<L, S, LAY, READ><<<nchunks, kRedBlock, 0, s>>>(static_cast<const S*>(src), chunks, boxes,
                                                                      partial);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
        k_totals_final<<<nbox, kRedBlock, 0, s>>>(partial, box_chunk_begin, out);
        return hipGetLastError();
    });
}

hipError_t launch_residual(int lat, int dtype, const void* src, int layout, int read, const double* rho_ref,
                           const double* u_ref, const ChunkDesc* chunks, int nchunks, const BoxDesc* boxes,
                           long long nsites, double* partial, double* out, bool sqrt_l2, hipStream_t s)
{
    return dispatch_ld(lat, dtype, [&](auto Lt, auto* Sp, auto) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        hipError_t e = by_layout(layout, read, [&](auto Lay, auto Read) -> hipError_t {
            constexpr int LAY = decltype(Lay)::value;
            constexpr int READ = decltype(Read)::value;
            k_residual_partial<L, S, LAY, READ><<<nchunks, kRedBlock, 0, s>>>(static_cast<const S*>(src), rho_ref, u_ref,
                                                                        chunks, boxes, nsites, partial);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
        k_residual_final<<<1, kRedBlock, 0, s>>>(partial, nchunks, out, sqrt_l2 ? 1 : 0);
        return hipGetLastError();
    });
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    const size_t g = (n + 255) / 256;
    if (g == 0 || g > 0x7fffffffu) return hipErrorInvalidValue;
    k_copy<<<unsigned(g), 256, 0, s>>>(static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), n);
    return hipGetLastError();
}

// Layout conversions of a single box's state between the natural layout and
// one of the in-place steps' layouts (layout_elem), into another buffer: a
// pure permutation of stored values (bit-exact).  TO_NATURAL: population i of
// site x is read at its element in LAYOUT and written to its natural element;
// otherwise the other way round.  One thread per site.
template <class L, class S, int LAYOUT, bool TO_NATURAL>
__global__ __launch_bounds__(256) void k_relayout(const S* __restrict__ src, S* __restrict__ dst, BoxDesc b)
{
    const int y = blockIdx.y;
    const int z = blockIdx.z;
    const int x = int(blockIdx.x) * int(blockDim.x) + int(threadIdx.x);
    if (x >= b.nx) return;
    const SitePos pos{(long long)z * b.ny + y, x, y, z};
    const long long nat = site_elem<L::Q>(pos, b.nx);
    const Around<L> at(pos, b);
    unroll<L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const long long e = layout_elem<L, LAYOUT, i>(at, b);
        const long long n = nat + (long long)mem_row<L>(i) * b.nx;
        if constexpr (TO_NATURAL) dst[n] = src[e];
        else dst[e] = src[n];
    });
}

hipError_t launch_relayout(int lat, int dtype, int layout, bool to_natural, const void* src, void* dst,
                           const StepGeom& geo, int block, hipStream_t s)
{
    if (layout == kNatural) return hipErrorInvalidValue;
    BoxDesc b{};
    b.nx = geo.nx;
    b.ny = geo.ny;
    b.nz = geo.nz;
    b.w = geo.nx;
    const dim3 grid(unsigned(geo.xblocks), unsigned(geo.ny), unsigned(geo.nz));
    return dispatch_ld(lat, dtype, [&](auto Lt, auto* Sp, auto) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return by_layout(layout, kReadCached, [&](auto Lay, auto) -> hipError_t {
            constexpr int LAY = decltype(Lay)::value;
            if constexpr (LAY != kNatural) {
                if (to_natural)
                    k_relayout<L, S, LAY, true><<<grid, block, 0, s>>>(static_cast<const S*>(src),
                                                                       static_cast<S*>(dst), b);
                else
                    k_relayout<L, S, LAY, false><<<grid, block, 0, s>>>(static_cast<const S*>(src),
                                                                        static_cast<S*>(dst), b);
                return hipGetLastError();
            }
            return hipErrorInvalidValue;
        });
    });
}

// ---------------------------------------------------------------------------
// Runtime-lattice entry points of the step kernels (instances compiled per
// lattice in step_<lattice>.hip and batch_<lattice>.hip).
// ---------------------------------------------------------------------------

// Calls f(L{}, (S*)nullptr) for a runtime (lattice, dtype).
template <class F>
static hipError_t by_pair(int lat, int dtype, F&& f)
{
    return dispatch_kind(lat, dtype, 2, kFiltered,
                         [&](auto Lt, auto* Sp, auto, auto) -> hipError_t { return f(Lt, Sp); });
}

hipError_t launch_step(int lat, int dtype, int K, int kind, const void* src, void* dst, const StepGeom& geo,
                       double omega, double theta, int block, bool pair, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return launch_step_l<L, S>(K, kind, src, dst, geo, omega, theta, block, pair, s);
    });
}

hipError_t launch_step2(int lat, int dtype, int K, int kind, const void* src, void* dst, const Step2Geom& geo,
                        double omega, double theta, int grid, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        if constexpr (std::is_same<L, D3Q15>::value || std::is_same<L, D3Q19>::value)
            return launch_step2_l<L, S>(K, kind, src, dst, geo, omega, theta, grid, s);
        else
            return hipErrorInvalidValue;
    });
}

hipError_t launch_step2_batch(int lat, int dtype, int K, int kind, const void* src, void* dst,
                              const ColumnDesc* columns, const ColumnStart* starts, int rounds, double theta,
                              int grid, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        if constexpr (std::is_same<L, D3Q15>::value || std::is_same<L, D3Q19>::value)
            return launch_step2_batch_l<L, S>(K, kind, src, dst, columns, starts, rounds, theta, grid, s);
        else
            return hipErrorInvalidValue;
    });
}

hipError_t launch_step_tile(int lat, int dtype, int K, int kind, const void* src, void* dst, const TileGeom& geo,
                            double omega, double theta, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) -> hipError_t {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        if constexpr (L::R == 1)
            return launch_step_tile_l<L, S>(K, kind, src, dst, geo, omega, theta, s);
        else
            return hipErrorInvalidValue;
    });
}

int vec_sites_per_lane(int lat, int dtype)
{
    int v = 0;
    (void)by_pair(lat, dtype, [&](auto Lt, auto* Sp) {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        v = vec_sites_l<L, S>();
        return hipSuccess;
    });
    return v;
}

hipError_t launch_step_vec(int lat, int dtype, int K, int kind, const void* src, void* dst, const VecGeom& geo,
                           double omega, double theta, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return launch_step_vec_l<L, S>(K, kind, src, dst, geo, omega, theta, s);
    });
}

hipError_t launch_step_ip(int lat, int dtype, int K, int kind, void* buf, bool from_natural, const StepGeom& geo,
                          double omega, double theta, int block, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return launch_step_ip_l<L, S>(K, kind, buf, from_natural, geo, omega, theta, block, s);
    });
}

hipError_t launch_step_tw(int lat, int dtype, int K, int kind, void* buf, bool even, const StepGeom& geo,
                          double omega, double theta, int block, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return launch_step_tw_l<L, S>(K, kind, buf, even, geo, omega, theta, block, s);
    });
}

hipError_t launch_step_batch(int lat, int dtype, int K, int kind, const void* src, void* dst, const TileDesc* tiles,
                             int ntiles, double theta, int block, int grid, bool aligned_rows, hipStream_t s)
{
    return by_pair(lat, dtype, [&](auto Lt, auto* Sp) {
        using L = decltype(Lt);
        using S = std::remove_pointer_t<decltype(Sp)>;
        return launch_step_batch_l<L, S>(K, kind, src, dst, tiles, ntiles, theta, block, grid, aligned_rows, s);
    });
}

}  // namespace lbm
