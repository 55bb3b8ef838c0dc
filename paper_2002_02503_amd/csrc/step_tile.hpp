// Several fused time steps per launch on a single box, for lattices whose
// velocity components are at most 1 in magnitude (D2Q9, D3Q15, D3Q19).
// Included by the per-lattice translation units, which instantiate
// launch_step_tile_l for one (lattice, storage type).
#pragma once

#include "device.hpp"
#include "step_launch.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// A block owns a tile of the box and takes `steps` steps on it in LDS.  Step 1
// runs on the tile and a ring of steps - 1 sites around it and pulls from HBM
// (or the caches); its results go to LDS in the storage type, so a read gives
// back exactly what a store to HBM and a reload would.  Each later step runs
// on a ring one site narrower and pulls from LDS; the last one writes the tile.
// Each site's arithmetic is k_step's on the same values, so the launch gives
// the bits of `steps` k_step launches.
// A launch whose sites do not fill the chip costs about 3 us whatever it does
// (launch, the latency of the loads, the collision's dependent chain), so
// small boxes take several steps for one launch and pay with the rings'
// arithmetic, on compute units that would otherwise idle.
// One LDS plane set, not two: a step reads all its pulls into registers, one
// site per thread, before any thread writes (two barriers).  Step 1 reads no
// LDS and loops over any number of sites.
// A tile of whole x-rows wraps inside itself and has no ring in x; its loads
// then use every byte of the lines they touch.
// ---------------------------------------------------------------------------

// Quotient and remainder of i / n for 0 <= i < 2^15 and 0 < n < 2^15: i + 1/2
// is at least 1/(2n) of n away from a multiple, the rounding of the product
// below i / n 2^-22.
__device__ __forceinline__ int small_div(int i, float inv_n)
{
    return int((float(i) + 0.5f) * inv_n);
}

template <class L, class S, int K, int KIND>
__global__ __launch_bounds__(1024) void k_step_tile(const S* __restrict__ src, S* __restrict__ dst, TileGeom geo,
                                                    typename Store<S>::R omega, typename Store<S>::R theta)
{
    using ST = Store<S>;
    using R = typename ST::R;
    constexpr bool PROJ = !std::is_same<R, double>::value;
    constexpr bool D3 = (L::D == 3);
    constexpr int Q = L::Q;
    static_assert(L::R == 1, "a ring of one site per step");
    extern __shared__ __align__(16) unsigned char tile_lds[];
    S* lds = reinterpret_cast<S*>(tile_lds);  // population i of region site s: lds[i * cap + s]

    const int tid = threadIdx.x, nthreads = blockDim.x;
    const int x0 = int(blockIdx.x) * geo.tx, y0 = int(blockIdx.y) * geo.ty, z0 = int(blockIdx.z) * geo.tz;
    const int w = min(geo.tx, geo.nx - x0), h = min(geo.ty, geo.ny - y0), d = min(geo.tz, geo.nz - z0);
    const int ring = geo.steps - 1;  // of step 1
    const bool rows = geo.tx == geo.nx;  // whole x-rows: periodic inside the tile, no ring in x
    const int ring_x = rows ? 0 : ring;
    // the stored region: step 1's sites, x fastest
    const int ex = w + 2 * ring_x, ey = h + 2 * ring, ez = D3 ? d + 2 * ring : 1;
    const int exy = ex * ey;
    const unsigned row_bytes = unsigned(geo.nx) * unsigned(sizeof(S));

    // Step 1.  Offsets are 32-bit bytes from src (the host checks the size).
    {
        const float inv_x = 1.0f / float(ex), inv_y = 1.0f / float(ey);
        const int n = exy * ez;
        for (int s = tid; s < n; s += nthreads) {
            const int r = small_div(s, inv_x);
            const int hx = s - r * ex;
            const int hz = D3 ? small_div(r, inv_y) : 0;
            const int hy = r - hz * ey;
            const int x = wrap_coord(x0 - ring_x + hx, geo.nx), y = wrap_coord(y0 - ring + hy, geo.ny);
            const int z = D3 ? wrap_coord(z0 - ring + hz, geo.nz) : 0;
            unsigned xo[3], yz[3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k) xo[k] = unsigned(wrap_coord(x + k - 1, geo.nx)) * unsigned(sizeof(S));
#pragma unroll
            for (int kz = 0; kz < 3; ++kz) {
                if (!D3 && kz != 1) continue;
                const int zr = D3 ? wrap_coord(z + kz - 1, geo.nz) * geo.ny : 0;
#pragma unroll
                for (int ky = 0; ky < 3; ++ky)
                    yz[kz][ky] = unsigned(zr + wrap_coord(y + ky - 1, geo.ny)) * (unsigned(Q) * row_bytes);
            }
            R g[Q];
            unroll<Q>([&](auto M) {  // in tile-row order
                constexpr int m = decltype(M)::value;
                constexpr int i = mem_pop<L>(m);
                constexpr int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
                const char* base = reinterpret_cast<const char*>(src) + (long long)m * row_bytes;
                g[i] = ST::get(reinterpret_cast<const S*>(base + (yz[1 - cz][1 - cy] + xo[1 - cx])));
            });
            collide_site<L, K, KIND, PROJ, R>(g, omega, theta);
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                ST::put(lds + i * geo.cap + s, g[i]);
            });
        }
    }
    __syncthreads();

    for (int t = 2; t <= geo.steps; ++t) {
        const int in = t - 1;  // this step's region inside the stored one
        const int in_x = rows ? 0 : in;
        const int sx = ex - 2 * in_x, sy = ey - 2 * in, sz = D3 ? ez - 2 * in : 1;
        const int n = sx * sy * sz;  // at most nthreads
        const bool active = tid < n;
        const int r = small_div(tid, 1.0f / float(sx));
        const int hx = tid - r * sx;
        const int hz = D3 ? small_div(r, 1.0f / float(sy)) : 0;
        const int hy = r - hz * sy;
        const int s = ((D3 ? hz + in : 0) * ey + hy + in) * ex + hx + in_x;
        // the stored sites at x - 1 and x + 1
        const int west = (rows && hx == 0) ? s + ex - 1 : s - 1, east = (rows && hx == ex - 1) ? s - ex + 1 : s + 1;
        R g[Q];
        if (active)
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
                const int from = (cx == 0) ? s : (cx > 0) ? west : east;
                g[i] = ST::get(lds + from + (i * geo.cap - cy * ex - cz * exy));
            });
        __syncthreads();  // every pull of this step is in registers
        if (active) {
            collide_site<L, K, KIND, PROJ, R>(g, omega, theta);
            if (t < geo.steps) {
                unroll<Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    ST::put(lds + i * geo.cap + s, g[i]);
                });
            } else {  // the tile's site (hx, hy, hz)
                const unsigned row = unsigned((z0 + hz) * geo.ny + y0 + hy);
                const unsigned o = row * (unsigned(Q) * row_bytes) + unsigned(x0 + hx) * unsigned(sizeof(S));
                unroll<Q>([&](auto M) {
                    constexpr int m = decltype(M)::value;
                    constexpr int i = mem_pop<L>(m);
                    char* base = reinterpret_cast<char*>(dst) + (long long)m * row_bytes;
                    ST::put(reinterpret_cast<S*>(base + o), g[i]);
                });
            }
        }
        __syncthreads();
    }
}

template <class L, class S>
hipError_t launch_step_tile_l(int K, int kind, const void* src, void* dst, const TileGeom& geo, double omega,
                              double theta, hipStream_t s)
{
    if constexpr (L::R == 1) {
        return dispatch_pair<L, S>(K, kind, [&](auto, auto*, auto Kc, auto Kind) -> hipError_t {
            using R = typename Store<S>::R;
            constexpr int KK = decltype(Kc)::value;
            constexpr int KD = decltype(Kind)::value;
            const dim3 grid(unsigned((geo.nx + geo.tx - 1) / geo.tx), unsigned((geo.ny + geo.ty - 1) / geo.ty),
                            unsigned((geo.nz + geo.tz - 1) / geo.tz));
            const size_t lds = size_t(geo.cap) * L::Q * sizeof(S);
            k_step_tile<L, S, KK, KD><<<grid, geo.block, lds, s>>>(static_cast<const S*>(src), static_cast<S*>(dst),
                                                                  geo, R(omega), R(theta));
            return hipGetLastError();
        });
    } else {
        return hipErrorInvalidValue;
    }
}

}  // namespace lbm
