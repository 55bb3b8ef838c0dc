// Two fused time steps per launch on a batch of boxes (lattices whose velocity
// components are at most 1 in magnitude, 3-D).  Included by the per-pair
// translation units, which instantiate launch_step2_batch_l.
#pragma once

#include "step2.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// The two-step kernel's walk (step2.hpp) over the columns of every box of a
// batch, in the blocked layout.  The host cuts the column-planes of all boxes, in
// memory order, into grid * rounds runs of equal cost; one launch has one block
// per compute unit, and block b takes the runs b, b + grid, ... in turn, run k
// from starts[k] up to starts[k + 1].  At any time the blocks then work on
// neighbouring columns: the two rows that two columns of a box share meet in an
// L2, and the reads spread over less memory.  Measured on 256 D3Q19 boxes of
// sides 16-64 (17.6 million sites), us per step with 1, 2, 4 and 8 rounds: FP32
// 415, 403, 368, 351 (one-step kernel 448), FP64 with 12 rounds 660 (1: 758;
// one-step 900).  Every cut costs two more planes of step 1, so short runs are not cut further
// (api.hip, build_columns).  Runs of z-chunks with the columns of a box side by
// side in z were no faster (4 rounds: 380), nor were smaller tiles with two
// blocks per compute unit (512 threads 438, 384 501).
// The one-step kernel (step_batch.hpp) reads and writes the state once per
// step; this one does it once per two.  A column of whole x-rows (boxes up to
// 128 sites wide) is one run of consecutive sites per plane, so loads and
// stores use whole lines but at the run's ends.
// An element's address is the box's base (uniform) plus a 32-bit offset formed
// at each access from the source site; the population's place in the block is
// the instruction's constant offset.  That needs 90 registers a lane against
// the single-box kernel's 160.
// ---------------------------------------------------------------------------

template <class L, class S, int K, int KIND>
__global__ __launch_bounds__(batch_columns_threads(sizeof(S))) void k_step2_batch(
    const S* __restrict__ src, S* __restrict__ dst, const ColumnDesc* __restrict__ columns,
    const ColumnStart* __restrict__ starts, int rounds, typename Store<S>::R theta)
{
    using ST = Store<S>;
    using R = typename ST::R;
    constexpr int Q = L::Q;
    constexpr int NT = batch_columns_threads(sizeof(S));
    static_assert(L::D == 3 && L::R == 1, "a one-site ring in x, y and z");
    __shared__ S lplane[2][Q][NT];

    const int tid = threadIdx.x;
    const unsigned nb = gridDim.x;
    // consecutive runs on one XCD (blocks are dealt to the eight in turn)
    const unsigned lb = (nb % 8 == 0) ? (blockIdx.x % 8) * (nb / 8) + blockIdx.x / 8 : blockIdx.x;
    int c = 0, za = 0;       // next column-plane
    ColumnStart last{0, 0};  // end of this block's current run
    for (int r = 0;; ++c, za = 0) {
        while (c > last.column || (c == last.column && za >= last.z)) {  // the run is done: the next one
            if (r == rounds) return;
            const ColumnStart first = starts[lb + r * nb];
            last = starts[lb + r * nb + 1];
            c = first.column;
            za = first.z;
            ++r;
        }
        const ColumnDesc b = columns[c];
        const int zb = (c < last.column) ? b.nz : last.z;
        const int wx = b.tx + 2;
        const int hy = int((float(tid) + 0.5f) * (1.0f / float(wx)));  // exact for tid < 2^10
        const int hx = tid - hy * wx;
        const bool owner = tid < b.tx * b.ty;
        const int oy = int((float(tid) + 0.5f) * (1.0f / float(b.tx)));
        const int ox = tid - oy * b.tx;
        const int oh = owner ? (oy + 1) * wx + ox + 1 : wx + 1;
        const int ohy[3] = {oh - wx, oh, oh + wx};
        const bool writer = owner && b.x0 + ox < b.nx && b.y0 + oy < b.ny;
        const int x = wrap_coord(b.x0 + hx - 1, b.nx), y = wrap_coord(b.y0 + min(hy, b.ty + 1) - 1, b.ny);
        int xw[3], yr[3];  // in-plane site offsets of the neighbours
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            xw[k] = wrap_coord(x + k - 1, b.nx);
            yr[k] = wrap_coord(y + k - 1, b.ny) * b.nx;
        }
        const int own = (b.y0 + oy) * b.nx + b.x0 + ox;
        const int plane = b.nx * b.ny;
        // byte offset of population 0 of a site: (l / 64) Q 64 + l % 64 elements
        auto offset = [](int l) -> unsigned {
            return (unsigned(l) + (unsigned(l) >> 6) * unsigned(64 * (Q - 1))) * unsigned(sizeof(S));
        };
        const char* from = reinterpret_cast<const char*>(src + b.mem);
        char* to = reinterpret_cast<char*>(dst + b.mem);
        auto pull = [&](int p, R(&g)[Q]) {
            int zo[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) zo[k] = wrap_coord(p + k - 1, b.nz) * plane;
            unroll<Q>([&](auto M) {  // in tile-row order
                constexpr int m = decltype(M)::value;
                constexpr int i = mem_pop<L>(m);
                constexpr int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
                const char* e = from + offset(zo[1 - cz] + yr[1 - cy] + xw[1 - cx]);
                g[i] = ST::get(reinterpret_cast<const S*>(e) + m * 64);
            });
        };
        auto put = [&](int p, const R(&h)[Q]) {
            if (!writer) return;
            S* e = reinterpret_cast<S*>(to + offset(wrap_coord(p, b.nz) * plane + own));
            unroll<Q>([&](auto M) {
                constexpr int m = decltype(M)::value;
                constexpr int i = mem_pop<L>(m);
                ST::put(e + m * 64, h[i]);
            });
        };
        walk_column<L, S, K, KIND, true>(lplane, za, zb, owner, ohy, R(b.omega), theta, pull, put);
        __syncthreads();  // the next column's first plane refills buffer 0
    }
}

template <class L, class S>
hipError_t launch_step2_batch_l(int K, int kind, const void* src, void* dst, const ColumnDesc* columns,
                                const ColumnStart* starts, int rounds, double theta, int grid, hipStream_t s)
{
    if constexpr (L::D == 3 && L::R == 1) {
        return dispatch_pair<L, S>(K, kind, [&](auto, auto*, auto Kc, auto Kind) -> hipError_t {
            using R = typename Store<S>::R;
            constexpr int KK = decltype(Kc)::value;
            constexpr int KD = decltype(Kind)::value;
            constexpr int NTHREADS = batch_columns_threads(sizeof(S));
            k_step2_batch<L, S, KK, KD><<<dim3(unsigned(grid)), NTHREADS, 0, s>>>(
                static_cast<const S*>(src), static_cast<S*>(dst), columns, starts, rounds, R(theta));
            return hipGetLastError();
        });
    } else {
        return hipErrorInvalidValue;
    }
}

}  // namespace lbm
