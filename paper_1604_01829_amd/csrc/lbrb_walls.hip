// lbrb_walls.hip -- the moving-wall link kernel and the hole mirrors (see lbrb_walls.h).
#include "lbrb_device.h"
#include "lbrb_layout.h"
#include "lbrb_walls.h"

namespace lbrb {

template <typename Real>
__global__ __launch_bounds__(256) void wall_links_kernel(Real* f, const WallLink* links,
                                                         int64_t n_links)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= n_links) return;
    const WallLink L = links[k];
    Real* p = f + pop_at(L.pop, L.g);
    *p = *p + (Real)L.delta;
}

template <typename Real>
void launch_wall_links(Real* f, const WallLink* links, int64_t n_links, hipStream_t s)
{
    if (n_links <= 0) return;
    const int64_t blocks = (n_links + 255) / 256;
    hipLaunchKernelGGL((wall_links_kernel<Real>), dim3((unsigned)blocks), dim3(256), 0, s, f,
                       links, n_links);
}

// one thread per stored node of the tiles that hold holes.  TRANSPOSED: the reverse pass's
// mirror, slot opp(i) of the hole takes population i of x (lambda_opp(i)(h) = lambda_i(h + c_i)),
// so that the transposed pull at a fluid node y = h - c_j reads, from the hole's slot j, its own
// lambda_opp(j)(y): the transpose of halfway bounce-back.
// Latency-bound: few nodes, a chain of dependent lookups.  So the lookups of all 18 neighbours
// go out together, round by round -- the 9 rows around the hole, then the marks and the
// populations, then the stores -- and only the tiles with holes are launched.  One neighbour
// after another (each store kept the next lookup waiting) a box of 45 x 37 x 61 nodes with two
// obstacles took 16.3 us, this 6.0 us.
template <typename Real, bool TRANSPOSED>
__global__ __launch_bounds__(kNodeBlock) void mirror_holes_kernel(Real* f, const ReplicaDesc* reps,
                                                                  const RowDesc* rows,
                                                                  const RowDesc* rowinfo,
                                                                  const NodeTile* tiles,
                                                                  const uint8_t* hole)
{
    __shared__ RowDesc tile_rows[kNodeBlock];
    const NodeTile t = tiles[blockIdx.x];
    const ReplicaDesc R = reps[t.replica];
    const int64_t local = t.begin + threadIdx.x;
    const int64_t g = R.base + local;
    const bool mine = (int)threadIdx.x < t.count && hole[g] != 0;
    int x, y, z;
    RowDesc self;
    locate_tile<true>(R, rows, t, local, tile_rows, x, y, z, self);
    if (!mine) return;
    // neighbour h + c_i in storage coordinates: direction k = i, or its exchange when the replica is
    // stored with axes x and z exchanged; Rows9 looks along -c, so slot 8 - r is row r's opposite
    Rows9 rw;
    load_rows9(rowinfo, R.row_base, R.ny, R.nz, y, z, rw);
    const bool sw = R.swap != 0;
    int32_t n[Q];       // the neighbour's local index, -1: not stored (a boundary node)
    uint8_t mark[Q];
    Real v[Q];
#pragma unroll
    for (int k = 1; k < Q; ++k) {
        const int r9 = (1 - cy_of(k)) + 3 * (1 - cz_of(k));
        const int off = wrap1(x + cx_of(k), R.nx) - rw.lo[r9];
        n[k] = (unsigned)off < (unsigned)rw.ln[r9] ? rw.st[r9] + off : -1;
        const int i = sw ? swap_xz_of(k) : k;
        const int64_t gx = n[k] >= 0 ? R.base + n[k] : g;
        mark[k] = hole[gx];                   // (of the hole itself where there is none)
        v[k] = f[pop_at(TRANSPOSED ? i : opposite_of(i), gx)];
    }
#pragma unroll
    for (int k = 1; k < Q; ++k) {
        const int i = sw ? swap_xz_of(k) : k;
        if (mark[k] == 0) f[pop_at(TRANSPOSED ? opposite_of(i) : i, g)] = v[k];   // a fluid node
    }
}

template <typename Real>
void launch_mirror_holes(Real* f, const ReplicaDesc* reps, const RowDesc* rows,
                         const RowDesc* rowinfo, const NodeTile* tiles, int32_t n_tiles,
                         const uint8_t* hole, hipStream_t s)
{
    if (n_tiles <= 0) return;
    hipLaunchKernelGGL((mirror_holes_kernel<Real, false>), dim3(n_tiles), dim3(kNodeBlock), 0, s, f,
                       reps, rows, rowinfo, tiles, hole);
}

template <typename Real>
void launch_mirror_holes_transposed(Real* lam, const ReplicaDesc* reps, const RowDesc* rows,
                                    const RowDesc* rowinfo, const NodeTile* tiles, int32_t n_tiles,
                                    const uint8_t* hole, hipStream_t s)
{
    if (n_tiles <= 0) return;
    hipLaunchKernelGGL((mirror_holes_kernel<Real, true>), dim3(n_tiles), dim3(kNodeBlock), 0, s,
                       lam, reps, rows, rowinfo, tiles, hole);
}

template void launch_mirror_holes<float>(float*, const ReplicaDesc*, const RowDesc*,
                                         const RowDesc*, const NodeTile*, int32_t,
                                         const uint8_t*, hipStream_t);
template void launch_mirror_holes<double>(double*, const ReplicaDesc*, const RowDesc*,
                                          const RowDesc*, const NodeTile*, int32_t,
                                          const uint8_t*, hipStream_t);
template void launch_mirror_holes_transposed<float>(float*, const ReplicaDesc*, const RowDesc*,
                                                    const RowDesc*, const NodeTile*, int32_t,
                                                    const uint8_t*, hipStream_t);
template void launch_mirror_holes_transposed<double>(double*, const ReplicaDesc*, const RowDesc*,
                                                     const RowDesc*, const NodeTile*, int32_t,
                                                     const uint8_t*, hipStream_t);
template void launch_wall_links<float>(float*, const WallLink*, int64_t, hipStream_t);
template void launch_wall_links<double>(double*, const WallLink*, int64_t, hipStream_t);

}  // namespace lbrb
