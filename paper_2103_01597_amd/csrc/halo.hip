// Periodic halo fill (Section 3.3): every halo cell of the padded grid
// takes the interior cell given by the mapping s' = ((s - r) mod n) + r on
// each axis, r the halo width (the stencil radius, 1..4); sides, edges and
// corners of all 8 fields are filled.  Bytes per fill: 2 * 8 * elem *
// (M^3 - N^3).
#include "mhd_internal.hpp"

namespace mhd {
namespace {

__device__ __forceinline__ int wrap_index(int s, int n, int r)
{
    int t = s - r;
    if (n < r) {  // a box thinner than its halo (uniform)
        t %= n;
        return (t < 0 ? t + n : t) + r;
    }
    return (t < 0 ? t + n : t >= n ? t - n : t) + r;
}

// One launch, every halo cell straight from the interior cell it maps to, so
// no part waits for another.  Workgroups [0, xblocks) fill the 2r halo columns
// of the interior rows; the rest copy whole rows of the halo (the 2r halo
// planes, then the 2r halo rows of the interior planes), x wrapped at both ends.
//
// X part: a workgroup covers 32 rows of the interior of one field, eight lanes
// per row (lane c < 2r fills column c of the left halo, c < r, or column c - r
// of the right halo).  Bound: the columns touch two cache lines per row for 2r
// cells.  Row part: consecutive lanes copy consecutive cells.
constexpr int HX_ROWS = 32, ROW_UNROLL = 4;

template <typename E>
__global__ __launch_bounds__(256) void k_halo(Grid g, unsigned xblocks, int lanes_log2,
                                                E* __restrict__ fields)
{
    const int r = g.r;
    E* f = fields + (int64_t)blockIdx.y * g.fstride;
    if (blockIdx.x < xblocks) {
        const int c = threadIdx.x & 7;
        if (c >= 2 * r) return;
        const int dst = c < r ? c : g.nx + c;  // padded halo column
        const int src = wrap_index(dst, g.nx, r);
        const int row = (int)blockIdx.x * HX_ROWS + (threadIdx.x >> 3);
        if (row >= g.ny * g.nz) return;
        const int z = row / g.ny, y = row - z * g.ny;
        E* p = f + ((r + z) * g.my + r + y) * g.mx;
        p[dst] = p[src];
        return;
    }
    // 2^lanes_log2 lanes per row, each copying up to ROW_UNROLL cells of it at once
    const int lanes = 1 << lanes_log2;
    int k = (int)(blockIdx.x - xblocks) * (256 >> lanes_log2) + ((int)threadIdx.x >> lanes_log2);
    int z, y;
    if (k < 2 * r * g.my) {
        z = k / g.my;
        y = k - z * g.my;
        if (z >= r) z += g.nz;
    } else {
        k -= 2 * r * g.my;
        z = k / (2 * r);
        y = k - z * (2 * r);
        if (z >= g.nz) return;
        z += r;
        if (y >= r) y += g.ny;
    }
    E* dst = f + (z * g.mxy + y * g.mx);
    const E* src = f + (wrap_index(z, g.nz, r) * g.mxy + wrap_index(y, g.ny, r) * g.mx);
    for (int x0 = (int)threadIdx.x & (lanes - 1); x0 < g.mx; x0 += ROW_UNROLL * lanes) {
        E v[ROW_UNROLL];
#pragma unroll
        for (int i = 0; i < ROW_UNROLL; ++i)
            if (x0 + i * lanes < g.mx) v[i] = src[wrap_index(x0 + i * lanes, g.nx, r)];
#pragma unroll
        for (int i = 0; i < ROW_UNROLL; ++i)
            if (x0 + i * lanes < g.mx) dst[x0 + i * lanes] = v[i];
    }
}

template <typename E>
void launch_halo_typed(const Grid& g, void* fields, hipStream_t st)
{
    const unsigned xblocks = (unsigned)(((int64_t)g.ny * g.nz + HX_ROWS - 1) / HX_ROWS);
    int lg = 5;  // lanes of a row: about a quarter of it, 32 to 256
    while (lg < 8 && (1 << lg) * ROW_UNROLL < g.mx) ++lg;
    const int64_t rows = (int64_t)2 * g.r * (g.my + g.nz), per_block = 256 >> lg;
    hipLaunchKernelGGL(k_halo<E>, dim3(xblocks + (unsigned)((rows + per_block - 1) / per_block), NQ),
                       dim3(256), 0, st, g, xblocks, lg, (E*)fields);
}

}  // namespace

hipError_t launch_halo(const Grid& g, void* fields, int elem_size, hipStream_t st)
{
    if (elem_size == 8) launch_halo_typed<uint64_t>(g, fields, st);
    else launch_halo_typed<uint32_t>(g, fields, st);
    return hipGetLastError();
}

}  // namespace mhd
