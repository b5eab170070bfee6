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

// a / d for a >= 0 and quotients below 2^20; inv: 1 / d within an ulp
__device__ __forceinline__ int quotient(int a, int d, float inv)
{
    const int q = (int)((float)a * inv), rem = a - q * d;
    return q + (rem >= d ? 1 : 0) - (rem < 0 ? 1 : 0);
}

// One launch, every halo cell straight from the interior cell it maps to, so
// no part waits for another.  The first NQ * rblocks workgroups copy whole rows of
// the halo (of each field the 2r halo planes, then the 2r halo rows of the interior
// planes), x wrapped at both ends; the rest fill the 2r halo columns of the
// interior rows.
//
// Row part: the rows of a field are cut into units of V cells (16 bytes, wherever
// the row starts; the last one of a row may be shorter), consecutive lanes copy
// consecutive units, ROW_UNROLL in flight per lane.  Only the units that hold halo
// columns are gathered cell by cell.  Lanes on rows of their own leave most of a
// workgroup idle where a row does not fill it, and one workgroup per row leaves
// the chip idle where rows are long and few (FP64 30000 x 8 x 8: 103 us, 69 now).
// X part: a workgroup covers 32 rows of the interior of one field, eight lanes
// per row (lane c < 2r fills column c of the left halo, c < r, or column c - r
// of the right halo).  Bound: the columns touch two cache lines per row for 2r
// cells.
// The two parts after one another, not field by field beside one another: the row
// copies stream and lose more from the x part's scattered lines than overlap gives
// (FP64 512^3 273 against 255 us, 256^3 49.5 against 47.7).  Three launches (x columns, then rows
// and planes with their halo columns filled) took 259 and 50.9, 32^3 11.3 against 6.4.
constexpr int HX_ROWS = 32, ROW_UNROLL = 4;

template <typename E>
__global__ __launch_bounds__(256) void k_halo(Grid g, unsigned rblocks, unsigned xblocks,
                                              E* __restrict__ fields)
{
    constexpr int V = 16 / sizeof(E);
    // (one access each; the hardware takes unaligned ones)
    typedef E Unit __attribute__((ext_vector_type(V), aligned(sizeof(E))));
    const int r = g.r;
    const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;  // the order of launch
    if (block >= NQ * rblocks) {
        const unsigned b = block - NQ * rblocks, q = b / xblocks;
        const int c = threadIdx.x & 7;
        if (c >= 2 * r) return;
        const int dst = c < r ? c : g.nx + c;  // padded halo column
        const int src = wrap_index(dst, g.nx, r);
        const int row = (int)(b - q * xblocks) * HX_ROWS + (threadIdx.x >> 3);
        if (row >= g.ny * g.nz) return;
        const int z = row / g.ny, y = row - z * g.ny;
        E* p = fields + (int64_t)q * g.fstride + ((r + z) * g.my + r + y) * g.mx;
        p[dst] = p[src];
        return;
    }
    const unsigned q = block / rblocks;
    E* f = fields + (int64_t)q * g.fstride;
    const int units = (g.mx + V - 1) / V, rows = 2 * r * (g.my + g.nz);
    const int begin = (int)(block - q * rblocks) * (256 * ROW_UNROLL), k0 = begin / units;
    const float inv_units = __builtin_amdgcn_rcpf((float)units),
                inv_my = __builtin_amdgcn_rcpf((float)g.my),
                inv_2r = __builtin_amdgcn_rcpf((float)(2 * r));
    Unit v[ROW_UNROLL];
    int at[ROW_UNROLL], left[ROW_UNROLL];  // the unit's cell (-1: none), and the row's cells from it on
#pragma unroll
    for (int i = 0; i < ROW_UNROLL; ++i) {
        const int u = begin - k0 * units + (int)threadIdx.x + i * 256;
        int k = quotient(u, units, inv_units);
        const int x = V * (u - k * units);
        k += k0;
        at[i] = -1;
        left[i] = g.mx - x;
        if (k >= rows) continue;
        int z, y;
        if (k < 2 * r * g.my) {
            z = quotient(k, g.my, inv_my);
            y = k - z * g.my;
            if (z >= r) z += g.nz;
        } else {
            k -= 2 * r * g.my;
            z = quotient(k, 2 * r, inv_2r);
            y = k - z * (2 * r);
            z += r;
            if (y >= r) y += g.ny;
        }
        at[i] = z * g.mxy + y * g.mx + x;
        const E* src = f + (wrap_index(z, g.nz, r) * g.mxy + wrap_index(y, g.ny, r) * g.mx);
        if (x >= r && x + V <= r + g.nx) {
            v[i] = *reinterpret_cast<const Unit*>(src + x);
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e) v[i][e] = src[wrap_index(min(x + e, g.mx - 1), g.nx, r)];
        }
    }
#pragma unroll
    for (int i = 0; i < ROW_UNROLL; ++i) {
        if (at[i] < 0) continue;
        if (left[i] >= V) {
            *reinterpret_cast<Unit*>(f + at[i]) = v[i];
        } else {
#pragma unroll
            for (int e = 0; e + 1 < V; ++e)
                if (e < left[i]) f[at[i] + e] = v[i][e];
        }
    }
}

template <typename E>
void launch_halo_typed(const Grid& g, void* fields, hipStream_t st)
{
    const int64_t unit = 16 / sizeof(E), per_block = 256 * ROW_UNROLL;
    const int64_t units = (int64_t)2 * g.r * (g.my + g.nz) * ((g.mx + unit - 1) / unit);
    const unsigned rblocks = (unsigned)((units + per_block - 1) / per_block);
    const unsigned xblocks = (unsigned)(((int64_t)g.ny * g.nz + HX_ROWS - 1) / HX_ROWS);
    // (NQ in the second dimension: a dimension holds fewer than 2^32 threads)
    hipLaunchKernelGGL(k_halo<E>, dim3(rblocks + xblocks, NQ), dim3(256), 0, st, g, rblocks, xblocks,
                       (E*)fields);
}

}  // namespace

hipError_t launch_halo(const Grid& g, void* fields, int elem_size, hipStream_t st)
{
    if (elem_size == 8) launch_halo_typed<uint64_t>(g, fields, st);
    else launch_halo_typed<uint32_t>(g, fields, st);
    return hipGetLastError();
}

}  // namespace mhd
