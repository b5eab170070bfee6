// Periodic halo fill (Section 3.3): every halo cell of the padded grid
// takes the interior cell given by the mapping s' = ((s - r) mod n) + r on
// each axis, r the halo width (the stencil radius, 1..4); sides, edges and
// corners of all 8 fields are filled.  Bytes per fill: 2 * 8 * elem *
// (M^3 - N^3).
#include "mhd_internal.hpp"

namespace mhd {
namespace {

// THIN: an axis may be thinner than its halo
template <bool THIN>
__device__ __forceinline__ int wrap_index(int s, int n, int r)
{
    int t = s - r;
    if (THIN) t %= n;
    return (t < 0 ? t + n : t >= n ? t - n : t) + r;
}

// a / d for a >= 0 and quotients below 2^20; inv: 1 / d within an ulp
__device__ __forceinline__ int quotient(int a, int d, float inv)
{
    const int q = (int)((float)a * inv), rem = a - q * d;
    return q + (rem >= d ? 1 : 0) - (rem < 0 ? 1 : 0);
}

// One launch, every halo cell straight from the interior cell it maps to, so
// no part waits for another.  Of each field the first rblocks workgroups copy whole
// rows of the halo (the 2r halo planes, then the 2r halo rows of the interior
// planes), x wrapped at both ends; the rest fill the 2r halo columns of the
// interior rows.  The fields are interleaved: consecutive workgroups go to the 8
// XCDs in turn, so each XCD walks one field and its L2 holds the lines that
// neighbouring workgroups share.
//
// Row part: the rows are cut into units of V cells (16 bytes, wherever the row
// starts; the last one of a row may be shorter), consecutive lanes copy consecutive
// units, so rows of any length fill the workgroups; only the units that hold halo
// columns are gathered cell by cell.  X part: a workgroup covers 32 rows of
// the interior, eight lanes per row (lane c < 2r fills column c of the left halo,
// c < r, or column c - r of the right halo).  Bound: the columns touch two cache
// lines per row for 2r cells.
//
// us, FP64, 512^3 / 256^3 / 32^3 in a step (three fills and three substeps) / 30000 x 8 x 8:
//   three launches (columns, then whole rows and planes)     258 / 50.9 / - / 73
//   one launch, field by field, columns beside the rows,
//   rows by lanes of their own, cell by cell                 271 / 48.2 / 43.4 / 102
//   units, four per lane, rows before columns, field by field 254 / 47.6 / 46.9 / 69
//   units, one per lane, the fields interleaved (now)        246 / 47.4 / 42.5 / 68
// (at 512^3 in a step, where the substep leaves lines in the caches: 247 -> 219)
constexpr int HX_ROWS = 32, HALO_THR = 256;

template <typename E, bool THIN>
__global__ __launch_bounds__(HALO_THR) void k_halo(Grid g, int rblocks, float inv_units, float inv_my,
                                                   float inv_2r, float inv_ny, E* __restrict__ fields)
{
    constexpr int V = 16 / sizeof(E);
    // (one access each; the hardware takes unaligned ones)
    typedef E Unit __attribute__((ext_vector_type(V), aligned(sizeof(E))));
    const int r = g.r;
    const int block = (int)(blockIdx.y * (gridDim.x / NQ) + blockIdx.x / NQ);
    E* f = fields + (int64_t)(blockIdx.x % NQ) * g.fstride;
    if (block >= rblocks) {
        const int c = threadIdx.x & 7;
        if (c >= 2 * r) return;
        const int dst = c < r ? c : g.nx + c;  // padded halo column
        const int src = wrap_index<THIN>(dst, g.nx, r);
        const int row = (block - rblocks) * HX_ROWS + (int)(threadIdx.x >> 3);
        if (row >= g.ny * g.nz) return;
        const int z = quotient(row, g.ny, inv_ny), y = row - z * g.ny;
        E* p = f + ((r + z) * g.my + r + y) * g.mx;
        p[dst] = p[src];
        return;
    }
    const int units = (g.mx + V - 1) / V;
    const int begin = block * HALO_THR, k0 = quotient(begin, units, inv_units);
    const int u = begin - k0 * units + (int)threadIdx.x, du = quotient(u, units, inv_units);
    const int x = V * (u - du * units);
    int k = k0 + du, z, y;  // the halo's row
    const bool planes = k < 2 * r * g.my;
    if (planes) {
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
    if (!planes && z >= r + g.nz) return;
    E* dst = f + (z * g.mxy + y * g.mx + x);
    const E* src = f + (wrap_index<THIN>(z, g.nz, r) * g.mxy + wrap_index<THIN>(y, g.ny, r) * g.mx);
    Unit v;  // (both kinds of unit in flight before either is stored)
    if (x >= r && x + V <= r + g.nx) {
        v = *reinterpret_cast<const Unit*>(src + x);
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = src[wrap_index<THIN>(min(x + e, g.mx - 1), g.nx, r)];
    }
    if (x + V <= g.mx) {
        *reinterpret_cast<Unit*>(dst) = v;
    } else {
#pragma unroll
        for (int e = 0; e + 1 < V; ++e)
            if (x + e < g.mx) dst[e] = v[e];
    }
}

template <typename E>
void launch_halo_typed(const Grid& g, void* fields, hipStream_t st)
{
    const int64_t row = (g.mx + 16 / sizeof(E) - 1) / (16 / sizeof(E));
    const int64_t units = 2 * g.r * ((int64_t)g.my + g.nz) * row;
    const int64_t rblocks = (units + HALO_THR - 1) / HALO_THR;
    const int64_t blocks = rblocks + ((int64_t)g.ny * g.nz + HX_ROWS - 1) / HX_ROWS;
    // (a dimension holds fewer than 2^32 threads; what the fold adds at the end has no row)
    const int64_t fold = (blocks >> 20) + 1;
    const dim3 grid((unsigned)(NQ * ((blocks + fold - 1) / fold)), (unsigned)fold);
    const bool thin = g.nx < g.r || g.ny < g.r || g.nz < g.r;
    hipLaunchKernelGGL((thin ? k_halo<E, true> : k_halo<E, false>), grid, dim3(HALO_THR), 0, st, g,
                       (int)rblocks, 1.0f / (float)row, 1.0f / (float)g.my, 1.0f / (float)(2 * g.r),
                       1.0f / (float)g.ny, (E*)fields);
}

}  // namespace

hipError_t launch_halo(const Grid& g, void* fields, int elem_size, hipStream_t st)
{
    if (elem_size == 8) launch_halo_typed<uint64_t>(g, fields, st);
    else launch_halo_typed<uint32_t>(g, fields, st);
    return hipGetLastError();
}

}  // namespace mhd
