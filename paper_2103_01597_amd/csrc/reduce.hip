// Deterministic reductions over the interior of one field, in one launch.
// Block b walks rows b, b + G, b + 2G, ... (G blocks) with each thread
// striding x by 256, then a fixed LDS tree, and writes its partial to pinned host
// memory; once the launch has ended the host combines the G partials in the same
// fixed tree (combine_partials).  FP64 accumulation throughout, so the result
// depends only on the data, never on timing, and nothing is kept from one call for
// the next: every partial that is read was written by the call's own launch.
//
// Bound by memory latency where a thread waits for each value before it fetches
// the next, so RED_AHEAD values are fetched at a time and then added in the same
// order (8 at a time: 3% slower at 256^3).  A call at 256^3 and 32^3, FP64: 58 and 23 us
// with one value at a time, a second launch for the partials and a copy of the result;
// 44 and 31 with the block that ends last combining the partials, which takes a count of
// ended blocks (one address for all of them, and a value that outlives the call);
// 38 and 21 now.
#include <math.h>

#include "mhd_internal.hpp"

namespace mhd {
namespace {

__host__ __device__ __forceinline__ double nan_max(double a, double b)
{
    return (isnan(a) || isnan(b)) ? __builtin_nan("") : (a > b ? a : b);
}
__host__ __device__ __forceinline__ double nan_min(double a, double b)
{
    return (isnan(a) || isnan(b)) ? __builtin_nan("") : (a < b ? a : b);
}

__host__ __device__ __forceinline__ double red_init(int op)
{
    if (op == MHD_RED_MIN) return __builtin_huge_val();
    if (op == MHD_RED_MAX) return -__builtin_huge_val();
    return 0.0;
}
__device__ __forceinline__ double red_map(double v, int op)
{
    switch (op) {
    case MHD_RED_SUMSQ: return v * v;
    case MHD_RED_SUMEXP: return exp(v);
    case MHD_RED_NONFINITE: return isfinite(v) ? 0.0 : 1.0;
    case MHD_RED_MAXABS: return fabs(v);
    default: return v;
    }
}
__host__ __device__ __forceinline__ double red_comb(double a, double b, int op)
{
    switch (op) {
    case MHD_RED_MAXABS:
    case MHD_RED_MAX: return nan_max(a, b);
    case MHD_RED_MIN: return nan_min(a, b);
    default: return a + b;
    }
}

constexpr int RED_THR = 256;

__device__ double block_tree(double v, int op, double* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int h = RED_THR / 2; h > 0; h >>= 1) {
        if (t < h)
            sh[t] = red_comb(sh[t], sh[t + h], op);
        __syncthreads();
    }
    return sh[0];
}

constexpr int RED_AHEAD = 16;

template <typename E, int op>
__global__ __launch_bounds__(RED_THR) void k_reduce(Grid g, const E* __restrict__ f,
                                                    double* __restrict__ partials)
{
    __shared__ double sh[RED_THR];
    double acc = red_init(op);
    const int G = gridDim.x, rows = g.ny * g.nz, t = threadIdx.x;
    const int dj = G % g.ny, dk = G / g.ny;
    int x = t, r = t < g.nx ? (int)blockIdx.x : rows;  // the thread's next value: row r = (j, k)
    int j = r % g.ny, k = r / g.ny;
    while (r < rows) {
        E v[RED_AHEAD];
        bool ok[RED_AHEAD];
#pragma unroll
        for (int u = 0; u < RED_AHEAD; ++u) {
            ok[u] = r < rows;  // past the end the first cell stands in
            v[u] = f[g.interior + (ok[u] ? (int64_t)k * g.mxy + j * g.mx + x : 0)];
            x += RED_THR;
            if (x >= g.nx) {
                x = t;
                r += G;
                j += dj;
                k += dk;
                if (j >= g.ny) {
                    j -= g.ny;
                    ++k;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < RED_AHEAD; ++u) {
            const double c = red_comb(acc, red_map(double(v[u]), op), op);
            acc = ok[u] ? c : acc;
        }
    }
    const double b = block_tree(acc, op, sh);
    if (t == 0) partials[blockIdx.x] = b;
}

template <typename E>
hipError_t launch_typed(const Grid& g, const E* f, int op, double* partials, hipStream_t st)
{
    const dim3 grid(reduce_blocks(g));
#define MHD_REDUCE(OP) \
    case OP: hipLaunchKernelGGL((k_reduce<E, OP>), grid, dim3(RED_THR), 0, st, g, f, partials); break
    switch (op) {
        MHD_REDUCE(MHD_RED_SUM);
        MHD_REDUCE(MHD_RED_SUMSQ);
        MHD_REDUCE(MHD_RED_MAXABS);
        MHD_REDUCE(MHD_RED_MIN);
        MHD_REDUCE(MHD_RED_MAX);
        MHD_REDUCE(MHD_RED_SUMEXP);
        MHD_REDUCE(MHD_RED_NONFINITE);
    default: return hipErrorInvalidValue;
    }
#undef MHD_REDUCE
    return hipGetLastError();
}

}  // namespace

int reduce_blocks(const Grid& g)
{
    const int64_t rows = (int64_t)g.ny * g.nz;
    return (int)(rows < REDUCE_BLOCKS ? rows : REDUCE_BLOCKS);
}

// partials: reduce_blocks(g) doubles of pinned host memory
hipError_t launch_reduce(const Grid& g, const void* field, int elem_size, int op, double* partials,
                         hipStream_t st)
{
    return elem_size == 8 ? launch_typed(g, (const double*)field, op, partials, st)
                          : launch_typed(g, (const float*)field, op, partials, st);
}

// As one block of RED_THR threads would: thread t takes partials t, t + RED_THR, ..., then
// the tree of block_tree.
double combine_partials(const double* partials, int n, int op)
{
    double v[RED_THR];
    for (int t = 0; t < RED_THR; ++t) {
        v[t] = red_init(op);
        for (int i = t; i < n; i += RED_THR) v[t] = red_comb(v[t], partials[i], op);
    }
    for (int h = RED_THR / 2; h > 0; h >>= 1)
        for (int t = 0; t < h; ++t) v[t] = red_comb(v[t], v[t + h], op);
    return v[0];
}

}  // namespace mhd
