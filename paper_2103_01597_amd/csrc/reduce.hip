// Deterministic reductions over the interior of one field, in one launch.
// Block b walks rows b, b + G, b + 2G, ... (G blocks) with each thread
// striding x by 256, then a fixed LDS tree; the block that ends last combines
// the G partials in the same fixed tree and writes the result to the host.
// FP64 accumulation throughout, so the result depends only on the data, never
// on timing.
//
// Bound by memory latency where a thread waits for each value before it fetches
// the next (256^3 FP64: 53 us, 2.5 TB/s), so RED_AHEAD values are fetched at a
// time and then added in the same order: 32 us, 4.2 TB/s (8 at a time: 33).  A
// second launch for the partials and a copy of the result cost 14 us more, with
// the gaps between them.
#include "mhd_internal.hpp"

namespace mhd {
namespace {

__device__ __forceinline__ double nan_max(double a, double b)
{
    return (isnan(a) || isnan(b)) ? __longlong_as_double(0x7ff8000000000000LL) : (a > b ? a : b);
}
__device__ __forceinline__ double nan_min(double a, double b)
{
    return (isnan(a) || isnan(b)) ? __longlong_as_double(0x7ff8000000000000LL) : (a < b ? a : b);
}

__device__ __forceinline__ double red_init(int op)
{
    if (op == MHD_RED_MIN) return __longlong_as_double(0x7ff0000000000000LL);   // +inf
    if (op == MHD_RED_MAX) return -__longlong_as_double(0x7ff0000000000000LL);  // -inf
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
__device__ __forceinline__ double red_comb(double a, double b, int op)
{
    switch (op) {
    case MHD_RED_MAXABS:
    case MHD_RED_MAX: return nan_max(a, b);
    case MHD_RED_MIN: return nan_min(a, b);
    default: return a + b;
    }
}

__device__ double block_tree(double v, int op, double* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h)
            sh[t] = red_comb(sh[t], sh[t + h], op);
        __syncthreads();
    }
    return sh[0];
}

constexpr int RED_AHEAD = 16;

template <typename E, int op>
__global__ __launch_bounds__(256) void k_reduce(Grid g, const E* __restrict__ f, double* partials,
                                                unsigned* ended, double* out)
{
    __shared__ double sh[256];
    __shared__ bool last;
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
            x += 256;
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
    if (t == 0) {
        __hip_atomic_store(partials + blockIdx.x, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // The partial has reached memory before the count does.  (Both bypass the
        // caches that are not shared, so no cache is written back or
        // invalidated for this; an acquire-release count does that in every
        // block, and the launch takes 66 us instead of 32.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = __hip_atomic_fetch_add(ended, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1u;
    }
    __syncthreads();
    if (!last) return;
    acc = red_init(op);
    for (int i = t; i < G; i += 256)
        acc = red_comb(acc, __hip_atomic_load(partials + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), op);
    const double total = block_tree(acc, op, sh);
    if (t == 0) {
        __hip_atomic_store(ended, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
        __hip_atomic_store(out, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <typename E>
hipError_t launch_typed(const Grid& g, const E* f, int op, double* partials, unsigned* ended,
                        double* out, hipStream_t st)
{
    const int64_t rows = (int64_t)g.ny * g.nz;
    const dim3 grid((unsigned)(rows < REDUCE_BLOCKS ? rows : REDUCE_BLOCKS));
#define MHD_REDUCE(OP) \
    case OP: hipLaunchKernelGGL((k_reduce<E, OP>), grid, dim3(256), 0, st, g, f, partials, ended, out); break
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

// partials: REDUCE_BLOCKS doubles of device memory; ended: a device counter
// that is zero before and after; result: memory of the host that the device
// writes.  Launches that share them must not overlap.
hipError_t launch_reduce(const Grid& g, const void* field, int elem_size, int op, double* partials,
                         unsigned* ended, double* result, hipStream_t st)
{
    return elem_size == 8 ? launch_typed(g, (const double*)field, op, partials, ended, result, st)
                          : launch_typed(g, (const float*)field, op, partials, ended, result, st);
}

}  // namespace mhd
