// Learned-closure kernels for gfx950 (declared in include/mhdnn.h).
//
// Periodic 3x3x3 convolutions run as implicit GEMMs on the BF16 matrix
// cores (FP32 accumulation).  A block owns a slab of 256 cells per plane
// (full periodic rows) and marches it through a chunk of planes, with a ring
// of planes (the slab plus one row on each side) in LDS and the next plane
// prefetched into registers:
//   * forward / data gradient (v_mfma_f32_16x16x32_bf16): M = output
//     channels, N = cells, K = 32 input channels of one tap, or 4 taps x 8
//     channels; see k_conv.
//   * weight gradient (v_mfma_f32_32x32x16_bf16, 9 waves): M = output
//     channels, N = input channels (or 4 taps x 8 channels for 8-channel
//     inputs), K = cells; wave w owns the taps of x shift w/3 - 1 and z
//     offset w%3 - 1; see k_wgrad.  Per-block partial sums go to a workspace that a second kernel reduces
//     in a fixed order (deterministic).
// MFMA lane layouts.  16x16x32: lane l holds A row l%16 and B column l%16 at
// K = 8(l/16)..8(l/16)+7; accumulator i of lane l is D[4(l/16) + i][l%16].
// 32x32x16: A row l%32 and B column l%32 at K = 8(l/32)..8(l/32)+7;
// accumulator r is D[8(r/4) + 4(l/32) + r%4][l%32].
#include <mutex>

#include "mhd_internal.hpp"
#include "../../include/mhdnn.h"

namespace mhd {

const Grid* ctx_grid(const mhd_ctx* ctx);
int ctx_precision(const mhd_ctx* ctx);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
// four consecutive channels of one cell, wherever the caller's buffer starts
// (one access each; the hardware takes unaligned ones)
typedef unsigned short u16x4 __attribute__((ext_vector_type(4), aligned(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Round-to-nearest-even FP32 -> BF16 (NaN stays NaN): one hardware
// conversion instruction on gfx950.
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// erfc(z) / 2 for z >= 0 as t exp(-z^2 + P(t)) / 2 with t = 1 / (1 + z/2)
// and P the degree-9 Chebyshev fit of Press et al. (Numerical Recipes,
// Sec. 6.2): relative error below 1.2e-7 in exact arithmetic, and branch
// free.  In FP32 the GELU built on it stays within 2e-5 relative error on
// [-12, 12], the negative tail included (where 1 + erf(x) would cancel).
__device__ __forceinline__ float half_erfc(float z)
{
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.5f * z);
    float p = 0.17087277f;
    p = fmaf(p, t, -0.82215223f);
    p = fmaf(p, t, 1.48851587f);
    p = fmaf(p, t, -1.13520398f);
    p = fmaf(p, t, 0.27886807f);
    p = fmaf(p, t, -0.18628806f);
    p = fmaf(p, t, 0.09678418f);
    p = fmaf(p, t, 0.37409196f);
    p = fmaf(p, t, 1.00002368f);
    p = fmaf(p, t, -1.26551223f);
    return 0.5f * t * __expf(fmaf(-z, z, p));
}
// Standard normal distribution function Phi(v) = erfc(-v / sqrt 2) / 2.
__device__ __forceinline__ float normal_cdf(float v)
{
    const float h = half_erfc(fabsf(v) * 0.70710678118654752f);
    return v >= 0.0f ? 1.0f - h : h;
}
// GELU(v) = v Phi(v) (exact-erf form) and its derivative Phi(v) + v phi(v).
__device__ __forceinline__ float gelu(float v) { return v * normal_cdf(v); }
__device__ __forceinline__ float gelu_grad(float v)
{
    return normal_cdf(v) + v * __expf(-0.5f * v * v) * 0.39894228040143268f;
}

__device__ __forceinline__ bf16x8 frag(const uint16_t* p)  // 16-byte aligned
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(p));
}

constexpr int NTHR = 256;

// ------------------------------------------------------------------ conv
// MODE 0: hidden layer (z, GELU(z) as BF16); 1: output layer (FP32);
// 2: data gradient (times GELU'(zprev), BF16).
//
// A block of CONV_THR threads owns a slab of CONV_CELLS / n full periodic
// rows and marches it through a chunk of zc planes; each of its 8 waves owns
// 64 of the slab plane's cells (four tiles of 16, whole rows: w % 4) and 16 of
// the output channels (w / 4).  With 8 output channels waves 4..7 only move
// planes.  The weights are the A operand and stay in registers for the whole
// march; the cells are the B operand, so that a lane ends with four
// consecutive output channels of a cell and stores them in one access.
//
// The bound is the instruction stream of a wave (LDS fragment reads, products,
// the rounding and GELU of the results) before memory (the bytes alone would take
// 0.45 to 0.48 of the time at the copy rate).  So:
//   * one fragment read serves the three taps along x: each has an accumulator
//     of its own over the unshifted cells, and the three are shifted and added
//     at the plane's end by DPP moves inside the rows of 16 lanes.  That is 9
//     (3) reads per tile and plane for 32 (8) input channels instead of 27
//     (14) of a shifted cell each, and no partial sums pass through LDS.
//   * the ring holds four planes, so one barrier per plane is enough.
//   * with 32 input channels waves w and w + 4 share a SIMD unit; one finishes
//     a plane right after its products, the other during the next plane, before
//     that one's products: one's epilogue then runs beside the other's matrix
//     instructions.  With 8 input channels the products are too few for that;
//     each wave's epilogue is interleaved with its own next products instead.
// 4 fields of 64^3 cells, 8 -> 32, 32 -> 32 and 32 -> 8 channels, forward: 62, 96
// and 54 us with a read per tap, 32x32x16 products and scalar stores; 52, 74 and 37
// now (data gradients of the last two: 97 and 58, now 78 and 50).  Without the
// skew 32 -> 32 takes 81; with it 8 -> 32 takes 62.
constexpr int CONV_THR = 512;
constexpr int WG_THR = 576;  // weight gradient: 9 waves, one per (dx, dz) tap triple
constexpr int CONV_CELLS = 256;  // cells per plane per block

// LDS row pitch (elements) per cell of the input ring, padded so that
// consecutive lanes' 16-byte fragment reads start an odd number of 16-byte
// units apart (no bank conflicts).
template <int CIN>
constexpr int conv_cp() { return CIN == 32 ? CIN + 8 : CIN; }

// Whether a plane's results pass through LDS, from where the block stores them in whole
// cache lines: 32 FP32 channels are a line per cell, of which a wave has half, and with
// 8 input channels nothing else takes as long as the stores.  Non-temporal ones: outputs
// beyond the 256 MB that the memory-side cache holds gain by it and smaller ones lose nothing.  us for 8 -> 32
// channels, FP32, of 2, 4, 6, 8 and 16 x 64^3 cells: half lines 17.2, 29.7, 65, 86, 203; whole lines
// 16.5, 27.8, 59, 92, 184; non-temporal 17.8, 28.5, 60, 55, 104.  (Waves with all channels of 32 cells
// and one store per channel, the kernel before: 17.7, 30.2, 62, 72, 154.)
template <int CIN, int MODE, int COUT>
constexpr bool conv_staged() { return CIN == 8 && MODE == 1 && COUT == 32; }
constexpr int STAGE_CP = 36;  // floats per cell there

// DPP moves within rows of 16 lanes (one tile of cells): lane x takes lane x -+ 1,
// the first (last) lane takes the last (first) lane of the tile before (after).
__device__ __forceinline__ float from_left(float v, float left_tile)
{
    const int edge = __builtin_amdgcn_update_dpp(0, __float_as_int(left_tile), 0x121, 0xf, 0xf, true);
    return __int_as_float(__builtin_amdgcn_update_dpp(edge, __float_as_int(v), 0x111, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_right(float v, float right_tile)
{
    const int edge = __builtin_amdgcn_update_dpp(0, __float_as_int(right_tile), 0x12f, 0xf, 0xf, true);
    return __int_as_float(__builtin_amdgcn_update_dpp(edge, __float_as_int(v), 0x101, 0xf, 0xf, false));
}

template <int CIN, int MODE, int LOGN, int COUT>
__global__ __launch_bounds__(CONV_THR) void k_conv(const uint16_t* __restrict__ x,
                                                   const uint16_t* __restrict__ w,
                                                   const float* __restrict__ bias,
                                                   const uint16_t* __restrict__ zprev, int nch,
                                                   int zc, uint16_t* __restrict__ out0,
                                                   uint16_t* __restrict__ out1,
                                                   float* __restrict__ outf)
{
    extern __shared__ __align__(16) uint16_t sm[];
    constexpr int CP = conv_cp<CIN>(), n = 1 << LOGN;
    constexpr int RY = CONV_CELLS >> LOGN;        // rows per slab
    constexpr int SLOT = (RY + 2) * n * CP;       // elements per ring plane
    constexpr int NV = (RY + 2) * n * CIN / 8;    // 16-byte vectors per ring plane
    uint16_t* lx = sm;                            // [4][RY+2][n][CP]; CIN 8: and one cell of zeros
    constexpr int slabs = n / RY;
    const int col_id = blockIdx.x / nch, ch_id = blockIdx.x - col_id * nch;
    const int b = col_id / slabs, y0 = (col_id - b * slabs) * RY;
    const int z0 = ch_id * zc, nz = min(zc, n - z0);
    constexpr size_t n3 = (size_t)n * n * n;
    const uint16_t* xb = x + (size_t)b * n3 * CIN;
    const int tid = threadIdx.x, l = tid & 63, q16 = l >> 4, c16 = l & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ch0 = 16 * (wv >> 2);               // this wave's output channels
    const int mbase = 64 * (wv & 3);              // and its cells of the slab plane

    // ---- A fragments (weights, [32][27][CIN] with output channels padded to
    // 32) for the whole march, tap t = 3 p + dxi, p = 3 (dz + 1) + (dy + 1):
    // lane l holds row l%16.  32 input channels: K chunk 8(l/16) of tap t.  8:
    // quarter l/16 takes pair p = 4 g + l/16, so that one product spans four.
    constexpr int NP = CIN == 32 ? 9 : 3;
    bf16x8 aw[NP][3];
#pragma unroll
    for (int g = 0; g < NP; ++g)
#pragma unroll
        for (int dxi = 0; dxi < 3; ++dxi) {
            const uint16_t* row = w + (size_t)(ch0 + c16) * 27 * CIN;
            if constexpr (CIN == 32) {
                aw[g][dxi] = frag(row + (3 * g + dxi) * 32 + 8 * q16);
            } else {
                const int p = 4 * g + q16;
                aw[g][dxi] = p < 9 ? frag(row + (3 * p + dxi) * 8) : bf16x8{};
            }
        }

    // ---- plane loads: vector i of ring plane z = rows y0-1 .. y0+RY (periodic).
    // Threads past the last vector skip it (MASKED), or move it once more, which
    // costs registers for the clamped places but leaves the loop without a branch.
    constexpr int NL = (NV + CONV_THR - 1) / CONV_THR;
    constexpr bool MASKED = CIN == 32 && NV % CONV_THR != 0;
    u16x8 pre[NL];
    unsigned src[NL];  // this lane's vectors within a plane,
    int dst[NL];       // and in the ring
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int i = tid + k * CONV_THR, e = (MASKED ? i : min(i, NV - 1)) * 8;
        const int cell = e / CIN, ch = e - cell * CIN;
        const int xx = cell & (n - 1), yy = (y0 - 1 + (cell >> LOGN) + n) & (n - 1);
        src[k] = (unsigned)(((yy << LOGN) + xx) * CIN + ch);
        dst[k] = cell * CP + ch;
    }
    auto mine = [&](int k) { return !MASKED || tid + k * CONV_THR < NV; };
    auto load = [&](int z) {
        const uint16_t* plane = xb + ((size_t)((z + n) & (n - 1)) << (2 * LOGN)) * CIN;
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (mine(k)) pre[k] = *reinterpret_cast<const u16x8*>(plane + src[k]);
    };
    auto store = [&](int sl) {
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (mine(k)) *reinterpret_cast<u16x8*>(lx + sl * SLOT + dst[k]) = pre[k];
    };
    if (CIN == 8 && tid < 8) lx[4 * SLOT + tid] = 0;
    load(z0 - 1);
    store(0);
    load(z0);
    store(1);
    load(z0 + 1);

    const int ch = ch0 + 4 * q16;  // first of this lane's four output channels
    float bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[i] = MODE != 2 && ch < COUT ? bias[ch + i] : 0.0f;
    // element of the outputs where the slab's plane z0 + p starts (uniform), and
    // this lane's channels of its first tile's cell from there
    auto out_plane = [&](int p) {
        return ((size_t)b * n3 + ((size_t)(z0 + p) << (2 * LOGN)) + ((size_t)y0 << LOGN)) * COUT;
    };
    const unsigned lane_out = (unsigned)((mbase + c16) * COUT + ch);
    constexpr bool STAGED = conv_staged<CIN, MODE, COUT>();
    float* stage = reinterpret_cast<float*>(lx + 4 * SLOT + 8);  // [2][CONV_CELLS][STAGE_CP]
    floatx4 res[4];
    u16x4 zp[4];
    auto finish = [&](int p) {  // plane z0 + p's results, four channels per lane and tile
        if (COUT < 32 && ch >= COUT) return;
        const size_t at = out_plane(p);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned o = lane_out + 16 * j * COUT;
            u16x4 a, g;
            floatx4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = res[j][i] + bv[i];
                if constexpr (MODE == 0) {
                    a[i] = f2bf(v[i]);
                    g[i] = f2bf(gelu(v[i]));
                } else if constexpr (MODE == 2) {
                    a[i] = f2bf(v[i] * gelu_grad(bf2f(zp[j][i])));
                }
            }
            if constexpr (STAGED)
                *reinterpret_cast<floatx4*>(stage + ((p & 1) * CONV_CELLS + mbase + 16 * j + c16) * STAGE_CP + ch) = v;
            else if constexpr (MODE == 1)
                *reinterpret_cast<f32x4u*>(outf + at + o) = v;
            else
                *reinterpret_cast<u16x4*>(out0 + at + o) = a;
            if constexpr (MODE == 0) *reinterpret_cast<u16x4*>(out1 + at + o) = g;
        }
    };
    auto flush = [&](int p) {  // plane z0 + p's staged results, a barrier after finish(p)
        if constexpr (STAGED) {
            float* out = outf + out_plane(p);
            const float* st = stage + (p & 1) * CONV_CELLS * STAGE_CP;
#pragma unroll
            for (int k = 0; k < CONV_CELLS * 8 / CONV_THR; ++k) {
                const int i = tid + k * CONV_THR;
                const f32x4u v = *reinterpret_cast<const floatx4*>(st + (i >> 3) * STAGE_CP + 4 * (i & 7));
                __builtin_nontemporal_store(v, reinterpret_cast<f32x4u*>(out + 4 * i));
            }
        }
    };
    int rbase[4];  // tile j's cell of this lane in the ring plane, row dy = -1
#pragma unroll
    for (int j = 0; j < 4; ++j) rbase[j] = (mbase + 16 * j + c16) * CP + (CIN == 32 ? 8 * q16 : 0);
    // the pre-activations of plane z0 + p's outputs (data gradient)
    auto load_zp = [&](int p) {
        if constexpr (MODE == 2) {
            if (COUT < 32 && ch >= COUT) return;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                zp[j] = *reinterpret_cast<const u16x4*>(zprev + out_plane(p) + (lane_out + 16 * j * COUT));
        }
    };
    auto products = [&](int p) {  // plane z0 + p
        // ring slot q holds the plane z0 - 1 + p' with p' = q (mod 4)
        floatx4 acc[3][4];  // [dx + 1][tile]
#pragma unroll
        for (int dxi = 0; dxi < 3; ++dxi)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[dxi][j] = floatx4{};
        const int sb[3] = {(p & 3) * SLOT, ((p + 1) & 3) * SLOT, ((p + 2) & 3) * SLOT};
#pragma unroll
        for (int g = 0; g < NP; ++g) {
            int off;  // ring offset of the fragments' (dz, dy) row relative to the cell
            bool pad = false;  // past the ninth pair: zeros (not a cell, which need not be finite)
            if constexpr (CIN == 32) {
                off = sb[g / 3] + (g % 3) * n * CP;
            } else {
                const int pr = min(4 * g + q16, 8), dz = pr / 3, dy = pr - 3 * dz;
                pad = 4 * g + q16 > 8;
                off = (dz == 0 ? sb[0] : dz == 1 ? sb[1] : sb[2]) + dy * n * CP;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bf16x8 v = frag(lx + (pad ? 4 * SLOT : off + rbase[j]));
#pragma unroll
                for (int dxi = 0; dxi < 3; ++dxi)
                    acc[dxi][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[g][dxi], v, acc[dxi][j], 0, 0, 0);
            }
        }
        // y(x) = D_-1(x - 1) + D_0(x) + D_+1(x + 1) along the periodic row, whose
        // n / 16 tiles are consecutive ones of this wave
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            constexpr int TPR = n / 16;  // tiles per row
            const int jl = j / TPR * TPR + (j + TPR - 1) % TPR, jr = j / TPR * TPR + (j + 1) % TPR;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                res[j][i] = acc[1][j][i] + from_left(acc[0][j][i], acc[0][jl][i]) +
                            from_right(acc[2][j][i], acc[2][jr][i]);
        }
    };
    // the instruction order of an epilogue and the products after it: a group's
    // fragments one group ahead, VPP vector instructions beside each product
    auto interleave = [&]() {
        constexpr int VPP = MODE == 1 ? 1 : 11;
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int g = 0; g < NP; ++g) {
            if (g + 1 < NP) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, VPP, 0);
            }
        }
    };
    // The plane after next is fetched and the next one put into the ring at each
    // plane's start; with four slots one barrier per plane is enough (a wave that
    // runs ahead overwrites the plane before the three that others still read).
    // Each plane's loads are issued before the stores of the plane finished
    // beside it, and no branch lies between (the last plane is fetched again
    // instead): the wait for the loads then counts past exactly those stores.
    // With a branch the compiler waits for all of them, on every plane.
    auto turn = [&](int p) {
        store((p + 2) & 3);  // plane z0+p+1
        __syncthreads();
        load(z0 + min(p + 2, nz));
    };
    turn(0);
    if (ch0 >= COUT) {  // no output channels: this wave only moves planes
        for (int p = 1; p < nz; ++p) turn(p);
    } else if (STAGED || (CIN == 32 && wv < 4)) {
        load_zp(0);
        products(0);
        finish(0);
        for (int p = 1; p < nz; ++p) {
            turn(p);
            flush(p - 1);
            load_zp(p);
            products(p);
            finish(p);
        }
        if constexpr (STAGED) {
            __syncthreads();
            flush(nz - 1);
        }
    } else {
        products(0);
        for (int p = 1; p < nz; ++p) {
            load_zp(p - 1);
            turn(p);
            finish(p - 1);
            products(p);
            if constexpr (CIN == 8) interleave();
        }
        load_zp(nz - 1);
        finish(nz - 1);
    }
}

// --------------------------------------------------------------- wgrad
// Weight gradient dW[o][t][c] = sum over cells of dz[cell][o] x[cell + off(t)][c]
// (and db[o] = sum dz[cell][o]) on the same slabs and z chunks as k_conv.
// M = output channels, N = input channels (or 4 (dz, dy) taps x 8 channels
// for 8-channel inputs), K = cells.  Over one full periodic x-row,
// sum_x dz(x) x(x + dx) = sum_q dz(q - dx) x(q): the x shift is taken by the
// dz operand, so that three x rows share its fragment.  Each block
// accumulates its chunk in registers and writes one partial sum per weight;
// k_wgrad_reduce adds the partials in a fixed order (deterministic).
//
// x is kept in a ring of four planes and dz in two alternating ones, both
// channels last as they come from memory, and a fragment (8 cells of one
// channel per lane) is two transposing reads: of each 16 lanes lane j names
// 4 channels of cell j/4, and lane i receives channel i of the 4 cells.  Each
// lane names its own cell, so the shift and its periodic wrap are part of the
// address.  The bound is the matrix cores (the 9 waves leave one SIMD unit
// with three) and the reads beside them.  With transposed planes, written by
// 2-byte LDS stores with three shifted copies of dz, those stores were: 4 x
// 64^3 cells, 8 -> 32, 32 -> 32 and 32 -> 8 channels took 74, 100 and 59 us;
// 41, 69 and 36 now.
//
// Bank layout: 4 consecutive cells' 32 bytes must lie in different banks.  32
// channels: the two halves of a cell's 64 bytes are exchanged in every other
// pair of cells.  8 channels: rows and planes are padded by 64 bytes, so that
// the two taps that 16 lanes read lie 64 bytes apart modulo the 128 read at a
// time.
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 frag_cells(const uint16_t* c0, const uint16_t* c4)
{
    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
    union {
        s16x4 h[2];
        bf16x8 v;
    } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)c0);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)c4);
    return u.v;
}

// Offset of channels c, c+1, .. of cell x within an LDS row of C channels
template <int C>
__device__ __forceinline__ int in_row(int x, int c)
{
    return x * C + (C == 32 ? c ^ ((x & 2) << 3) : c);
}
// LDS elements of a row and of a ring plane of x
template <int CIN>
constexpr int wg_row(int n) { return n * CIN + (CIN == 8 ? 32 : 0); }
template <int CIN>
constexpr int wg_slot(int n) { return (CONV_CELLS / n + 2) * wg_row<CIN>(n) + (CIN == 8 ? 32 : 0); }

template <int CIN, int COUT, int LOGN>
__global__ __launch_bounds__(WG_THR) void k_wgrad(const uint16_t* __restrict__ x,
                                                    const uint16_t* __restrict__ dz, int nch,
                                                    int zc, float* __restrict__ ws,
                                                    float* __restrict__ wsb)
{
    extern __shared__ __align__(16) uint16_t sm[];
    constexpr int n = 1 << LOGN, RY = CONV_CELLS >> LOGN;
    constexpr int ROW = wg_row<CIN>(n), SLOT = wg_slot<CIN>(n), DPLANE = CONV_CELLS * COUT;
    uint16_t* xs = sm;             // [4 planes][RY + 2][n][CIN]
    uint16_t* ds = sm + 4 * SLOT;  // [2 planes][RY][n][COUT]
    float* bsum = reinterpret_cast<float*>(ds + 2 * DPLANE);  // [WG_THR][8]
    constexpr int slabs = n / RY;
    const int col_id = blockIdx.x / nch, ch_id = blockIdx.x - col_id * nch;
    const int b = col_id / slabs, y0 = (col_id - b * slabs) * RY;
    const int z0 = ch_id * zc, nz = min(zc, n - z0);
    constexpr size_t n3 = (size_t)n * n * n;
    const uint16_t* xb = x + (size_t)b * n3 * CIN;
    const uint16_t* db = dz + (size_t)b * n3 * COUT + ((size_t)y0 << LOGN) * COUT;
    const int tid = threadIdx.x, l = tid & 63, h = l >> 5, col = l & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- plane loads (16-byte vectors of 8 channels of one cell)
    constexpr int NVX = (RY + 2) * n * CIN / 8, NLX = (NVX + WG_THR - 1) / WG_THR;
    constexpr int NVD = CONV_CELLS * COUT / 8, NLD = (NVD + WG_THR - 1) / WG_THR;
    u16x8 px[NLX], pd[NLD];
    auto load_x = [&](int z) {
        const uint16_t* plane = xb + ((size_t)((z + n) & (n - 1)) << (2 * LOGN)) * CIN;
#pragma unroll
        for (int k = 0; k < NLX; ++k) {
            const int i = tid + k * WG_THR;
            if (i < NVX) {
                const int cell = i / (CIN / 8), cg = (i - cell * (CIN / 8)) * 8;
                const int yy = (y0 - 1 + (cell >> LOGN) + n) & (n - 1);
                px[k] = *reinterpret_cast<const u16x8*>(
                    plane + (((yy << LOGN) + (cell & (n - 1))) * CIN + cg));
            }
        }
    };
    auto store_x = [&](int sl) {
#pragma unroll
        for (int k = 0; k < NLX; ++k) {
            const int i = tid + k * WG_THR;
            if (i < NVX) {
                const int cell = i / (CIN / 8), cg = (i - cell * (CIN / 8)) * 8;
                *reinterpret_cast<u16x8*>(xs + sl * SLOT + (cell >> LOGN) * ROW +
                                          in_row<CIN>(cell & (n - 1), cg)) = px[k];
            }
        }
    };
    auto load_dz = [&](int z) {
        const uint16_t* plane = db + ((size_t)z << (2 * LOGN)) * COUT;
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            const int i = tid + k * WG_THR;
            if (i < NVD) pd[k] = *reinterpret_cast<const u16x8*>(plane + i * 8);
        }
    };
    float bacc[8] = {};  // bias partials of this thread's 8 output channels
    auto store_dz = [&](int sl) {
#pragma unroll
        for (int k = 0; k < NLD; ++k) {
            const int i = tid + k * WG_THR;
            if (i < NVD) {
                const int cell = i / (COUT / 8), og = (i - cell * (COUT / 8)) * 8;
#pragma unroll
                for (int q = 0; q < 8; ++q) bacc[q] += bf2f(pd[k][q]);
                *reinterpret_cast<u16x8*>(ds + sl * DPLANE + in_row<COUT>(cell, og)) = pd[k];
            }
        }
    };

    // accumulator sets of wave wv (9 waves): CIN 32: the taps with x shift
    // dx = wv/3 - 1 and z offset dz = wv%3 - 1, one set per dy = -1, 0, 1, so
    // the three share each dz fragment; CIN 8: tap group g = wv (g = 3*dxi +
    // gi, gi selects 4 of the 9 (dz, dy) pairs).  CIN 32 with 8 output
    // channels: the 32 rows of the one set are (dx shift, o) pairs, rows
    // 8 (dx + 1) + o, the last 8 rows unused, for the taps with dz = wv%3 - 1
    // and dy = wv/3 - 1 (three times fewer products than three sets of 8
    // channels padded to 32).
    constexpr bool PACK_DX = CIN == 32 && COUT == 8;
    constexpr int NSET = CIN == 32 && !PACK_DX ? 3 : 1;
    floatx16 acc[NSET];
#pragma unroll
    for (int i = 0; i < NSET; ++i) acc[i] = floatx16{};

    // ---- what this lane names for a chunk of 16 cells from q0 in a row, in
    // its two reads (t = 0, 1): cell q0 + 8h + 4t + jc, channels (or tap and
    // channels) j4 .. j4 + 3 of the operand's 32
    const int jc = (l & 15) >> 2, j4 = 16 * ((l >> 4) & 1) + 4 * (l & 3);
    // dz at q - dx: only the first cell of a row (dx = 1) and the last one
    // (dx = -1) wrap, in the row's first and last chunk.  Output channels past
    // COUT repeat others and are not written.
    const int s = PACK_DX ? min(j4 >> 3, 2) : wv / 3;  // dx + 1
    const int o4 = COUT == 8 ? j4 & 7 : j4, e0 = 8 * h + jc + 1 - s, e1 = e0 + 4;
    // (e0 + 16: the pattern of in_row repeats every 4 cells)
    const int d0 = in_row<COUT>(e0 + 16, o4) - 16 * COUT, d0_first = d0 + (e0 < 0 ? n * COUT : 0);
    const int d1 = in_row<COUT>(e1, o4), d1_last = d1 - (e1 > 15 ? n * COUT : 0);
    // x: the ring plane dz + 1 and the offset in it
    const int pr = min(4 * (wv % 3) + (j4 >> 3), 8);  // CIN 8: (dz, dy) pair, the last repeated
    const int xz = CIN == 8 ? pr / 3 : wv % 3, xy = CIN == 8 ? pr % 3 : PACK_DX ? wv / 3 : 0;
    const int xo = xy * ROW + in_row<CIN>(8 * h + jc, CIN == 8 ? j4 & 7 : j4);

    load_x(z0 - 1);
    store_x(0);
    load_x(z0);
    store_x(1);
    load_x(z0 + 1);
    load_dz(z0);
    for (int p = 0; p < nz; ++p) {
        store_x((p + 2) & 3);  // plane z0+p+1 replaces plane z0+p-3
        store_dz(p & 1);       // plane z0+p
        __syncthreads();       // (all waves are past the products of plane z0+p-1)
        if (p + 1 < nz) {
            load_x(z0 + p + 2);
            load_dz(z0 + p + 1);
        }
        const uint16_t* xl = xs + ((p + xz) & 3) * SLOT + xo;
        const uint16_t* dl = ds + (p & 1) * DPLANE;
#pragma unroll
        for (int kc = 0; kc < CONV_CELLS / 16; ++kc) {
            const int rr = kc * 16 >> LOGN, q0 = kc * 16 & (n - 1);
            const uint16_t* dk = dl + kc * 16 * COUT;
            const bf16x8 a = frag_cells(dk + (q0 == 0 ? d0_first : d0),
                                        dk + (q0 + 16 == n ? d1_last : d1));
            const uint16_t* xk = xl + rr * ROW + q0 * CIN;
#pragma unroll
            for (int si = 0; si < NSET; ++si)  // dy = si - 1
                acc[si] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    a, frag_cells(xk + si * ROW, xk + si * ROW + 4 * CIN), acc[si], 0, 0, 0);
        }
    }

    // ---- this block's partial sums: ws[block][t][o][c], wsb[block][o]
    float* wb = ws + (size_t)blockIdx.x * 27 * 32 * 32;
#pragma unroll
    for (int si = 0; si < NSET; ++si) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = 8 * (r >> 2) + 4 * h + (r & 3);
            if (!PACK_DX && o >= COUT) continue;
            int t, c, oo = o;
            if constexpr (PACK_DX) {
                if (o >= 24) continue;
                oo = o & 7;
                t = 9 * (wv % 3) + 3 * (wv / 3) + (o >> 3);
                c = col;
            } else if constexpr (CIN == 32) {
                t = 9 * (wv % 3) + 3 * si + wv / 3;  // t = 9 (dz+1) + 3 (dy+1) + (dx+1)
                c = col;
            } else {
                const int tg = col >> 3, pr = 4 * (wv % 3) + tg;
                if (pr >= 9) continue;
                t = 9 * (pr / 3) + 3 * (pr % 3) + wv / 3;
                c = col & 7;
            }
            wb[(t * 32 + oo) * 32 + c] = acc[si][r];
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) bsum[tid * 8 + q] = bacc[q];
    __syncthreads();
    if (tid < COUT) {  // output channel o = tid: threads with og = 8 (o / 8), in order
        const int g = tid >> 3, q = tid & 7;
        float sacc = 0.0f;
        for (int j = g; j < (NVD < WG_THR ? NVD : WG_THR); j += COUT / 8) sacc += bsum[j * 8 + q];
        wsb[blockIdx.x * 32 + tid] = sacc;
    }
}

// Outputs per workgroup of k_wgrad_reduce: NTHR threads = RED_SEGS waves of
// RED_OUT lanes, wave k summing the k-th quarter of the blocks' partials.
constexpr int RED_SEGS = 4, RED_OUT = NTHR / RED_SEGS;

__global__ __launch_bounds__(NTHR) void k_wgrad_reduce(const float* __restrict__ ws,
                                                       const float* __restrict__ wsb, int nblocks,
                                                       int cin, int cout, float* __restrict__ dw,
                                                       float* __restrict__ dbias)
{
    // One lane per weight (then per bias) in each of the RED_SEGS waves;
    // wave k adds the partials of blocks [k q, (k+1) q) in block order,
    // fetched 8 at a time, and the RED_SEGS segment sums are then added in
    // segment order (deterministic)
    __shared__ float part[RED_SEGS][RED_OUT];
    const int lane = threadIdx.x % RED_OUT, seg = threadIdx.x / RED_OUT;
    const int i = blockIdx.x * RED_OUT + lane;
    const int nw = cout * 27 * cin;
    const bool valid = i < nw + cout;
    float s = 0.0f;
    if (valid) {
        const float* src;
        size_t stride;
        if (i < nw) {
            const int o = i / (27 * cin), rem = i - o * 27 * cin, t = rem / cin, c = rem - t * cin;
            src = ws + (size_t)(t * 32 + o) * 32 + c;
            stride = 27 * 32 * 32;
        } else {
            src = wsb + (i - nw);
            stride = 32;
        }
        const int q = (nblocks + RED_SEGS - 1) / RED_SEGS;
        const int b0 = seg * q, b1 = min(b0 + q, nblocks);
        int bk = b0;
        for (; bk + 8 <= b1; bk += 8) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = src[(size_t)(bk + j) * stride];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
        for (; bk < b1; ++bk) s += src[(size_t)bk * stride];
    }
    part[seg][lane] = s;
    __syncthreads();
    if (seg == 0 && valid) {
        float t = part[0][lane];
#pragma unroll
        for (int k = 1; k < RED_SEGS; ++k) t += part[k][lane];
        if (i < nw)
            dw[i] = t;
        else
            dbias[i - nw] = t;
    }
}

// ------------------------------------------------------------ elementwise
// Several arrays in one launch: launches, not work, are what a training step's
// updates of six small arrays and preparations of three layers cost: nine
// launches, two now (backward pass at 4 x 64^3 308 -> 298 us).  Block b serves the part whose blocks begin at
// or before b (uniform).  N: 1 where there is one array, which needs no search and few
// kernel arguments, else MAX_PARTS.
constexpr int MAX_PARTS = 8;
template <typename P, int N>
struct Parts {
    P part[N];
    int first[N];  // first block of each part
};
template <typename P, int N>
__device__ __forceinline__ P part_of_block(const Parts<P, N>& s, int& block)
{
    int k = 0;
#pragma unroll
    for (int q = 1; q < N; ++q) k += (int)blockIdx.x >= s.first[q];
    block = blockIdx.x - s.first[k];
    return s.part[k];
}
// blocks(part) blocks each; parts past count get none
template <int N, typename P, typename F>
Parts<P, N> make_parts(const P* parts, int count, F blocks)
{
    Parts<P, N> s{};
    int at = 0;
    for (int k = 0; k < N; ++k) {
        s.first[k] = at;
        if (k < count) {
            s.part[k] = parts[k];
            at += blocks(parts[k]);
        }
    }
    return s;
}

template <int N>
__global__ void k_prepare_weights(Parts<mhdnn_weights_part, N> s)
{
    int block;
    const mhdnn_weights_part a = part_of_block(s, block);
    const float* __restrict__ w = a.w;
    const int cin = a.cin, cout = a.cout, i = block * blockDim.x + threadIdx.x;
    if (i < 32 * 27 * cin) {  // w_pad[o][t][c]
        const int o = i / (27 * cin), rem = i - o * 27 * cin;
        a.w_pad[i] = o < cout ? f2bf(w[o * 27 * cin + rem]) : (uint16_t)0;
    }
    if (a.wt_pad && i < 32 * 27 * cout) {  // wt_pad[c][t][o] = w[o][26 - t][c]
        const int c = i / (27 * cout), rem = i - c * 27 * cout, t = rem / cout, o = rem - t * cout;
        a.wt_pad[i] = c < cin ? f2bf(w[(o * 27 + (26 - t)) * cin + c]) : (uint16_t)0;
    }
}

struct Vec8 {
    float v[8];
};

__global__ void k_pack(const float* __restrict__ src, const float* __restrict__ sub,
                       int64_t bstride, int64_t fstride,
                       int64_t origin, int64_t row, int64_t plane, int n, int logn, int batch,
                       Vec8 mean, Vec8 inv_std, uint16_t* __restrict__ out)
{
    const int64_t n3 = (int64_t)n * n * n;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n3 * batch) return;
    const int64_t b = i / n3, cell = i - b * n3;
    const int64_t xx = cell & (n - 1), yy = (cell >> logn) & (n - 1), zz = cell >> (2 * logn);
    const int64_t o = b * bstride + origin + zz * plane + yy * row + xx;
    u16x8 v;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        float f = src[o + q * fstride];
        if (sub) f -= sub[o + q * fstride];
        v[q] = f2bf((f - mean.v[q]) * inv_std.v[q]);
    }
    reinterpret_cast<u16x8*>(out)[i] = v;
}

// Guarded correction: guard[0] counts the cells whose corrected value
// would not be finite (reset by k_guard_reset, filled by k_guard_check),
// guard[1] the corrections refused so far.  k_apply then leaves the state
// untouched when guard[0] != 0 -- the plain method's step stands.
__global__ void k_guard_reset(int* __restrict__ guard)
{
    if (threadIdx.x == 0) guard[0] = 0;
}

__global__ void k_guard_check(Grid g, const float* __restrict__ f, const float* __restrict__ comp,
                              const float* __restrict__ y, Vec8 scale, int* __restrict__ guard)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;  // interior cell, x fastest
    const int n3 = g.nx * g.ny * g.nz;
    bool bad = false;
    if (i < n3) {
        const int xx = i % g.nx, yy = (i / g.nx) % g.ny, zz = i / (g.nx * g.ny);
        const int c = g.interior + zz * g.mxy + yy * g.mx + xx;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t o = q * g.fstride + c;
            const float add = y[(int64_t)i * 8 + q] * scale.v[q];
            float cc = comp ? comp[o] : 0.0f;
            const float t = comp ? kahan_add(f[o], add, cc) : f[o] + add;
            bad |= !isfinite(t) || !isfinite(cc);
        }
    }
    const unsigned long long m = __ballot(bad);
    if (m && (threadIdx.x & 63) == 0) atomicAdd(guard, __popcll(m));
}

__global__ void k_apply(Grid g, float* __restrict__ f, float* __restrict__ comp,
                        const float* __restrict__ y, Vec8 scale, int* __restrict__ guard)
{
    if (guard && guard[0] != 0) {  // uniform over the launch
        if (blockIdx.x == 0 && threadIdx.x == 0) guard[1] += 1;
        return;
    }
    const int i = blockIdx.x * blockDim.x + threadIdx.x;  // interior cell, x fastest
    const int n3 = g.nx * g.ny * g.nz;
    if (i >= n3) return;
    const int xx = i % g.nx, yy = (i / g.nx) % g.ny, zz = i / (g.nx * g.ny);
    const int c = g.interior + zz * g.mxy + yy * g.mx + xx;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t o = q * g.fstride + c;
        const float add = y[(int64_t)i * 8 + q] * scale.v[q];
        if (comp) {
            float cc = comp[o];
            f[o] = kahan_add(f[o], add, cc);
            comp[o] = cc;
        } else {
            f[o] = f[o] + add;
        }
    }
}

template <typename E>
__global__ void k_box4(Grid g, const E* __restrict__ fine, float* __restrict__ coarse)
{
    const int nc = g.nx / 4;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int nc3 = nc * nc * nc;
    if (i >= nc3 * 8) return;
    const int q = i / nc3, cell = i - q * nc3;
    const int I = cell % nc, J = (cell / nc) % nc, K = cell / (nc * nc);
    const E* f = fine + q * g.fstride + g.interior;
    double s = 0.0;
    for (int c = 0; c < 4; ++c)
        for (int b = 0; b < 4; ++b)
            for (int a = 0; a < 4; ++a)
                s += (double)f[(4 * K + c) * g.mxy + (4 * J + b) * g.mx + 4 * I + a];
    coarse[i] = (float)(s / 64.0);
}

// Loss and output gradient of one batch: y channels-last [b][cell][q],
// target field-major [b][q][cell] times tscale[q].
__global__ __launch_bounds__(NTHR) void k_mse(const float* __restrict__ y,
                                              const float* __restrict__ t, Vec8 tscale, int logn3,
                                              int64_t count, uint16_t* __restrict__ dy,
                                              float* __restrict__ part)
{
    __shared__ float sh[NTHR];
    const float scale = 2.0f / (float)count, inv = 1.0f / (float)count;
    const int64_t n3 = (int64_t)1 << logn3;
    float acc = 0.0f;
    for (int64_t i = (int64_t)blockIdx.x * NTHR + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * NTHR) {
        // the scaled target is rounded before the difference (no fused multiply-add)
#pragma clang fp contract(off)
        const int q = (int)(i & 7);
        const int64_t bc = i >> 3, b = bc >> logn3, cell = bc & (n3 - 1);
        const float d = y[i] - t[(b * 8 + q) * n3 + cell] * tscale.v[q];
        dy[i] = f2bf(scale * d);
        acc += d * d * inv;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int hh = NTHR / 2; hh > 0; hh >>= 1) {
        if (threadIdx.x < hh) sh[threadIdx.x] += sh[threadIdx.x + hh];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Training pair from a coarse step: x = S - C_now (the step's tendency),
// d = C_next - S (what the step misses); S in the coarse solver's padded
// layout, C and the outputs unpadded field-major.
__global__ void k_pair(Grid g, const float* __restrict__ S, const float* __restrict__ cnow,
                       const float* __restrict__ cnext, float* __restrict__ x,
                       float* __restrict__ d)
{
    const int64_t n3 = (int64_t)g.nx * g.ny * g.nz;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // q * n3 + cell
    if (i >= 8 * n3) return;
    const int q = (int)(i / n3);
    const int64_t cell = i - q * n3;
    const int xx = (int)(cell % g.nx), yy = (int)((cell / g.nx) % g.ny), zz = (int)(cell / ((int64_t)g.nx * g.ny));
    const float sv = S[q * g.fstride + g.interior + (int64_t)zz * g.mxy + (int64_t)yy * g.mx + xx];
    x[i] = sv - cnow[i];
    d[i] = cnext[i] - sv;
}

constexpr int STAT_BLOCKS = 256;  // blocks per field in the statistics pass

// Per-field FP64 partial sums over samples [p][8][n3]: of x (mean == NULL)
// or of (x - mean[q])^2.  Block b of field q covers a fixed interleaved set
// of elements; partials[q][b].
__global__ __launch_bounds__(NTHR) void k_stats(const float* __restrict__ x, int64_t npairs,
                                                int64_t n3, const double* __restrict__ mean,
                                                double* __restrict__ partials)
{
    __shared__ double sh[NTHR];
    const int q = blockIdx.y;
    const double m = mean ? mean[q] : 0.0;
    const int64_t per = npairs * n3;
    double acc = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * NTHR + threadIdx.x; j < per;
         j += (int64_t)STAT_BLOCKS * NTHR) {
        const int64_t p = j / n3, cell = j - p * n3;
        const double v = (double)x[(p * 8 + q) * n3 + cell];
        acc += mean ? (v - m) * (v - m) : v;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int hh = NTHR / 2; hh > 0; hh >>= 1) {
        if (threadIdx.x < hh) sh[threadIdx.x] += sh[threadIdx.x + hh];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[q * STAT_BLOCKS + blockIdx.x] = sh[0];
}

// out[q] = (sum of partials[q][*] in order) / count (then sqrt if `root`).
__global__ void k_stats_final(const double* __restrict__ partials, double count, int root,
                              double* __restrict__ out)
{
    const int q = threadIdx.x;
    if (q >= 8) return;
    double s = 0.0;
    for (int b = 0; b < STAT_BLOCKS; ++b) s += partials[q * STAT_BLOCKS + b];
    s /= count;
    out[q] = root ? sqrt(s) : s;
}

template <int N>
__global__ void k_adam(Parts<mhdnn_adam_part, N> s, float lr, float b1, float b2, float eps, float c1,
                       float c2)
{
    int block;
    const mhdnn_adam_part a = part_of_block(s, block);
    const int64_t i = (int64_t)block * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    // (all four in flight before the first store, which the compiler must take to alias them)
    const float gi = a.g[i], m0 = a.m[i], v0 = a.v[i], p0 = a.p[i];
    const float mi = b1 * m0 + (1.0f - b1) * gi;
    const float vi = b2 * v0 + (1.0f - b2) * gi * gi;
    a.m[i] = mi;
    a.v[i] = vi;
    a.p[i] = p0 - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

int ilog2(int n)
{
    int l = 0;
    while ((1 << l) < n) ++l;
    return (1 << l) == n ? l : -1;
}

bool conv_n_ok(int n) { return n == 16 || n == 32 || n == 64; }

int status(hipError_t e) { return e == hipSuccess ? MHD_OK : MHD_ERR_DEVICE; }

size_t wgrad_lds(int cin, int cout, int n)
{
    return 2 * (4 * (cin == 32 ? wg_slot<32>(n) : wg_slot<8>(n)) + 2 * CONV_CELLS * cout) +
           4 * WG_THR * 8;
}

// Slabs of CONV_CELLS cells per plane and z chunks of zc planes, so that
// about one block per CU (256) marches at once: blocks = columns * nch.
void conv_chunks(int n, int batch, int& columns, int& nch, int& zc)
{
    columns = batch * (n / (CONV_CELLS / n));
    nch = (256 + columns - 1) / columns;
    nch = nch < 1 ? 1 : nch > n / 4 ? n / 4 : nch;
    zc = (n + nch - 1) / nch;
    nch = (n + zc - 1) / zc;
}

template <int CIN, int MODE, int LOGN, int COUT>
constexpr size_t conv_lds()
{
    constexpr int n = 1 << LOGN;
    return 2 * (4 * (CONV_CELLS / n + 2) * n * conv_cp<CIN>() + 8) +
           (conv_staged<CIN, MODE, COUT>() ? 4 * 2 * CONV_CELLS * STAGE_CP : 0);
}

template <int CIN, int MODE, int LOGN, int COUT>
hipError_t launch_conv_n(const uint16_t* x, const uint16_t* w, const float* bias,
                         const uint16_t* zp, int batch, uint16_t* o0, uint16_t* o1,
                         float* of, hipStream_t st)
{
    // once per instantiation (thread-safe static initialisation)
    static const hipError_t attr =
        hipFuncSetAttribute((const void*)k_conv<CIN, MODE, LOGN, COUT>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)conv_lds<CIN, MODE, LOGN, COUT>());
    if (attr != hipSuccess) return attr;
    int columns, nch, zc;
    conv_chunks(1 << LOGN, batch, columns, nch, zc);
    hipLaunchKernelGGL((k_conv<CIN, MODE, LOGN, COUT>), dim3(columns * nch), dim3(CONV_THR),
                       (conv_lds<CIN, MODE, LOGN, COUT>()), st, x, w, bias, zp, nch, zc, o0, o1, of);
    return hipGetLastError();
}

template <int CIN, int MODE>
hipError_t launch_conv(const uint16_t* x, const uint16_t* w, const float* bias, const uint16_t* zp,
                       int n, int batch, int cout, uint16_t* o0, uint16_t* o1, float* of,
                       hipStream_t st)
{
#define MHDNN_LAUNCH(LOGN)                                                                     \
    (cout == 32 ? launch_conv_n<CIN, MODE, LOGN, 32>(x, w, bias, zp, batch, o0, o1, of, st)     \
                : launch_conv_n<CIN, MODE, LOGN, 8>(x, w, bias, zp, batch, o0, o1, of, st))
    switch (n) {
    case 16: return MHDNN_LAUNCH(4);
    case 32: return MHDNN_LAUNCH(5);
    default: return MHDNN_LAUNCH(6);
    }
#undef MHDNN_LAUNCH
}

template <int CIN, int COUT, int LOGN>
hipError_t launch_wgrad_n(const uint16_t* x, const uint16_t* dz, int blocks, int nch, int zc,
                          float* ws, float* wsb, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(
        (const void*)k_wgrad<CIN, COUT, LOGN>, hipFuncAttributeMaxDynamicSharedMemorySize,
        (int)wgrad_lds(CIN, COUT, 1 << LOGN));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((k_wgrad<CIN, COUT, LOGN>), dim3(blocks), dim3(WG_THR),
                       wgrad_lds(CIN, COUT, 1 << LOGN), st, x, dz, nch, zc, ws, wsb);
    return hipGetLastError();
}

template <int CIN, int COUT>
hipError_t launch_wgrad(const uint16_t* x, const uint16_t* dz, int n, int batch, float* ws,
                        float* dw, float* db, hipStream_t st)
{
    int columns, nch, zc;
    conv_chunks(n, batch, columns, nch, zc);
    const int blocks = columns * nch;
    float* wsb = ws + (size_t)blocks * 27 * 32 * 32;
    hipError_t e = n == 16   ? launch_wgrad_n<CIN, COUT, 4>(x, dz, blocks, nch, zc, ws, wsb, st)
                   : n == 32 ? launch_wgrad_n<CIN, COUT, 5>(x, dz, blocks, nch, zc, ws, wsb, st)
                             : launch_wgrad_n<CIN, COUT, 6>(x, dz, blocks, nch, zc, ws, wsb, st);
    if (e != hipSuccess) return e;
    const int total = COUT * 27 * CIN + COUT;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((total + RED_OUT - 1) / RED_OUT), dim3(NTHR), 0, st, ws,
                       wsb, blocks, CIN, COUT, dw, db);
    return hipGetLastError();
}

}  // namespace
}  // namespace mhd

// ------------------------------------------------------ no-alloc wgrad
// Workspace of mhdnn_conv3d_wgrad_noalloc: a file-scope device array (each
// GPU the library runs on holds its own copy until the process ends).  Its
// device address is looked up once per device, with that device current,
// and only that address is ever handed to a kernel.  Every partial the
// reduction reads is written by the weight-gradient kernel of the same
// call, so nothing needs clearing between calls.
static __device__ __align__(256) float scratch[MHDNN_WGRAD_SCRATCH_FLOATS];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex scratch_mutex;
float* scratch_ptr[SCRATCH_MAX_DEVICES] = {};

int scratch_of_current_device(float** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return MHD_ERR_NO_DEVICE;
    if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return MHD_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
            return MHD_ERR_DEVICE;
        scratch_ptr[dev] = static_cast<float*>(p);
    }
    *out = scratch_ptr[dev];
    return MHD_OK;
}
}  // namespace

using namespace mhd;

extern "C" {

int mhdnn_box_filter4(const void* fine_ctx, const void* fine_fields, float* coarse, void* stream)
{
    if (!fine_ctx || !fine_fields || !coarse) return MHD_ERR_INVALID;
    const mhd_ctx* ctx = (const mhd_ctx*)fine_ctx;
    const Grid g = *ctx_grid(ctx);
    if (g.nx != g.ny || g.nx != g.nz || g.nx % 4 != 0) return MHD_ERR_INVALID;
    const int nc = g.nx / 4, total = nc * nc * nc * 8;
    hipStream_t st = (hipStream_t)stream;
    if (ctx_precision(ctx) == MHD_F64)
        hipLaunchKernelGGL(k_box4<double>, dim3((total + 255) / 256), dim3(256), 0, st, g,
                           (const double*)fine_fields, coarse);
    else
        hipLaunchKernelGGL(k_box4<float>, dim3((total + 255) / 256), dim3(256), 0, st, g,
                           (const float*)fine_fields, coarse);
    return status(hipGetLastError());
}

int mhdnn_pack(const float* src, const float* sub, int64_t batch_stride, int64_t field_stride,
               int64_t origin, int64_t row, int64_t plane, int32_t n, int32_t batch,
               const float* mean, const float* inv_std, uint16_t* x_bf16, void* stream)
{
    if (!src || !mean || !inv_std || !x_bf16 || batch < 1 || ilog2(n) < 0) return MHD_ERR_INVALID;
    Vec8 mm, is;
    for (int q = 0; q < 8; ++q) {
        mm.v[q] = mean[q];
        is.v[q] = inv_std[q];
    }
    const int64_t total = (int64_t)n * n * n * batch;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, src, sub, batch_stride, field_stride, origin, row, plane, n,
                       ilog2(n), batch, mm, is, x_bf16);
    return status(hipGetLastError());
}

int mhdnn_conv3d_fwd(const uint16_t* x, const uint16_t* w_pad, const float* bias, int32_t n,
                     int32_t batch, int32_t cin, int32_t cout, int32_t mode, uint16_t* z_bf16,
                     uint16_t* a_bf16, float* y_f32, void* stream)
{
    if (!x || !w_pad || !bias || !conv_n_ok(n) || batch < 1) return MHD_ERR_INVALID;
    if ((cin != 8 && cin != 32) || (cout != 8 && cout != 32)) return MHD_ERR_INVALID;
    if (mode == 0 && (!z_bf16 || !a_bf16)) return MHD_ERR_INVALID;
    if (mode == 1 && !y_f32) return MHD_ERR_INVALID;
    if (mode != 0 && mode != 1) return MHD_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    if (mode == 0)
        e = cin == 32 ? launch_conv<32, 0>(x, w_pad, bias, nullptr, n, batch, cout, z_bf16, a_bf16,
                                           nullptr, st)
                      : launch_conv<8, 0>(x, w_pad, bias, nullptr, n, batch, cout, z_bf16, a_bf16,
                                          nullptr, st);
    else
        e = cin == 32 ? launch_conv<32, 1>(x, w_pad, bias, nullptr, n, batch, cout, nullptr,
                                           nullptr, y_f32, st)
                      : launch_conv<8, 1>(x, w_pad, bias, nullptr, n, batch, cout, nullptr,
                                          nullptr, y_f32, st);
    return status(e);
}

int mhdnn_conv3d_dgrad(const uint16_t* dz, const uint16_t* wt_pad, const uint16_t* zprev,
                       int32_t n, int32_t batch, int32_t cin_dz, int32_t cprev, uint16_t* dprev,
                       void* stream)
{
    if (!dz || !wt_pad || !zprev || !dprev || !conv_n_ok(n) || batch < 1) return MHD_ERR_INVALID;
    if ((cin_dz != 8 && cin_dz != 32) || (cprev != 8 && cprev != 32)) return MHD_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = cin_dz == 32
                       ? launch_conv<32, 2>(dz, wt_pad, nullptr, zprev, n, batch, cprev, dprev,
                                            nullptr, nullptr, st)
                       : launch_conv<8, 2>(dz, wt_pad, nullptr, zprev, n, batch, cprev, dprev,
                                           nullptr, nullptr, st);
    return status(e);
}

int64_t mhdnn_wgrad_workspace_floats(int32_t n, int32_t batch)
{
    if (!conv_n_ok(n) || batch < 1) return 0;
    int columns, nch, zc;
    conv_chunks(n, batch, columns, nch, zc);
    return (int64_t)columns * nch * (27 * 32 * 32 + 32);
}

int mhdnn_conv3d_wgrad(const uint16_t* x, const uint16_t* dz, int32_t n, int32_t batch,
                       int32_t cin, int32_t cout, float* workspace, float* dw, float* db,
                       void* stream)
{
    if (!x || !dz || !workspace || !dw || !db || !conv_n_ok(n) || batch < 1) return MHD_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    if (cin == 8 && cout == 32) e = launch_wgrad<8, 32>(x, dz, n, batch, workspace, dw, db, st);
    else if (cin == 32 && cout == 32) e = launch_wgrad<32, 32>(x, dz, n, batch, workspace, dw, db, st);
    else if (cin == 32 && cout == 8) e = launch_wgrad<32, 8>(x, dz, n, batch, workspace, dw, db, st);
    else if (cin == 8 && cout == 8) e = launch_wgrad<8, 8>(x, dz, n, batch, workspace, dw, db, st);
    else return MHD_ERR_INVALID;
    return status(e);
}

int mhdnn_conv3d_wgrad_noalloc(const uint16_t* x, const uint16_t* dz, int32_t n, int32_t batch,
                               int32_t cin, int32_t cout, float* dw, float* db, void* stream)
{
    if (!x || !dz || !dw || !db || !conv_n_ok(n) || batch < 1 || batch > 65536)
        return MHD_ERR_INVALID;
    const bool shape_ok = (cin == 8 || cin == 32) && (cout == 8 || cout == 32);
    if (!shape_ok || mhdnn_wgrad_workspace_floats(n, batch) > MHDNN_WGRAD_SCRATCH_FLOATS)
        return MHD_ERR_INVALID;
    float* ws = nullptr;
    const int rc = scratch_of_current_device(&ws);
    if (rc != MHD_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    if (cin == 8 && cout == 32) e = launch_wgrad<8, 32>(x, dz, n, batch, ws, dw, db, st);
    else if (cin == 32 && cout == 32) e = launch_wgrad<32, 32>(x, dz, n, batch, ws, dw, db, st);
    else if (cin == 32 && cout == 8) e = launch_wgrad<32, 8>(x, dz, n, batch, ws, dw, db, st);
    else e = launch_wgrad<8, 8>(x, dz, n, batch, ws, dw, db, st);
    return status(e);
}

int mhdnn_prepare_weights(const float* w, int32_t cin, int32_t cout, uint16_t* w_pad,
                          uint16_t* wt_pad, void* stream)
{
    const mhdnn_weights_part one = {w, w_pad, wt_pad, cin, cout};
    return mhdnn_prepare_weights_parts(&one, 1, stream);
}

int mhdnn_prepare_weights_parts(const mhdnn_weights_part* parts, int32_t count, void* stream)
{
    if (!parts || count < 0 || count > MAX_PARTS) return MHD_ERR_INVALID;
    for (int k = 0; k < count; ++k) {
        const mhdnn_weights_part& a = parts[k];
        if (!a.w || !a.w_pad || (a.cin != 8 && a.cin != 32) || (a.cout != 8 && a.cout != 32))
            return MHD_ERR_INVALID;
    }
    if (count == 0) return MHD_OK;
    int total = 0;
    auto blocks = [](const mhdnn_weights_part& a) {
        return (32 * 27 * (a.cin > a.cout ? a.cin : a.cout) + 255) / 256;
    };
    for (int k = 0; k < count; ++k) total += blocks(parts[k]);
    hipStream_t st = (hipStream_t)stream;
    if (count == 1)
        hipLaunchKernelGGL(k_prepare_weights<1>, dim3(total), dim3(256), 0, st, make_parts<1>(parts, count, blocks));
    else
        hipLaunchKernelGGL(k_prepare_weights<MAX_PARTS>, dim3(total), dim3(256), 0, st,
                           make_parts<MAX_PARTS>(parts, count, blocks));
    return status(hipGetLastError());
}

int mhdnn_mse(const float* y, const float* target, const float* tscale, int32_t n, int32_t batch,
              uint16_t* dy_bf16, float* loss_partials, void* stream)
{
    if (!y || !target || !tscale || !dy_bf16 || !loss_partials || batch < 1) return MHD_ERR_INVALID;
    const int logn = ilog2(n);
    if (logn < 0) return MHD_ERR_INVALID;
    Vec8 ts;
    for (int q = 0; q < 8; ++q) ts.v[q] = tscale[q];
    const int64_t count = ((int64_t)batch << (3 * logn)) * 8;
    hipLaunchKernelGGL(k_mse, dim3(256), dim3(NTHR), 0, (hipStream_t)stream, y, target, ts,
                       3 * logn, count, dy_bf16, loss_partials);
    return status(hipGetLastError());
}

int mhdnn_pair(const void* coarse_ctx, const void* stepped, const float* c_now,
               const float* c_next, float* x_out, float* d_out, void* stream)
{
    if (!coarse_ctx || !stepped || !c_now || !c_next || !x_out || !d_out) return MHD_ERR_INVALID;
    const mhd_ctx* ctx = (const mhd_ctx*)coarse_ctx;
    if (ctx_precision(ctx) == MHD_F64) return MHD_ERR_INVALID;
    const Grid g = *ctx_grid(ctx);
    const int64_t total = 8LL * g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_pair, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, g, (const float*)stepped, c_now, c_next, x_out, d_out);
    return status(hipGetLastError());
}

int64_t mhdnn_field_stats_workspace_doubles(void) { return 8 * STAT_BLOCKS; }

int mhdnn_field_stats(const float* x, int64_t npairs, int64_t n3, double* workspace,
                      double* mean_std, void* stream)
{
    if (!x || !workspace || !mean_std || npairs < 1 || n3 < 1) return MHD_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    const double count = (double)npairs * (double)n3;
    hipLaunchKernelGGL(k_stats, dim3(STAT_BLOCKS, 8), dim3(NTHR), 0, st, x, npairs, n3,
                       (const double*)nullptr, workspace);
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(64), 0, st, (const double*)workspace, count,
                       0, mean_std);
    hipLaunchKernelGGL(k_stats, dim3(STAT_BLOCKS, 8), dim3(NTHR), 0, st, x, npairs, n3,
                       (const double*)mean_std, workspace);
    hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(64), 0, st, (const double*)workspace, count,
                       1, mean_std + 8);
    return status(hipGetLastError());
}

int mhdnn_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1,
               float b2, float eps, int32_t t, void* stream)
{
    const mhdnn_adam_part one = {p, g, m, v, n};
    return mhdnn_adam_parts(&one, 1, lr, b1, b2, eps, t, stream);
}

int mhdnn_adam_parts(const mhdnn_adam_part* parts, int32_t count, float lr, float b1, float b2,
                     float eps, int32_t t, void* stream)
{
    if (!parts || count < 0 || count > MAX_PARTS || t < 1) return MHD_ERR_INVALID;
    auto blocks = [](const mhdnn_adam_part& a) { return a.n / 256 + (a.n % 256 != 0); };
    int64_t total = 0;
    for (int k = 0; k < count; ++k) {
        const mhdnn_adam_part& a = parts[k];
        if (!a.p || !a.g || !a.m || !a.v || a.n < 0) return MHD_ERR_INVALID;
        total += blocks(a);
        if (total > INT32_MAX) return MHD_ERR_INVALID;  // more than 2 TB of parameters
    }
    if (total == 0) return MHD_OK;
    const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    const dim3 grid((unsigned)total);
    hipStream_t st = (hipStream_t)stream;
    if (count == 1)
        hipLaunchKernelGGL(k_adam<1>, grid, dim3(256), 0, st, make_parts<1>(parts, count, blocks), lr, b1, b2,
                           eps, c1, c2);
    else
        hipLaunchKernelGGL(k_adam<MAX_PARTS>, grid, dim3(256), 0, st, make_parts<MAX_PARTS>(parts, count, blocks),
                           lr, b1, b2, eps, c1, c2);
    return status(hipGetLastError());
}

int mhdnn_apply(const void* ctx_, void* fields, void* comp, const float* y, const float* scale,
                int32_t* guard, void* stream)
{
    if (!ctx_ || !fields || !y || !scale) return MHD_ERR_INVALID;
    const mhd_ctx* ctx = (const mhd_ctx*)ctx_;
    if (ctx_precision(ctx) == MHD_F64) return MHD_ERR_INVALID;
    const Grid g = *ctx_grid(ctx);
    Vec8 sc;
    for (int q = 0; q < 8; ++q) sc.v[q] = scale[q];
    const int n3 = g.nx * g.ny * g.nz;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((n3 + 255) / 256), block(256);
    if (guard) {
        hipLaunchKernelGGL(k_guard_reset, dim3(1), dim3(64), 0, st, (int*)guard);
        hipLaunchKernelGGL(k_guard_check, grid, block, 0, st, g, (const float*)fields,
                           (const float*)comp, y, sc, (int*)guard);
    }
    hipLaunchKernelGGL(k_apply, grid, block, 0, st, g, (float*)fields, (float*)comp, y, sc,
                       (int*)guard);
    return status(hipGetLastError());
}

}  // extern "C"
