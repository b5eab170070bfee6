// Fused RHS + RK3 substep, LDS-tiled z-marching kernel with two wave groups
// per cell (gfx950).
//
// A workgroup owns a 32 x 8 column tile and marches it through the planes of
// its box, one plane at a time.  On chip, for stencil radius r:
//   * an LDS ring of r + 1 halo'd planes (t .. t+r) of all 8 fields, each the
//     tile plus r cells on every side in x and y (38 x 14 at r = 3);
//   * x, y and xy derivatives of plane t read the ring's plane t;
//   * z derivatives use the thread's own column: planes t-r .. t-1 from a
//     register history, t .. t+r from the ring;
//   * the xz / yz mixed derivatives are differences of x (or y) differences
//     taken on planes t +- m:  Dxz f(t) = sum_m w_m [d_m(t+m) - d_m(t-m)],
//     d_m(p) = f(x+m, p) - f(x-m, p): the t+m halves come from the ring, the
//     t-m halves were formed when plane t-m was current and are carried in r
//     running accumulators per mixed combination.
// Each input value is fetched from HBM once per tile plus the tile halo;
// neighbouring tiles of one round run concurrently on the same XCD (see
// tile_of_block), so halo fetches mostly hit its L2.  Stencil weights are the
// integers W1, W2 of the central formulas of order 2r (exact as literals) with
// one scale factor per axis or plane.
//
// Each cell is served by two threads in different waves:
//   group F (waves 0-3): lnrho, ux, uy, uz -- their derivatives, Eq. B.1
//                        and Eq. B.2, and their 2N updates;
//   group M (waves 4-7): ss, Ax, Ay, Az -- their derivatives, Eqs. B.3 and
//                        B.4, and their 2N updates.
// FP64 at r = 4 uses a 32 x 4 tile (256 threads): its ring of five 40 x 12
// planes and the hand-over area take 159 of the 160 KB of LDS.
// Each group loads, stores and differentiates only its own four fields and
// evaluates its own equations but for the terms that need the other group's
// derivatives; those go through LDS:
//   F -> M (5 values): grad lnrho, lap lnrho, the viscous heating;
//   M -> F (4 values): the force j x B / rho - cs^2 grad s / cp, and cs^2
// (FP32 storage: 6 and 6 values, see physics_late).
// (M reads lnrho and u themselves from the ring).  A plane costs two barriers:
//   derivatives and own equations of plane t, the loads of plane t+r+1 issued
//   between their first steps; both groups write their values
//   -- barrier (plane t read, the values visible) --
//   the other group's values are read; plane t+r+1 goes into plane t's slot
//   -- barrier (plane t+r+1 visible, the hand-over area free) --
//   right-hand sides completed, 2N update and stores of plane t.
//
// What bounds it, at 512^3, FP64, sixth order.  With all vector-memory
// instructions of a plane in one burst after the physics (loads, then stores)
// the later group stalled in that burst for half of the plane (5000 of 10500
// clocks) while the earlier one waited at the barrier: 9.1 ms per substep.
// Spread over the plane, with 9 values handed over instead of 17, each step's
// LDS reads issued ahead of the step before it, and the march started without
// warm-up planes, it takes 7.9 ms.  No single unit is full: of the clocks (2.05 GHz
// on average) the SIMDs issue VALU instructions in 45%, the LDS is busy in 49% and
// the address units in 39%, and waves wait for an instruction 22% of their time.
// Leaving out the stencil's LDS reads alone gives 7.4 ms, its arithmetic alone 7.7.
// A third wave per SIMD (three groups: u, A, and lnrho with s) changes nothing
// (7.8-7.9 ms), nor do wave priorities; non-temporal stores cost 6%.
// FP32 storage with compensation is nearest to VALU issue (65% of the clocks): the
// second derivatives' sums are FP64 and their inputs FP32.  One thread per cell for
// all 8 fields, two workgroups to a CU, took 22.0 ms per step at 512^3, halo fills
// included, sixth order (21.8 and 21.6 at second and fourth); the two groups take 20.6
// (18.5, 19.4) although only one workgroup is resident.
#pragma once

#include <type_traits>

#include "mhd_internal.hpp"
#include "rk3_common.hpp"

namespace mhd {

namespace {

// Whether each group evaluates all of its equations after the hand-over, from
// the other's derivatives, rather than its own terms before it.  FP32 storage
// does: the terms are then rounded and added as in every other kernel of the
// library (rhs_flow, rhs_entropy_induction), while in FP64 a term's rounding is
// far below what a caller can see, and the shorter hand-over pays (512^3: 17
// values 8.2, 9 values 7.9 ms per substep).  With its terms handed over like
// those of FP64, one step of FP32C at 512^3 changed 40% of the register values
// by a rounding; now four of the eight fields keep every bit.
// What FP64 gives up: the two halves of the pressure gradient meet after the
// hand-over, so where they cancel exactly (s = -lnrho with cp = 1) the rounding of
// one product is left, 2e-16 of it, and not zero.
template <int PREC>
constexpr bool physics_late() { return PREC != MHD_F64; }
template <int PREC>
constexpr int nxf() { return physics_late<PREC>() ? 6 : 5; }  // values F hands to M
template <int PREC>
constexpr int nxm() { return physics_late<PREC>() ? 6 : 4; }  // values M hands to F
// Per precision and stencil radius RAD: the tile plane of TX x TY cells
// (TY = 4 for FP64 at RAD = 4, whose 5-plane ring of a 32 x 8 tile would not
// fit the LDS; 8 otherwise), the halo'd tile plane (38 x 14 = 532 cells at
// RAD = 3) and the LDS ring of RAD + 1 such planes of all 8 fields.
template <int PREC, int RAD>
struct SRing {
    static constexpr bool SMALL = PREC == MHD_F64 && RAD == 4;
    static constexpr int TX = 32;
    static constexpr int TY = (SMALL ? 128 : 256) / TX;
    static constexpr int NC = TX * TY;   // cells per tile plane
    static constexpr int NTH = 2 * NC;   // threads: two groups of NC
    static constexpr int HX = TX + 2 * RAD, HY = TY + 2 * RAD, PLANE = HX * HY;
    static constexpr int SLOT = NQ * PLANE;
    static constexpr int NSLOT = RAD + 1;
};

template <int PREC, int RAD>
constexpr size_t ring_bytes()
{
    return sizeof(typename Prec<PREC>::T) * SRing<PREC, RAD>::NSLOT * SRing<PREC, RAD>::SLOT;
}
// Whether two workgroups share a CU: plain FP32 up to r = 3, whose rings and
// registers allow it (82, 128 and 124-128; the 128 at r = 2 leave one pointer of
// group M in scratch memory, read back once per plane).  us per step at 256^3 with
// one and two: orders 2, 4, 6 1890 -> 1735, 1873 -> 1830, 1973 -> 1878.
// The other precisions fit two at r = 1 only and lose by it, as the halo reads
// of two tiles find less in L2: FP64 3150 -> 3240, FP32C 2440 -> 2567.  They
// ask for more than half of the 160 KB where the ring is smaller.
template <int PREC, int RAD>
constexpr bool two_resident() { return PREC == MHD_F32 && RAD <= 3; }
// Whether two share one only where the tiles are ragged (see ragged_tiles).
template <int PREC, int RAD>
constexpr bool two_if_ragged() { return PREC == MHD_F32C && RAD == 1; }
template <int PREC, int RAD>
constexpr size_t lds_needed()
{
    return ring_bytes<PREC, RAD>() +
           sizeof(typename Prec<PREC>::Rt) * (nxf<PREC>() + nxm<PREC>()) * SRing<PREC, RAD>::NC;
}
template <int PREC, int RAD>
constexpr size_t lds_bytes()
{
    constexpr size_t need = lds_needed<PREC, RAD>();
    return two_resident<PREC, RAD>() || need > 84 * 1024 ? need : 84 * 1024;
}

static_assert(SRing<MHD_F64, 4>::NC % 64 == 0 && SRing<MHD_F32, 1>::NC % 64 == 0,
              "each group must be whole waves");

// Per-axis scale factors of the integer-weight stencils.
// (Sized by the radius: the kernel keeps these in scalar registers, which
// are scarce.)
template <int RAD>
struct Scales {
    double d1[3];     // 1/(DEN1 h_a)
    double d2[3];     // 1/(DEN2 h_a^2)
    double mxy;       // 1/(4 DEN2 h_x h_y)
    double wxz[RAD];  // W2(r, m)/(4 DEN2 h_x h_z), m = 1..r
    double wyz[RAD];  // W2(r, m)/(4 DEN2 h_y h_z)
};

// Eqs. B.1 and B.2 as group F sees them before the hand-over: out[0] = d lnrho/dt
// and out[1..3] = du/dt without the entropy part of the pressure gradient and
// the Lorentz force (which group M hands over as one force, with cs^2) and
// without -cs^2 grad lnrho; heat: the viscous heating 2 nu S:S + zeta (div u)^2.
template <typename Rt>
__device__ __forceinline__ void rhs_flow_own(const Derivs<Rt>& d, const Phys& P, Rt out[4], Rt& heat)
{
    Rt S[3][3], divu, SS;
    shear(d.gu, S, divu, SS);
    const Rt nu = Rt(P.nu), zeta = Rt(P.zeta);
    const Rt u[3] = {d.ux, d.uy, d.uz};
    out[0] = -(u[0] * d.gl[0] + u[1] * d.gl[1] + u[2] * d.gl[2]) - divu;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const Rt adv = u[0] * d.gu[a][0] + u[1] * d.gu[a][1] + u[2] * d.gu[a][2];
        const Rt Sgl = S[a][0] * d.gl[0] + S[a][1] * d.gl[1] + S[a][2] * d.gl[2];
        out[1 + a] = nu * (d.lapu[a] + d.gdu[a] * Rt(1.0 / 3.0) + Rt(2) * Sgl) - adv + zeta * d.gdu[a];
    }
    heat = Rt(2) * nu * SS + zeta * divu * divu;
}

// What group M keeps of Eq. B.3 across the hand-over.
template <typename Rt>
struct EntropyOwn {
    Rt hs[3];  // gamma grad s / cp
    Rt kr;     // K / rho
    Rt inv_T;
};

// Eqs. B.3 and B.4 as group M sees them before the hand-over: out[1..3] =
// dA/dt, out[0] = ds/dt without the terms in grad lnrho, lap lnrho and the viscous
// heating; force = j x B / rho - cs^2 grad s / cp for Eq. B.2.
template <typename Rt>
__device__ __forceinline__ void rhs_entropy_own(const Derivs<Rt>& d, const Phys& P, EntropyOwn<Rt>& own,
                                                Rt out[4], Rt force[3], Rt& cs2)
{
    Rt B[3], J[3], jxB[3];
    magnetic(d, P, B, J, jxB);
    const Rt gamma = Rt(P.gamma), inv_cp = Rt(P.inv_cp), gm1 = Rt(P.gamma_m1), eta = Rt(P.eta);
    const Rt u[3] = {d.ux, d.uy, d.uz};
    const Rt inv_rho = exp(-d.lnrho);
    cs2 = Rt(P.cs0sq) * exp(gamma * d.ss * inv_cp + gm1 * (d.lnrho - Rt(P.lnrho0)));
    own.inv_T = Rt(P.cp_gm1) / cs2;
    own.kr = Rt(P.K) * inv_rho;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        own.hs[a] = gamma * d.gs[a] * inv_cp;
        force[a] = jxB[a] * inv_rho - cs2 * (d.gs[a] * inv_cp);
    }
    const Rt jj = J[0] * J[0] + J[1] * J[1] + J[2] * J[2];
    const Rt udgs = u[0] * d.gs[0] + u[1] * d.gs[1] + u[2] * d.gs[2];
    out[0] = own.kr * (gamma * d.laps * inv_cp) +
             own.inv_T * ((Rt(P.hc) + eta * Rt(P.mu0) * jj) * inv_rho) - udgs;
    out[1] = u[1] * B[2] - u[2] * B[1] + eta * d.lapA[0];
    out[2] = u[2] * B[0] - u[0] * B[2] + eta * d.lapA[1];
    out[3] = u[0] * B[1] - u[1] * B[0] + eta * d.lapA[2];
}

// The rest of Eq. B.3, with what group F hands over.
template <typename Rt>
__device__ __forceinline__ void rhs_entropy_other(const Phys& P, const EntropyOwn<Rt>& own,
                                                  const Rt gl[3], Rt lapl, Rt heat, Rt& out)
{
    const Rt gm1 = Rt(P.gamma_m1);
    Rt glnT2 = Rt(0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const Rt g = own.hs[a] + gm1 * gl[a];
        glnT2 += g * g;
    }
    out += own.kr * (gm1 * lapl + glnT2) + own.inv_T * heat;
}

// MULTI: the launch covers the several boxes of `plan` and each workgroup
// takes its box and tile grid from there; otherwise one box, `box` and `map`
// (a separate instantiation, so that the single-box march is compiled as if
// the plan did not exist).  PAIRS: most of each halo'd plane is fetched and
// stored into the ring as pairs of x-neighbours (one 16-byte load and LDS
// store per pair in FP64, about half the load instructions); the launch
// guarantees that every pair is aligned (even padded row length, even box x0,
// aligned f_in).
template <int PREC, int RAD, bool MULTI, bool PAIRS>
__global__ __launch_bounds__((SRing<PREC, RAD>::NTH), (two_resident<PREC, RAD>() ? 4 : 1)) void k_rk3_split(Grid g, const Phys* __restrict__ P_dev, Scales<RAD> sc, TileMap map, int s,
                                                     const typename Prec<PREC>::T* __restrict__ fin,
                                                     typename Prec<PREC>::T* __restrict__ fout,
                                                     typename Prec<PREC>::T* __restrict__ w,
                                                     typename Prec<PREC>::T* __restrict__ comp,
                                                     double dt, Box box, TilePlan plan)
{
    int multi_tile = 0;
    if constexpr (MULTI) {
        const int tile_g = tile_of_block(blockIdx.x, plan.tiles, plan.round);
        if (tile_g == NO_TILE) return;  // the whole workgroup exits together
        int x0, x1, y0, y1, z0, z1, ntx, nty, zc;
        plan_box(plan, box_of_tile(tile_g, plan), tile_g, x0, x1, y0, y1, z0, z1, ntx, nty, zc,
                 multi_tile);
        box = Box{x0, x1, y0, y1, z0, z1};
        map.ntx = ntx;
        map.nty = nty;
        map.zc = zc;
    }
    // the box's bounds as plain scalars (a struct captured by the lambdas
    // below costs registers)
    const int bx0 = box.x0, bx1 = box.x1, by0 = box.y0, by1 = box.y1;
    using T = typename Prec<PREC>::T;
    using Rt = typename Prec<PREC>::Rt;
    using D2 = typename Prec<PREC>::D2;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* __restrict__ lds = reinterpret_cast<T*>(smem_raw);
    // hand-over area past the ring: F's NXF values per cell, then M's NXM
    Rt* __restrict__ xch = reinterpret_cast<Rt*>(smem_raw + ring_bytes<PREC, RAD>());  // [NXF + NXM][NC]
    using RG = SRing<PREC, RAD>;
    constexpr int TY = RG::TY, NC = RG::NC;
    constexpr int HX = RG::HX, PLANE = RG::PLANE, SLOT = RG::SLOT;
    constexpr int NSLOT = RG::NSLOT;
    constexpr bool LATE = physics_late<PREC>();
    constexpr int NXF = nxf<PREC>(), NXM = nxm<PREC>();

    const int tile = MULTI ? multi_tile : tile_of_block(blockIdx.x, map);
    if (tile == NO_TILE) return;  // the whole workgroup exits together
    // tile = (chunk * nty + ty) * ntx + tx; the chunk marches its own z range
    const int per_chunk = map.ntx * map.nty, ch = tile / per_chunk, txy = tile - ch * per_chunk;
    const int tx = txy % map.ntx, ty = txy / map.ntx;
    const int bz0 = box.z0 + ch * map.zc, bz1 = min(bz0 + map.zc, box.z1);
    constexpr int TX = RG::TX;
    const int x0 = bx0 + tx * TX, y0 = by0 + ty * TY;
    // group index, made visibly wave-uniform so that the two groups' code
    // paths (each with its own registers and the same barriers) are scalar
    // branches
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / NC);
    const int tid = threadIdx.x - grp * NC, lx = tid % TX, ly = tid / TX;
    const bool active = (x0 + lx < bx1) && (y0 + ly < by1);

    auto field_ptr = [&](auto* base, int q) { return base + q * g.fstride; };
    auto at = [](auto* p, unsigned idx) {
        using Pt = decltype(p);
        using C = typename std::conditional<std::is_const<typename std::remove_pointer<Pt>::type>::value,
                                            const char*, char*>::type;
        return reinterpret_cast<Pt>(reinterpret_cast<C>(p) + idx * (unsigned)sizeof(T));
    };

    // The whole march runs in one of two instantiations, one per group, so
    // that each group's registers are allocated for its own path only.  Both
    // execute the same sequence of barriers.
    auto march = [&](auto group_tag) {
        constexpr int G = decltype(group_tag)::value;
        // ---- per-thread load slots of the halo'd tile plane (clamped into the
        // padded grid for ragged tiles); each group loads its own four fields
        constexpr int q0 = 4 * G;  // first of the group's fields
        // Load units of the halo'd tile plane: with PAIRS, the first NFP * NC
        // pairs of x-neighbours (rows of HX cells are HX / 2 pairs; one 2-element
        // load and LDS store each), then NFE * NC cells one by one; without,
        // every cell one by one.  The NEE cells per field that do not fill the
        // group's threads are spread over them for all four fields together
        // (one load under a mask at RAD = 3, not one per field).  Ragged tiles
        // clamp the places to the last column and row that the box's cells read,
        // so that no line beyond them is fetched (a 3 x 256 x 256 slab, FP32C: 145 us
        // with the padded grid's end as the limit, here and for the idle threads' own
        // cells below; 102 now).
        typedef T Pair __attribute__((ext_vector_type(2)));
        constexpr int HP = HX / 2;
        constexpr int NFP = PAIRS ? (PLANE / 2) / NC : 0;   // pair slots per thread
        constexpr int CELLS0 = 2 * NFP * NC;                 // cells the pair slots cover
        constexpr int NFE = (PLANE - CELLS0) / NC, NEE = (PLANE - CELLS0) % NC;
        constexpr int NXS = (4 * NEE + NC - 1) / NC;         // left-over slots per thread
        const int xlast = bx1 + 2 * RAD - 1, ylast = by1 + 2 * RAD - 1;  // (padded)
        unsigned poff[NFP > 0 ? NFP : 1], coff[NFE > 0 ? NFE : 1];
        const T* xptr[NXS > 0 ? NXS : 1];
        int xlds[NXS > 0 ? NXS : 1];
#pragma unroll
        for (int k = 0; k < NFP; ++k) {
            const int p = tid + k * NC, r = p / HP, c = 2 * (p - r * HP);
            const int px = min(x0 + c, xlast & ~1), py = min(y0 + r, ylast);
            poff[k] = (unsigned)(py * g.mx + px);
        }
#pragma unroll
        for (int k = 0; k < NFE; ++k) {
            const int e = CELLS0 + tid + k * NC, r = e / HX, c = e - r * HX;
            const int px = min(x0 + c, xlast), py = min(y0 + r, ylast);
            coff[k] = (unsigned)(py * g.mx + px);
        }
#pragma unroll
        for (int k = 0; k < NXS; ++k) {
            const int i = min(tid + k * NC, 4 * NEE - 1), k4 = i / NEE;
            const int e = CELLS0 + NFE * NC + (i - k4 * NEE), r = e / HX, c = e - r * HX;
            const int px = min(x0 + c, xlast), py = min(y0 + r, ylast);
            xptr[k] = fin + (q0 + k4) * g.fstride + (py * g.mx + px);
            xlds[k] = (q0 + k4) * PLANE + e;
        }

        Pair prep[4][NFP > 0 ? NFP : 1];
        T prec_[4][NFE > 0 ? NFE : 1], prex[NXS > 0 ? NXS : 1];
        // field k4 of the group on plane t, and the left-over cells of all four:
        // their load units into registers
        auto load_field = [&](int k4, int t) {
            const unsigned zo = (unsigned)((t + RAD) * g.mxy);
            const T* f = field_ptr(fin, q0 + k4);
#pragma unroll
            for (int k = 0; k < NFP; ++k) prep[k4][k] = *reinterpret_cast<const Pair*>(at(f, poff[k] + zo));
#pragma unroll
            for (int k = 0; k < NFE; ++k) prec_[k4][k] = *at(f, coff[k] + zo);
        };
        auto load_rest = [&](int t) {
            const int64_t zo = (int64_t)(t + RAD) * g.mxy;
#pragma unroll
            for (int k = 0; k < NXS; ++k)
                if ((k + 1) * NC <= 4 * NEE || tid + k * NC < 4 * NEE) prex[k] = xptr[k][zo];
        };
        auto store_plane = [&](int slot) {
            T* base = lds + slot * SLOT + q0 * PLANE;
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {
#pragma unroll
                for (int k = 0; k < NFP; ++k) reinterpret_cast<Pair*>(base + k4 * PLANE)[tid + k * NC] = prep[k4][k];
#pragma unroll
                for (int k = 0; k < NFE; ++k) base[k4 * PLANE + CELLS0 + tid + k * NC] = prec_[k4][k];
            }
#pragma unroll
            for (int k = 0; k < NXS; ++k)
                if ((k + 1) * NC <= 4 * NEE || tid + k * NC < 4 * NEE) lds[slot * SLOT + xlds[k]] = prex[k];
        };

        // V(slot, q, dy, dx): field q of the ring slot at offset (dx, dy) from the
        // thread's cell.  Addressed from the cell's stencil corner so that every
        // offset is a non-negative constant the LDS instructions take as an immediate.
        const int corner = ly * HX + lx;  // cell (x - RAD, y - RAD) within a plane
        auto V = [&](int slot, int q, int dy, int dx) -> T {
            return lds[(slot * SLOT + corner) + (q * PLANE + (dy + RAD) * HX + (dx + RAD))];
        };

        // ---- z state of the group's fields: own-column history (t-RAD .. t-1),
        // indexed by field within the group, and the carried past halves of the
        // group's three xz/yz mixed combinations (past[cb][k]: output t+1+k):
        //   F: 0 Dxz uz, 1 Dyz uz, 2 Dxz ux + Dyz uy
        //   M: 0 Dxz Az, 1 Dyz Az, 2 Dxz Ax + Dyz Ay
        T hist[RAD][4];
        D2 past[3][RAD];

        // ring slot of plane p: p + SOFS > 0 for every plane the march touches
        // (p >= bz0), so an unsigned modulo gives the slot (an AND when NSLOT
        // is a power of two)
        constexpr int SOFS = 4 * NSLOT;
        auto slot_of = [](int p) { return (int)((unsigned)(p + SOFS) % (unsigned)NSLOT); };

        // the thread's cell on plane bz0, clamped into the box for the idle
        // threads of ragged tiles (which load, but never store)
        const unsigned cell0 = (unsigned)(g.interior + bz0 * g.mxy + min(y0 + ly, by1 - 1) * g.mx +
                                          min(x0 + lx, bx1 - 1));

        // ---- start of the march: planes bz0 .. bz0+RAD into the ring, and the
        // z state of plane bz0 from global memory, summed in the order in which
        // the march itself forms it (so that a chunk boundary changes no bit)
        {
            auto F = [&](int q, int dz, int dy, int dx) -> T {
                return *at(field_ptr(fin, q), cell0 + (unsigned)(dz * g.mxy + dy * g.mx + dx));
            };
            // one field's plane bz0 - j added to the past halves of outputs
            // bz0 .. bz0 + RAD - j
            auto add = [&](int q, int dir, int cb, bool first_of_combo, int j) {
                const double* wm = dir == 0 ? sc.wxz : sc.wyz;
#pragma unroll
                for (int m = RAD; m >= 1; --m) {
                    if (m < j) continue;
                    const D2 dd = dir == 0 ? D2(F(q, -j, 0, m)) - D2(F(q, -j, 0, -m))
                                           : D2(F(q, -j, m, 0)) - D2(F(q, -j, -m, 0));
                    D2& acc = past[cb][m - j];
                    acc = first_of_combo && m == RAD ? D2(wm[m - 1]) * dd : fmadd(D2(wm[m - 1]), dd, acc);
                }
            };
#pragma unroll
            for (int k = 0; k <= RAD; ++k) {
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) load_field(k4, bz0 + k);
                load_rest(bz0 + k);
                store_plane(slot_of(bz0 + k));
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = RAD; j >= 1; --j) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) hist[RAD - j][k4] = F(q0 + k4, -j, 0, 0);
                add(q0 + 3, 0, 0, true, j);
                add(q0 + 3, 1, 1, true, j);
                add(q0 + 1, 0, 2, true, j);
                add(q0 + 2, 1, 2, false, j);
            }
            __syncthreads();  // the first RAD + 1 planes are visible
        }

        const int nplanes = bz1 - bz0;
        // (a lambda that the loop calls: the compiler needs fewer registers than
        // for the same text as the loop's body, and the FP64 kernels at r = 2
        // and 3 ran 3.5% faster)
        auto plane_step = [&](const int u) {
            const int t = bz0 + u;
            // plane t + RAD + 1 is fetched while the derivatives begin; the chunk's
            // last plane fetches its newest one again rather than branch
            const int tn = t + RAD + (u + 1 < nplanes ? 1 : 0);
            const unsigned cell = cell0 + (unsigned)(u * g.mxy);
            const int s0 = slot_of(t);
            Derivs<Rt> d;
            T fc[4], wold[4] = {}, cc[4] = {};
            Rt rhs[4];
            EntropyOwn<Rt> own;
            Rt S[3][3], divu, SS, B[3], J[3];  // LATE only
            {
                int sl[RAD + 1];  // ring slots of planes t .. t+RAD
#pragma unroll
                for (int k = 0; k <= RAD; ++k) sl[k] = slot_of(t + k);

                if (s > 0) {
#pragma unroll
                    for (int k4 = 0; k4 < 4; ++k4) wold[k4] = *at(field_ptr(w, q0 + k4), cell);
                }
                if constexpr (PREC == MHD_F32C) {
#pragma unroll
                    for (int k4 = 0; k4 < 4; ++k4) cc[k4] = *at(field_ptr(comp, q0 + k4), cell);
                }
                load_rest(tn);
                // ---- what one field's derivatives read: the axis lines of plane t and
                // the own column (A), the planar diagonals and the x or y line of
                // the future planes (B), both lines of the future planes (C)
                auto rdA = [&](LineA<T, RAD>& L, int q) {
#pragma unroll
                    for (int m = 1; m <= RAD; ++m) {
                        L.x[0][m - 1] = V(s0, q, 0, -m);
                        L.x[1][m - 1] = V(s0, q, 0, m);
                        L.y[0][m - 1] = V(s0, q, -m, 0);
                        L.y[1][m - 1] = V(s0, q, m, 0);
                        L.z[m - 1] = V(sl[m], q, 0, 0);
                    }
                    L.c = V(s0, q, 0, 0);
                };
                auto rdF = [&](T f[2][RAD], int q, int dir) {
#pragma unroll
                    for (int m = 1; m <= RAD; ++m) {
                        f[0][m - 1] = dir == 0 ? V(sl[m], q, 0, -m) : V(sl[m], q, -m, 0);
                        f[1][m - 1] = dir == 0 ? V(sl[m], q, 0, m) : V(sl[m], q, m, 0);
                    }
                };
                auto rdB = [&](LineB<T, RAD>& L, int q, int dir) {
#pragma unroll
                    for (int m = 1; m <= RAD; ++m) {
                        L.d[0][m - 1] = V(s0, q, m, m);
                        L.d[1][m - 1] = V(s0, q, -m, -m);
                        L.d[2][m - 1] = V(s0, q, -m, m);
                        L.d[3][m - 1] = V(s0, q, m, -m);
                    }
                    rdF(L.f, q, dir);
                };
                auto rdC = [&](LineC<T, RAD>& L, int q) {
                    rdF(L.fx, q, 0);
                    rdF(L.fy, q, 1);
                };
                // first derivative along x (0) or y (1), or z (2); LATE: not yet scaled
                // (scaled beside its use, where the compiler fuses the product as
                // it does in the other kernels)
                auto first = [&](const LineA<T, RAD>& L, int k4, int dir) -> Rt {
                    auto g1 = [&](int m) -> Rt {
                        if (dir == 2) return Rt(L.z[m - 1]) - Rt(hist[RAD - m][k4]);
                        return dir == 0 ? Rt(L.x[1][m - 1]) - Rt(L.x[0][m - 1])
                                        : Rt(L.y[1][m - 1]) - Rt(L.y[0][m - 1]);
                    };
                    Rt acc = Rt(W1(RAD, 1)) * g1(1);
#pragma unroll
                    for (int m = 2; m <= RAD; ++m) acc += Rt(W1(RAD, m)) * g1(m);
                    return LATE ? acc : acc * Rt(sc.d1[dir]);
                };
                auto second = [&](const LineA<T, RAD>& L, int k4, D2& xx, D2& yy, D2& zz) {
                    const D2 f0 = D2(W2(RAD, 0)) * D2(L.c);
                    D2 ax = D2(W2(RAD, 1)) * (D2(L.x[1][0]) + D2(L.x[0][0]));
#pragma unroll
                    for (int m = 2; m <= RAD; ++m) ax += D2(W2(RAD, m)) * (D2(L.x[1][m - 1]) + D2(L.x[0][m - 1]));
                    xx = (ax + f0) * D2(sc.d2[0]);
                    D2 ay = D2(W2(RAD, 1)) * (D2(L.y[1][0]) + D2(L.y[0][0]));
#pragma unroll
                    for (int m = 2; m <= RAD; ++m) ay += D2(W2(RAD, m)) * (D2(L.y[1][m - 1]) + D2(L.y[0][m - 1]));
                    yy = (ay + f0) * D2(sc.d2[1]);
                    D2 az = D2(W2(RAD, 1)) * (D2(L.z[0]) + D2(hist[RAD - 1][k4]));
#pragma unroll
                    for (int m = 2; m <= RAD; ++m) az += D2(W2(RAD, m)) * (D2(L.z[m - 1]) + D2(hist[RAD - m][k4]));
                    zz = (az + f0) * D2(sc.d2[2]);
                };
                auto dxy = [&](const LineB<T, RAD>& L) -> D2 {
                    auto e = [&](int m) {
                        return (D2(L.d[0][m - 1]) + D2(L.d[1][m - 1])) - (D2(L.d[2][m - 1]) + D2(L.d[3][m - 1]));
                    };
                    D2 acc = D2(W2(RAD, 1)) * e(1);
#pragma unroll
                    for (int m = 2; m <= RAD; ++m) acc += D2(W2(RAD, m)) * e(m);
                    return acc * D2(sc.mxy);
                };
                // The xz (dir 0) / yz (dir 1) mixed derivative of the group's
                // combination cb is its future half (future) minus the carried past
                // half; carry() returns that past half and adds plane t's own
                // differences to the past halves of outputs t+1 .. t+RAD.
                auto carry = [&](const LineA<T, RAD>& L, int dir, int cb, bool first_of_combo) -> D2 {
                    const double* wm = dir == 0 ? sc.wxz : sc.wyz;
                    const D2 p0 = past[cb][0];
#pragma unroll
                    for (int m = 1; m <= RAD; ++m) {
                        const D2 wd = D2(wm[m - 1]);
                        const D2 e = dir == 0 ? D2(L.x[1][m - 1]) - D2(L.x[0][m - 1])
                                              : D2(L.y[1][m - 1]) - D2(L.y[0][m - 1]);
                        if (!first_of_combo)
                            past[cb][m - 1] = fmadd(wd, e, past[cb][m - 1]);
                        else
                            past[cb][m - 1] = m < RAD ? fmadd(wd, e, past[cb][m < RAD ? m : 0]) : wd * e;
                    }
                    return p0;
                };
                auto future = [&](const T f[2][RAD], int dir) -> D2 {
                    const double* wm = dir == 0 ? sc.wxz : sc.wyz;
                    D2 res = D2(wm[0]) * (D2(f[1][0]) - D2(f[0][0]));
#pragma unroll
                    for (int m = 2; m <= RAD; ++m) res += D2(wm[m - 1]) * (D2(f[1][m - 1]) - D2(f[0][m - 1]));
                    return res;
                };
#define MHD_PHASE_FENCE() __builtin_amdgcn_sched_barrier(0)
                auto pin_past = [&](int cb) {
#pragma unroll
                    for (int k = 0; k < RAD; ++k) pin(past[cb][k]);
                };
                // the field's centre value (the 2N update's f_in) and the history shift
                auto centre = [&](const LineA<T, RAD>& L, int k4) {
                    fc[k4] = L.c;
#pragma unroll
                    for (int k = 0; k + 1 < RAD; ++k) hist[k][k4] = hist[k + 1][k4];
                    hist[RAD - 1][k4] = fc[k4];
                    return Rt(fc[k4]);
                };
                // ---- the group's fields in turn; each step first issues the next
                // step's LDS reads, so that they are in flight during its arithmetic
                const Phys P = *P_dev;
                LineA<T, RAD> A0, A1, A2, A3;
                LineB<T, RAD> B1, B2;
                LineC<T, RAD> C3;
                D2 grad[3], mix, mix2;  // F: grad(div u); M: mu0 j
                D2 xx, yy, zz;
                rdA(A0, q0);
                load_field(0, tn);
                load_field(1, tn);
                // The loads go out over the first four steps, early enough to land
                // before the ring store (one field per step up to the last one:
                // order 8 at 256^3 4340 -> 4085 us per step, the others 0-1%); at
                // r = 1 the plane is short and all go first (3150 -> 3000 us).
                constexpr bool SPREAD = RAD > 1;
                if constexpr (!SPREAD) {
                    load_field(2, tn);
                    load_field(3, tn);
                }
                MHD_PHASE_FENCE();
                // lnrho / ss
                rdA(A1, q0 + 1);
                MHD_PHASE_FENCE();
                {
                    Rt(&gr)[3] = G == 0 ? d.gl : d.gs;
                    Rt& lap = G == 0 ? d.lapl : d.laps;
#pragma unroll
                    for (int a = 0; a < 3; ++a) gr[a] = first(A0, 0, a);
                    second(A0, 0, xx, yy, zz);
                    lap = Rt(xx + yy + zz);
                    (G == 0 ? d.lnrho : d.ss) = centre(A0, 0);
                    pin(gr[0], gr[1], gr[2], lap);
                }
                MHD_PHASE_FENCE();
                // ux / Ax: axis lines
                rdB(B1, q0 + 1, 0);
                if constexpr (SPREAD) load_field(2, tn);
                MHD_PHASE_FENCE();
                mix = carry(A1, 0, 2, true);
                second(A1, 1, xx, yy, zz);
                if constexpr (G == 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.gu[0][a] = first(A1, 1, a);
                    d.lapu[0] = Rt(xx + yy + zz);
                    grad[0] = xx;
                    d.ux = centre(A1, 1);
                    pin(d.gu[0][0], d.gu[0][1], d.gu[0][2], d.lapu[0], grad[0], mix);
                } else {
                    d.dAx_dy = first(A1, 1, 1);
                    d.dAx_dz = first(A1, 1, 2);
                    d.lapA[0] = Rt(xx + yy + zz);
                    grad[0] = -(yy + zz);
                    centre(A1, 1);
                    pin(d.dAx_dy, d.dAx_dz, d.lapA[0], grad[0], mix);
                }
                pin_past(2);
                MHD_PHASE_FENCE();
                // ux / Ax: mixed
                rdA(A2, q0 + 2);
                if constexpr (SPREAD) load_field(3, tn);
                MHD_PHASE_FENCE();
                grad[1] = dxy(B1);
                grad[2] = future(B1.f, 0) - mix;
                pin(grad[1], grad[2]);
                MHD_PHASE_FENCE();
                // uy / Ay: axis lines
                rdB(B2, q0 + 2, 1);
                MHD_PHASE_FENCE();
                carry(A2, 1, 2, false);
                second(A2, 2, xx, yy, zz);
                if constexpr (G == 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.gu[1][a] = first(A2, 2, a);
                    d.lapu[1] = Rt(xx + yy + zz);
                    grad[1] += yy;
                    d.uy = centre(A2, 2);
                    pin(d.gu[1][0], d.gu[1][1], d.gu[1][2], d.lapu[1], grad[1]);
                } else {
                    d.dAy_dx = first(A2, 2, 0);
                    d.dAy_dz = first(A2, 2, 2);
                    d.lapA[1] = Rt(xx + yy + zz);
                    grad[1] -= xx + zz;
                    centre(A2, 2);
                    pin(d.dAy_dx, d.dAy_dz, d.lapA[1], grad[1]);
                }
                pin_past(2);
                MHD_PHASE_FENCE();
                // uy / Ay: mixed
                rdA(A3, q0 + 3);
                MHD_PHASE_FENCE();
                grad[0] += dxy(B2);
                grad[2] += future(B2.f, 1);
                pin(grad[0], grad[2]);
                MHD_PHASE_FENCE();
                // uz / Az: axis lines
                rdC(C3, q0 + 3);
                MHD_PHASE_FENCE();
                mix = carry(A3, 0, 0, true);
                mix2 = carry(A3, 1, 1, true);
                second(A3, 3, xx, yy, zz);
                if constexpr (G == 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.gu[2][a] = first(A3, 3, a);
                    d.lapu[2] = Rt(xx + yy + zz);
                    grad[2] += zz;
                    d.uz = centre(A3, 3);
                    pin(d.gu[2][0], d.gu[2][1], d.gu[2][2], d.lapu[2], grad[2], mix, mix2);
                } else {
                    d.dAz_dx = first(A3, 3, 0);
                    d.dAz_dy = first(A3, 3, 1);
                    d.lapA[2] = Rt(xx + yy + zz);
                    grad[2] -= xx + yy;
                    centre(A3, 3);
                    pin(d.dAz_dx, d.dAz_dy, d.lapA[2], grad[2], mix, mix2);
                }
                pin_past(0);
                pin_past(1);
                MHD_PHASE_FENCE();
                // uz / Az: mixed
                if constexpr (G == 1) {
                    // group F's fields at this cell, straight from its ring plane
                    d.lnrho = Rt(V(s0, 0, 0, 0));
                    d.ux = Rt(V(s0, 1, 0, 0));
                    d.uy = Rt(V(s0, 2, 0, 0));
                    d.uz = Rt(V(s0, 3, 0, 0));
                } else if constexpr (LATE) {
                    d.ss = Rt(V(s0, 4, 0, 0));  // and the entropy of group M's
                }
                MHD_PHASE_FENCE();
                grad[0] += future(C3.fx, 0) - mix;
                grad[1] += future(C3.fy, 1) - mix2;
                pin(grad[0], grad[1]);
                MHD_PHASE_FENCE();
                if constexpr (G == 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.gdu[a] = Rt(grad[a]);
                    if constexpr (LATE) {
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            d.gl[b] *= Rt(sc.d1[b]);
#pragma unroll
                            for (int a = 0; a < 3; ++a) d.gu[a][b] *= Rt(sc.d1[b]);
                        }
                    }
                    Rt v[NXF] = {d.gl[0], d.gl[1], d.gl[2], d.lapl};
                    if constexpr (LATE) {
                        shear(d.gu, S, divu, SS);
                        v[4] = SS;
                        v[NXF - 1] = divu;
                    } else {
                        rhs_flow_own(d, P, rhs, v[4]);
                    }
#pragma unroll
                    for (int i = 0; i < NXF; ++i) xch[i * NC + tid] = v[i];
                } else {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.jmu[a] = Rt(grad[a]);
                    Rt v[NXM];
                    if constexpr (LATE) {
                        const Rt sx = Rt(sc.d1[0]), sy = Rt(sc.d1[1]), sz = Rt(sc.d1[2]);
                        d.dAx_dy *= sy; d.dAx_dz *= sz;
                        d.dAy_dx *= sx; d.dAy_dz *= sz;
                        d.dAz_dx *= sx; d.dAz_dy *= sy;
                        d.gs[0] *= sx; d.gs[1] *= sy; d.gs[2] *= sz;
                        Rt jxB[3];
                        magnetic(d, P, B, J, jxB);
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            v[a] = d.gs[a];
                            v[NXM - 3 + a] = jxB[a];
                        }
                    } else {
                        rhs_entropy_own(d, P, own, rhs, v, v[3]);
                    }
#pragma unroll
                    for (int i = 0; i < NXM; ++i) xch[(NXF + i) * NC + tid] = v[i];
                }
#undef MHD_PHASE_FENCE
            }

            // Every read of plane t is done and both groups' values are visible:
            // each group fetches the other's values and plane t+RAD+1 replaces
            // plane t in the ring.
            __syncthreads();
            constexpr int NIN = G == 0 ? NXM : NXF;
            Rt in[NIN];
#pragma unroll
            for (int i = 0; i < NIN; ++i) in[i] = xch[((G == 0 ? NXF : 0) + i) * NC + tid];
            store_plane(slot_of(t + RAD + 1));
            __syncthreads();  // plane t+RAD+1 visible; the hand-over area is free

            // The right-hand sides completed, and the 2N update.
            if constexpr (LATE) {
                if constexpr (G == 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.gs[a] = in[a];
                    rhs_flow(d, *P_dev, S, divu, in + 3, rhs);
                } else {
#pragma unroll
                    for (int a = 0; a < 3; ++a) d.gl[a] = in[a];
                    d.lapl = in[3];
                    rhs_entropy_induction(d, *P_dev, in[NIN - 1], in[4], B, J, rhs);
                }
            } else if constexpr (G == 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) rhs[1 + a] += in[a] - in[3] * d.gl[a];
            } else {
                rhs_entropy_other(*P_dev, own, in, in[3], in[4], rhs[0]);
            }
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {
                T wnew, fnew, cnew = cc[k4];
                rk_values<PREC>(s, fc[k4], wold[k4], rhs[k4], dt, wnew, fnew, cnew);
                if (active) {
                    *at(field_ptr(w, q0 + k4), cell) = wnew;
                    *at(field_ptr(fout, q0 + k4), cell) = fnew;
                    if constexpr (PREC == MHD_F32C) *at(field_ptr(comp, q0 + k4), cell) = cnew;
                }
            }
        };
        for (int u = 0; u < nplanes; ++u) plane_step(u);
    };
    if (grp == 0)
        march(std::integral_constant<int, 0>{});
    else
        march(std::integral_constant<int, 1>{});
}

// Whether the boxes fill less than 0.8 of their tiles' columns.  Such tiles ask less
// of the memory system, latency bounds the march, and a second workgroup per CU pays
// where whole tiles lose by it.  us per step, FP32C second order, with one and two
// (share of the columns): 16 x 500 x 500 925 -> 812 (0.50), 40 x 400 x 300 1050 -> 986 (0.63),
// 100^3 159 -> 144 (0.75), 300 x 20 x 400 461 -> 441 (0.78); 200^3 1338 -> 1402 (0.89),
// 256^3 2409 -> 2545 (1).
bool ragged_tiles(const Box* bx, int nbox, int tx, int ty)
{
    int64_t cells = 0, tiles = 0;
    for (int k = 0; k < nbox; ++k) {
        const int64_t nx = bx[k].x1 - bx[k].x0, ny = bx[k].y1 - bx[k].y0, nz = bx[k].z1 - bx[k].z0;
        cells += nx * ny * nz;
        tiles += (nx + tx - 1) / tx * ((ny + ty - 1) / ty) * nz;
    }
    return 10 * cells < 8 * tiles * tx * ty;
}

template <int PREC, int RAD>
hipError_t launch_one(const Grid& g, const Phys& P, const Phys* P_dev, const Box* bx, int nbox,
                      int s, const void* f_in, void* f_out, void* w, void* comp, double dt,
                      hipStream_t st)
{
    using T = typename Prec<PREC>::T;
    const bool two = two_if_ragged<PREC, RAD>() &&
                     ragged_tiles(bx, nbox, SRing<PREC, RAD>::TX, SRing<PREC, RAD>::TY);
    const size_t lds = two ? lds_needed<PREC, RAD>() : lds_bytes<PREC, RAD>();
    // pair fetches, where they measured faster: FP64 (9.51 -> 9.36 ms per substep
    // before the loads were spread), FP32 storage up to order 6 (512^3 step
    // 21.3 -> 20.8 ms with compensation, 15.5 -> 14.5 plain, both before the physics
    // moved behind the hand-over; 20.6 and 15.0 since), not at order 8
    // (256^3 step 3.05 -> 3.10 ms)
    constexpr bool PAIRS_OK = PREC == MHD_F64 || RAD < 4;
    // once per instantiation (thread-safe static initialisation): the LDS
    // limit of every variant, and the workgroups resident at once (a round)
    struct Setup {
        hipError_t err;
        int round, round_two;
    };
    static const Setup setup = []() -> Setup {
        const void* kernels[4] = {(const void*)k_rk3_split<PREC, RAD, false, false>,
                                  (const void*)k_rk3_split<PREC, RAD, true, false>, nullptr,
                                  nullptr};
        if constexpr (PAIRS_OK) {
            kernels[2] = (const void*)k_rk3_split<PREC, RAD, false, PAIRS_OK>;
            kernels[3] = (const void*)k_rk3_split<PREC, RAD, true, PAIRS_OK>;
        }
        hipError_t e = hipSuccess;
        for (int k = 0; k < 4 && e == hipSuccess; ++k)
            if (kernels[k])
                e = hipFuncSetAttribute(kernels[k], hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)lds_bytes<PREC, RAD>());
        int per_cu = 0, two_per_cu = 0, dev = 0, cus = 0;
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_rk3_split<PREC, RAD, false, false>,
                                                             SRing<PREC, RAD>::NTH, lds_bytes<PREC, RAD>());
        if (e == hipSuccess && two_if_ragged<PREC, RAD>())
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&two_per_cu, k_rk3_split<PREC, RAD, false, false>,
                                                             SRing<PREC, RAD>::NTH, lds_needed<PREC, RAD>());
        if (e == hipSuccess) e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        return Setup{e, per_cu * cus, min(two_per_cu, 2) * cus};
    }();
    if (setup.err != hipSuccess) return setup.err;
    const int round = two ? setup.round_two : setup.round;
    const TilePlan plan =
        plan_tiles(bx, nbox, SRing<PREC, RAD>::TX, SRing<PREC, RAD>::TY, round);
    Scales<RAD> sc{};
    for (int a = 0; a < 3; ++a) {
        sc.d1[a] = P.inv_h[a] / DEN1(RAD);
        sc.d2[a] = P.inv_h[a] * P.inv_h[a] / DEN2(RAD);
    }
    sc.mxy = P.inv_h[0] * P.inv_h[1] / (4.0 * DEN2(RAD));
    for (int k = 1; k <= RAD; ++k) {
        sc.wxz[k - 1] = W2(RAD, k) * P.inv_h[0] * P.inv_h[2] / (4.0 * DEN2(RAD));
        sc.wyz[k - 1] = W2(RAD, k) * P.inv_h[1] * P.inv_h[2] / (4.0 * DEN2(RAD));
    }
    const dim3 grid(plan_blocks(plan)), block(SRing<PREC, RAD>::NTH);
    const bool pairs = PAIRS_OK && pairs_aligned(g, bx, nbox, f_in, sizeof(T));
#define MHD_SPLIT_LAUNCH(MULTI, PAIRS, MAP, BOX, PLAN)                                          \
    hipLaunchKernelGGL((k_rk3_split<PREC, RAD, MULTI, PAIRS>), grid, block, lds, st, g, P_dev, sc, \
                       MAP, s, (const T*)f_in, (T*)f_out, (T*)w, (T*)comp, dt, BOX, PLAN)
    if (pairs) {
        if constexpr (PAIRS_OK) {
            if (nbox == 1)
                MHD_SPLIT_LAUNCH(false, PAIRS_OK, plan_map(plan), plan.box[0], TilePlan{});
            else
                MHD_SPLIT_LAUNCH(true, PAIRS_OK, TileMap{}, Box{}, plan);
        }
    } else if (nbox == 1) {
        MHD_SPLIT_LAUNCH(false, false, plan_map(plan), plan.box[0], TilePlan{});
    } else {
        MHD_SPLIT_LAUNCH(true, false, TileMap{}, Box{}, plan);
    }
#undef MHD_SPLIT_LAUNCH
    return hipGetLastError();
}

}  // namespace
}  // namespace mhd
