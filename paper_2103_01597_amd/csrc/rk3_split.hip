// The fused RHS + RK3 substep (rk3_march.hpp): the FP64 instantiations, and the
// choice of an instantiation by precision and stencil radius.
#include "rk3_march.hpp"

namespace mhd {

// The FP32-storage instantiations (rk3_tiled.hip).
hipError_t launch_rk3_f32(const Grid& g, const Phys& P, const Phys* P_dev, int precision,
                          const Box* bx, int nbox, int s, const void* f_in, void* f_out, void* w,
                          void* comp, double dt, hipStream_t st);

// P (host copy) sets the stencil scales; P_dev (device copy of the same
// values) is what the kernel's physics reads.  The stencil radius is the
// grid's halo width g.r (1..4).  One launch updates the nbox (1..MAX_BOXES)
// disjoint, non-empty boxes bx.
hipError_t launch_rk3_march(const Grid& g, const Phys& P, const Phys* P_dev, int precision,
                            const Box* bx, int nbox, int s, const void* f_in, void* f_out,
                            void* w, void* comp, double dt, hipStream_t st)
{
    if (precision != MHD_F64)
        return launch_rk3_f32(g, P, P_dev, precision, bx, nbox, s, f_in, f_out, w, comp, dt, st);
    static_assert(lds_bytes<MHD_F64, 3>() <= 160 * 1024 && lds_bytes<MHD_F64, 4>() <= 160 * 1024,
                  "FP64 ring exceeds the LDS");
    switch (g.r) {
    case 1: return launch_one<MHD_F64, 1>(g, P, P_dev, bx, nbox, s, f_in, f_out, w, nullptr, dt, st);
    case 2: return launch_one<MHD_F64, 2>(g, P, P_dev, bx, nbox, s, f_in, f_out, w, nullptr, dt, st);
    case 3: return launch_one<MHD_F64, 3>(g, P, P_dev, bx, nbox, s, f_in, f_out, w, nullptr, dt, st);
    case 4: return launch_one<MHD_F64, 4>(g, P, P_dev, bx, nbox, s, f_in, f_out, w, nullptr, dt, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mhd
