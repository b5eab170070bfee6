// The fused RHS + RK3 substep (rk3_march.hpp): the FP32-storage instantiations,
// compensated (FP32C) and plain (FP32).
#include "rk3_march.hpp"

namespace mhd {

hipError_t launch_rk3_f32(const Grid& g, const Phys& P, const Phys* P_dev, int precision,
                          const Box* bx, int nbox, int s, const void* f_in, void* f_out, void* w,
                          void* comp, double dt, hipStream_t st)
{
    const bool c = precision == MHD_F32C;
#define MHD_LAUNCH(PREC, RAD) \
    launch_one<PREC, RAD>(g, P, P_dev, bx, nbox, s, f_in, f_out, w, c ? comp : nullptr, dt, st)
    switch (g.r) {
    case 1: return c ? MHD_LAUNCH(MHD_F32C, 1) : MHD_LAUNCH(MHD_F32, 1);
    case 2: return c ? MHD_LAUNCH(MHD_F32C, 2) : MHD_LAUNCH(MHD_F32, 2);
    case 3: return c ? MHD_LAUNCH(MHD_F32C, 3) : MHD_LAUNCH(MHD_F32, 3);
    case 4: return c ? MHD_LAUNCH(MHD_F32C, 4) : MHD_LAUNCH(MHD_F32, 4);
    default: return hipErrorInvalidValue;
    }
#undef MHD_LAUNCH
}

}  // namespace mhd
