// Dispatch over the compiled variants of chip2d_kernel for one element type and kind of cut.
// Included by launch_chip2d_{even,ragged}_{f64,f32}.hip.
#include "chip2d_kernel.h"

namespace jk {

template <typename T, bool RAGGED>
static hipError_t chip2d_dispatch(int rr, const Chip2dLaunch &a)
{
    const dim3 grid((unsigned)(a.p.x.nb * a.p.y.nb)), block(BLK_WAVES * WAVE);
#define JK_L(RR_, LT_, LB_)                                                                                                  \
    if constexpr (chip2d_compiled(RR_, sizeof(T) == 8, RAGGED)) if (rr == RR_) {                                             \
        hipLaunchKernelGGL((chip2d_kernel<T, RR_, LT_, LB_, RAGGED>), grid, block, 0, a.st, a.g, a.p, (T *)a.in, (T *)a.out);\
        return hipGetLastError();                                                                                            \
    }
    JK_CHIP2D_VARIANTS(JK_L)
#undef JK_L
    return hipErrorInvalidValue;
}

}  // namespace jk
