// Dispatch over the compiled variants of blocks2d_kernel for one element type.
// Included by launch_blocks2d_f64.hip and launch_blocks2d_f32.hip.
#include "blocks2d_kernel.h"

namespace jk {

template <typename T>
static hipError_t blocks2d_dispatch(int c, int rw, const Blocks2dLaunch &a)
{
    const dim3 grid((unsigned)(a.p.x.nb * a.p.y.nb)), block(BLK_WAVES * WAVE);
#define JK_L(C_, RW_, E64_, E32_)                                                                                                 \
    if (c == C_ && rw == RW_) {                                                                                              \
        hipLaunchKernelGGL((blocks2d_kernel<T, C_, RW_>), grid, block, 0, a.st, a.g, a.p, (T *)a.in, (T *)a.out);            \
        return hipGetLastError();                                                                                            \
    }
    JK_BLOCKS2D_VARIANTS(JK_L)
    if constexpr (sizeof(T) == 4) { JK_BLOCKS2D_VARIANTS_F32(JK_L) }
#undef JK_L
    return hipErrorInvalidValue;
}

}  // namespace jk
