// Dispatch over the compiled variants of blocks3d_kernel for one element type.
// Included by launch_blocks3d_f64.hip and launch_blocks3d_f32.hip.
#include "blocks3d_kernel.h"

namespace jk {

template <typename T>
static hipError_t blocks3d_dispatch(int c, int rz, int ry, const Blocks3dLaunch &a)
{
    const dim3 grid((unsigned)(a.p.z.nb * a.p.y.nb)), block(BLK_WAVES * WAVE);
    T *ga = (T *)a.in, *gb = (T *)a.out;
#define JK_L(C_, RZ_, RY_, ...)                                                                                              \
    if (c == C_ && rz == RZ_ && ry == RY_) {                                                                                 \
        if (a.p.nx == WAVE * C_)                                                                                             \
            hipLaunchKernelGGL((blocks3d_kernel<T, C_, RZ_, RY_, true>), grid, block, 0, a.st, a.g, a.p, ga, gb);            \
        else hipLaunchKernelGGL((blocks3d_kernel<T, C_, RZ_, RY_, false>), grid, block, 0, a.st, a.g, a.p, ga, gb);          \
        return hipGetLastError();                                                                                            \
    }
    JK_BLOCKS3D_VARIANTS(JK_L)
    if constexpr (sizeof(T) == 4) { JK_BLOCKS3D_VARIANTS_F32(JK_L) }
#undef JK_L
    return hipErrorInvalidValue;
}

}  // namespace jk
