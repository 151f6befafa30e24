// Dispatch over the compiled variants of chip3d_kernel for one element type, of those with some number of cells per lane.
// Included by launch_chip3d_c{1,2,4}_{f64,f32}.hip.
#include "chip3d_kernel.h"

namespace jk {

template <typename T, int C>
static hipError_t chip3d_dispatch(int rz, int ry, int nxw, const Chip3dLaunch &a)
{
    const int per_workgroup = nxw == 2 ? 1 : 2, nb = a.p.z.nb * a.p.y.nb;
    const dim3 grid((unsigned)((nb + per_workgroup - 1) / per_workgroup)), block(BLK_WAVES * WAVE);
#define JK_L(C_, RZ_, RY_, NXW_)                                                                                             \
    if constexpr (C == C_) if (rz == RZ_ && ry == RY_ && nxw == NXW_) {                                                      \
        hipLaunchKernelGGL((chip3d_kernel<T, C_, RZ_, RY_, NXW_>), grid, block, 0, a.st, a.g, a.p, (T *)a.in, (T *)a.out);   \
        return hipGetLastError();                                                                                            \
    }
    JK_CHIP3D_VARIANTS(JK_L)
    if constexpr (sizeof(T) == 4) { JK_CHIP3D_VARIANTS_F32(JK_L) }
#undef JK_L
    return hipErrorInvalidValue;
}

}  // namespace jk
