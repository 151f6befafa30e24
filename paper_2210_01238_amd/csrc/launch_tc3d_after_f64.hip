#include "launchers.h"
namespace jk {
hipError_t launch_tc3d_after_f64(const LaunchArgs &a)
{
    constexpr int LEVELS = TC3D_MAX;
    hipLaunchKernelGGL((sweep3d_tc_kernel<double, MODE_AFTER, LEVELS, tc3d_rows_per_wave(LEVELS), TC3D_WAVES, 2>), dim3(a.nwg), dim3(TC3D_WAVES * WAVE), 0, a.st,
                       a.g, a.sp, a.aux, (const double *)a.src, (double *)a.dst, a.partial);
    return hipGetLastError();
}
}
