#include "launch_tp.inc.h"
namespace jk {
hipError_t launch_tp_f32(int depth, int mode, const LaunchArgs &a) { return tp_dispatch<float, false>(depth, mode, a); }
}
