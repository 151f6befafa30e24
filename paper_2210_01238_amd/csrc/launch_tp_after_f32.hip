#include "launch_tp.inc.h"
namespace jk {
hipError_t launch_tp_after_f32(int levels, int mode, const LaunchArgs &a) { return tp_dispatch<float, true>(levels, mode, a); }
}
