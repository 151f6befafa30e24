#include "launch_tp.inc.h"
namespace jk {
hipError_t launch_tp_after_f64(int levels, int mode, const LaunchArgs &a) { return tp_dispatch<double, true>(levels, mode, a); }
}
