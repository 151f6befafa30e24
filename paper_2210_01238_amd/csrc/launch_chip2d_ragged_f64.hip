#include "launch_chip2d.inc.h"
namespace jk {
hipError_t launch_chip2d_ragged_f64(int rr, const Chip2dLaunch &a) { return chip2d_dispatch<double, true>(rr, a); }
}
