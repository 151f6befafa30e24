#include "launch_chip2d.inc.h"
namespace jk {
hipError_t launch_chip2d_ragged_f32(int rr, const Chip2dLaunch &a) { return chip2d_dispatch<float, true>(rr, a); }
}
