#include "launch_blocks3d.inc.h"
namespace jk {
hipError_t launch_blocks3d_f64(int c, int rz, int ry, const Blocks3dLaunch &a) { return blocks3d_dispatch<double>(c, rz, ry, a); }
}
