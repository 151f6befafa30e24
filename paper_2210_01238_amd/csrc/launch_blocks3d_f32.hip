#include "launch_blocks3d.inc.h"
namespace jk {
hipError_t launch_blocks3d_f32(int c, int rz, int ry, const Blocks3dLaunch &a) { return blocks3d_dispatch<float>(c, rz, ry, a); }
}
