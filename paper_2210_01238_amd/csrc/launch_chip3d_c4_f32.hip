#include "launch_chip3d.inc.h"
namespace jk {
hipError_t launch_chip3d_c4_f32(int rz, int ry, int nxw, const Chip3dLaunch &a) { return chip3d_dispatch<float, 4>(rz, ry, nxw, a); }
}
