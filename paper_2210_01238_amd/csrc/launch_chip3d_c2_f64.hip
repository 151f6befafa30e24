#include "launch_chip3d.inc.h"
namespace jk {
hipError_t launch_chip3d_c2_f64(int rz, int ry, int nxw, const Chip3dLaunch &a) { return chip3d_dispatch<double, 2>(rz, ry, nxw, a); }
}
