#include "launch_chip3d.inc.h"
namespace jk {
hipError_t launch_chip3d_c1_f64(int rz, int ry, int nxw, const Chip3dLaunch &a) { return chip3d_dispatch<double, 1>(rz, ry, nxw, a); }
}
