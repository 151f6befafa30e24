#include "launch_blocks2d.inc.h"
namespace jk {
hipError_t launch_blocks2d_f64(int c, int rw, const Blocks2dLaunch &a) { return blocks2d_dispatch<double>(c, rw, a); }
}
