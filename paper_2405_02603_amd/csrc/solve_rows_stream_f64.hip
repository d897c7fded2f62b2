// Launcher of the streaming forward row pass (double, rows below 384).
#include "solve_launch.hpp"

namespace fsp {
template hipError_t launch_p1<double, true>(int, int, const RowArgs&, int, hipStream_t);
}  // namespace fsp
