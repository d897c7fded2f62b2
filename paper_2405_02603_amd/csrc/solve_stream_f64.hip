// Launchers of the streaming forms (double): the forward row pass (rows below 384), the inverse axis-1 pass.
#include "solve_launch.hpp"

namespace fsp {
template hipError_t launch_p1<double, true>(int, int, const RowArgs&, int, hipStream_t);
template hipError_t launch_p4_stream<double>(int, int, const ColArgs&, int, hipStream_t);
}  // namespace fsp
