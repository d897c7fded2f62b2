// Whole-solve kernel of tiny grids (double).
#include "tiny_kernel.hpp"

namespace fsp {
template hipError_t launch_tiny<double>(const TinyArgs&, int, hipStream_t);
}  // namespace fsp
