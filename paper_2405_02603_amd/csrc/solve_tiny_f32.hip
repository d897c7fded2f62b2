// Whole-solve kernel of tiny grids (float).
#include "tiny_kernel.hpp"

namespace fsp {
template hipError_t launch_tiny<float>(const TinyArgs&, int, hipStream_t);
}  // namespace fsp
