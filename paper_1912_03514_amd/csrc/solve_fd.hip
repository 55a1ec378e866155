// Instances of the persistent solve kernel: A in FP32, inner operator in FP64.
#include "solve_pick.hpp"

namespace mihs {
template SolveKernel pick_kernel_typed<float, double>(int, bool, bool);
}  // namespace mihs
