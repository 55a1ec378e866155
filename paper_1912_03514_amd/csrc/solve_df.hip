// Instances of the persistent solve kernel: A in FP64, inner operator in FP32.
#include "solve_pick.hpp"

namespace mihs {
template SolveKernel pick_kernel_typed<double, float>(int, bool, bool);
}  // namespace mihs
