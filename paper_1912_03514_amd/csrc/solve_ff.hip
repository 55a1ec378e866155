// Instances of the persistent solve kernel: A in FP32, inner operator in FP32.
#include "solve_pick.hpp"

namespace mihs {
template SolveKernel pick_kernel_typed<float, float>(int, bool, bool);
}  // namespace mihs
