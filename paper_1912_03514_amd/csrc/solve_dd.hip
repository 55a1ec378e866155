// Instances of the persistent solve kernel: A in FP64, inner operator in FP64.
#include "solve_pick.hpp"

namespace mihs {
template SolveKernel pick_kernel_typed<double, double>(int, bool, bool);
}  // namespace mihs
