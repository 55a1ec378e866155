// Definition behind the explicit instances of the solve_*.hip files.
#pragma once

#include "solve_kernel.hpp"

namespace mihs {

template <typename TA, typename TS>
SolveKernel pick_kernel_typed(int ept, bool gram, bool res) {
  if (gram) return res ? pick_by_ept<TA, TS, true, true>(ept) : pick_by_ept<TA, TS, true, false>(ept);
  return res ? pick_by_ept<TA, TS, false, true>(ept) : pick_by_ept<TA, TS, false, false>(ept);
}

}  // namespace mihs
