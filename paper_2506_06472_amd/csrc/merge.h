// Neighbours in the schedule that go out in one launch.
#pragma once
#include <cstdint>
#include <vector>

#include "analysis.h"
#include "program.h"

namespace tio {

// Per kernel: how many from it on one launch does (1: itself alone; kernels inside a launch: 1).  at: per kernel and role, where the
// operand lies in the arena (ignored for absent ones).  Host only.
std::vector<int> merged_launches(const Program &prog, const Plan &plan, const std::vector<std::vector<uint64_t>> &at);

}  // namespace tio
