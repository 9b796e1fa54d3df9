// A plan's fused blocks, shared by the planners (sv_plan.cpp) and the code
// that runs them (sv_api.hip).  Plain C++, no HIP.
#pragma once

#include <cstdint>
#include <vector>

struct SvBlock {
  int k = 0;
  int ngates = 0;
  bool diag = true;
  std::vector<int32_t> tuple;    // ordered logical targets (ascending)
  std::vector<double> matrix;    // complex128 interleaved, 2^k x 2^k
  bool swap = false;             // a layout-swap block: no matrix, tuple[j] goes to physical bit dest[j]
  std::vector<int32_t> dest;
};

struct sv_plan {
  int n = 0;
  std::vector<SvBlock> blocks;
};
