// Launch of a gate chain (device side of sv_chain_host.h).
#pragma once

#include <hip/hip_runtime.h>

#include "sv_chain_host.h"

namespace sv {
namespace chain {

// Runs a fused step on the 2^n state psi; gate[i].op are offsets from ops, in device memory.
hipError_t launch(int n, const Step &s, float2 *psi, const char *ops, hipStream_t st);

}  // namespace chain
}  // namespace sv
