// Launch of a fused tile pass (device side of sv_pass_host.h).
#pragma once

#include <hip/hip_runtime.h>

#include "sv_pass_host.h"

namespace sv {
namespace pass {

// Runs f on the 2^n state psi; data_dev holds f.data in device memory, 256-byte aligned.
hipError_t launch(int n, const Fused &f, float2 *psi, const char *data_dev, hipStream_t st);

}  // namespace pass
}  // namespace sv
