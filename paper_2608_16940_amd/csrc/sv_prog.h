// Launch of a gate program (device side of sv_prog_host.h).
#pragma once

#include <hip/hip_runtime.h>

#include "sv_prog_host.h"

namespace sv {
namespace prog {

hipError_t launch(const Args &a, float2 *psi, hipStream_t st);

}  // namespace prog
}  // namespace sv
