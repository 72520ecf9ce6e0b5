// Launchers of the block form of the FP32 linear V-cycle (internal).
#pragma once

#include <hip/hip_runtime.h>

namespace mr {

struct LinDownArgs;
struct LinUpArgs;
struct LinTail2Args;
hipError_t launch_lin_down(const LinDownArgs& a, hipStream_t s);
hipError_t launch_lin_up(const LinUpArgs& a, hipStream_t s);
hipError_t launch_lin_tail2(const LinTail2Args& a, hipStream_t s);

}  // namespace mr
