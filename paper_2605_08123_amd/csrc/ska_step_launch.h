// Launches of the step kernel, one function per storage type and head dimension: its instances are most of the library, so each of
// the six has an object of its own (ska_step_launch.hip), which are compiled side by side.
#pragma once
#include <hip/hip_runtime.h>

// args: StepArgs, shape: StepShape (ska_step.h).  SKA_EUNSUPPORTED: no such instance, or a chain's workgroups do not fit the device
// together; nothing has been launched.  The caller holds the library's lock.
#define SKA_DECLARE_STEPS(NAME) extern "C" __attribute__((visibility("hidden"))) int NAME(const void *args, const void *shape, int N, hipStream_t st, int dev)
SKA_DECLARE_STEPS(ska_launch_steps_f32_32);
SKA_DECLARE_STEPS(ska_launch_steps_f32_64);
SKA_DECLARE_STEPS(ska_launch_steps_f32_128);
SKA_DECLARE_STEPS(ska_launch_steps_bf16_32);
SKA_DECLARE_STEPS(ska_launch_steps_bf16_64);
SKA_DECLARE_STEPS(ska_launch_steps_bf16_128);
