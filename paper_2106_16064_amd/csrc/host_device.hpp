// Functions that host code compiles too, so that they can be tried without a GPU.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define DGSP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define DGSP_HOST_DEVICE inline
#endif
