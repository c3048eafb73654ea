// Functions that the kernels and checks on the host share (not installed; compiles without HIP).
#pragma once

#ifdef __HIPCC__
#define CDL_ANYWHERE __host__ __device__ __forceinline__
#else
#define CDL_ANYWHERE inline
#endif
