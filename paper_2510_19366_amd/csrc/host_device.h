// Functions that the compiler of the kernels and one of host programs (tests) both take.
#pragma once
#ifdef __HIPCC__
#define MP_HD __host__ __device__ __forceinline__
#else
#define MP_HD inline
#endif
