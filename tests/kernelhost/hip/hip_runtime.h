// Host stand-in for the device side of <hip/hip_runtime.h>, enough to compile
// csrc/kernels.h for the CPU and call its address computations thread by
// thread (test infrastructure).  Cross-lane operations are declared only: the
// functions called here use none but readfirstlane, whose argument is the
// same on every lane.
#pragma once
#include <stdint.h>

#define __device__
#define __global__ static  // unused here: not emitted
#define __shared__ static
#define __forceinline__ inline
#define __align__(n) __attribute__((aligned(n)))
#define __launch_bounds__(...)

struct Dim3 {
  uint32_t x, y, z;
};
inline Dim3 threadIdx, blockIdx, blockDim, gridDim;

inline uint64_t __umul64hi(uint64_t a, uint64_t b) { return uint64_t((unsigned __int128)a * b >> 64); }
template <class T>
T __shfl_up(T, int, int);
void __syncthreads();
void __threadfence_system();
uint64_t __ballot(int);
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
int atomicOr(int *, int);
int atomicMax(int *, int);

#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __builtin_amdgcn_s_sleep(n) ((void)(n))
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_mbcnt_lo(m, v) (v)
#define __builtin_amdgcn_mbcnt_hi(m, v) (v)
