// Host stand-in for <hip/hip_runtime.h>, used only by the CPU tests that
// compile headers holding kernels (shared_currents.h, shared_adjoint.h) for
// the host: clang's HIP mode reads the kernels and their launches, none of
// which is instantiated, and the device functions become plain inline
// functions.  The hardware estimates of 1/x and 1/sqrt(x) get the relative
// error ESTIMATE_ERROR (the Newton steps take it out), so that what the steps
// leave is seen.
#pragma once
#define __host__ __attribute__((host))
#define __device__ __attribute__((device))
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <functional>
#include <random>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#define __global__ __attribute__((global))
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#ifndef ESTIMATE_ERROR
#define ESTIMATE_ERROR 1e-8
#endif
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_rcp(x) ((1.0 + ESTIMATE_ERROR) / (x))
#define __builtin_amdgcn_rsq(x) ((1.0 + ESTIMATE_ERROR) / std::sqrt(x))
#define __builtin_amdgcn_mov_dpp(x, c, r, b, z) (x)
struct HostPair {
  unsigned v[2];
  __device__ unsigned operator[](int k) const { return v[k]; }
};
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) (HostPair{{(a), (b)}})
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) (HostPair{{(a), (b)}})
__device__ inline void __syncthreads() {}
__device__ inline int __all(int x) { return x; }
struct HostIndex {
  unsigned x;
};
static HostIndex threadIdx, blockIdx, gridDim;
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
typedef struct ihipStream_t* hipStream_t;
typedef int hipError_t;
extern "C" unsigned __hipPushCallConfiguration(dim3, dim3, size_t = 0, hipStream_t = nullptr);
extern "C" hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t);
// the empty asm statements that hide values from the optimiser name registers
// of the device
#define volatile
#define asm(...) ((void)0)
