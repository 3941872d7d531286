// Stand-in for the HIP runtime header: enough of the device language to compile
// the pass kernels as ordinary C++ and run them on the host one lane after
// another (lane_races.cpp).  Buffer loads return zero and stores do nothing;
// shared memory is static storage, so that a compiler's memory-access
// instrumentation sees it; a workgroup barrier ends the lane's epoch.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <type_traits>

#define __host__
#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
// (the kernels' only asm statements are empty ones on a vector register)
#define asm
#define volatile(...)

struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
struct int2 { int x, y; };
struct uint3_host { unsigned x, y, z; };
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
inline uint3_host threadIdx{}, blockIdx{}, gridDim{}, blockDim{};
inline int lane_epoch = 0;  // barriers this lane has passed

__attribute__((no_sanitize("thread"), noinline)) inline void __syncthreads() { ++lane_epoch; }
inline int __syncthreads_or(int v) { __syncthreads(); return v; }
inline int __any(int v) { return v; }
template <class T> T __shfl_xor(T v, int, int) { return v; }
inline int __float_as_int(float f) { return __builtin_bit_cast(int, f); }
inline float __int_as_float(int i) { return __builtin_bit_cast(float, i); }
using std::max;
using std::min;

struct __amdgpu_buffer_rsrc_t {};
typedef int host_v2i __attribute__((ext_vector_type(2)));
inline __amdgpu_buffer_rsrc_t __builtin_amdgcn_make_buffer_rsrc(void*, short, int, int) { return {}; }
inline host_v2i __builtin_amdgcn_raw_buffer_load_b64(__amdgpu_buffer_rsrc_t, int, int, int) { return 0; }
inline int __builtin_amdgcn_raw_buffer_load_b32(__amdgpu_buffer_rsrc_t, int, int, int) { return 0; }
inline void __builtin_amdgcn_raw_buffer_store_b64(host_v2i, __amdgpu_buffer_rsrc_t, int, int, int) {}
inline void __builtin_amdgcn_raw_buffer_store_b32(int, __amdgpu_buffer_rsrc_t, int, int, int) {}
inline int __builtin_amdgcn_mov_dpp(int v, int, int, int, bool) { return v; }
inline int __builtin_amdgcn_ds_swizzle(int v, int) { return v; }
inline void __builtin_amdgcn_fence(int, const char*) {}
inline void __builtin_amdgcn_wave_barrier() {}
inline void __builtin_amdgcn_sched_barrier(int) {}

using hipError_t = int;
using hipStream_t = void*;
enum { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum { hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor };
struct hipFuncAttributes { size_t sharedSizeBytes; };
inline int hipGetLastError() { return 0; }
inline int hipGetDevice(int*) { return 1; }
inline int hipDeviceGetAttribute(int*, int, int) { return 1; }
inline int hipOccupancyMaxActiveBlocksPerMultiprocessor(int*, const void*, int, size_t) { return 1; }
inline int hipFuncGetAttributes(hipFuncAttributes*, const void*) { return 1; }
#define hipLaunchKernelGGL(...) ((void)0)
