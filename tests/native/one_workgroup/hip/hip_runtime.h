// The HIP names that step_kernels.hip uses, for one workgroup on the CPU: every
// thread is a fiber, a barrier or a lane exchange is where fibers change over
// (sampler.cpp has the scheduler).  Nothing here is part of the library.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
struct int4 { int x, y, z, w; };
struct float2 { float x, y; };
typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1 };
static inline hipError_t hipGetLastError() { return hipSuccess; }
#define hipLaunchKernelGGL(...) ((void)0)

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static

struct FiberIdx { operator unsigned() const; };
struct FiberIdx3 { FiberIdx x; };
extern FiberIdx3 threadIdx;
extern dim3 blockIdx, blockDim, gridDim;
void __syncthreads();
uint32_t exchange(uint32_t v, int lane_xor);
static inline float __shfl_xor(float v, int x) { return __builtin_bit_cast(float, exchange(__builtin_bit_cast(uint32_t, v), x)); }
static inline int __shfl_xor(int v, int x) { return (int)exchange((uint32_t)v, x); }
static inline int atomicAdd(int* p, int v) { const int o = *p; *p += v; return o; }
using std::max;
using std::min;

// named by helpers of common.h that the kernels run here do not reach
template <typename... A> static inline int unreached(A...) { __builtin_trap(); }
struct Unreached2 { unsigned v[2]; unsigned operator[](int i) const { return v[i]; } };
template <typename... A> static inline Unreached2 unreached2(A...) { __builtin_trap(); }
#define __builtin_amdgcn_permlane16_swap unreached2
#define __builtin_amdgcn_permlane32_swap unreached2
#define __builtin_amdgcn_update_dpp unreached
#define __builtin_amdgcn_mov_dpp unreached
