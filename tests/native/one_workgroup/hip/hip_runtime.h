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
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidDevice, hipDeviceAttributeMultiprocessorCount, hipFuncAttributeMaxDynamicSharedMemorySize };
static inline hipError_t hipGetLastError() { return hipSuccess; }
template <typename... A> static inline hipError_t hipGetDevice(A...) { return hipErrorInvalidDevice; }
template <typename... A> static inline hipError_t hipDeviceGetAttribute(A...) { return hipErrorInvalidDevice; }
template <typename... A> static inline hipError_t hipFuncSetAttribute(A...) { return hipErrorInvalidDevice; }
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
#define __builtin_amdgcn_readfirstlane unreached
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_sched_group_barrier(...) ((void)0)
struct Anything { template <typename T> operator T() const { __builtin_trap(); } };
template <typename... A> static inline Anything anything(A...) { __builtin_trap(); }
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16 anything
#define __builtin_amdgcn_mfma_f32_16x16x4f32 anything
#define __builtin_amdgcn_cvt_pk_fp8_f32 unreached

// Buffer descriptors (base, stride 0, bytes, flags) and a 16-byte load through one, which returns the address that it would
// read, twice: zeros where lane and wavefront offset together are past the descriptor's end.
typedef unsigned int BufferVec __attribute__((ext_vector_type(4)));
struct Buffer { const char* base; uint64_t bytes; };
#define __amdgpu_buffer_rsrc_t Buffer
static inline Buffer __builtin_amdgcn_make_buffer_rsrc(const char* base, short, int bytes, int) { return Buffer{base, (uint32_t)bytes}; }
static inline BufferVec __builtin_amdgcn_raw_buffer_load_b128(Buffer b, int voff, int soff, int) {
    const uint64_t off = (uint64_t)(uint32_t)voff + (uint32_t)soff, at = off + 16 <= b.bytes ? (uint64_t)(b.base + off) : 0;
    return BufferVec{(uint32_t)at, (uint32_t)(at >> 32), (uint32_t)at, (uint32_t)(at >> 32)};
}
