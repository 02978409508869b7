// What csrc/kernels.h takes from HIP, for a CPU compiler: enough to run fetch_kv_small lane by lane (small_fetch.cpp).  The rest only
// has to parse.  Nothing here is part of the product library or ever reaches a GPU.
#pragma once
#include <stdint.h>

#define __host__
#define __device__
#define __global__ static
#define __shared__ static
#define __launch_bounds__(...)

struct dim3 { uint32_t x = 1, y = 1, z = 1; };
extern dim3 threadIdx, blockIdx, gridDim;               // of the lane that is running

void __syncthreads();
uint64_t __ballot(bool pred);
uint32_t read_lane(uint32_t x, uint32_t k);
inline uint32_t __lane_id() { return threadIdx.x & 63; }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline uint64_t wall_clock64() { return 0; }
uint32_t __shfl_xor(uint32_t, int);
uint32_t __shfl_up(uint32_t, int);
void __threadfence_system();
template <typename T> T atomicAdd(T *p, T v) { T old = *p; *p += v; return old; }
template <typename T> T atomicOr(T *p, T v) { T old = *p; *p |= v; return old; }
template <typename T> T atomicMax(T *p, T v) { T old = *p; if (v > old) *p = v; return old; }
inline uint32_t atomicAdd(uint32_t *p, int v) { uint32_t old = *p; *p += v; return old; }

#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (void)(*(p) = (v))
#define __hip_atomic_fetch_add(p, v, order, scope) atomicAdd(p, v)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_readlane(x, k) read_lane(x, k)
#define __builtin_amdgcn_s_setprio(n) ((void)0)
extern const char *kernel_arguments;                    // laid out as a launch would have them
#define __builtin_amdgcn_kernarg_segment_ptr() ((const __attribute__((address_space(4))) void *)kernel_arguments)
#define __builtin_amdgcn_global_store_b128(p, v, scope) (void)(*(p) = (v))
