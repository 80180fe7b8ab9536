// Stand-in for the HIP runtime header that lets a kernel source of the library be compiled for the
// CPU: a workgroup's threads are fibers, run one after another from barrier to barrier in an order
// that the caller picks.  Only what ka_square.hip and ka_cube.hip (and the headers they include) need.
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>
#include <functional>
#include <type_traits>

using std::max;
using std::min;

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct int4 { int x, y, z, w; };
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize };
typedef void *hipStream_t;
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }

namespace cpu {
extern dim3 thread, block, block_dim, grid_dim;
extern char dynamic_lds[160 << 10];
void barrier();
void launch(dim3 grid, dim3 block, const std::function<void()> &kernel);
}  // namespace cpu

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __align__(n) alignas(n)
#define __launch_bounds__(...)
#define threadIdx cpu::thread
#define blockIdx cpu::block
#define blockDim cpu::block_dim
#define gridDim cpu::grid_dim
#define __syncthreads() cpu::barrier()
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) cpu::launch(grid, block, [&] { kernel(__VA_ARGS__); })

#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x)
#define __builtin_amdgcn_bitop3_b32(a, b, c, table) cpu::bitop3(a, b, c, table)
namespace cpu {
inline uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c, uint32_t table)
{
  uint32_t r = 0;
  for (uint32_t k = 0; k < 8; ++k)
    if (table >> k & 1) r |= (k & 4 ? a : ~a) & (k & 2 ? b : ~b) & (k & 1 ? c : ~c);
  return r;
}
}  // namespace cpu
inline uint64_t __umul64hi(uint64_t a, uint64_t b) { return (uint64_t)(((unsigned __int128)a * b) >> 64); }

// Named by device functions that these kernels do not call.
#define __builtin_amdgcn_mov_dpp(...) (abort(), 0)
#define __builtin_amdgcn_ds_swizzle(...) (abort(), 0)
#define __builtin_amdgcn_alignbit(...) (abort(), 0u)
#define __builtin_amdgcn_permlane32_swap(...) cpu::no_swap()
#define __hip_atomic_fetch_or(...) abort()
namespace cpu {
struct Pair {
  uint32_t operator[](int) const { abort(); }
};
inline Pair no_swap() { abort(); }
}  // namespace cpu
inline int __lane_id() { abort(); }
template <typename T>
T __shfl_xor(T, int) { abort(); }
inline int __popc(uint32_t x) { return __builtin_popcount(x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
