// Shared host/device helpers of the gfx950 library: error reporting, a bump allocator
// for the caller's workspace, wave64/block scans, fill kernels.  Internal; the public
// interface is include/ginex.h.
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "ginex.h"

namespace ginex {

constexpr int WAVE = 64;

void set_error(const char* fmt, ...);
int32_t fail(int32_t code, const char* fmt, ...);

#define GINEX_HIP(call)                                                              \
  do {                                                                               \
    hipError_t e_ = (call);                                                          \
    if (e_ != hipSuccess)                                                            \
      return ::ginex::fail(GINEX_ERR_HIP, "%s failed: %s (%s:%d)", #call,            \
                           hipGetErrorString(e_), __FILE__, __LINE__);               \
  } while (0)

#define GINEX_LAUNCH_CHECK() GINEX_HIP(hipGetLastError())

// Bump allocator over the caller's workspace.  Run once with base == nullptr to measure
// and once with the real pointer to carve; both runs take the same path, so the size
// query and the call can never disagree.
struct Arena {
  char* base;
  size_t used = 0;
  explicit Arena(void* b) : base(static_cast<char*>(b)) {}
  template <typename T>
  T* take(size_t count) {
    used = (used + 255) & ~size_t(255);
    T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
    used += count * sizeof(T);
    return p;
  }
};

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- device helpers -------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return threadIdx.x & (WAVE - 1); }

// A neighbour's value by DPP, without the LDS round trip of a shuffle: 0 where the control names no lane, or not in
// these rows of 16.
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_or_zero(T v) {
  static_assert(std::is_integral_v<T> && (sizeof(T) == 4 || sizeof(T) == 8), "whole words");
  if constexpr (sizeof(T) == 4) {
    return (T)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
  } else {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)v >> 32), CTRL, ROWS, 0xF, false);
    return (T)((uint64_t)hi << 32 | lo);
  }
}

// Inclusive scan across the 64 lanes of a wave (all of them active): inside the rows of 16, then the last lane of a
// row to the next one, and of the first half to the second.  With a shuffle a step, six trips through LDS that wait for
// each other, the smallest changeset call took 272 us instead of 242 (its one workgroup 103 of them, some 20 barriers and
// scans an iteration), sampling on a graph of 1 M nodes 297 instead of 286.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
  v += dpp_or_zero<0x111, 0xF>(v);   // row_shr:1
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);   // row_bcast:15
  v += dpp_or_zero<0x143, 0xC>(v);   // row_bcast:31
  return v;
}

template <typename T>
__device__ __forceinline__ T wave_reduce_sum(T v) {
  v = wave_inclusive_scan(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, WAVE - 1);
  if constexpr (sizeof(T) == 4) return (T)lo;
  else return (T)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), WAVE - 1) << 32 | lo);
}

// The value of the lane to the left (right); the first (last) lane keeps its own.  All lanes active.
__device__ __forceinline__ uint32_t from_left(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138, 0xF, 0xF, false);   // wave_shr:1
}
__device__ __forceinline__ uint32_t from_right(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130, 0xF, 0xF, false);   // wave_shl:1
}
// The value of one lane, the same for all.
__device__ __forceinline__ uint32_t of_lane(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ uint64_t of_lane(uint64_t v, int lane) {
  return (uint64_t)of_lane((uint32_t)(v >> 32), lane) << 32 | of_lane((uint32_t)v, lane);
}
__device__ __forceinline__ int32_t of_lane(int32_t v, int lane) { return (int32_t)of_lane((uint32_t)v, lane); }

// Exclusive scan over a block of THREADS threads (a multiple of 64, at most 1024).
// `total` receives the block sum in every thread.  `smem` needs THREADS/64 + 1 slots.
template <typename T, int THREADS>
__device__ __forceinline__ T block_exclusive_scan(T v, T* smem, T& total) {
  constexpr int NW = THREADS / WAVE;
  const int w = threadIdx.x / WAVE;
  T inc = wave_inclusive_scan(v);
  if (lane_id() == WAVE - 1) smem[w] = inc;
  __syncthreads();
  if (threadIdx.x < WAVE) {
    T s = threadIdx.x < NW ? smem[threadIdx.x] : T(0);
    T si = wave_inclusive_scan(s);
    if (threadIdx.x < NW) smem[threadIdx.x] = si - s;
    if (threadIdx.x == NW - 1) smem[NW] = si;
  }
  __syncthreads();
  T base = smem[w];
  total = smem[NW];
  __syncthreads();
  return base + inc - v;
}

template <typename T>
__global__ void k_fill(T* p, int64_t n, T value) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = value;
}

template <typename T>
inline hipError_t fill_async(T* p, int64_t n, T value, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = ceil_div(n, 256 * 8);
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, st, p, n, value);
  return hipGetLastError();
}

// A full mix (the finaliser of MurmurHash3).
__device__ __forceinline__ uint32_t hash_mix(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  return h ^ (h >> 16);
}

// Several arrays cleared in one launch: calls on few ids are a chain of launches of a few microseconds
// each (a changeset call clears up to eleven arrays).
struct Zeros {
  static constexpr int MOST = 12;
  uint32_t* at[MOST];
  int64_t words[MOST];
  int used = 0;
  template <typename T>
  Zeros& add(T* p, int64_t n) {
    static_assert(sizeof(T) % sizeof(uint32_t) == 0, "whole words");
    at[used] = reinterpret_cast<uint32_t*>(p);
    words[used++] = n * (int64_t)(sizeof(T) / sizeof(uint32_t));
    return *this;
  }
};

static __global__ void k_zero(Zeros z) {
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int a = 0; a < z.used; ++a)
    for (int64_t i = first; i < z.words[a]; i += stride) z.at[a][i] = 0;
}

inline hipError_t zero_async(const Zeros& z, hipStream_t st) {
  int64_t longest = 0;
  for (int a = 0; a < z.used; ++a) longest = z.words[a] > longest ? z.words[a] : longest;
  if (longest == 0) return hipSuccess;
  const int64_t blocks = ceil_div(longest, 256 * 8);
  hipLaunchKernelGGL(k_zero, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, z);
  return hipGetLastError();
}

}  // namespace ginex
