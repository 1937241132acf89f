// Small results on their way from the device to the host: through pinned memory that a kernel writes, instead of a copy
// to pageable memory.  A call waits for some words two to four times (how many rows there are, the cuts, the offsets of
// its lists), and such a copy with the wait behind it takes 23 us, a kernel's stores and the wait 13 (1 word or
// 400; the wait alone is 11).  Sampling 151 -> 124 us (16 384 nodes), 233 -> 201 (3 M), the smallest changeset call 245 ->
// 215, LRU of 1.4 M accesses 494 -> 436.
#pragma once

#include <cstring>

#include "common.hpp"

namespace ginex {

// Blocks of pinned memory, made when first needed and kept for later calls of any thread: at most HOST_BLOCKS of them,
// one to a call at a time.  Null where there is none, and with GINEX_PINNED=0 (the copy then goes to pageable memory).
// core.cpp
constexpr size_t HOST_BLOCK_BYTES = 64 << 10;
constexpr int HOST_BLOCKS = 16;
void* host_block_take();
void host_block_give(void* block);

struct ReturnParts {
  static constexpr int MOST = 4;
  const uint32_t* from[MOST];
  uint32_t* to[MOST];
  int32_t words[MOST];
  int used;
};

constexpr int RETURN_THREADS = 1024;
static __global__ __launch_bounds__(RETURN_THREADS) void k_return(ReturnParts parts) {
  for (int a = 0; a < parts.used; ++a)
    for (int i = threadIdx.x; i < parts.words[a]; i += RETURN_THREADS) parts.to[a][i] = parts.from[a][i];
}

// get() names words to bring over, wait() brings them as they are then and waits for the stream.
class Returns {
 public:
  explicit Returns(bool pinned = true) : block_(pinned ? host_block_take() : nullptr) {}
  ~Returns() {
    if (block_ && !lost_) host_block_give(block_);
  }
  Returns(const Returns&) = delete;
  Returns& operator=(const Returns&) = delete;

  template <typename T>
  void get(T* to, const void* from, size_t count = 1) {
    static_assert(sizeof(T) % sizeof(uint32_t) == 0, "whole words");
    if (count == 0) return;
    to_[used_] = to;
    from_[used_] = from;
    bytes_[used_++] = sizeof(T) * count;
  }

  hipError_t wait(hipStream_t st) {
    size_t all = 0;
    for (int a = 0; a < used_; ++a) all += bytes_[a];
    const bool pinned = block_ && all <= HOST_BLOCK_BYTES;
    if (pinned && used_ > 0) {
      ReturnParts parts{};
      parts.used = used_;
      char* at = static_cast<char*>(block_);
      for (int a = 0; a < used_; ++a) {
        parts.from[a] = static_cast<const uint32_t*>(from_[a]);
        parts.to[a] = reinterpret_cast<uint32_t*>(at);
        parts.words[a] = (int32_t)(bytes_[a] / sizeof(uint32_t));
        at += bytes_[a];
      }
      hipLaunchKernelGGL(k_return, dim3(1), dim3(RETURN_THREADS), 0, st, parts);
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    } else {
      for (int a = 0; a < used_; ++a)
        if (hipError_t e = hipMemcpyAsync(to_[a], from_[a], bytes_[a], hipMemcpyDeviceToHost, st); e != hipSuccess)
          return e;
    }
    lost_ = pinned && used_ > 0;                   // (a kernel that was not waited for may still write)
    const hipError_t e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    lost_ = false;
    if (pinned) {
      const char* at = static_cast<const char*>(block_);
      for (int a = 0; a < used_; ++a) {
        memcpy(to_[a], at, bytes_[a]);
        at += bytes_[a];
      }
    }
    used_ = 0;
    return hipSuccess;
  }

 private:
  void* const block_;
  bool lost_ = false;
  int used_ = 0;
  void* to_[ReturnParts::MOST];
  const void* from_[ReturnParts::MOST];
  size_t bytes_[ReturnParts::MOST];
};

}  // namespace ginex
