// Device-wide building blocks written for wave64: exclusive scan and a stable LSD radix
// sort of 64-bit words on a chosen bit range.  Internal header; every function enqueues
// on the given stream and never synchronises or allocates.
#pragma once

#include "common.hpp"

namespace ginex {

// ---------------------------------------------------------------------------------
// Exclusive scan of uint32 counters (two kernels, or three, recursive on the tile sums).
// ---------------------------------------------------------------------------------
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

// What else is done with the results, SCAN_ITEMS of them from `base` on at a time (a launch for a few words of them
// costs 4 us, and some 30 where it is the seventh before a wait).
struct ScanOnly {
  template <typename T>
  __device__ __forceinline__ void operator()(int64_t, const T (&)[SCAN_ITEMS], int64_t) const {}
};

template <typename T, typename Done>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_tiles(T* __restrict__ data, int64_t n,
                                                             T* __restrict__ tile_sums, Done done) {
  __shared__ T smem[SCAN_THREADS / WAVE + 1];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  T v[SCAN_ITEMS];
  T sum = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    v[i] = (base + i < n) ? data[base + i] : T(0);
    sum += v[i];
  }
  T total;
  T run = block_exclusive_scan<T, SCAN_THREADS>(sum, smem, total);
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const T next = run + v[i];
    v[i] = run;
    if (base + i < n) data[base + i] = run;
    run = next;
  }
  done(base, v, n);
  if (threadIdx.x == 0 && tile_sums) tile_sums[blockIdx.x] = total;
}

// SCANNED: the tiles' sums are bases already; else a block adds up those in front of its own, up to SCAN_SUMS of
// them, so that the scan of the sums is no launch of its own (a launch of one block in a chain: 5 us and
// the wait for the one before; by one block altogether 45 056 counters took 42 us, three launches 14).
constexpr int64_t SCAN_SUMS = 1024;

template <typename T, bool SCANNED, typename Done>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_add(T* __restrict__ data, int64_t n,
                                                           const T* __restrict__ tile_bases, Done done) {
  T add = 0;
  if (SCANNED) {
    add = tile_bases[blockIdx.x];
  } else {
    __shared__ T smem[SCAN_THREADS / WAVE + 1];
    for (int q = threadIdx.x; q < (int)blockIdx.x; q += SCAN_THREADS) add += tile_bases[q];
    T total;
    block_exclusive_scan<T, SCAN_THREADS>(add, smem, total);
    add = total;
  }
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  T v[SCAN_ITEMS];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    v[i] = add;
    if (base + i < n) data[base + i] = v[i] += data[base + i];
  }
  done(base, v, n);
}

// Scratch elements needed by exclusive_scan_inplace for n elements.
inline int64_t scan_scratch_elems(int64_t n) {
  int64_t total = 0;
  while (n > SCAN_TILE) {
    n = ceil_div(n, SCAN_TILE);
    total += n;
  }
  return total + 1;
}

// data[i] <- sum of data[0..i).  `scratch` holds scan_scratch_elems(n) elements.
template <typename T, typename Done = ScanOnly>
inline hipError_t exclusive_scan_inplace(T* data, int64_t n, T* scratch, hipStream_t st, Done done = Done{}) {
  if (n <= 0) return hipSuccess;
  const int64_t tiles = ceil_div(n, SCAN_TILE);
  if (tiles == 1) {
    hipLaunchKernelGGL((k_scan_tiles<T, Done>), dim3(1), dim3(SCAN_THREADS), 0, st, data, n, (T*)nullptr, done);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_scan_tiles<T, ScanOnly>), dim3((unsigned)tiles), dim3(SCAN_THREADS), 0, st, data, n,
                     scratch, ScanOnly{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (tiles <= SCAN_SUMS) {
    hipLaunchKernelGGL((k_scan_add<T, false, Done>), dim3((unsigned)tiles), dim3(SCAN_THREADS), 0, st, data, n,
                       scratch, done);
    return hipGetLastError();
  }
  e = exclusive_scan_inplace<T>(scratch, tiles, scratch + tiles, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_scan_add<T, true, Done>), dim3((unsigned)tiles), dim3(SCAN_THREADS), 0, st, data, n,
                     scratch, done);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Occurrence histogram: count[v] += number of times v occurs in values[0..n).  With the CSR
// rows holding in-neighbours this is the out-degree of every node.  Entries outside
// [0, bins) are counted in *bad and skipped.  `values` may live in host-pinned memory.
// ---------------------------------------------------------------------------------
static __global__ __launch_bounds__(256) void k_occurrences(const int32_t* __restrict__ values,
                                                            int64_t n, int64_t bins,
                                                            uint32_t* __restrict__ count,
                                                            unsigned long long* __restrict__ bad) {
  const int64_t span = (int64_t)gridDim.x * 256;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += span) {
    const int32_t v = values[e];
    if ((uint32_t)v < (uint64_t)bins) atomicAdd(&count[v], 1u);
    else atomicAdd(bad, 1ull);
  }
}

inline hipError_t occurrences_async(const int32_t* values, int64_t n, int64_t bins, uint32_t* count,
                                    unsigned long long* bad, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = ceil_div(n, (int64_t)256 * 16);
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_occurrences, dim3((unsigned)blocks), dim3(256), 0, st, values, n, bins, count,
                     bad);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Stable LSD radix sort of uint64 words on bits [bit_lo, bit_hi), at most 8 bits per pass and the same
// number in every pass (9 bits: see RS_WIDE_BITS), or one less in the last ones: 27 bits as 7 + 7 + 7 + 6 instead of 8 +
// 8 + 8 + 3 halve the counters that are scanned and double the runs that are written (33 M pairs: 1.22 -> 1.02 ms).
// Each pass: (1) per-tile digit histogram, (2) exclusive scan of the digit-major
// histogram, (3) scatter.  In the scatter a wave owns a contiguous run of its tile and
// ranks its 64 keys per step with ballot-built peer masks, so equal digits keep their
// input order; keys are then staged in LDS in digit order and written out in runs.
// ---------------------------------------------------------------------------------
constexpr int RS_THREADS = 256;
constexpr int RS_ITEMS = 16;                    // keys per thread
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;  // 4096 keys, 32 KB of LDS staging
constexpr int RS_BITS = 8;
constexpr int RS_BINS = 1 << RS_BITS;           // at most
// Wide tiles, four times the keys (128 KB of LDS staging), have room for a bit more with runs of the same length, which
// is a pass less for 17, 18 and 25 to 27 bits; one block to a CU hides less, though.  Histogram, scan and scatter of all passes
// over 27 bits, narrow and wide: 33 M words 710 us and 709, 67 M 1 413 and 1 354, 100 M 2 143 and 1 987; 154 M, 26
// bits, 3 700 and 2 940.  And whatever the digit where there are so many words that the runs of narrow tiles are written more
// slowly (a scatter by 7 bits: 33 M 97 and 131 us, 100 M 311 and 367, 154 M 690 and 559).
constexpr int RS_WIDE_THREADS = 1024;
constexpr int RS_WIDE_BITS = 9;
constexpr int64_t RS_WIDE_MIN = int64_t(1) << 26, RS_WIDE_ALWAYS = int64_t(1) << 27;

// Where a pass reads its words: an array of words, or (the first pass of a sort of
// (value, position) pairs) an array of 32-bit values, word j = value j << 32 | j, so that the
// pairs need not be written out and read back first.
struct RadixWords {
  const uint64_t* in;
  __device__ __forceinline__ uint64_t operator()(int64_t j) const { return in[j]; }
};
struct RadixValuesWithPositions {
  const int32_t* values;
  __device__ __forceinline__ uint64_t operator()(int64_t j) const {
    return ((uint64_t)(uint32_t)values[j] << 32) | (uint64_t)j;
  }
};

template <typename Source, int BITS, int THREADS>
static __global__ __launch_bounds__(THREADS) void k_radix_hist(Source in, int64_t n, int shift,
                                                               int64_t tiles,
                                                               uint32_t* __restrict__ hist) {
  constexpr int BINS = 1 << BITS;
  __shared__ uint32_t bins[BINS];
  if (threadIdx.x < BINS) bins[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (THREADS * RS_ITEMS);
  uint32_t digit[RS_ITEMS];
#pragma unroll
  for (int i = 0; i < RS_ITEMS; ++i) {
    const int64_t j = base + i * THREADS + threadIdx.x;
    digit[i] = (uint32_t)(in(j < n ? j : n - 1) >> shift) & (BINS - 1);
  }
#pragma unroll
  for (int i = 0; i < RS_ITEMS; ++i)
    if (base + i * THREADS + threadIdx.x < n) atomicAdd(&bins[digit[i]], 1u);
  __syncthreads();
  if (threadIdx.x < BINS) hist[(int64_t)threadIdx.x * tiles + blockIdx.x] = bins[threadIdx.x];
}

template <typename Source, int BITS, int THREADS>
static __global__ __launch_bounds__(THREADS) void k_radix_scatter(
    Source in, uint64_t* __restrict__ out, int64_t n, int shift, int64_t tiles,
    const uint32_t* __restrict__ hist_scanned) {
  constexpr int BINS = 1 << BITS, WAVES = THREADS / WAVE, TILE = THREADS * RS_ITEMS;
  static_assert(BINS <= THREADS, "a thread per digit");
  typedef typename std::conditional<(WAVES > 4), uint16_t, uint32_t>::type Count;   // (LDS is short for many waves)
  static_assert(WAVES <= 4 || TILE - WAVE * RS_ITEMS <= 0xFFFF, "keys of a digit in the waves in front");
  __shared__ uint64_t staged[TILE];
  __shared__ Count wave_count[WAVES][BINS];
  __shared__ uint32_t digit_start[BINS];   // start of each digit inside the tile
  __shared__ uint32_t digit_dst[BINS];     // global destination of the digit's run, less its start (modulo 2^32)
  __shared__ uint32_t scan_smem[THREADS / WAVE + 1];

  const int w = threadIdx.x / WAVE;
  const int lane = lane_id();
  for (int i = threadIdx.x; i < WAVES * BINS; i += THREADS) (&wave_count[0][0])[i] = 0;
  __syncthreads();

  const int64_t tile_base = (int64_t)blockIdx.x * TILE;
  const int64_t wave_base = tile_base + (int64_t)w * (WAVE * RS_ITEMS);
  uint64_t key[RS_ITEMS];
  uint32_t rank[RS_ITEMS];  // rank among the wave's keys with the same digit
  // all reads first (the barrier below holds the compiler back from moving one in front of it), and
  // without a branch around each, behind which its value would be waited for: beyond the end the last
  // word again.  33 M words: 183 -> 125 us per pass
#pragma unroll
  for (int i = 0; i < RS_ITEMS; ++i) {
    const int64_t j = wave_base + i * WAVE + lane;
    key[i] = in(j < n ? j : n - 1);
  }
#pragma unroll
  for (int i = 0; i < RS_ITEMS; ++i) {
    const bool valid = wave_base + i * WAVE + lane < n;
    const uint32_t d = (uint32_t)(key[i] >> shift) & (BINS - 1);
    // lanes with the same digit: of every bit's ballot m, or of ~m, as the own bit (all ones or none in x) says.  Five
    // instructions a bit (with a select between m and ~m, which the compiler makes eight of, 7 bits of 33 M words took 121 us
    // instead of 97: the kernel is as near its arithmetic as its memory)
    const uint64_t all = __ballot(valid);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);
      const uint64_t m = __ballot(x != 0);
      lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, x, 0x90);           // lo & ~(m ^ x)
      hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), x, 0x90);
    }
    const uint64_t peers = (uint64_t)hi << 32 | lo;
    const uint32_t before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    const int leader = __ffsll((unsigned long long)peers) - 1;
    uint32_t prev = 0;
    if (valid && lane == leader) {
      prev = wave_count[w][d];
      wave_count[w][d] = (Count)(prev + __popcll(peers));
    }
    __builtin_amdgcn_wave_barrier();  // keep the LDS update ahead of the next step's read
    prev = __shfl(prev, leader < 0 ? 0 : leader, WAVE);
    rank[i] = prev + before;
  }
  __syncthreads();

  // thread t owns digit t: turn per-wave counts into per-wave starts, get tile totals
  {
    const int d = threadIdx.x;
    uint32_t run = 0;
    if (d < BINS)
#pragma unroll
      for (int ww = 0; ww < WAVES; ++ww) {
        const uint32_t c = wave_count[ww][d];
        wave_count[ww][d] = (Count)run;
        run += c;
      }
    uint32_t total;
    const uint32_t start = block_exclusive_scan<uint32_t, THREADS>(run, scan_smem, total);
    if (d < BINS) {
      digit_start[d] = start;
      digit_dst[d] = hist_scanned[(int64_t)d * tiles + blockIdx.x] - start;
    }
  }
  __syncthreads();

#pragma unroll
  for (int i = 0; i < RS_ITEMS; ++i) {
    const int64_t j = wave_base + i * WAVE + lane;
    if (j < n) {
      const uint32_t d = (uint32_t)(key[i] >> shift) & (BINS - 1);
      staged[digit_start[d] + wave_count[w][d] + rank[i]] = key[i];
    }
  }
  __syncthreads();

  const int64_t remaining = n - tile_base;
  const int count = remaining < TILE ? (int)remaining : TILE;
  for (int i = threadIdx.x; i < count; i += THREADS) {
    const uint64_t k = staged[i];
    const uint32_t d = (uint32_t)(k >> shift) & (BINS - 1);
    out[digit_dst[d] + (uint32_t)i] = k;
  }
}

struct RadixPlan {
  int64_t tiles;
  int64_t hist_elems;   // uint32 counters (+ scan scratch) the sort needs
};

inline RadixPlan radix_plan(int64_t n) {
  RadixPlan p;
  p.tiles = n > 0 ? ceil_div(n, RS_TILE) : 1;
  const int64_t h = p.tiles * RS_BINS;
  p.hist_elems = h + scan_scratch_elems(h);
  return p;
}

template <int BITS, int THREADS, typename Source>
inline hipError_t radix_pass_bits(Source in, uint64_t* out, int64_t n, int shift, uint32_t* hist, hipStream_t st) {
  const int64_t tiles = ceil_div(n, THREADS * RS_ITEMS), h = tiles << BITS;
  hipLaunchKernelGGL((k_radix_hist<Source, BITS, THREADS>), dim3((unsigned)tiles), dim3(THREADS), 0, st, in, n,
                     shift, tiles, hist);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = exclusive_scan_inplace<uint32_t>(hist, h, hist + h, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_radix_scatter<Source, BITS, THREADS>), dim3((unsigned)tiles), dim3(THREADS), 0, st, in,
                     out, n, shift, tiles, hist);
  return hipGetLastError();
}

// A pass over `bits` bits (the digit may be wider than that: the bits above are zero or not sorted by): its digit and
// whether its tiles are wide.
struct RadixDigit {
  int bits;
  bool wide;
};
inline RadixDigit radix_digit(int64_t n, int bits) {
  if (bits > RS_BITS) return {RS_WIDE_BITS, true};
  if (n >= RS_WIDE_ALWAYS) return {bits == 8 ? 8 : 7, true};
  return {bits < 5 ? 5 : bits, false};
}

// Afterwards hist[d * tiles] is where the words of digit d start.
inline int64_t radix_tiles(int64_t n, int bits) {
  return ceil_div(n, (radix_digit(n, bits).wide ? RS_WIDE_THREADS : RS_THREADS) * RS_ITEMS);
}

template <typename Source>
inline hipError_t radix_pass(Source in, uint64_t* out, int64_t n, int shift, int bits, uint32_t* hist, hipStream_t st) {
  const RadixDigit d = radix_digit(n, bits);
  if (d.wide) {
    if (d.bits == RS_WIDE_BITS) return radix_pass_bits<RS_WIDE_BITS, RS_WIDE_THREADS>(in, out, n, shift, hist, st);
    if (d.bits == 8) return radix_pass_bits<8, RS_WIDE_THREADS>(in, out, n, shift, hist, st);
    return radix_pass_bits<7, RS_WIDE_THREADS>(in, out, n, shift, hist, st);
  }
  if (d.bits == 8) return radix_pass_bits<8, RS_THREADS>(in, out, n, shift, hist, st);
  if (d.bits == 7) return radix_pass_bits<7, RS_THREADS>(in, out, n, shift, hist, st);
  if (d.bits == 6) return radix_pass_bits<6, RS_THREADS>(in, out, n, shift, hist, st);
  return radix_pass_bits<5, RS_THREADS>(in, out, n, shift, hist, st);
}

// Bits of pass `k` of the passes that cover `bits`: as even as possible, the wider ones first.
inline int radix_passes(int bits, int64_t n) {
  const int narrow = (bits + RS_BITS - 1) / RS_BITS, wide = (bits + RS_WIDE_BITS - 1) / RS_WIDE_BITS;
  return n >= RS_WIDE_MIN && wide < narrow ? wide : narrow;
}
inline int radix_pass_width(int bits, int passes, int k) { return bits / passes + (k < bits % passes ? 1 : 0); }

// Sorts `n` words by bits [bit_lo, bit_hi).  `a` holds the input, `b` is a buffer of the
// same size; returns (through *sorted) which of the two holds the result.  The total
// number of keys must stay below 2^32 (uint32 histogram).
inline hipError_t radix_sort_u64(uint64_t* a, uint64_t* b, int64_t n, int bit_lo, int bit_hi,
                                 uint32_t* hist, hipStream_t st, uint64_t** sorted) {
  *sorted = a;
  if (n <= 1) return hipSuccess;
  const int passes = radix_passes(bit_hi - bit_lo, n);
  for (int k = 0, shift = bit_lo; k < passes; ++k) {
    const int bits = radix_pass_width(bit_hi - bit_lo, passes, k);
    const hipError_t e = radix_pass(RadixWords{a}, b, n, shift, bits, hist, st);
    if (e != hipSuccess) return e;
    uint64_t* t = a; a = b; b = t;
    shift += bits;
  }
  *sorted = a;
  return hipSuccess;
}

// The words (values[j] << 32 | j), j in [0, n), sorted by bits [32, bit_hi) of the word, that
// is by the low bits of the value; equal values keep the order of their positions.  `a` and
// `b` are two buffers of n words; *sorted tells which of them holds the result.
inline hipError_t radix_sort_values_with_positions(const int32_t* values, uint64_t* a, uint64_t* b,
                                                   int64_t n, int bit_hi, uint32_t* hist,
                                                   hipStream_t st, uint64_t** sorted) {
  *sorted = a;
  if (n <= 0) return hipSuccess;
  const int passes = radix_passes(bit_hi - 32, n);
  int shift = 32;
  for (int k = 0; k < passes; ++k) {
    const int bits = radix_pass_width(bit_hi - 32, passes, k);
    hipError_t e;
    if (k == 0) {
      e = radix_pass(RadixValuesWithPositions{values}, a, n, shift, bits, hist, st);
    } else {
      e = radix_pass(RadixWords{a}, b, n, shift, bits, hist, st);
      uint64_t* t = a; a = b; b = t;
    }
    if (e != hipSuccess) return e;
    shift += bits;
  }
  *sorted = a;
  return hipSuccess;
}

}  // namespace ginex
