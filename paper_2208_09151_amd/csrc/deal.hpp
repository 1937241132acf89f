// Results in node order to the positions of their accesses, for many accesses.  Included by changeset.hip only.
//
// A word stored to a random place costs a transaction of its own on the way to memory, at 66 G/s as long
// as the memory-side cache collects them, at 25 G/s beyond, so k_stay_ends takes a launch per 2^25 positions, each of
// which reads all pairs.  Here they are read once:
//   k_stay_deal   a block per tile of DEAL_TILE node-sorted accesses sorts its results by window of
//                 2^WINDOW_SHIFT positions in LDS and writes them back to back, with the start of every window inside
//                 the tile
//   k_collect     many blocks of one XCD per window read the window's share of every tile and store the
//                 words at their places, in a stretch of 2 MB at a time
// 164 M accesses: 0.96 + 2.06 ms against 4.36, so 200 x 820 000 goes from 20 310 to 18 970 us a call.  The stores
// still reach memory one by one (36 bytes written for a word of 8), which is what bounds k_collect.
// (Windows of 2^14 positions put together in LDS by a workgroup each: 0.25 + 0.28 ms for 33 M, and shares of one or two
// words for 164 M.)
#pragma once

constexpr int DEAL_THREADS = 1024;
constexpr int DEAL_ITEMS = 16;
constexpr int DEAL_TILE = DEAL_THREADS * DEAL_ITEMS;   // 128 KB of words in LDS
constexpr int WINDOW_SHIFT = 18;                       // 2 MB of 8-byte words, half of an L2
constexpr int DEAL_WINDOWS = 2048;                     // at most: LDS counters of a tile, and 20 bits beside 32 + 12
constexpr int64_t DEAL_TOTAL_MAX = (int64_t)DEAL_WINDOWS << WINDOW_SHIFT;
constexpr int COLLECT_ENTRIES = 2048;                  // of a window, to a block
constexpr int COLLECT_TILES = TB;                      // shares a block lays out at a time
constexpr int COLLECT_ITEMS = 8;

// Accesses from which this pays: 0.37 + 0.81 ms against 1.34 for 67 M on 20 M nodes, 0.62 + 1.21 against 2.3 or more
// for 101 M; for 33 M, one direct launch, 0.25 + 0.39 against 0.49.
constexpr int64_t DEAL_MIN = int64_t(1) << 26;

struct Dealt {
  uint64_t* words;         // [total] a tile's results by window
  uint16_t* start;         // [tiles][windows + 1] start of every window inside the tile
  int64_t total;
  int32_t windows;
};

inline int64_t deal_tiles(int64_t total) { return ceil_div(total, DEAL_TILE); }
inline int64_t deal_windows(int64_t total) { return ceil_div(total, int64_t(1) << WINDOW_SHIFT); }
inline size_t deal_start_bytes(int64_t total) {
  return sizeof(uint16_t) * (size_t)(deal_tiles(total) * (deal_windows(total) + 1));
}

// The block's tile, in three steps that all threads take: clear, a place for every result, results out.
struct DealShared {
  uint64_t words[DEAL_TILE];
  uint32_t count[DEAL_WINDOWS];
  uint32_t scan[DEAL_THREADS / WAVE + 1];
};
constexpr uint32_t NOT_DEALT = 0xFFFFFFFFu;

__device__ __forceinline__ void deal_clear(const Dealt& d, DealShared& sh) {
  for (int w = threadIdx.x; w < d.windows; w += DEAL_THREADS) sh.count[w] = 0;
  __syncthreads();
}

// Window and place among the tile's results for it, of a result for position p.
__device__ __forceinline__ uint32_t deal_place(DealShared& sh, uint32_t p) {
  const uint32_t w = p >> WINDOW_SHIFT;
  return w << 16 | atomicAdd(&sh.count[w], 1u);    // (at most 2^11 windows and 2^14 results)
}

__device__ __forceinline__ void deal_out(const Dealt& d, DealShared& sh, const uint64_t (&word)[DEAL_ITEMS],
                                         const uint32_t (&at)[DEAL_ITEMS]) {
  __syncthreads();
  constexpr int PER = DEAL_WINDOWS / DEAL_THREADS;
  uint32_t c[PER], mine = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int w = threadIdx.x * PER + q;
    c[q] = w < d.windows ? sh.count[w] : 0u;
    mine += c[q];
  }
  uint32_t total;
  uint32_t run = block_exclusive_scan<uint32_t, DEAL_THREADS>(mine, sh.scan, total);
  uint16_t* const start = d.start + (int64_t)blockIdx.x * (d.windows + 1);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int w = threadIdx.x * PER + q;
    if (w < d.windows) {
      sh.count[w] = run;
      start[w] = (uint16_t)run;
      run += c[q];
    }
  }
  if (threadIdx.x == 0) start[d.windows] = (uint16_t)total;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < DEAL_ITEMS; ++k)
    if (at[k] != NOT_DEALT) sh.words[sh.count[at[k] >> 16] + (at[k] & 0xFFFFu)] = word[k];
  __syncthreads();
  uint64_t* const out = d.words + (int64_t)blockIdx.x * DEAL_TILE;
  for (uint32_t x = threadIdx.x; x < total; x += DEAL_THREADS) out[x] = sh.words[x];
}

// put(window's first position, word) for every word of the window.  A block per COLLECT_ENTRIES positions of a
// window, all blocks of a window on one XCD (blocks go to the eight XCDs in turn).
template <typename Put>
__global__ __launch_bounds__(TB) void k_collect(Dealt d, int64_t tiles, int32_t parts, Put put) {
  extern __shared__ int32_t lds_off[];
  __shared__ uint16_t s_coarse[IterFinder::COARSE + 1];
  __shared__ uint32_t s_end[COLLECT_TILES];
  __shared__ int32_t s_shift[COLLECT_TILES];
  __shared__ uint32_t smem[TB / WAVE + 1];
  const int32_t m = blockIdx.x / 8, part = m % parts, window = m / parts * 8 + blockIdx.x % 8;
  if (window >= d.windows) return;
  const IterFinder iteration = iter_finder(lds_off, s_coarse, put.off, put.S);
  const int64_t per = (tiles + parts - 1) / parts;
  const int64_t first = part * per, last = first + per < tiles ? first + per : tiles;
  for (int64_t t0 = first; t0 < last; t0 += COLLECT_TILES) {
    const int64_t t = t0 + threadIdx.x;
    uint32_t lo = 0, hi = 0;
    if (t < last) {
      lo = d.start[t * (d.windows + 1) + window];
      hi = d.start[t * (d.windows + 1) + window + 1];
    }
    uint32_t total;
    const uint32_t before = block_exclusive_scan<uint32_t, TB>(hi - lo, smem, total);
    s_end[threadIdx.x] = before + hi - lo;
    s_shift[threadIdx.x] = (int32_t)threadIdx.x * DEAL_TILE + (int32_t)lo - (int32_t)before;
    __syncthreads();
    const uint64_t* const words = d.words + t0 * DEAL_TILE;
    const int tiles_here = last - t0 < COLLECT_TILES ? (int)(last - t0) : COLLECT_TILES;
    for (uint32_t x0 = threadIdx.x; x0 < total; x0 += TB * COLLECT_ITEMS) {
      uint64_t word[COLLECT_ITEMS];
#pragma unroll
      for (int k = 0; k < COLLECT_ITEMS; ++k) {
        const uint32_t x = x0 + k * TB < total ? x0 + k * TB : x0;
        int a = 0, z = tiles_here - 1;             // the first tile whose shares end behind x
        while (a < z) {
          const int mid = (a + z) >> 1;
          if (s_end[mid] > x) z = mid; else a = mid + 1;
        }
        word[k] = words[s_shift[a] + (int32_t)x];
      }
#pragma unroll
      for (int k = 0; k < COLLECT_ITEMS; ++k)
        if (x0 + k * TB < total) put((int64_t)window << WINDOW_SHIFT, word[k], iteration);
    }
    __syncthreads();                               // the shares are laid out anew
  }
}

template <typename Put>
inline void collect_async(const Dealt& d, const Put& put, size_t lds, hipStream_t st) {
  const int32_t parts = (1 << WINDOW_SHIFT) / COLLECT_ENTRIES;
  hipLaunchKernelGGL(k_collect<Put>, dim3((unsigned)(ceil_div(d.windows, 8) * 8 * parts)), dim3(TB), lds, st, d,
                     deal_tiles(d.total), parts, put);
}
