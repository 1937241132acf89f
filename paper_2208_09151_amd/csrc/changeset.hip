// Changeset precomputation on gfx950 (Ginex Section 3.4, lists of Section 3.3).
//
// Part 1, next accessed iteration of every access, fully parallel:
//   (node, flat position) pairs are radix-sorted by node (stable, so each node's accesses
//   stay in iteration order); an access's successor in the sorted array tells its next
//   accessed iteration, the head of each node's run tells the node's first access.
// Part 2, C_0: run heads (first iteration, node) sorted by first iteration; the first
//   `cap` of them fill cache lines 0..cap-1.
// Part 3, the recurrence C_{i+1} = f_Belady(union(C_i, ids_i)).  For up to 2 048 iterations
//   hits, misses, insertions and evictions follow from the trace and the start state at once,
//   and only the lines are handed on iteration by iteration (stays.hpp; a carried cache that
//   holds every row of the superbatch: the part "without a loop" below).  Beyond 2 048
//   iterations, for LRU where an iteration is longer than the cache, and for the smallest carried caches a loop
//   over the state, serial over iterations and parallel inside one (small.hpp: the same in one
//   workgroup, for the smallest fresh caches).  The cache is full from C_0 on (otherwise everything fitted and
//   nothing ever changes), so iteration i must drop exactly as many candidates as it had
//   misses.  Keys are (next iteration, incoming?, node id); next iterations take only
//   S-i distinct values, so a histogram per next iteration (kept incrementally for the
//   residents, rebuilt for the incoming rows) finds the threshold bucket j*; only inside
//   j* does the id order matter, and there the k-th smallest id is found by setting the
//   members' bits in a bitmap over node ids and locating the k-th set bit through per-part
//   counts.  Evicted lines and inserted positions are then compacted in line / position
//   order and paired.
//   Both ways also serve a superbatch that resumes from the cache state of the previous one
//   (C_0 given instead of computed, Belady only); LRU has other keys.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "common.hpp"
#include "primitives.hpp"
#include "returns.hpp"

namespace ginex {
namespace {

constexpr int TB = 256;
constexpr int BIG = 1024;          // threads of the single-block kernels
constexpr int TOUCH_ITEMS = 8;     // accesses per thread in the touch kernel
constexpr int PART_SHIFT = 16;     // a part of a bitmap covers 2^16 node ids ...
constexpr int PART_WORDS = 1 << (PART_SHIFT - 5);   // ... in 2048 words

enum { MODE_NONE = 0, MODE_ALL = 1, MODE_SELECT = 2 };

struct Ctrl {        // decisions of the running iteration (device memory)
  int32_t jstar;     // threshold bucket (S+1: nothing is dropped)
  int32_t mode_in;   // incoming rows of bucket j*: none / all / ids <= T are inserted
  int32_t mode_res;  // resident rows of bucket j*: all / ids <= T are kept
  int32_t keep;      // how many members of the selected class stay
  int32_t T;         // id threshold of the select
  int32_t n_change;  // evictions (= insertions) of the iteration
  int32_t use_dead;  // the select runs on the standing bitmap of dead residents
  int32_t marked;    // bit 0: residents of bucket j* have their bits in the scratch bitmap,
                     // bit 1: incoming rows of bucket j* in theirs (both are cleared in k_flags)
};
enum { MARKED_RES = 1, MARKED_IN = 2 };
// State::fault (device, one word): set when a launch sequence that leaves the live select out
// meets an iteration that needs it (cannot happen when every row of the superbatch fits the
// cache beside the rows it already holds; checked by the host after the loop).

struct State {
  int32_t* res_id;      // [cap] node held by each cache line
  int32_t* res_next;    // [cap] its next accessed iteration (S = never)
  int32_t* addr;        // [N] line of a node or -1
  uint32_t* rhist;      // [S+1] residents per next iteration
  uint32_t* ihist;      // [S+1] incoming rows of the running iteration per next iteration
  uint32_t* bitmap;     // [words] select scratch (residents of bucket j*), all zero between iterations
  uint32_t* sel_part;   // [parts] its set bits per part, all zero between iterations
  uint32_t* bitmap_in;  // [words] the same for the incoming rows of bucket j*
  uint32_t* sel_part_in;
  uint32_t* dead_bits;  // [words] residents that are never accessed again, kept up to date
  uint32_t* dead_part;  // [parts] its set bits per part, kept up to date
  Ctrl* ctrl;
  int32_t* fault;
  uint64_t* evict_words;  // bit l%64 of word l/64: line l is evicted in this iteration
  uint32_t* evict_tiles;  // evictions per tile of EVICT_TILE lines
  uint32_t* in_tiles;     // insertions per tile of positions in ids_i
  int32_t* acc_line;      // [longest iteration] line of each access of the running iteration, -1 = miss
  uint64_t* pair;         // [max_change] meeting point of the t-th eviction and the t-th insertion
  int64_t cap, num_nodes;
  int64_t words, parts;   // of the two bitmaps
  int32_t S;
  int64_t max_change;     // entries of pair
  int32_t lru;            // 0: Belady keys (next accessed iteration), 1: LRU keys
  int32_t dead_scatter;   // evictions among the dead residents are found from the id bitmap
                          // (large caches) instead of by a pass over all cache lines
  int32_t dead_only;      // every eviction falls among the dead residents: no live select
};

// Iteration that holds flat position p: the largest i with off[i] <= p.  `off` is the
// block's LDS copy of ids_offsets (total ids < 2^31, so 32 bits do).
__device__ __forceinline__ int32_t iter_of(const int32_t* off, int32_t S, int32_t p) {
  int32_t lo = 0, hi = S;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (off[mid] <= p) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ void load_offsets(int32_t* lds_off, const int64_t* __restrict__ off,
                                             int32_t S) {
  for (int j = threadIdx.x; j <= S; j += blockDim.x) lds_off[j] = (int32_t)off[j];
  __syncthreads();
}

// The same from the iteration of every 2^shift-th position: the search is over the iterations between two of
// these, one or two steps instead of eight among 200 iterations.  For kernels that search for every access and
// are not bound by something else (33 M accesses, 200 iterations: k_stays_walk 486 -> 402 us, k_stays_links 308 ->
// 285, k_heads_write 82 -> 65; k_stay_ends, bound by its stores, 490 -> 530: not there).
struct IterFinder {
  static constexpr int COARSE = 128;
  const int32_t* off;
  const uint16_t* coarse;              // [COARSE + 1]
  int shift;
  __device__ __forceinline__ int32_t operator()(uint32_t p) const {
    const uint32_t b = p >> shift;
    int32_t lo = coarse[b], hi = coarse[b + 1] + 1;
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if (off[mid] <= (int32_t)p) lo = mid; else hi = mid;
    }
    return lo;
  }
};

__device__ __forceinline__ IterFinder iter_finder(int32_t* lds_off, uint16_t* coarse, const int64_t* __restrict__ off,
                                                  int32_t S) {
  load_offsets(lds_off, off, S);
  const int32_t total = lds_off[S];
  int shift = 0;
  while ((total >> shift) >= IterFinder::COARSE) ++shift;
  for (int t = threadIdx.x; t <= IterFinder::COARSE; t += blockDim.x) {
    const int64_t p = (int64_t)t << shift;
    coarse[t] = (uint16_t)iter_of(lds_off, S, p < total ? (int32_t)p : total);
  }
  __syncthreads();
  return {lds_off, coarse, shift};
}

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* red) {
  v = wave_reduce_sum(v);
  __syncthreads();  // red may still be read from an earlier call
  if (lane_id() == 0) red[threadIdx.x / WAVE] = v;
  __syncthreads();
  uint32_t s = 0;
  for (int w = 0; w < (int)blockDim.x / WAVE; ++w) s += red[w];
  return s;
}

// ---- part 1 -----------------------------------------------------------------------

constexpr int LOOK_ITEMS = 8;
constexpr int LOOK_TILE = TB * LOOK_ITEMS;

// The offsets of the iterations, in the launch's arguments as far as they have room, and what is to be cleared: one
// launch instead of a copy to the device and one (a copy costs the host as much as two launches, and the
// device the wait for it).
struct NearOffsets {
  static constexpr int MOST = 384;
  int32_t at[MOST + 1];                // (accesses are below 2^31)
};

__global__ __launch_bounds__(TB) void k_begin(NearOffsets near, int32_t S, int64_t* __restrict__ off, Zeros z) {
  for (int i = threadIdx.x; i <= S; i += TB) off[i] = near.at[i];
  for (int a = 0; a < z.used; ++a)
    for (int64_t i = threadIdx.x; i < z.words[a]; i += TB) z.at[a][i] = 0;
}

// number of run heads (= distinct nodes) per tile of the sorted pairs, and a zero behind them
__global__ __launch_bounds__(TB) void k_count_heads(const uint64_t* __restrict__ sorted, int64_t n,
                                                    uint32_t* __restrict__ head_tiles) {
  __shared__ uint32_t red[TB / WAVE];
  uint32_t heads = 0;
  const int64_t base = (int64_t)blockIdx.x * LOOK_TILE;
  uint64_t here[LOOK_ITEMS], left[LOOK_ITEMS];   // (beyond the end the last pair, which is not counted)
#pragma unroll
  for (int i = 0; i < LOOK_ITEMS; ++i) {
    int64_t j = base + i * TB + threadIdx.x;
    j = j < n ? j : n - 1;
    here[i] = sorted[j];
    left[i] = sorted[j > 0 ? j - 1 : 0];
  }
#pragma unroll
  for (int i = 0; i < LOOK_ITEMS; ++i) {
    const int64_t j = base + i * TB + threadIdx.x;
    if (j < n) heads += j == 0 || (uint32_t)(left[i] >> 32) != (uint32_t)(here[i] >> 32);
  }
  heads = wave_reduce_sum(heads);
  if (lane_id() == 0) red[threadIdx.x / WAVE] = heads;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int w = 0; w < TB / WAVE; ++w) s += red[w];
    head_tiles[blockIdx.x] = s;
    if (blockIdx.x == 0) head_tiles[gridDim.x] = 0;
  }
}

// Precondition check (only when asked for): ids inside [0, num_nodes) and no id twice in
// one iteration.  In the node-sorted pairs a repeated id shows up as two neighbours of the
// same node whose positions fall into the same iteration.  counts[0] = out of range,
// counts[1] = repeats.
__global__ __launch_bounds__(TB) void k_validate(const uint64_t* __restrict__ sorted, int64_t n,
                                                 const int64_t* __restrict__ off, int32_t S,
                                                 int64_t num_nodes,
                                                 unsigned long long* __restrict__ counts) {
  extern __shared__ int32_t lds_off[];
  load_offsets(lds_off, off, S);
  const int64_t j = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (j >= n) return;
  const uint64_t cur = sorted[j];
  const uint32_t v = (uint32_t)(cur >> 32);
  if ((int64_t)v >= num_nodes) atomicAdd(&counts[0], 1ull);
  if (j + 1 < n) {
    const uint64_t r = sorted[j + 1];
    if ((uint32_t)(r >> 32) == v &&
        iter_of(lds_off, S, (int32_t)(r & 0xFFFFFFFFu)) ==
            iter_of(lds_off, S, (int32_t)(cur & 0xFFFFFFFFu)))
      atomicAdd(&counts[1], 1ull);
  }
}

// next_iter of every access: the iteration of its right neighbour in the sorted order if
// that is the same node, else S ("never")
__global__ __launch_bounds__(TB) void k_look_right(const uint64_t* __restrict__ sorted, int64_t n,
                                                   const int64_t* __restrict__ off, int32_t S,
                                                   int32_t* __restrict__ next_iter) {
  extern __shared__ int32_t lds_off[];
  load_offsets(lds_off, off, S);
  const int64_t base = (int64_t)blockIdx.x * LOOK_TILE;
#pragma unroll
  for (int i = 0; i < LOOK_ITEMS; ++i) {
    const int64_t j = base + i * TB + threadIdx.x;
    if (j < n) {
      const uint64_t cur = sorted[j];
      int32_t nxt = S;
      if (j + 1 < n) {
        const uint64_t r = sorted[j + 1];
        if ((uint32_t)(r >> 32) == (uint32_t)(cur >> 32))
          nxt = iter_of(lds_off, S, (int32_t)(r & 0xFFFFFFFFu));
      }
      next_iter[cur & 0xFFFFFFFFu] = nxt;
    }
  }
}

// heads[r] = (first iteration << 32 | node) for the r-th distinct node (ascending id).  A wave takes
// LOOK_ITEMS * 64 consecutive pairs, 64 at a time (with a thread per eight consecutive ones every read
// of a wave touched 32 cache lines: 173 us for 33 M pairs, 81 us this way).
__global__ __launch_bounds__(TB) void k_heads_write(const uint64_t* __restrict__ sorted, int64_t n,
                                                    const int64_t* __restrict__ off, int32_t S,
                                                    const uint32_t* __restrict__ head_bases,
                                                    uint64_t* __restrict__ heads) {
  extern __shared__ int32_t lds_off[];
  __shared__ uint32_t s_heads[TB / WAVE];
  __shared__ uint16_t s_coarse[IterFinder::COARSE + 1];
  const IterFinder iteration = iter_finder(lds_off, s_coarse, off, S);
  const int lane = lane_id(), wave = threadIdx.x / WAVE;
  const int64_t base = (int64_t)blockIdx.x * LOOK_TILE + wave * (WAVE * LOOK_ITEMS);
  uint64_t here[LOOK_ITEMS];
#pragma unroll
  for (int i = 0; i < LOOK_ITEMS; ++i) {
    const int64_t j = base + i * WAVE + lane;
    here[i] = j < n ? sorted[j] : ~0ull;         // behind the end: an id that no access has
  }
  uint32_t before = base > 0 && base - 1 < n ? (uint32_t)(sorted[base - 1] >> 32) : 0xFFFFFFFFu;
  uint64_t is_head[LOOK_ITEMS];
  uint32_t count = 0;
#pragma unroll
  for (int i = 0; i < LOOK_ITEMS; ++i) {
    const uint32_t v = (uint32_t)(here[i] >> 32);
    uint32_t left = from_left(v);
    if (lane == 0) left = before;
    before = of_lane(v, WAVE - 1);
    is_head[i] = __ballot(v != left && v != 0xFFFFFFFFu);
    count += __popcll(is_head[i]);
  }
  if (lane == 0) s_heads[wave] = count;
  __syncthreads();
  uint32_t at = head_bases[blockIdx.x];
  for (int w = 0; w < wave; ++w) at += s_heads[w];
#pragma unroll
  for (int i = 0; i < LOOK_ITEMS; ++i) {
    if (is_head[i] >> lane & 1)
      heads[at + __popcll(is_head[i] & ((1ull << lane) - 1))] =
          ((uint64_t)(uint32_t)iteration((uint32_t)here[i]) << 32) | (here[i] >> 32);
    at += __popcll(is_head[i]);
  }
}

// ---- part 2 -----------------------------------------------------------------------

// (*last: the last of them, for the way that needs the heads' room)
__global__ __launch_bounds__(TB) void k_init_state(const uint64_t* __restrict__ heads,
                                                   int64_t count, int32_t* __restrict__ init_ids,
                                                   State st, uint64_t* __restrict__ last) {
  extern __shared__ uint32_t lds_hist[];  // S+1 bins
  for (int j = threadIdx.x; j <= st.S; j += TB) lds_hist[j] = 0;
  __syncthreads();
  const int64_t span = (int64_t)gridDim.x * TB;
  for (int64_t s = (int64_t)blockIdx.x * TB + threadIdx.x; s < count; s += span) {
    const uint64_t h = heads[s];
    const int32_t v = (int32_t)(h & 0xFFFFFFFFu);
    // Belady: the key of a prefetched row is its first access; LRU: it has not been used
    // yet, which is the oldest possible key
    const int32_t first = st.lru ? st.S : (int32_t)(h >> 32);
    if (s == count - 1) *last = h;
    init_ids[s] = v;
    st.res_id[s] = v;
    st.res_next[s] = first;
    st.addr[v] = (int32_t)s;
    atomicAdd(&lds_hist[first], 1u);
  }
  __syncthreads();
  for (int j = threadIdx.x; j <= st.S; j += TB)
    if (lds_hist[j]) atomicAdd(&st.rhist[j], lds_hist[j]);
}

// first_of[node] = first iteration that accesses the node (the array is preset to S, "never")
__global__ __launch_bounds__(TB) void k_scatter_first(const uint64_t* __restrict__ heads,
                                                      int64_t count,
                                                      int32_t* __restrict__ first_of) {
  const int64_t r = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (r < count) first_of[heads[r] & 0xFFFFFFFFu] = (int32_t)(heads[r] >> 32);
}

// The state a superbatch starts from when the cache is carried over: line s holds
// start_ids[s], keyed by the row's first access in this superbatch.  A row that is never
// accessed is a dead resident from the start.  bad[0] counts ids outside [0, num_nodes) and
// ids that occur twice (both are skipped).
__global__ __launch_bounds__(TB) void k_init_state_resume(const int32_t* __restrict__ start_ids,
                                                          const int32_t* __restrict__ first_of,
                                                          State st,
                                                          unsigned long long* __restrict__ bad) {
  extern __shared__ uint32_t lds_hist[];  // S+1 bins
  for (int j = threadIdx.x; j <= st.S; j += TB) lds_hist[j] = 0;
  __syncthreads();
  const int64_t span = (int64_t)gridDim.x * TB;
  for (int64_t s = (int64_t)blockIdx.x * TB + threadIdx.x; s < st.cap; s += span) {
    const int32_t v = start_ids[s];
    if (v < 0 || v >= st.num_nodes || atomicCAS(&st.addr[v], -1, (int32_t)s) != -1) {
      atomicAdd(bad, 1ull);
      continue;
    }
    const int32_t first = first_of[v];
    st.res_id[s] = v;
    st.res_next[s] = first;
    atomicAdd(&lds_hist[first], 1u);
    if (first == st.S) atomicOr(&st.dead_bits[(uint32_t)v >> 5], 1u << ((uint32_t)v & 31));
  }
  __syncthreads();
  for (int j = threadIdx.x; j <= st.S; j += TB)
    if (lds_hist[j]) atomicAdd(&st.rhist[j], lds_hist[j]);
}

// The same without keys, for the ways that do not loop over the state.  What they need of a carried state:
// which rows it holds, the lines of those the superbatch accesses, and its dead rows.  The rows
// come in no order, so every access below is to a random place; the kernel above makes three of
// them per line, two of them atomics on the memory side (2.05 ms for 27.75 M lines of 111 M nodes),
// these one read of a 14 MB bitmap, one byte stored, and a table entry stored for the rows that are
// accessed (0.99 ms in the order of the lines; dealt by the upper eight bits of the id first: 0.17 + 0.41
// ms; the passes around it 0.17).  Where a stretch of ids so dealt has room for its bits in LDS, they are put together
// there, see k_hold_stretch.  Whether all rows are distinct and in range shows in the number of bytes or bits set.
constexpr int HOLD_ITEMS = 8;
// Lines are dealt from here on, and where the free buffer of the sort has a word for each.  k_hold, 2^20 lines:
// dealt 16 + 11 us and the scans of the counters (10), in their own order 19; 2^21: 20 + 28 (and 10)
// against 51; 2^22: 28 + 54 (and 10) against 128.  That is where its line lies; k_hold_stretch, which takes the dealt
// words up to 2^27 nodes, would pay below it, too: calls of four accesses to a line on 5, 20 and 110 M nodes, in
// their own order and dealt, 2^18 lines 598, 623, 689 and 592, 619, 659 us; 2^20 827, 933, 1 034 and 800, 892,
// 956; 2^21 1 355, 1 475, 1 595 and 1 328, 1 409, 1 496.
constexpr int64_t HOLD_DEAL_MIN = int64_t(1) << 22;

// A stretch of the ids as they are dealt is shared by up to four blocks, each of which reads all of its words and takes
// those of its own ids: the lines crowd where the cache was filled up, every id of some stretches and one in six of the others.
// A part of the dead rows' counts is not divided.
constexpr int HOLD_SHIFT_MIN = PART_SHIFT, HOLD_SHIFT_MAX = 19, HOLD_SHARE_MAX = 2;   // (2^17 ids to a block at most)

// how many of the heads have an id below x (a wave: all lanes take part, and get it)
__device__ __forceinline__ int64_t heads_below(const uint64_t* __restrict__ heads, int64_t count, int64_t x) {
  int64_t lo = 0, hi = count;            // it is in [lo, hi]
  while (lo < hi) {
    const int64_t step = (hi - lo + WAVE - 1) / WAVE, at = lo + lane_id() * step;
    const int n = __popcll(__ballot(at < hi && (int64_t)(uint32_t)heads[at < hi ? at : lo] < x));
    if (n == 0) return lo;               // (the lanes below: ids ascend)
    const int64_t next = lo + n * step;
    lo += (n - 1) * step + 1;
    hi = next < hi ? next : hi;
  }
  return lo;
}

// All of it for one share of a stretch of 2^shift ids, 2^share of them: accessed and held rows as bits in LDS, the table
// entries of rows that are both, then the words, the dead rows and their part counts.  in: the words (v << 32 | line) by
// stretch, that of digit d from starts[d * tiles] on.  27.75 M lines of 111 M nodes, a third of them in 22 of 212
// stretches: 313 us, where k_accessed_bits, k_hold, k_held_words and what they have cleared take 105, 413, 40 and 25 (the
// call 2 724 -> 2 479); one block to a stretch 414, the fullest 22 at work alone in the end.
__global__ __launch_bounds__(BIG) void k_hold_stretch(const uint64_t* __restrict__ in, const uint32_t* __restrict__ starts,
                                                      int64_t tiles, int32_t digits, int shift, int share, State st,
                                                      const uint64_t* __restrict__ heads, int64_t count,
                                                      uint32_t* __restrict__ accessed,
                                                      uint32_t* __restrict__ held_bits,
                                                      unsigned long long* __restrict__ rows) {
  constexpr int BITS = HOLD_SHIFT_MAX - HOLD_SHARE_MAX, MOST = 1 << (BITS - 5), PARTS = 1 << (BITS - PART_SHIFT);
  __shared__ uint32_t s_accessed[MOST], s_held[MOST];
  __shared__ uint32_t s_dead[PARTS], s_rows;
  __shared__ int64_t s_range[2];
  // (blocks go to the eight XCDs in turn; the shares of a stretch to the same one)
  const int32_t m = blockIdx.x / 8, d = (m >> share) * 8 + blockIdx.x % 8, words = 1 << (shift - share - 5);
  const int64_t first_id = ((int64_t)d << shift) + ((int64_t)(m & ((1 << share) - 1)) << (shift - share));
  if (first_id >= st.num_nodes) return;
  const uint32_t base = (uint32_t)first_id;
  const int64_t span = st.num_nodes - first_id < words * 32 ? st.num_nodes - first_id : words * 32;
  for (int x = threadIdx.x; x < words; x += BIG) s_accessed[x] = s_held[x] = 0;
  if (threadIdx.x < PARTS) s_dead[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_rows = 0;
  if (threadIdx.x < 2 * WAVE) {
    const int64_t at = heads_below(heads, count, (int64_t)base + (threadIdx.x < WAVE ? 0 : span));
    if (lane_id() == 0) s_range[threadIdx.x / WAVE] = at;
  }
  __syncthreads();
  const int64_t last = s_range[1];
  for (int64_t r0 = s_range[0] + threadIdx.x; r0 < last; r0 += BIG * HOLD_ITEMS) {
    uint32_t v[HOLD_ITEMS];
#pragma unroll
    for (int t = 0; t < HOLD_ITEMS; ++t) v[t] = (uint32_t)heads[r0 + t * BIG < last ? r0 + t * BIG : r0] - base;
#pragma unroll
    for (int t = 0; t < HOLD_ITEMS; ++t)
      if (r0 + t * BIG < last && v[t] < (uint32_t)span) atomicOr(&s_accessed[v[t] >> 5], 1u << (v[t] & 31));
  }
  __syncthreads();
  const int64_t end = d + 1 < digits ? starts[(d + 1) * tiles] : st.cap;
  uint64_t next[HOLD_ITEMS];               // (asked for while the ones before are put in)
  auto ask = [&](int64_t x0) {
#pragma unroll
    for (int t = 0; t < HOLD_ITEMS; ++t) next[t] = in[x0 + t * BIG < end ? x0 + t * BIG : 0];   // (a branch would be a wait)
  };
  int64_t x0 = starts[d * tiles] + threadIdx.x;
  ask(x0);
  for (; x0 < end; x0 += BIG * HOLD_ITEMS) {
    uint32_t v[HOLD_ITEMS], word[HOLD_ITEMS];
    int32_t line[HOLD_ITEMS];
#pragma unroll
    for (int t = 0; t < HOLD_ITEMS; ++t) {
      v[t] = (uint32_t)(next[t] >> 32) - base;
      line[t] = (int32_t)(uint32_t)next[t];
      // (out of range: shows in the number of rows held)
      if (x0 + t * BIG >= end || v[t] >= (uint32_t)span) v[t] = 0xFFFFFFFFu;
    }
    ask(x0 + BIG * HOLD_ITEMS);
#pragma unroll
    for (int t = 0; t < HOLD_ITEMS; ++t) word[t] = s_accessed[v[t] != 0xFFFFFFFFu ? v[t] >> 5 : 0];
#pragma unroll
    for (int t = 0; t < HOLD_ITEMS; ++t) {
      if (v[t] == 0xFFFFFFFFu) continue;
      atomicOr(&s_held[v[t] >> 5], 1u << (v[t] & 31));
      if (word[t] >> (v[t] & 31) & 1u) st.addr[base + v[t]] = line[t];
    }
  }
  __syncthreads();
  uint32_t mine = 0;
  for (int x0 = 0; x0 < words; x0 += BIG) {                       // (whole waves, each in one part)
    const int x = x0 + threadIdx.x;
    const int64_t w = (int64_t)(base >> 5) + x;
    uint32_t held = 0, dead = 0;
    if (x < words && w < st.words) {
      held = s_held[x];
      dead = held & ~s_accessed[x];
      accessed[w] = s_accessed[x];
      held_bits[w] = held;
      st.dead_bits[w] = dead;
    }
    mine += __popc(held);
    const uint32_t sum = wave_reduce_sum((uint32_t)__popc(dead));
    if (lane_id() == 0 && sum) atomicAdd(&s_dead[x / PART_WORDS], sum);
  }
  mine = wave_reduce_sum(mine);
  if (lane_id() == 0 && mine) atomicAdd(&s_rows, mine);
  __syncthreads();
  const int64_t part = (int64_t)(base >> PART_SHIFT) + threadIdx.x;
  if (threadIdx.x < (words + PART_WORDS - 1) / PART_WORDS && part < st.parts) st.dead_part[part] = s_dead[threadIdx.x];
  if (threadIdx.x == 0 && s_rows) atomicAdd(rows, (unsigned long long)s_rows);
}

// bit v of `bits` for every head (heads in id order, so a word's bits are neighbours: a wave
// gathers them and stores words that are its own)
__global__ __launch_bounds__(TB) void k_accessed_bits(const uint64_t* __restrict__ heads, int64_t count,
                                                      uint32_t* __restrict__ bits) {
  const int64_t r = (int64_t)blockIdx.x * TB + threadIdx.x;
  const uint32_t v = r < count ? (uint32_t)heads[r] : 0xFFFFFFFFu;
  const uint32_t w = v >> 5;
  uint32_t word = r < count ? 1u << (v & 31) : 0u;
  const int lane = lane_id();
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    const uint32_t other = __shfl_down(word, d, WAVE), ow = __shfl_down(w, d, WAVE);
    if (lane + d < WAVE && ow == w) word |= other;
  }
  const uint32_t left = from_left(w);   // (every lane takes part)
  const bool leads = lane == 0 || left != w;
  const uint32_t last = of_lane(w, WAVE - 1);
  if (r >= count || !leads) return;
  if (lane == 0 || w == last) atomicOr(&bits[w], word);   // the word may have bits in the next wave, too
  else bits[w] = word;
}

// held[v] = 1 and, for the rows that are accessed, addr[v] = line, for the words (v << 32 | line).
// In the order of the lines every access is a random one.  Where the words come dealt by the upper bits
// of v (DEALT), an XCD takes an eighth of them, and what its blocks touch at a time stays in its L2.
template <bool DEALT, typename Source>
__global__ __launch_bounds__(TB) void k_hold(Source in, int64_t cap, int64_t num_nodes,
                                             const uint32_t* __restrict__ accessed,
                                             uint8_t* __restrict__ held, int32_t* __restrict__ addr) {
  // (blocks go to the eight XCDs in turn)
  const int64_t b = DEALT ? (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8 : blockIdx.x;
  const int64_t base = b * (TB * HOLD_ITEMS) + threadIdx.x;
  int32_t v[HOLD_ITEMS], line[HOLD_ITEMS];
  uint32_t word[HOLD_ITEMS];
#pragma unroll
  for (int t = 0; t < HOLD_ITEMS; ++t) {
    const int64_t s = base + t * TB;
    const uint64_t w = s < cap ? in(s) : ~0ull;
    v[t] = (int32_t)(w >> 32);
    line[t] = (int32_t)w;
  }
#pragma unroll
  for (int t = 0; t < HOLD_ITEMS; ++t) {
    if (v[t] >= num_nodes) v[t] = -1;    // shows in the number of rows held
    word[t] = v[t] >= 0 ? accessed[(uint32_t)v[t] >> 5] : 0u;
  }
#pragma unroll
  for (int t = 0; t < HOLD_ITEMS; ++t) {
    if (v[t] < 0) continue;
    held[v[t]] = 1;
    if (word[t] >> (v[t] & 31) & 1u) addr[v[t]] = line[t];
  }
}

// The bytes as bits; the dead rows (held, not accessed) and their part counts; the number of rows held.
// A block per part.
__global__ __launch_bounds__(TB) void k_held_words(const uint8_t* __restrict__ held, State st,
                                                   const uint32_t* __restrict__ accessed,
                                                   uint32_t* __restrict__ held_bits,
                                                   unsigned long long* __restrict__ rows) {
  __shared__ uint32_t red[TB / WAVE];
  uint32_t all = 0, dead = 0;
  for (int t = threadIdx.x; t < PART_WORDS; t += TB) {
    const int64_t w = (int64_t)blockIdx.x * PART_WORDS + t;
    if (w >= st.words) break;
    uint32_t word = 0;
    const uint32_t* bytes = reinterpret_cast<const uint32_t*>(held) + w * 8;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t x = bytes[q];       // four bytes of 0 or 1
      word |= ((x | x >> 7 | x >> 14 | x >> 21) & 15u) << (4 * q);
    }
    const uint32_t gone = word & ~accessed[w];
    held_bits[w] = word;
    st.dead_bits[w] = gone;
    all += __popc(word);
    dead += __popc(gone);
  }
  const uint32_t n_dead = block_sum_u32(dead, red), n_all = block_sum_u32(all, red);
  if (threadIdx.x == 0) {
    st.dead_part[blockIdx.x] = n_dead;
    if (n_all) atomicAdd(rows, (unsigned long long)n_all);
  }
}

// rhist of a carried state: the rows held by their first access; bin S, the rows never accessed, gets
// what is left (counted down from cap by every block)
__global__ __launch_bounds__(TB) void k_held_hist(const uint64_t* __restrict__ heads, int64_t count,
                                                  const uint32_t* __restrict__ held_bits, State st) {
  extern __shared__ uint32_t lds_hist[];  // S bins
  for (int j = threadIdx.x; j < st.S; j += TB) lds_hist[j] = 0;
  __syncthreads();
  const int64_t span = (int64_t)gridDim.x * TB;
  for (int64_t r = (int64_t)blockIdx.x * TB + threadIdx.x; r < count; r += span) {
    const uint64_t h = heads[r];
    const uint32_t v = (uint32_t)h;
    if (held_bits[v >> 5] >> (v & 31) & 1u) atomicAdd(&lds_hist[h >> 32], 1u);
  }
  __syncthreads();
  uint32_t mine = 0;
  for (int j = threadIdx.x; j < st.S; j += TB)
    if (lds_hist[j]) {
      atomicAdd(&st.rhist[j], lds_hist[j]);
      mine += lds_hist[j];
    }
  mine = wave_reduce_sum(mine);
  if (lane_id() == 0 && mine) atomicSub(&st.rhist[st.S], mine);
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&st.rhist[st.S], (uint32_t)st.cap);
}

// addr of the dead rows from lo_id up: the only ones of them that can be evicted
__global__ __launch_bounds__(TB) void k_dead_lines(State st, const uint32_t* __restrict__ accessed,
                                                   int64_t lo_id) {
  const int64_t span = (int64_t)gridDim.x * TB;
  for (int64_t s = (int64_t)blockIdx.x * TB + threadIdx.x; s < st.cap; s += span) {
    const int32_t v = st.res_id[s];
    if (v >= lo_id && !(accessed[(uint32_t)v >> 5] >> (v & 31) & 1u)) st.addr[v] = (int32_t)s;
  }
}

// addr[node of rank r] = r for the first `count` heads (C_0 when everything fits)
__global__ __launch_bounds__(TB) void k_scatter_rank(const uint64_t* __restrict__ heads,
                                                     int64_t count, int32_t* __restrict__ addr) {
  const int64_t r = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (r < count) addr[heads[r] & 0xFFFFFFFFu] = (int32_t)r;
}

// src_line[p] = addr[ids[p]]: every accessed row is resident, nothing ever changes
__global__ __launch_bounds__(TB) void k_lookup_lines(const int32_t* __restrict__ ids, int64_t n,
                                                     const int32_t* __restrict__ addr,
                                                     int32_t* __restrict__ src_line) {
  constexpr int ITEMS = 4;
  const int64_t base = (int64_t)blockIdx.x * (TB * ITEMS) + threadIdx.x;
  int32_t v[ITEMS];
#pragma unroll
  for (int t = 0; t < ITEMS; ++t) {
    const int64_t p = base + t * TB;
    v[t] = ids[p < n ? p : 0];
  }
#pragma unroll
  for (int t = 0; t < ITEMS; ++t) v[t] = addr[v[t]];
#pragma unroll
  for (int t = 0; t < ITEMS; ++t) {
    const int64_t p = base + t * TB;
    if (p < n) src_line[p] = v[t];
  }
}

// miss_count[i] = |ids_i| (a cache without lines: every access misses)
__global__ __launch_bounds__(TB) void k_iteration_lengths(const int64_t* __restrict__ off, int32_t S,
                                                          int64_t* __restrict__ miss_count) {
  const int32_t i = blockIdx.x * TB + threadIdx.x;
  if (i < S) miss_count[i] = off[i + 1] - off[i];
}

__global__ __launch_bounds__(TB) void k_copy_init(const uint64_t* __restrict__ heads, int64_t count,
                                                  int32_t* __restrict__ init_ids) {
  const int64_t s = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (s < count) init_ids[s] = (int32_t)(heads[s] & 0xFFFFFFFFu);
}

// ---- part 3 -----------------------------------------------------------------------
//
// The loop over the state (more iterations than stays.hpp takes, LRU with iterations longer than the cache,
// the smallest calls).  One iteration of
// the recurrence is six dependent launches:
//   k_touch      hits get their new key, hits and misses are histogrammed by key, the line of
//                every access (or -1) is kept for the later phases and for the executor
//   k_threshold  one block: walks the histograms down from "never", fixes the threshold
//                bucket j*, what happens inside it and the size of the changeset; when the
//                evictions fall among the dead residents (the usual case of a large cache)
//                it also finds the id threshold T, from part counts of the standing dead-row
//                bitmap that are kept up to date wherever a bit changes
//   k_mark       otherwise: the members of the selected class of bucket j* set their bit in a
//                scratch bitmap over node ids and count themselves per part
//   k_find       one block: T = the keep-th set bit, from the part counts
//   k_flags      eviction flags per cache line (dead residents of a large cache: the bits above
//                T of their bitmap are turned into line flags through the address table
//                instead) and insertion counts per tile of accesses; the scratch bitmap is
//                cleared by the members that set it
//   k_emit_pair  both lists in their order (every block sums the tile counts in front of it:
//                no scan launch), and the cache state of C_{i+1}: the t-th insertion takes
//                the line of the t-th eviction, the two sides meeting in one 64-bit word per
//                t that the second to arrive completes
// A carried cache that has room for every row of the superbatch never needs k_mark and k_find
// (all evictions fall among the dead rows): its iterations are four launches.
// No phase makes a pass over a whole bitmap or scans all tiles in one block: the cost of an
// iteration follows its accesses and, unless the dead-row path applies, the cache lines.
// Measured and dropped earlier: a single cooperative kernel with grid.sync() between the
// phases (about 0.1 ms per barrier on 1024 blocks), and running the single-block phases in
// the last block to finish of the launch before them with a device-wide fence per block
// (writes back and invalidates L2 on this multi-XCD part: three to four times slower).

// ready[i] = number of prefetched rows whose first access lies in iterations 0..i: the
// prefix of C_0 (it is ordered by first access) that iteration i can touch.
__global__ __launch_bounds__(TB) void k_init_ready(const uint64_t* __restrict__ heads,
                                                   int64_t n_init, int32_t S,
                                                   int64_t* __restrict__ ready) {
  const int32_t i = blockIdx.x * TB + threadIdx.x;
  if (i >= S) return;
  int64_t lo = 0, hi = n_init;   // first rank whose first access is later than i
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int32_t)(heads[mid] >> 32) <= i) lo = mid + 1; else hi = mid;
  }
  ready[i] = lo;
}

struct Iter {           // what a phase needs to know about the running iteration
  const int32_t* ids;   // ids_i
  const int32_t* next;  // next accessed iteration of each access of ids_i (Belady keys)
  int64_t n;            // |ids_i|
  int32_t i;
  int32_t key;          // >= 0: every access of the iteration takes this key (LRU: S-1-i,
                        // smaller = used more recently); < 0: the key is next[p]
  int32_t lo_bin;       // smallest bucket a candidate of this iteration can fall into
  int32_t* src_line;    // out (may be null): cache line of each access in C_i, -1 for a miss
};

__device__ __forceinline__ int32_t key_of(const Iter& it, int64_t p) {
  return it.key >= 0 ? it.key : it.next[p];
}

struct Outputs {
  int32_t* in_ids;
  int32_t* out_ids;
  int32_t* in_positions;
  int64_t cs_capacity;
  int64_t* cs_offsets;
  int64_t* miss_count;
};

// Sum of counts[0 .. n) by the whole block.
__device__ __forceinline__ uint32_t block_prefix_of(const uint32_t* __restrict__ counts, int64_t n,
                                                    uint32_t* red) {
  uint32_t s = 0;
  for (int64_t q = threadIdx.x; q < n; q += TB) s += counts[q];
  return block_sum_u32(s, red);
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
  const uint32_t lo = __shfl((uint32_t)v, src, WAVE);
  const uint32_t hi = __shfl((uint32_t)(v >> 32), src, WAVE);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ void dead_bit_set(const State& st, uint32_t v) {
  atomicOr(&st.dead_bits[v >> 5], 1u << (v & 31));
  atomicAdd(&st.dead_part[v >> PART_SHIFT], 1u);
}

// Refresh the keys of the hits, histogram hits and misses by key, keep every access's line.
// lds: 2*(S+1) counters.  One block covers TB*TOUCH_ITEMS accesses.
__global__ __launch_bounds__(TB) void k_touch(State st, Iter it, unsigned long long* miss_out) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t red[TB / WAVE];
  uint32_t* hr = lds;
  uint32_t* hi = lds + st.S + 1;
  for (int j = threadIdx.x; j < 2 * (st.S + 1); j += TB) lds[j] = 0;
  __syncthreads();
  uint32_t misses = 0;
  const int64_t base = (int64_t)blockIdx.x * (TB * TOUCH_ITEMS);
  // id, then address-table entry, then the line's state: the reads of one level are issued
  // for all items before any is used, so that they are in flight together.  An item beyond
  // the end repeats the block's first item (in range) and is skipped when it is processed.
  int32_t v[TOUCH_ITEMS], line[TOUCH_ITEMS], nx[TOUCH_ITEMS];
#pragma unroll
  for (int t = 0; t < TOUCH_ITEMS; ++t) {
    int64_t p = base + t * TB + threadIdx.x;
    p = p < it.n ? p : base;
    v[t] = it.ids[p];
    nx[t] = key_of(it, p);
  }
#pragma unroll
  for (int t = 0; t < TOUCH_ITEMS; ++t) line[t] = st.addr[v[t]];
#pragma unroll
  for (int t = 0; t < TOUCH_ITEMS; ++t) {
    const int64_t p = base + t * TB + threadIdx.x;
    if (p < it.n) {
      st.acc_line[p] = line[t];
      if (it.src_line) it.src_line[p] = line[t];   // the state is C_i here
    }
  }
  int32_t old_key[TOUCH_ITEMS];
  if (st.lru) {
#pragma unroll
    for (int t = 0; t < TOUCH_ITEMS; ++t) old_key[t] = line[t] >= 0 ? st.res_next[line[t]] : 0;
  }
#pragma unroll
  for (int t = 0; t < TOUCH_ITEMS; ++t) {
    if (base + t * TB + threadIdx.x >= it.n) continue;
    if (line[t] >= 0) {
      // An LRU hit leaves a bucket that is still walked (an older one): take it out of
      // the count there; counters wrap, the flush below adds them modulo 2^32.  A Belady
      // hit leaves bucket i, which no later iteration looks at.
      if (st.lru) atomicSub(&hr[old_key[t]], 1u);
      st.res_next[line[t]] = nx[t];
      atomicAdd(&hr[nx[t]], 1u);
      // the row's last access: a dead resident from now on
      if (nx[t] == st.S && !st.lru) dead_bit_set(st, (uint32_t)v[t]);
    } else {
      atomicAdd(&hi[nx[t]], 1u);
      ++misses;
    }
  }
  const uint32_t total = block_sum_u32(misses, red);
  for (int j = it.lo_bin + threadIdx.x; j <= st.S; j += TB) {
    if (hr[j]) atomicAdd(&st.rhist[j], hr[j]);
    if (hi[j]) atomicAdd(&st.ihist[j], hi[j]);
  }
  if (threadIdx.x == 0 && total) atomicAdd(miss_out, (unsigned long long)total);
}

// One block of NT threads.  Walks the buckets from "never" downwards until as many
// candidates as there were misses are dropped; fixes the threshold bucket, what happens
// inside it, the size of the changeset, and rolls the resident histogram forward to C_{i+1}.
template <int NT>
__device__ void p_threshold(const State& st, int32_t i, int32_t lo_bin, const int64_t* miss_count,
                            int64_t* cs_offsets) {
  __shared__ int64_t smem[NT / WAVE + 1];
  __shared__ int32_t s_jstar;
  __shared__ uint32_t s_kept;
  const int32_t S = st.S;
  const int64_t n_drop = miss_count[i];
  const int32_t bins = S - lo_bin + 1;            // buckets lo_bin .. S, walked as r = S - j
  const int32_t per = (bins + NT - 1) / NT;
  const int32_t r0 = threadIdx.x * per;
  int64_t mine = 0;
  for (int32_t r = r0; r < r0 + per && r < bins; ++r)
    mine += (int64_t)st.rhist[S - r] + st.ihist[S - r];
  int64_t total;
  int64_t before = block_exclusive_scan<int64_t, NT>(mine, smem, total);
  if (threadIdx.x == 0) {
    // default: nothing is dropped (no misses); overwritten below by the thread that
    // finds the threshold bucket
    s_jstar = S + 1;
    s_kept = 0;
    Ctrl c{};
    c.jstar = S + 1;
    c.mode_in = MODE_ALL;
    c.mode_res = MODE_ALL;
    c.T = -1;
    *st.ctrl = c;
    cs_offsets[i + 1] = cs_offsets[i];
  }
  __syncthreads();
  if (n_drop > 0) {
    for (int32_t r = r0; r < r0 + per && r < bins; ++r) {
      const int32_t j = S - r;
      const int64_t R = st.rhist[j], I = st.ihist[j];
      if (before <= n_drop && before + R + I > n_drop) {
        const int64_t rem = n_drop - before;  // still to drop, all from bucket j
        Ctrl c{};
        c.jstar = j;
        int64_t from_res = 0;
        if (rem == 0) {
          c.mode_in = MODE_ALL; c.mode_res = MODE_ALL;
        } else if (rem < I) {
          c.mode_in = MODE_SELECT; c.mode_res = MODE_ALL; c.keep = (int32_t)(I - rem);
        } else if (rem == I) {
          c.mode_in = MODE_NONE; c.mode_res = MODE_ALL;
        } else {
          c.mode_in = MODE_NONE; c.mode_res = MODE_SELECT;
          from_res = rem - I;
          c.keep = (int32_t)(R - from_res);
          // in the "never" bucket the members are exactly the dead residents, whose
          // bitmap is maintained incrementally: no marking pass is needed
          c.use_dead = j == S && !st.lru;
        }
        c.T = -1;
        // evictions inside j*; those of the buckets above j* are added after the barrier
        s_jstar = j;
        s_kept = (uint32_t)(R + I - rem);
        c.n_change = (int32_t)from_res;
        *st.ctrl = c;
      }
      before += R + I;
    }
  }
  __syncthreads();
  const int32_t jstar = s_jstar;
  // residents evicted from the buckets above j*, and the histogram of C_{i+1}
  int64_t above = 0;
  for (int32_t r = r0; r < r0 + per && r < bins; ++r) {
    const int32_t j = S - r;
    if (j > jstar) {
      above += st.rhist[j];
      st.rhist[j] = 0;
    } else if (j == jstar) {
      st.rhist[j] = s_kept;
    } else {
      st.rhist[j] += st.ihist[j];
    }
    st.ihist[j] = 0;
  }
  int64_t above_total;
  block_exclusive_scan<int64_t, NT>(above, smem, above_total);
  if (threadIdx.x == 0 && n_drop > 0) {
    st.ctrl->n_change += (int32_t)above_total;
    cs_offsets[i + 1] = cs_offsets[i] + st.ctrl->n_change;
  }
  __syncthreads();
}

// One block of NT threads: the position of the keep-th set bit (1-based, from the bottom) of
// `bits`, found through `part` (set bits per PART_WORDS words); -1 if there are fewer set bits.
// Every thread gets the result.  With `trim`, the part counts are rewritten to what remains
// once every bit above that position is cleared.
template <int NT>
__device__ int32_t p_kth_set_bit(const uint32_t* __restrict__ bits, uint32_t* __restrict__ part,
                                 int64_t parts, int64_t words, int64_t keep, bool trim) {
  __shared__ int64_t smem[NT / WAVE + 1];
  __shared__ int64_t s_part, s_before;
  __shared__ int32_t s_found;
  // 1. the part that holds the keep-th set bit
  const int64_t per = (parts + NT - 1) / NT;
  const int64_t q0 = threadIdx.x * per;
  int64_t mine = 0;
  for (int64_t q = q0; q < q0 + per && q < parts; ++q) mine += part[q];
  int64_t total;
  int64_t before = block_exclusive_scan<int64_t, NT>(mine, smem, total);
  if (threadIdx.x == 0) {
    s_part = -1;
    s_found = -1;
  }
  __syncthreads();
  for (int64_t q = q0; q < q0 + per && q < parts; ++q) {
    const int64_t cnt = part[q];
    if (before < keep && before + cnt >= keep) {
      s_part = q;
      s_before = before;
    }
    before += cnt;
  }
  __syncthreads();
  if (s_part < 0) return -1;  // fewer set bits than asked for (uniform over the block)
  if (trim) {
    for (int64_t q = q0; q < q0 + per && q < parts; ++q)
      if (q > s_part) part[q] = 0;
      else if (q == s_part) part[q] = (uint32_t)(keep - s_before);
  }
  // 2. the word inside that part, then the bit inside the word
  constexpr int WPT = PART_WORDS / NT;
  const int64_t w0 = s_part * PART_WORDS + (int64_t)threadIdx.x * WPT;
  int64_t cntw = 0;
  for (int t = 0; t < WPT; ++t)
    if (w0 + t < words) cntw += __popc(bits[w0 + t]);
  int64_t tot2;
  int64_t bw = s_before + block_exclusive_scan<int64_t, NT>(cntw, smem, tot2);
  for (int t = 0; t < WPT; ++t)
    if (w0 + t < words) {
      uint32_t word = bits[w0 + t];
      const int pc = __popc(word);
      if (bw < keep && bw + pc >= keep) {
        int need = (int)(keep - bw);  // the need-th set bit of this word, 1-based
        int bit = 0;
        while (true) {
          bit = __ffs(word) - 1;
          if (--need == 0) break;
          word &= word - 1;
        }
        s_found = (int32_t)((w0 + t) * 32 + bit);
      }
      bw += pc;
    }
  __syncthreads();
  return s_found;
}

// T of the running iteration = the id whose bit is the keep-th set bit of `bits`.
template <int NT>
__device__ void p_bits_find(const State& st, const uint32_t* __restrict__ bits,
                            uint32_t* __restrict__ part, bool trim) {
  Ctrl* c = st.ctrl;
  const int32_t T = p_kth_set_bit<NT>(bits, part, st.parts, st.words, c->keep, trim);
  if (threadIdx.x == 0 && T >= 0) c->T = T;   // fewer set bits than asked for cannot happen: T stays -1
  __syncthreads();
}

__global__ __launch_bounds__(BIG) void k_threshold(State st, int32_t i, int32_t lo_bin, Outputs o,
                                                   int64_t evict_tiles) {
  p_threshold<BIG>(st, i, lo_bin, o.miss_count, o.cs_offsets);
  Ctrl c = *st.ctrl;   // written by this block, in front of the barrier that ends p_threshold
  // k_mark will set the bits of the selected class only
  c.marked = (c.mode_res == MODE_SELECT && !c.use_dead ? MARKED_RES : 0) |
             (c.mode_in == MODE_SELECT ? MARKED_IN : 0);
  if (threadIdx.x == 0) st.ctrl->marked = c.marked;
  if (st.dead_only && !c.use_dead && threadIdx.x == 0 &&
      (c.mode_res == MODE_SELECT || c.mode_in == MODE_SELECT))
    *st.fault = 1;
  if (c.use_dead) {
    p_bits_find<BIG>(st, st.dead_bits, st.dead_part, true);
    if (st.dead_scatter)     // the scatter counts evictions per tile with atomics
      for (int64_t q = threadIdx.x; q < evict_tiles; q += BIG) st.evict_tiles[q] = 0;
  }
}

__global__ __launch_bounds__(BIG) void k_find(State st) {
  const Ctrl c = *st.ctrl;
  if (c.use_dead || (c.mode_res != MODE_SELECT && c.mode_in != MODE_SELECT)) return;
  if (c.mode_res == MODE_SELECT) p_bits_find<BIG>(st, st.bitmap, st.sel_part, false);
  else p_bits_find<BIG>(st, st.bitmap_in, st.sel_part_in, false);
}

constexpr int MARK_ITEMS = 8;   // lines / accesses per thread in the mark phases

// ---- Belady: what an iteration decides without looking at the cache ---------------------------
//
// The candidates of iteration i per next-use bucket are the residents that the iteration does
// not access (a histogram R_i that rolls forward by the rule of p_threshold) plus the
// iteration's accesses by their new key (a histogram H_i of next_iter alone), and the number
// to drop is the iteration's length minus R_i[i], the residents keyed to it.  So the threshold
// bucket j* of every iteration, the number of rows to drop from it, and R_{i+1} follow from S
// histograms of the trace.  stays.hpp turns them into the changesets.
#include "deal.hpp"
#include "stays.hpp"
#include "lines.hpp"
#include "fits.hpp"
#include "small.hpp"

// H[i][k] = accesses of iteration i whose next accessed iteration is k.  blockIdx.y = iteration.
__global__ __launch_bounds__(TB) void k_key_hists(const uint64_t* __restrict__ ends,
                                                  const int64_t* __restrict__ off, int32_t S,
                                                  uint32_t* __restrict__ hists) {
  extern __shared__ uint32_t lds_h[];   // S + 1 bins
  const int32_t i = blockIdx.y;
  const int64_t lo = off[i], n = off[i + 1] - lo;
  const int64_t base = (int64_t)blockIdx.x * (TB * TOUCH_ITEMS);
  if (base >= n) return;                // uniform
  for (int j = threadIdx.x; j <= S; j += TB) lds_h[j] = 0;
  __syncthreads();
  uint64_t w[TOUCH_ITEMS];
#pragma unroll
  for (int t = 0; t < TOUCH_ITEMS; ++t) {
    const int64_t p = base + t * TB + threadIdx.x;
    w[t] = ends[lo + (p < n ? p : base)];
  }
#pragma unroll
  for (int t = 0; t < TOUCH_ITEMS; ++t)
    if (base + t * TB + threadIdx.x < n) atomicAdd(&lds_h[stay_next(w[t])], 1u);
  __syncthreads();
  for (int j = i + 1 + threadIdx.x; j <= S; j += TB)
    if (lds_h[j]) atomicAdd(&hists[(int64_t)i * (S + 1) + j], lds_h[j]);
}

// One block of NT threads: the thresholds of all iterations, one after the other.  rhist holds R_0
// (the residents of the start state by key).  Bins are walked as r = S - j, PER consecutive r to a
// thread, which keeps their counts in registers.
template <int NT, int PER>
__global__ __launch_bounds__(NT) void k_static_roll(State st, const uint32_t* __restrict__ hists,
                                                    const int64_t* __restrict__ off,
                                                    Cut* __restrict__ cuts,
                                                    int64_t* __restrict__ miss_count) {
  __shared__ uint32_t slots[2][NT / WAVE];
  __shared__ int32_t s_cut[2][3];                     // j*, rem, candidates of bucket j* that stay
  __shared__ uint32_t s_due[2];                       // residents keyed to the iteration
  const int32_t S = st.S;
  const int r0 = threadIdx.x * PER;
  uint32_t res[PER], ahead[PER];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int j = S - (r0 + t);
    res[t] = j >= 0 ? st.rhist[j] : 0u;
    ahead[t] = j > 0 ? hists[j] : 0u;                 // requested an iteration ahead from here on
    if (j == 0) s_due[0] = res[t];
  }
  int64_t n_ahead = off[1] - off[0];
  __syncthreads();
  for (int32_t i = 0; i < S; ++i) {
    const int now = i & 1;
    const int64_t drop = n_ahead - (int64_t)s_due[now];   // the misses: the cache is full
    uint32_t cand[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int j = S - (r0 + t);
      cand[t] = j > i ? res[t] + ahead[t] : 0u;       // (no candidate has a key up to i)
      mine += cand[t];
    }
    if (i + 1 < S) {
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int j = S - (r0 + t);
        ahead[t] = j > i + 1 ? hists[(int64_t)(i + 1) * (S + 1) + j] : 0u;
      }
      n_ahead = off[i + 2] - off[i + 1];
    }
    if (threadIdx.x == 0) {
      s_cut[now][0] = S + 1;
      s_cut[now][1] = 0;
    }
    // exclusive prefix over the threads with one barrier
    const uint32_t inc = wave_inclusive_scan(mine);
    if (lane_id() == WAVE - 1) slots[now][threadIdx.x / WAVE] = inc;
    __syncthreads();
    int64_t before = inc - mine;
    for (int q = 0; q < (int)(threadIdx.x / WAVE); ++q) before += slots[now][q];
    if (drop > 0)
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        if (before <= drop && before + cand[t] > drop) {
          s_cut[now][0] = S - (r0 + t);
          s_cut[now][1] = (int32_t)(drop - before);
          s_cut[now][2] = (int32_t)(cand[t] - (drop - before));
        }
        before += cand[t];
      }
    __syncthreads();
    const int32_t jstar = s_cut[now][0], rem = s_cut[now][1];
    if (threadIdx.x == 0) {
      Cut c{};
      c.jstar = jstar;
      c.rem = rem;
      c.T = -1;
      if (jstar == S) c.n_res = (uint32_t)s_cut[now][2];   // for k_never_parts
      else if (rem > 0) c.T = s_cut[now][2] + rem;         // members of the bucket, for the host
      cuts[i] = c;
      miss_count[i] = drop;
    }
    // R_{i+1}: everything below j* stays, bucket j* loses rem, everything above goes
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int j = S - (r0 + t);
      res[t] = j < jstar ? cand[t] : j == jstar ? cand[t] - (uint32_t)rem : 0u;
      if (j == i + 1) s_due[now ^ 1] = res[t];
    }
    __syncthreads();
  }
}

constexpr int EVICT_TILE = WAVE * WAVE;   // cache lines per tile: 64 flag words of 64 lines

// Set the bit of every member of the selected class in bucket j* (distinct ids in an all-zero bitmap, so
// no atomic needs its result) and count it in its part.  A graph of up to MARK_PARTS parts has only a
// few cache lines of part counts, on which an atomic per member queues up (1 M nodes, 80 k members: 152 us):
// there a block counts in LDS first (8 us).
constexpr int MARK_PARTS = 256;

struct Marker {
  uint32_t *bits, *part, *lds;
  __device__ __forceinline__ void operator()(uint32_t v) const {
    atomicOr(&bits[v >> 5], 1u << (v & 31));
    atomicAdd(lds ? &lds[v >> PART_SHIFT] : &part[v >> PART_SHIFT], 1u);
  }
};

// blocks [0, res_blocks): residents, the next in_blocks blocks: incoming rows; only one
// class is selected, and none when the select runs on the dead rows.
__global__ __launch_bounds__(TB) void k_mark(State st, Iter it, int64_t res_blocks) {
  __shared__ uint32_t s_part[MARK_PARTS];
  const Ctrl c = *st.ctrl;
  const bool residents = (int64_t)blockIdx.x < res_blocks;
  if (c.use_dead || (residents ? c.mode_res : c.mode_in) != MODE_SELECT) return;   // uniform
  const bool in_lds = st.parts <= MARK_PARTS;
  const Marker mark{residents ? st.bitmap : st.bitmap_in, residents ? st.sel_part : st.sel_part_in,
                    in_lds ? s_part : nullptr};
  for (int x = threadIdx.x; x < MARK_PARTS; x += TB) s_part[x] = 0;
  __syncthreads();
  if (residents) {
    const int64_t base = (int64_t)blockIdx.x * (TB * MARK_ITEMS);
#pragma unroll
    for (int t = 0; t < MARK_ITEMS; ++t) {
      const int64_t s = base + t * TB + threadIdx.x;
      if (s < st.cap && st.res_next[s] == c.jstar) mark((uint32_t)st.res_id[s]);
    }
  } else {
    const int64_t base = ((int64_t)blockIdx.x - res_blocks) * (TB * MARK_ITEMS);
#pragma unroll
    for (int t = 0; t < MARK_ITEMS; ++t) {
      const int64_t p = base + t * TB + threadIdx.x;
      if (p < it.n && st.acc_line[p] < 0 && key_of(it, p) == c.jstar) mark((uint32_t)it.ids[p]);
    }
  }
  __syncthreads();
  if (in_lds)
    for (int x = threadIdx.x; x < st.parts; x += TB)
      if (s_part[x]) atomicAdd(&mark.part[x], s_part[x]);
}

// Large caches, evictions among the dead residents only (the usual case once a cache is
// full): the evicted rows are the set bits above T of the standing dead-row bitmap, a short
// stretch at its upper end, so they are found from there and their lines flagged through
// the address table, instead of reading the key and id of every cache line.  The flag
// words are all zero when the phase starts (the emit phase clears what it consumes), the
// tile counts were zeroed by k_threshold; the bits above T leave the bitmap here.
__device__ void p_dead_scatter(const State& st, const Ctrl& c, int64_t vb, int64_t vblocks) {
  // the stretch above T is short as a rule, so a small grid strides over it from T's word on
  const int64_t t_word = c.T < 0 ? 0 : c.T >> 5;   // T = -1: every dead row goes
  for (int64_t w = t_word + vb * TB + threadIdx.x; w < st.words; w += vblocks * TB) {
    const uint32_t all = st.dead_bits[w];
    uint32_t bits = all;
    if (c.T >= 0 && w == t_word) bits &= (c.T & 31) == 31 ? 0u : ~((2u << (c.T & 31)) - 1u);
    if (!bits) continue;
    st.dead_bits[w] = all & ~bits;
    while (bits) {
      const int32_t v = (int32_t)(w * 32 + (__ffs(bits) - 1));
      bits &= bits - 1;
      const int32_t line = st.addr[v];   // a dead row is resident, so this is its line
      if (line >= 0) {
        atomicOr((unsigned long long*)&st.evict_words[line >> 6], 1ull << (line & 63));
        atomicAdd(&st.evict_tiles[line / EVICT_TILE], 1u);
      }
    }
  }
}

__device__ __forceinline__ bool evicts(const Ctrl& c, int32_t next, int32_t id) {
  return next > c.jstar || (next == c.jstar && c.mode_res == MODE_SELECT && id > c.T);
}

__device__ __forceinline__ bool inserts(const Ctrl& c, int32_t next, int32_t id) {
  return next < c.jstar ||
         (next == c.jstar && (c.mode_in == MODE_ALL || (c.mode_in == MODE_SELECT && id <= c.T)));
}

// Eviction flags of one tile of cache lines.  A wave reads 64 consecutive lines at a time
// (coalesced) and its ballot is a 64-bit flag word; the four waves of the block share the
// tile's 64 words.  The tile's total goes to evict_tiles.  Residents that marked themselves
// for the select take their word of the scratch bitmap back to zero.
__device__ void p_evict_flags(const State& st, const Ctrl& c, int64_t vb) {
  __shared__ uint32_t red[TB / WAVE];
  constexpr int PER_WAVE = WAVE / (TB / WAVE);
  const int64_t first_word = vb * WAVE + (threadIdx.x / WAVE) * PER_WAVE;
  const bool unmark = c.marked & MARKED_RES;
  // all keys of the wave's 16 x 64 lines first, so that the loads are in flight together;
  // a line beyond the end repeats line 0 and is masked out below
  int32_t next[PER_WAVE];
#pragma unroll
  for (int g = 0; g < PER_WAVE; ++g) {
    const int64_t line = (first_word + g) * WAVE + lane_id();
    next[g] = st.res_next[line < st.cap ? line : 0];
  }
  uint32_t cnt = 0;
#pragma unroll
  for (int g = 0; g < PER_WAVE; ++g) {
    const int64_t line = (first_word + g) * WAVE + lane_id();
    bool out = false;
    if (line < st.cap && next[g] >= c.jstar) {   // the common case needs no look at the node id
      const int32_t id = st.res_id[line];
      out = evicts(c, next[g], id);
      if (unmark && next[g] == c.jstar) st.bitmap[(uint32_t)id >> 5] = 0;
    }
    const uint64_t word = __ballot(out);
    if ((first_word + g) * WAVE < st.cap && lane_id() == 0) {
      st.evict_words[first_word + g] = word;
      cnt += __popcll(word);
    }
  }
  const uint32_t total = block_sum_u32(cnt, red);
  if (threadIdx.x == 0) st.evict_tiles[vb] = total;
}

constexpr int IN_ITEMS = 8;        // accesses per thread in the insertion phases

// Insertions per tile of TB*IN_ITEMS accesses; incoming rows that marked themselves for the
// select take their word of the scratch bitmap back to zero.
__device__ void p_in_count(const State& st, const Ctrl& c, const Iter& it, int64_t vb) {
  __shared__ uint32_t red[TB / WAVE];
  const int64_t base = (vb * TB + threadIdx.x) * IN_ITEMS;
  const bool unmark = c.marked & MARKED_IN;
  // line, key and id of all items first (an item beyond the end repeats item 0 of the
  // iteration and is not counted)
  int32_t line[IN_ITEMS], key[IN_ITEMS], v[IN_ITEMS];
#pragma unroll
  for (int t = 0; t < IN_ITEMS; ++t) {
    const int64_t p = base + t < it.n ? base + t : 0;
    line[t] = st.acc_line[p];
    key[t] = key_of(it, p);
    v[t] = it.ids[p];
  }
  uint32_t cnt = 0;
#pragma unroll
  for (int t = 0; t < IN_ITEMS; ++t)
    if (base + t < it.n && line[t] < 0 && key[t] <= c.jstar) {
      cnt += inserts(c, key[t], v[t]);
      if (unmark && key[t] == c.jstar) st.bitmap_in[(uint32_t)v[t] >> 5] = 0;
    }
  const uint32_t total = block_sum_u32(cnt, red);
  if (threadIdx.x == 0) st.in_tiles[vb] = total;
}

// blocks [0, evict_tiles): eviction flags and counts per tile, by a pass over the tile's lines
// or, dead rows of a large cache, by the scatter from the bitmap (the blocks then stride over
// the stretch above T); the next in_tiles blocks: insertions per tile; one more block takes
// the part counts of the scratch bitmap back to zero.
__global__ __launch_bounds__(TB) void k_flags(State st, Iter it, int64_t evict_tiles,
                                              int64_t in_tiles) {
  const Ctrl c = *st.ctrl;
  const int64_t vb = blockIdx.x;
  if (vb < evict_tiles) {
    if (st.dead_scatter && c.use_dead) {
      if (c.n_change > 0) p_dead_scatter(st, c, vb, evict_tiles);
    } else if (c.n_change > 0 || (c.marked & MARKED_RES)) {
      p_evict_flags(st, c, vb);
    }
  } else if (vb < evict_tiles + in_tiles) {
    if (c.n_change > 0 || (c.marked & MARKED_IN)) p_in_count(st, c, it, vb - evict_tiles);
  } else {
    if (c.marked & MARKED_RES)
      for (int64_t q = threadIdx.x; q < st.parts; q += TB) st.sel_part[q] = 0;
    if (c.marked & MARKED_IN)
      for (int64_t q = threadIdx.x; q < st.parts; q += TB) st.sel_part_in[q] = 0;
  }
}

// ---- the last phase: lists and the state of C_{i+1} ----------------------------------------
//
// The t-th insertion takes the line of the t-th eviction.  The two sides compute their ranks
// independently; they meet in pair[t], one 64-bit word (iteration tag, side, line or
// position) that each side swaps in atomically: the side that finds the other's word there
// knows line and position and writes the line's new state.  Everything that crosses from one
// block to another travels inside that word, so no fence is needed; the state arrays are
// read by the next launch.
constexpr uint64_t PAIR_EVICT = 1ull << 39;

__device__ __forceinline__ uint64_t pair_tag(int32_t i) { return (uint64_t)(i + 1) << 40; }

__device__ __forceinline__ void finish_line(const State& st, int32_t line, int32_t v, int32_t key) {
  st.res_id[line] = v;
  st.res_next[line] = key;
  st.addr[v] = line;
}

// One wave per tile of 64 flag words: the evicted lines in line order.  The tile's set bits
// are dealt to the lanes round-robin by rank (lane l takes the l-th, (l+64)-th ... set bit,
// located through the wave's running popcounts), so that the chain of dependent memory
// operations behind every eviction is as long for a clustered tile as for an even one.
// A small cache has few tiles, and under LRU an iteration may evict most of their lines: `split` waves
// (a multiple of a block's) share a tile there, so that a wave has a few rounds to go instead of up to 64
// (k_emit_pair on 104 857 lines, 28 k changes an iteration: 53 us with one wave per tile, 10 us with 16).
__device__ void p_evict_emit(const State& st, const Ctrl& c, const Iter& it, const Outputs& o,
                             int64_t vb, int64_t tiles, int32_t split) {
  __shared__ uint32_t red[TB / WAVE];
  constexpr int TPB = TB / WAVE;                 // tiles per block, or waves of one tile
  const int64_t first_tile = vb * TPB / split;
  const int w = split == 1 ? threadIdx.x / WAVE : 0;
  const uint32_t share = split == 1 ? 0u : (uint32_t)((vb * TPB + threadIdx.x / WAVE) % split);
  const int64_t tile = first_tile + w;
  // the block's own tiles first: most blocks of a large cache have nothing to emit
  uint32_t own[TPB];
  uint32_t any = 0;
#pragma unroll
  for (int k = 0; k < TPB; ++k) {
    own[k] = first_tile + k < tiles && (split == 1 || k == 0) ? st.evict_tiles[first_tile + k] : 0;
    any |= own[k];
  }
  if (!any) return;                              // uniform over the block
  const int64_t word_at = tile * WAVE + lane_id();
  const uint64_t word = tile < tiles && word_at * WAVE < st.cap ? st.evict_words[word_at] : 0;
  uint32_t tile_base = block_prefix_of(st.evict_tiles, first_tile, red);
#pragma unroll
  for (int k = 0; k < TPB; ++k)
    if (k < w) tile_base += own[k];
  if (tile >= tiles) return;                     // uniform over the wave
  const bool scattered = st.dead_scatter && c.use_dead;
  if (st.dead_scatter && word) st.evict_words[word_at] = 0;   // consumed: zero for the next scatter
  const uint32_t mine = (uint32_t)__popcll(word);
  const uint32_t incl = wave_inclusive_scan(mine);
  const uint32_t total = of_lane(incl, WAVE - 1);
  const int64_t dst = o.cs_offsets[it.i];
  const uint64_t tag = pair_tag(it.i);
  for (uint32_t k0 = share * WAVE; k0 < total; k0 += split * WAVE) {   // uniform trip count: shuffles inside
    const uint32_t k = k0 + lane_id();
    int lo = 0, hi = WAVE - 1;                   // the first word whose running count exceeds k
#pragma unroll
    for (int step = 0; step < 6; ++step) {
      const int mid = (lo + hi) >> 1;
      if (__shfl(incl, mid, WAVE) > k) hi = mid; else lo = mid + 1;
    }
    const int j = lo < WAVE ? lo : WAVE - 1;
    uint64_t bits = shfl_u64(word, j);
    const uint32_t before = __shfl(incl, j, WAVE) - __shfl(mine, j, WAVE);
    if (k >= total) continue;
    for (uint32_t r = k - before; r > 0; --r) bits &= bits - 1;
    const int32_t line = (int32_t)((tile * WAVE + j) * WAVE + (__ffsll((unsigned long long)bits) - 1));
    const uint32_t at = tile_base + k;
    const int32_t gone = st.res_id[line];
    const int32_t key = st.res_next[line];
    if (dst + at < o.cs_capacity) o.out_ids[dst + at] = gone;
    st.addr[gone] = -1;
    if (key == st.S && !st.lru && !scattered) {   // a dead resident leaves the standing bitmap
      atomicAnd(&st.dead_bits[(uint32_t)gone >> 5], ~(1u << ((uint32_t)gone & 31)));
      // (its part count was rewritten by k_threshold when the dead rows were selected from)
      if (!c.use_dead) atomicSub(&st.dead_part[(uint32_t)gone >> PART_SHIFT], 1u);
    }
    if (at < st.max_change) {
      // the reads of this line's old state are complete (their values were used above)
      // before the word is swapped in: from then on the other side may rewrite the line
      __asm__ volatile("" ::: "memory");
      const uint64_t other = atomicExch((unsigned long long*)&st.pair[at],
                                        tag | PAIR_EVICT | (uint32_t)line);
      if ((other & ~((1ull << 40) - 1)) == tag) {
        const int64_t p = (int64_t)(other & 0xFFFFFFFFull);
        finish_line(st, line, it.ids[p], key_of(it, p));
      }
    }
  }
}

// The inserted positions of one tile of accesses in position order; the block's insertions
// are first gathered in LDS by rank and then dealt one to a thread, for the same reason as
// above.
__device__ void p_in_emit(const State& st, const Ctrl& c, const Iter& it, const Outputs& o,
                          int64_t vb) {
  __shared__ uint32_t smem[TB / WAVE + 1];
  __shared__ uint32_t red[TB / WAVE];
  __shared__ int32_t s_pos[TB * IN_ITEMS];
  if (st.in_tiles[vb] == 0) return;              // uniform over the block
  const int64_t base = (vb * TB + threadIdx.x) * IN_ITEMS;
  uint32_t flags = 0, cnt = 0;
  int32_t v[IN_ITEMS], key[IN_ITEMS], line[IN_ITEMS];
#pragma unroll
  for (int t = 0; t < IN_ITEMS; ++t) {
    const int64_t p = base + t < it.n ? base + t : 0;
    line[t] = st.acc_line[p];
    key[t] = key_of(it, p);
    v[t] = it.ids[p];
  }
#pragma unroll
  for (int t = 0; t < IN_ITEMS; ++t)
    if (base + t < it.n && line[t] < 0 && inserts(c, key[t], v[t])) {
      flags |= 1u << t;
      ++cnt;
    }
  uint32_t total;
  uint32_t rank = block_exclusive_scan<uint32_t, TB>(cnt, smem, total);
  const uint32_t tile_base = block_prefix_of(st.in_tiles, vb, red);
#pragma unroll
  for (int t = 0; t < IN_ITEMS; ++t)
    if (flags >> t & 1) s_pos[rank++] = threadIdx.x * IN_ITEMS + t;   // position inside the tile
  __syncthreads();
  const int64_t dst = o.cs_offsets[it.i];
  const uint64_t tag = pair_tag(it.i);
  const int64_t tile_first = vb * (int64_t)(TB * IN_ITEMS);
  for (uint32_t k = threadIdx.x; k < total; k += TB) {
    const int64_t p = tile_first + s_pos[k];
    const uint32_t at = tile_base + k;
    const int32_t id = it.ids[p];
    const int32_t nk = key_of(it, p);
    if (dst + at < o.cs_capacity) {
      o.in_ids[dst + at] = id;
      o.in_positions[dst + at] = (int32_t)p;
    }
    if (at < st.max_change) {
      const uint64_t other = atomicExch((unsigned long long*)&st.pair[at], tag | (uint32_t)p);
      if ((other & ~((1ull << 40) - 1)) == tag)
        finish_line(st, (int32_t)(other & 0xFFFFFFFFull), id, nk);
    }
  }
}

__global__ __launch_bounds__(TB) void k_emit_pair(State st, Iter it, Outputs o, int64_t evict_tiles,
                                                  int64_t evict_blocks, int32_t split) {
  const Ctrl c = *st.ctrl;
  if (c.n_change <= 0) return;
  if ((int64_t)blockIdx.x < evict_blocks) p_evict_emit(st, c, it, o, blockIdx.x, evict_tiles, split);
  else p_in_emit(st, c, it, o, blockIdx.x - evict_blocks);
}

// popcount of one part of a bitmap (the part counts of the dead-row bitmap after a resumed
// superbatch's start state has been marked)
__global__ __launch_bounds__(TB) void k_part_count(const uint32_t* __restrict__ bits, int64_t words,
                                                   uint32_t* __restrict__ part) {
  __shared__ uint32_t red[TB / WAVE];
  const int64_t base = (int64_t)blockIdx.x * PART_WORDS;
  uint32_t cnt = 0;
  for (int t = threadIdx.x; t < PART_WORDS; t += TB)
    if (base + t < words) cnt += __popc(bits[base + t]);
  const uint32_t total = block_sum_u32(cnt, red);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// ---- part 3 without a loop over the state: a carried cache that holds the whole superbatch ----
//
// When the carried cache has a line for every distinct row of the superbatch, an iteration
// never evicts a row that is still needed (the live candidates alone never exceed the
// capacity), so:
//   * hits and misses are known up front: an access misses iff it is the first access of a row
//     the start state does not hold; it is inserted iff the row is accessed again later
//     (otherwise it ranks behind every resident and bypasses the cache);
//   * a row keeps one line for the whole superbatch, the start line or the one it is given;
//   * iteration i evicts the n_i dead residents with the largest ids, n_i = its insertions,
//     where a resident is dead once its last access has passed (or from the start).
// The insertion lists are therefore a compaction over all accesses, and only the choice of
// the evicted rows is sequential.  All of them lie at the upper end of the id space: with M
// evictions in total, none has an id below lo_id, the M-th largest id among the rows that are
// dead from the start (they alone would supply M victims, and later arrivals only raise the
// thresholds).  The rows from lo_id up that are ever dead residents (the M rows dead from the
// start, and the rows that die during the superbatch: a few thousand, however wide that id
// range has become) are the candidates; they are numbered in id order, and which iteration evicts
// which of them, and from which line, follows for all iterations together (victims.hpp).
// What the path cannot take (more than PLAN_CAND_MAX candidates, an iteration with more than
// PLAN_SORT_MAX insertions, S above PLAN_S_MAX, fewer rows dead from the start than
// insertions) goes the way of any other cache (stays.hpp, or the loop above).
constexpr int PLAN_CAND_WORDS = 16384;              // words of a bitmap ...
constexpr int PLAN_CAND_MAX = PLAN_CAND_WORDS * 32; // ... over at most 524 288 candidates
constexpr int PLAN_SORT_MAX = 4096;      // evictions of one iteration that are ordered in LDS
constexpr int PLAN_RANK_DIRECT = 256;    // up to here every eviction is compared with every other
constexpr int PLAN_S_MAX = 2048;         // iterations (LDS histograms of k_plan_heads)
enum { PLAN_M = 0, PLAN_MAX_N = 1, PLAN_LO_ID = 2, PLAN_DEAD = 3, PLAN_TAIL = 4, PLAN_FAILED = 5,
       PLAN_WHERE = 6, PLAN_CANDS = 7, PLAN_FULLEST = 8, PLAN_SCALARS = 9 };

struct Plan {
  uint32_t* ins_bits;    // [ceil(total / 32)] bit p: access p (flat position) is an insertion
  uint32_t* ins_tiles;   // insertions per tile of TB words, then their exclusive scan
  uint32_t* ins_base;    // [ceil(total / 32)] insertions in front of each word (tiles that have any)
  int32_t* ins_cand;     // [distinct rows] candidate number of each inserted row, -1 = not one
  int64_t* scalars;      // [PLAN_SCALARS]
  uint32_t* cand_tiles;  // candidates per tile of TB words of the id bitmap, then their scan
  uint32_t* cand_base;   // [words] candidates in front of each word of the id bitmap (from lo_id's word on)
  int32_t* cand_id;      // [PLAN_CAND_MAX] candidates in id order
  int32_t* cand_line;    // [PLAN_CAND_MAX] their cache line, -1 while not resident
  uint32_t* cand_dead;   // [PLAN_CAND_WORDS] bit c: candidate c is dead from the start
  uint32_t* arr_off;     // [S + 2] candidates that die in iteration d: count at d + 1, then offsets
  uint32_t* arr_cur;     // [S + 1] fill cursors
  int32_t* arr_cand;     // [PLAN_CAND_MAX] their numbers, grouped by iteration; then the evicted ones (victims.hpp)
  int64_t ins_words, ins_tile_count, cand_tile_count;
};

// Pass over the node-sorted accesses: the head of a run is the row's first access.  If the
// start state does not hold the row, that access misses, and it is an insertion if the run
// goes on.  Misses per iteration go to miss_count, insertions per iteration to
// cs_offsets[i + 1] (scanned afterwards) and to the bitmap over positions.
// (Large blocks, two to a CU: every block adds its counts to the same few lines in the end, 0.2 G/s for each of them.  A wave
// takes LOOK_ITEMS * 64 consecutive pairs and passes ids on to the neighbours.  33 M pairs, 200 iterations: 1 024 blocks
// of 256, each pair read three times, 170 us, this 146)
constexpr int64_t PLAN_HEADS_TILE = BIG * LOOK_ITEMS, PLAN_HEADS_BLOCKS = 512;
__global__ __launch_bounds__(BIG) void k_plan_heads(const uint64_t* __restrict__ sorted, int64_t n,
                                                    const int64_t* __restrict__ off, int32_t S,
                                                    const uint32_t* __restrict__ held,
                                                    int32_t* __restrict__ addr,
                                                    uint32_t* __restrict__ ins_bits,
                                                    unsigned long long* __restrict__ miss_count,
                                                    unsigned long long* __restrict__ cs_offsets) {
  extern __shared__ int32_t lds_plan[];   // offsets [S+1], misses [S], insertions [S]
  int32_t* lds_off = lds_plan;
  uint32_t* h_miss = reinterpret_cast<uint32_t*>(lds_plan + S + 1);
  uint32_t* h_ins = h_miss + S;
  for (int j = threadIdx.x; j < 2 * S; j += BIG) h_miss[j] = 0;
  load_offsets(lds_off, off, S);
  const int lane = lane_id();
  for (int64_t base = blockIdx.x * PLAN_HEADS_TILE + threadIdx.x / WAVE * (WAVE * LOOK_ITEMS); base < n;
       base += gridDim.x * PLAN_HEADS_TILE) {     // uniform over the wave
    // all pairs first, then the words that say which rows are held, so that the reads of a kind are in flight
    // together (with a wait for every such word, inside a branch, 270 us for 33 M pairs instead of 147)
    uint64_t here[LOOK_ITEMS + 1];
#pragma unroll
    for (int i = 0; i <= LOOK_ITEMS; ++i) {
      const int64_t j = base + i * WAVE + (i < LOOK_ITEMS ? lane : 0);
      here[i] = sorted[j < n ? j : n - 1];
    }
    uint32_t before = (uint32_t)(sorted[base > 0 ? base - 1 : 0] >> 32);
    uint32_t word[LOOK_ITEMS], head = 0, more = 0;   // bit i: item i
#pragma unroll
    for (int i = 0; i < LOOK_ITEMS; ++i) {
      const int64_t j = base + i * WAVE + lane;
      const uint32_t v = (uint32_t)(here[i] >> 32);
      uint32_t left = from_left(v), right = from_right(v);
      const uint32_t next = of_lane((uint32_t)(here[i + 1] >> 32), 0);
      if (lane == 0) left = before;
      if (lane == WAVE - 1) right = next;
      before = of_lane(v, WAVE - 1);
      head |= (j < n && (j == 0 || left != v) ? 1u : 0u) << i;
      more |= (j + 1 < n && right == v ? 1u : 0u) << i;
    }
#pragma unroll
    for (int i = 0; i < LOOK_ITEMS; ++i) word[i] = held[head >> i & 1u ? (uint32_t)(here[i] >> 32) >> 5 : 0u];
#pragma unroll
    for (int i = 0; i < LOOK_ITEMS; ++i) {
      const uint32_t v = (uint32_t)(here[i] >> 32);
      if (!(head >> i & 1u) || (word[i] >> (v & 31) & 1u)) continue;   // not the head of a run, or held
      addr[v] = -1;                       // (until it is inserted, if it is)
      const int32_t p = (int32_t)(uint32_t)here[i];
      const int32_t it = iter_of(lds_off, S, p);
      atomicAdd(&h_miss[it], 1u);
      if (more >> i & 1u) {
        atomicAdd(&h_ins[it], 1u);
        atomicOr(&ins_bits[p >> 5], 1u << (p & 31));
      }
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < S; j += BIG) {
    if (h_miss[j]) atomicAdd(&miss_count[j], (unsigned long long)h_miss[j]);
    if (h_ins[j]) atomicAdd(&cs_offsets[j + 1], (unsigned long long)h_ins[j]);
  }
}

// One block: cs_offsets from the insertion counts, their total M and maximum, the number of
// rows that are dead from the start, lo_id (num_nodes when nothing is evicted, -1 when the
// rows dead from the start are fewer than M) and the first sorted access of a row >= lo_id.
__global__ __launch_bounds__(BIG) void k_plan_scan(State st, const uint64_t* __restrict__ sorted,
                                                   int64_t n, int64_t* __restrict__ cs_offsets,
                                                   int64_t* __restrict__ scalars) {
  __shared__ int64_t smem[BIG / WAVE + 1];
  const int32_t S = st.S;
  const int32_t per = (S + BIG - 1) / BIG;
  const int32_t j0 = threadIdx.x * per;
  int64_t mine = 0, largest = 0;
  for (int32_t j = j0; j < j0 + per && j < S; ++j) {
    const int64_t c = cs_offsets[j + 1];
    mine += c;
    largest = c > largest ? c : largest;
  }
  int64_t M;
  int64_t run = block_exclusive_scan<int64_t, BIG>(mine, smem, M);
  for (int32_t j = j0; j < j0 + per && j < S; ++j) {
    run += cs_offsets[j + 1];
    cs_offsets[j + 1] = run;
  }
  // the largest count: waves first, then thread 0 over the waves
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) {
    const int64_t o = __shfl_xor(largest, d, WAVE);
    largest = o > largest ? o : largest;
  }
  if (lane_id() == 0) smem[threadIdx.x / WAVE] = largest;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t m = 0;
    for (int w = 0; w < BIG / WAVE; ++w) m = smem[w] > m ? smem[w] : m;
    scalars[PLAN_MAX_N] = m;
    scalars[PLAN_M] = M;
    scalars[PLAN_FAILED] = 0;
    scalars[PLAN_WHERE] = 0;
  }
  __syncthreads();
  const int64_t pper = (st.parts + BIG - 1) / BIG;
  int64_t dead_mine = 0;
  for (int64_t q = threadIdx.x * pper; q < (threadIdx.x + 1) * pper && q < st.parts; ++q)
    dead_mine += st.dead_part[q];
  int64_t dead;
  block_exclusive_scan<int64_t, BIG>(dead_mine, smem, dead);
  int32_t lo_id = (int32_t)st.num_nodes;
  if (M >= 1)   // uniform
    lo_id = dead >= M ? p_kth_set_bit<BIG>(st.dead_bits, st.dead_part, st.parts, st.words,
                                            dead - M + 1, false)
                      : -1;
  if (threadIdx.x == 0) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if ((int64_t)(sorted[mid] >> 32) < (int64_t)lo_id) lo = mid + 1; else hi = mid;
    }
    scalars[PLAN_TAIL] = lo;
    scalars[PLAN_LO_ID] = lo_id;
    scalars[PLAN_DEAD] = dead;
  }
}

// set bits per tile of TB words, and a zero behind them (where the scan leaves their sum)
__global__ __launch_bounds__(TB) void k_bit_tiles(const uint32_t* __restrict__ bits, int64_t words,
                                                  uint32_t* __restrict__ tiles) {
  __shared__ uint32_t red[TB / WAVE];
  const int64_t w = (int64_t)blockIdx.x * TB + threadIdx.x;
  const uint32_t total = block_sum_u32(w < words ? (uint32_t)__popc(bits[w]) : 0u, red);
  if (threadIdx.x == 0) tiles[blockIdx.x] = total;
  if (threadIdx.x == 0 && blockIdx.x == 0) tiles[gridDim.x] = 0;
}

constexpr uint32_t INS_DENSE = TB * 4;     // insertions of a tile of TB words

// in_ids / in_positions of the whole superbatch: the set bits of ins_bits in position order
// (iterations are consecutive stretches of positions, so this is iteration by iteration and
// inside an iteration by position, as the lists are defined).
__global__ __launch_bounds__(TB) void k_ins_emit(const uint32_t* __restrict__ bits, int64_t words,
                                                 const uint32_t* __restrict__ tile_base,
                                                 const int32_t* __restrict__ ids,
                                                 const int64_t* __restrict__ off, int32_t S,
                                                 int32_t* __restrict__ in_ids,
                                                 int32_t* __restrict__ in_positions,
                                                 uint32_t* __restrict__ ins_base,
                                                 uint64_t* __restrict__ ins_pairs,
                                                 int32_t* __restrict__ ins_cand) {
  extern __shared__ int32_t lds_off[];
  __shared__ uint32_t smem[TB / WAVE + 1];
  const uint32_t first = tile_base[blockIdx.x];
  if (tile_base[blockIdx.x + 1] == first) return;   // nothing in this tile (uniform)
  load_offsets(lds_off, off, S);
  const int64_t w = (int64_t)blockIdx.x * TB + threadIdx.x;
  uint32_t word = w < words ? bits[w] : 0u;
  uint32_t total;
  uint32_t rank = first + block_exclusive_scan<uint32_t, TB>((uint32_t)__popc(word), smem, total);
  if (w < words && ins_pairs) ins_pairs[w] = (uint64_t)rank << 32 | word;   // (see InsIndex)
  if (w < words && !ins_pairs) ins_base[w] = rank;
  if (total > INS_DENSE) {   // uniform
    // many of a word's bits are set: a position to a thread, so that neighbours write side by side (LRU of
    // 24 x 800 000 accesses, nearly all inserted: 50 us, a word to a thread 550)
    __shared__ uint32_t s_word[TB], s_rank[TB];
    __shared__ uint16_t s_iter[TB];                    // of the word's first position
    s_word[threadIdx.x] = word;
    s_rank[threadIdx.x] = rank;
    s_iter[threadIdx.x] = (uint16_t)(word ? iter_of(lds_off, S, (int32_t)(w * 32)) : 0);
    __syncthreads();
    const int64_t p0 = (int64_t)blockIdx.x * TB * 32;
    constexpr int ITEMS = 8;                           // reads in flight
    for (int x0 = threadIdx.x; x0 < TB * 32; x0 += TB * ITEMS) {
      int32_t v[ITEMS];
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const int x = x0 + k * TB;
        v[k] = s_word[x >> 5] >> (x & 31) & 1u ? ids[p0 + x] : 0;   // (positions behind the last one have no bit)
      }
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const int x = x0 + k * TB;
        const uint32_t bits_here = s_word[x >> 5];
        if (!(bits_here >> (x & 31) & 1u)) continue;
        const int32_t p = (int32_t)(p0 + x);
        const uint32_t at = s_rank[x >> 5] + __popc(bits_here & ((1u << (x & 31)) - 1u));
        int32_t i = s_iter[x >> 5];
        while (i + 1 < S && lds_off[i + 1] <= p) ++i;
        in_ids[at] = v[k];
        in_positions[at] = p - lds_off[i];
        if (ins_cand) ins_cand[at] = -1;
      }
    }
    return;
  }
  int32_t i = word ? iter_of(lds_off, S, (int32_t)(w * 32)) : 0;
  while (word) {
    const int32_t p = (int32_t)(w * 32 + (__ffs(word) - 1));
    word &= word - 1;
    while (i + 1 < S && lds_off[i + 1] <= p) ++i;
    in_ids[rank] = ids[p];
    in_positions[rank] = p - lds_off[i];
    if (ins_cand) ins_cand[rank] = -1;
    ++rank;
  }
}

// src_line of the insertions: their row arrives with this access
__global__ __launch_bounds__(TB) void k_ins_lines(const uint32_t* __restrict__ bits, int64_t words,
                                                  int32_t* __restrict__ src_line) {
  const int64_t w = (int64_t)blockIdx.x * TB + threadIdx.x;
  uint32_t word = w < words ? bits[w] : 0u;
  while (word) {
    src_line[w * 32 + (__ffs(word) - 1)] = -1;
    word &= word - 1;
  }
}

// The id bitmap of the candidates, from lo_id's word on: first the rows dead from the start ...
// (lo_id comes from the device-side scalars: this and the next two kernels run before the host
// has read them, so that the host learns the exact number of candidates with the same copy)
__global__ __launch_bounds__(TB) void k_cand_start(const uint32_t* __restrict__ dead_bits,
                                                   int64_t words, int64_t num_nodes,
                                                   const int64_t* __restrict__ scalars,
                                                   uint32_t* __restrict__ cand_bits) {
  const int64_t lo_id = scalars[PLAN_LO_ID];
  if (lo_id < 0 || lo_id >= num_nodes) return;      // nothing is evicted, or this path is not taken
  const int64_t span = (int64_t)gridDim.x * TB;
  for (int64_t w = (lo_id >> 5) + (int64_t)blockIdx.x * TB + threadIdx.x; w < words; w += span) {
    uint32_t word = dead_bits[w];
    if (w == (lo_id >> 5)) word &= ~((1u << (lo_id & 31)) - 1u);
    cand_bits[w] = word;
  }
}

// Is sorted[j] the last access of a row that is resident when it dies?  (A row the start state
// does not hold is resident only if it was inserted, that is, if it has an earlier access.)
__device__ __forceinline__ bool plan_arrival(const uint64_t* __restrict__ sorted, int64_t n,
                                             int64_t j, const uint32_t* __restrict__ held,
                                             const int32_t* off, int32_t S,
                                             int32_t& v, int32_t& d, bool& inserted) {
  const uint64_t cur = sorted[j];
  v = (int32_t)(cur >> 32);
  if (j + 1 < n && (int32_t)(sorted[j + 1] >> 32) == v) return false;
  const bool earlier = j > 0 && (int32_t)(sorted[j - 1] >> 32) == v;
  inserted = !(held[(uint32_t)v >> 5] >> (v & 31) & 1u);
  if (!earlier && inserted) return false;
  d = iter_of(off, S, (int32_t)(cur & 0xFFFFFFFFu));
  return true;
}

// ... then (PLACE = false) the rows >= lo_id that die during the superbatch, counted per
// iteration at arr_off[d + 1].  PLACE = true, after the candidates are numbered: their numbers
// go to arr_cand at the cursors, d to `when`, and a row that is inserted during this call leaves its number
// with its insertion record (with arr_ids, the rows themselves go there instead, and nothing
// else is written).  A block works on one stretch of the sorted pairs and counts
// per iteration in LDS first, so that the counters and cursors in global memory, a few
// addresses that every arrival would otherwise meet at, see one atomic per block and iteration.
// lds: S + 1 offsets, S counters.
template <bool PLACE>
__global__ __launch_bounds__(TB) void k_plan_arrivals(const uint64_t* __restrict__ sorted, int64_t n,
                                                      const int64_t* __restrict__ scalars,
                                                      const uint32_t* __restrict__ held,
                                                      const int64_t* __restrict__ off, int32_t S,
                                                      uint32_t* __restrict__ cand_bits,
                                                      const uint32_t* __restrict__ cand_base,
                                                      int64_t num_nodes, Plan pl, int32_t* __restrict__ when,
                                                      int32_t* __restrict__ arr_ids) {
  extern __shared__ int32_t lds_off[];
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(lds_off + S + 1);
  const int64_t lo_id = scalars[PLAN_LO_ID];
  if (lo_id < 0 || lo_id >= num_nodes) return;
  for (int d = threadIdx.x; d < S; d += TB) s_cnt[d] = 0;
  load_offsets(lds_off, off, S);
  const int64_t lo_word = lo_id >> 5;
  const int64_t tail = scalars[PLAN_TAIL];
  const int64_t per = (((n - tail + gridDim.x - 1) / gridDim.x + TB - 1) / TB) * TB;
  const int64_t first = tail + (int64_t)blockIdx.x * per;
  const int64_t last = first + per < n ? first + per : n;
  for (int64_t j = first + threadIdx.x; j < last; j += TB) {
    int32_t v, d;
    bool inserted;
    if (!plan_arrival(sorted, n, j, held, lds_off, S, v, d, inserted)) continue;
    if (!PLACE) atomicOr(&cand_bits[(uint32_t)v >> 5], 1u << (v & 31));
    atomicAdd(&s_cnt[d], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < S; d += TB) {
    const uint32_t c = s_cnt[d];
    if (!PLACE) {
      if (c) atomicAdd(&pl.arr_off[d + 1], c);
    } else {
      s_cnt[d] = c ? atomicAdd(&pl.arr_cur[d], c) : 0u;   // the block's places in the iteration's list
    }
  }
  if (!PLACE) return;
  __syncthreads();
  for (int64_t j = first + threadIdx.x; j < last; j += TB) {
    int32_t v, d;
    bool inserted;
    if (!plan_arrival(sorted, n, j, held, lds_off, S, v, d, inserted)) continue;
    if (arr_ids) {                                   // the stepped path wants the rows themselves
      arr_ids[atomicAdd(&s_cnt[d], 1u)] = v;
      continue;
    }
    const uint32_t below = (1u << (v & 31)) - 1u;
    const uint32_t c = cand_base[((uint32_t)v >> 5) - lo_word] + __popc(cand_bits[(uint32_t)v >> 5] & below);
    // (the host takes this path only with at most PLAN_CAND_MAX candidates: c is below that)
    if (c >= (uint32_t)PLAN_CAND_MAX) continue;
    pl.arr_cand[atomicAdd(&s_cnt[d], 1u)] = (int32_t)c;
    when[c] = d;
    if (inserted) {
      int64_t h = j;                                 // the row's first access is its insertion
      while (h > 0 && (int32_t)(sorted[h - 1] >> 32) == v) --h;
      const uint32_t p = (uint32_t)(sorted[h] & 0xFFFFFFFFu);
      pl.ins_cand[pl.ins_base[p >> 5] + __popc(pl.ins_bits[p >> 5] & ((1u << (p & 31)) - 1u))] = (int32_t)c;
    }
  }
}

// Numbers the candidates in id order: cand_base per bitmap word, id, start line (-1 for a row
// that is inserted during this call), the dead-from-the-start flag and, for these, when they die (before iteration
// 0; the others: S until their own is known) per candidate.
__global__ __launch_bounds__(TB) void k_cand_emit(const uint32_t* __restrict__ cand_bits,
                                                  const uint32_t* __restrict__ dead_bits,
                                                  int64_t lo_word, int64_t nwords,
                                                  const uint32_t* __restrict__ tile_base,
                                                  const int32_t* __restrict__ addr, Plan pl,
                                                  int32_t* __restrict__ when, int32_t S) {
  __shared__ uint32_t smem[TB / WAVE + 1];
  const int64_t w = (int64_t)blockIdx.x * TB + threadIdx.x;
  uint32_t word = w < nwords ? cand_bits[lo_word + w] : 0u;
  const uint32_t dead = w < nwords ? dead_bits[lo_word + w] : 0u;
  uint32_t total;
  uint32_t c = tile_base[blockIdx.x] + block_exclusive_scan<uint32_t, TB>((uint32_t)__popc(word), smem, total);
  if (w < nwords) pl.cand_base[w] = c;
  while (word) {
    const int b = __ffs(word) - 1;
    word &= word - 1;
    if (c < (uint32_t)PLAN_CAND_MAX) {
      const int32_t v = (int32_t)((lo_word + w) * 32 + b);
      pl.cand_id[c] = v;
      pl.cand_line[c] = addr[v];
      when[c] = dead >> b & 1 ? 0 : S;
      if (dead >> b & 1) atomicOr(&pl.cand_dead[c >> 5], 1u << (c & 31));
    }
    ++c;
  }
}

// One block: arr_off <- offsets (arr_off[i] .. arr_off[i + 1] are the candidates that die in
// iteration i), arr_cur <- the same, as cursors.
__global__ __launch_bounds__(BIG) void k_plan_arrival_offsets(uint32_t* __restrict__ arr_off,
                                                              uint32_t* __restrict__ arr_cur,
                                                              int32_t S,
                                                              int64_t* __restrict__ scalars) {
  __shared__ uint32_t smem[BIG / WAVE + 1];
  const int32_t per = (S + BIG - 1) / BIG;
  const int32_t j0 = threadIdx.x * per;
  uint32_t mine = 0;
  for (int32_t j = j0; j < j0 + per && j < S; ++j) mine += arr_off[j + 1];
  uint32_t total;
  uint32_t run = block_exclusive_scan<uint32_t, BIG>(mine, smem, total);
  for (int32_t j = j0; j < j0 + per && j < S; ++j) {
    arr_cur[j] = run;
    run += arr_off[j + 1];
    arr_off[j + 1] = run;
  }
  // the candidates: the M rows dead from the start and the rows that die during the superbatch
  if (threadIdx.x == 0) scalars[PLAN_CANDS] = scalars[PLAN_M] + (int64_t)total;
}

#include "victims.hpp"

// ---- the same regime with more candidates or evictions than those arrays hold ------------------
//
// Hits, misses and insertions are known up front as above; the choice of the evicted rows runs
// on the standing bitmap of dead rows in global memory instead, three launches per iteration
// that evicts: k_step_find (one block: the id T above which the iteration's n dead rows lie),
// k_step_scatter (their bits leave the bitmap, their lines are flagged), k_step_emit (the
// flagged lines in line order take the iteration's insertions; other blocks set the bits of the
// rows that die in the next iteration).  No pass touches the accesses.

// The rows of arr_ids[a0, a1) are dead residents from now on.
// (The list of an iteration comes in ascending stretches, so neighbouring lanes mostly fall
// into the same part of the bitmap: the first lane of each run adds the run's length to the
// part's count, instead of one atomic per row on a few hundred addresses.)
__device__ __forceinline__ void step_arrivals(const State& st, const int32_t* __restrict__ arr_ids,
                                              uint32_t a0, uint32_t a1, int64_t vb, int64_t vblocks) {
  const int lane = lane_id();
  for (int64_t first = a0 + vb * TB + (threadIdx.x - lane); first < a1; first += vblocks * TB) {
    const int64_t a = first + lane;                // whole waves stay in the loop together
    const bool valid = a < a1;
    const uint32_t v = valid ? (uint32_t)arr_ids[a] : 0u;
    const uint32_t part = valid ? v >> PART_SHIFT : 0xFFFFFFFFu;
    if (valid) atomicOr(&st.dead_bits[v >> 5], 1u << (v & 31));
    const uint32_t prev = from_left(part);
    const bool leader = valid && (lane == 0 || prev != part);
    const uint64_t leaders = __ballot(leader);
    const int valid_lanes = __popcll(__ballot(valid));   // the valid lanes are the lowest ones
    if (leader) {
      const uint64_t higher = lane == WAVE - 1 ? 0ull : leaders & ~((2ull << lane) - 1ull);
      const int next = higher ? __ffsll((unsigned long long)higher) - 1 : valid_lanes;
      atomicAdd(&st.dead_part[part], (uint32_t)(next - lane));
    }
  }
}

__global__ __launch_bounds__(TB) void k_step_arrive(State st, const int32_t* __restrict__ arr_ids,
                                                    uint32_t a0, uint32_t a1) {
  step_arrivals(st, arr_ids, a0, a1, blockIdx.x, gridDim.x);
}

// One block.  n rows are evicted: the n dead rows with the largest ids.
__global__ __launch_bounds__(BIG) void k_step_find(State st, int64_t n, int64_t evict_tiles) {
  __shared__ int64_t smem[BIG / WAVE + 1];
  int64_t mine = 0;
  for (int64_t q = threadIdx.x; q < st.parts; q += BIG) mine += st.dead_part[q];
  int64_t total;
  block_exclusive_scan<int64_t, BIG>(mine, smem, total);
  const int64_t keep = total - n;
  int32_t T = -1;
  if (keep > 0) {
    T = p_kth_set_bit<BIG>(st.dead_bits, st.dead_part, st.parts, st.words, keep, true);
  } else {
    for (int64_t q = threadIdx.x; q < st.parts; q += BIG) st.dead_part[q] = 0;
  }
  if (threadIdx.x == 0) {
    if (keep < 0) *st.fault = 1;   // fewer dead rows than insertions: cannot happen in this regime
    Ctrl c{};
    c.jstar = st.S;
    c.mode_in = MODE_ALL;
    c.mode_res = MODE_SELECT;
    c.keep = (int32_t)keep;
    c.T = T;
    c.n_change = (int32_t)n;
    c.use_dead = 1;
    *st.ctrl = c;
  }
  for (int64_t q = threadIdx.x; q < evict_tiles; q += BIG) st.evict_tiles[q] = 0;
}

__global__ void k_step_verdict(const int32_t* __restrict__ fault, int64_t* __restrict__ scalars) {
  if (*fault) {
    scalars[PLAN_FAILED] = 8;
    scalars[PLAN_WHERE] = -1;
  }
}

__global__ __launch_bounds__(TB) void k_step_scatter(State st) {
  const Ctrl c = *st.ctrl;
  p_dead_scatter(st, c, blockIdx.x, gridDim.x);
}

// blocks [0, evict_blocks): a block per TB flag words (TB / WAVE tiles), the evicted lines in
// line order; the t-th of them takes the t-th insertion of the iteration, whose list starts
// at in_ids[dst].  The evicted lines crowd in few tiles (where rows come and go), so the
// block's evictions are dealt to all its threads by rank: a thread finds the flag word of its
// rank in the block's running popcounts (LDS), then the bit inside the word.
// The other blocks: the rows that die in the next iteration.
__global__ __launch_bounds__(TB) void k_step_emit(State st, int64_t evict_tiles, int64_t evict_blocks,
                                                  int64_t dst, const int32_t* __restrict__ in_ids,
                                                  int32_t* __restrict__ out_ids,
                                                  const int32_t* __restrict__ arr_ids, uint32_t a0,
                                                  uint32_t a1) {
  __shared__ uint32_t red[TB / WAVE];
  __shared__ uint32_t smem[TB / WAVE + 1];
  __shared__ uint64_t s_word[TB];
  __shared__ uint32_t s_incl[TB];
  if ((int64_t)blockIdx.x >= evict_blocks) {
    step_arrivals(st, arr_ids, a0, a1, blockIdx.x - evict_blocks, gridDim.x - evict_blocks);
    return;
  }
  constexpr int TPB = TB / WAVE;
  const int64_t first_tile = (int64_t)blockIdx.x * TPB;
  uint32_t any = 0;
#pragma unroll
  for (int k = 0; k < TPB; ++k)
    any |= first_tile + k < evict_tiles ? st.evict_tiles[first_tile + k] : 0;
  if (!any) return;                                // uniform over the block
  const int64_t word_at = first_tile * WAVE + threadIdx.x;
  const uint64_t word = word_at < evict_tiles * WAVE && word_at * WAVE < st.cap
                            ? st.evict_words[word_at] : 0;
  if (word) st.evict_words[word_at] = 0;           // consumed: zero for the next scatter
  const uint32_t mine = (uint32_t)__popcll(word);
  uint32_t total;
  const uint32_t before_me = block_exclusive_scan<uint32_t, TB>(mine, smem, total);
  s_word[threadIdx.x] = word;
  s_incl[threadIdx.x] = before_me + mine;
  const int64_t base = dst + block_prefix_of(st.evict_tiles, first_tile, red);   // (barriers inside)
  for (uint32_t r = threadIdx.x; r < total; r += TB) {
    int lo = 0, hi = TB - 1;                       // the first word whose running count exceeds r
#pragma unroll
    for (int step = 0; step < 8; ++step) {
      const int mid = (lo + hi) >> 1;
      if (s_incl[mid] > r) hi = mid; else lo = mid + 1;
    }
    uint64_t bits = s_word[lo];
    for (uint32_t skip = r - (s_incl[lo] - (uint32_t)__popcll(bits)); skip > 0; --skip) bits &= bits - 1;
    const int32_t line = (int32_t)((first_tile * WAVE + lo) * WAVE + (__ffsll((unsigned long long)bits) - 1));
    const int64_t at = base + r;
    const int32_t gone = st.res_id[line];
    const int32_t comes = in_ids[at];
    out_ids[at] = gone;
    // (the evicted row keeps its entry of the address table: it is never accessed again, and the
    // lookup after the last iteration finds the line it had)
    st.addr[comes] = line;
    st.res_id[line] = comes;
  }
}

struct Workspace {
  uint64_t *pairs_a, *pairs_b, *heads_a, *heads_b;
  uint32_t* key_hists;      // [S x (S + 1)] accesses per iteration and next accessed iteration (S <= STATIC_S_MAX),
                            // later the table of stays.hpp
  Cut* cuts;                // [S]
  uint32_t* hist;
  uint32_t* head_tiles;
  int32_t* next_iter;
  int32_t* first_of;
  int64_t* d_offsets;
  int64_t* d_ready;         // [S], and behind it
  int64_t* d_cs_offsets;
  unsigned long long* d_counts;
  State st;
  Plan plan;
  int64_t look_tiles, evict_tiles, in_tiles, max_heads, max_change;
  size_t bytes;
};

int bits_for(int64_t values) {  // bits needed to hold 0 .. values-1
  int b = 1;
  while (b < 63 && (int64_t(1) << b) < values) ++b;
  return b;
}

Workspace carve(void* base, int64_t num_nodes, int64_t total, int32_t S, int64_t cap,
                int64_t max_n) {
  Arena a(base);
  Workspace w{};
  const int64_t t = total > 0 ? total : 1;
  w.max_heads = t < num_nodes ? t : num_nodes;
  w.pairs_a = a.take<uint64_t>(t);
  w.pairs_b = a.take<uint64_t>(t);
  w.heads_a = a.take<uint64_t>(w.max_heads);   // (these three side by side, see stays_run)
  w.heads_b = a.take<uint64_t>(w.max_heads);
  w.next_iter = a.take<int32_t>(t);
  w.hist = a.take<uint32_t>(radix_plan(t).hist_elems);
  w.look_tiles = ceil_div(t, LOOK_TILE);
  w.head_tiles = a.take<uint32_t>(w.look_tiles + 1 + scan_scratch_elems(w.look_tiles + 1));
  w.key_hists = a.take<uint32_t>(S <= STATIC_S_MAX ? (size_t)S * (S + 1) : 0);
  w.cuts = a.take<Cut>(S);
  w.first_of = a.take<int32_t>(num_nodes);   // resumed superbatches only
  w.d_offsets = a.take<int64_t>(S + 1);
  w.d_ready = a.take<int64_t>(S + S + 1);
  w.d_cs_offsets = w.d_ready ? w.d_ready + S : nullptr;
  w.d_counts = a.take<unsigned long long>(2);
  State& st = w.st;
  const int64_t c = cap > 0 ? cap : 1;
  st.cap = cap;
  st.num_nodes = num_nodes;
  st.S = S;
  st.res_id = a.take<int32_t>(c);
  st.res_next = a.take<int32_t>(c);
  st.addr = a.take<int32_t>(num_nodes);
  st.rhist = a.take<uint32_t>(S + 2);
  st.ihist = a.take<uint32_t>(S + 2);
  st.words = ceil_div(num_nodes, 32);
  st.parts = ceil_div(st.words, PART_WORDS);
  st.bitmap = a.take<uint32_t>(st.words);
  st.dead_bits = a.take<uint32_t>(st.words);
  st.sel_part = a.take<uint32_t>(st.parts);
  st.bitmap_in = a.take<uint32_t>(st.words);
  st.sel_part_in = a.take<uint32_t>(st.parts);
  st.dead_part = a.take<uint32_t>(st.parts);
  st.ctrl = a.take<Ctrl>(1);
  st.fault = a.take<int32_t>(1);
  w.evict_tiles = ceil_div(c, (int64_t)EVICT_TILE);
  st.evict_words = a.take<uint64_t>(w.evict_tiles * WAVE);
  w.in_tiles = ceil_div(max_n > 0 ? max_n : 1, (int64_t)TB * IN_ITEMS);
  st.evict_tiles = a.take<uint32_t>(w.evict_tiles);
  st.in_tiles = a.take<uint32_t>(w.in_tiles);
  w.max_change = max_n < c ? max_n : c;
  if (w.max_change < 1) w.max_change = 1;
  st.acc_line = a.take<int32_t>(max_n > 0 ? max_n : 1);
  st.pair = a.take<uint64_t>(w.max_change);
  st.max_change = w.max_change;
  Plan& pl = w.plan;
  pl.ins_words = ceil_div(t, 32);
  pl.ins_tile_count = ceil_div(pl.ins_words, TB);
  pl.cand_tile_count = ceil_div(st.words, TB);
  pl.ins_bits = a.take<uint32_t>(pl.ins_words);
  pl.ins_tiles = a.take<uint32_t>(pl.ins_tile_count + 1 + scan_scratch_elems(pl.ins_tile_count + 1));
  pl.ins_base = a.take<uint32_t>(pl.ins_words);
  pl.ins_cand = a.take<int32_t>(w.max_heads);
  pl.scalars = a.take<int64_t>(PLAN_SCALARS);
  pl.cand_tiles = a.take<uint32_t>(pl.cand_tile_count + 1 + scan_scratch_elems(pl.cand_tile_count + 1));
  pl.cand_base = a.take<uint32_t>(st.words);
  pl.cand_id = a.take<int32_t>(PLAN_CAND_MAX);
  pl.cand_line = a.take<int32_t>(PLAN_CAND_MAX);
  pl.cand_dead = a.take<uint32_t>(PLAN_CAND_WORDS);
  pl.arr_off = a.take<uint32_t>(S + 2);
  pl.arr_cur = a.take<uint32_t>(S + 1);
  pl.arr_cand = a.take<int32_t>(PLAN_CAND_MAX);
  w.bytes = (a.used + 255) & ~size_t(255);
  return w;
}

int32_t check_shape(int64_t num_nodes, int64_t total, int32_t S, int64_t cap, const char* who) {
  if (num_nodes <= 0 || num_nodes > INT32_MAX)
    return fail(GINEX_ERR_ARG, "%s: num_nodes=%lld out of range", who, (long long)num_nodes);
  if (S < 1 || S > 8191) return fail(GINEX_ERR_ARG, "%s: S=%d outside [1, 8191]", who, S);
  if (total < 0 || total > INT32_MAX)
    return fail(GINEX_ERR_ARG, "%s: total ids=%lld outside [0, 2^31)", who, (long long)total);
  if (cap < 0 || cap > INT32_MAX)
    return fail(GINEX_ERR_ARG, "%s: cap=%lld out of range", who, (long long)cap);
  return GINEX_OK;
}

}  // namespace
}  // namespace ginex

using namespace ginex;

extern "C" size_t ginex_changeset_workspace_bytes(int64_t num_nodes, int64_t total_ids, int32_t S,
                                                  int64_t cap) {
  if (check_shape(num_nodes, total_ids, S, cap, "ginex_changeset_workspace_bytes")) return 0;
  // the longest iteration is not known here: bound it by the total (and by num_nodes,
  // since the ids of one iteration are distinct)
  const int64_t max_n = total_ids < num_nodes ? total_ids : num_nodes;
  return carve(nullptr, num_nodes, total_ids, S, cap, max_n).bytes;
}

namespace ginex {
namespace {

// Selects by many blocks at a time: their counters sit in an array of the planned path.
constexpr int64_t WIDE_AT_ONCE = PLAN_CAND_MAX / (CUT_DIGITS * CUT_BINS);

// Belady's thresholds and cuts, from the histograms (see stays.hpp); *never: bucket "never" is cut.  jobs: read by a
// copy to the device that is not waited for here, so the caller keeps it until it has waited.
int32_t stays_cuts(const Workspace& w, const Stays& q, const int64_t* ids_offsets, int64_t* miss_count, bool* never,
                   std::vector<int32_t>& jobs, Returns& back, hipStream_t st) {
  const State& state = w.st;
  const Plan& pl = w.plan;
  const int32_t S = q.S;
  if (S < 256)
    hipLaunchKernelGGL((k_static_roll<256, 1>), dim3(1), dim3(256), 0, st, state, w.key_hists,
                       w.d_offsets, w.cuts, miss_count);
  else
    hipLaunchKernelGGL((k_static_roll<BIG, 3>), dim3(1), dim3(BIG), 0, st, state, w.key_hists,
                       w.d_offsets, w.cuts, miss_count);
  hipLaunchKernelGGL(k_stay_table, dim3((unsigned)(S / WAVE + 1)), dim3(WAVE),
                     sizeof(int32_t) * S, st, w.cuts, S, w.key_hists);
  GINEX_LAUNCH_CHECK();
  std::vector<Cut> cuts(S);
  back.get(cuts.data(), w.cuts, S);
  GINEX_HIP(back.wait(st));

  // the levels: a cut waits for the cuts of the bucket its own iteration's accesses come from, and for
  // the earlier cuts of its bucket
  std::vector<int32_t> level_of_bucket(S + 1, 0);
  std::vector<std::vector<int32_t>> levels;
  for (int32_t t = 0; t < S; ++t) {
    const Cut& c = cuts[t];
    if (c.jstar == S) *never = true;
    if (c.jstar >= S || c.rem == 0) continue;
    const int32_t l = std::max(level_of_bucket[t], level_of_bucket[c.jstar]);   // (levels count from 1)
    level_of_bucket[c.jstar] = l + 1;
    if ((int32_t)levels.size() <= l) levels.resize(l + 1);
    levels[l].push_back(t);
  }
  auto length = [&](int32_t i) { return ids_offsets[i + 1] - ids_offsets[i]; };
  auto wide = [&](int32_t t) { return cuts[t].T > CUT_WIDE; };   // (members of its bucket, see k_static_roll)
  size_t most_jobs = 0;
  for (auto& level : levels) {
    std::stable_partition(level.begin(), level.end(), wide);
    jobs.insert(jobs.end(), level.begin(), level.end());
    most_jobs = std::max(most_jobs, level.size());
  }
  int32_t* const d_jobs = reinterpret_cast<int32_t*>(pl.arr_off);   // [S + 2], not used on this way
  if (most_jobs > Jobs::MOST)
    GINEX_HIP(hipMemcpyAsync(d_jobs, jobs.data(), sizeof(int32_t) * jobs.size(), hipMemcpyHostToDevice, st));
  uint32_t* const digit_counts = reinterpret_cast<uint32_t*>(pl.arr_cand);
  const int32_t* at = d_jobs;
  for (const auto& level : levels) {
    int64_t blocks = 1, most_members = 1, wides = 0;
    for (const int32_t t : level) {
      blocks = std::max(blocks, ceil_div(length(t) + length(cuts[t].jstar), CUT_TILE));
      most_members = std::max<int64_t>(most_members, cuts[t].T);
      wides += wide(t);
    }
    const int64_t count = (int64_t)level.size();
    Jobs now{most_jobs > Jobs::MOST ? at : nullptr, {}};
    if (!now.far) std::copy(level.begin(), level.end(), now.near);
    hipLaunchKernelGGL(k_cut_members, dim3((unsigned)blocks, (unsigned)count), dim3(TB), 0, st, q, now);
    for (int64_t first = 0; first < wides; first += WIDE_AT_ONCE) {
      const int64_t n = std::min(WIDE_AT_ONCE, wides - first);
      const dim3 grid((unsigned)std::min<int64_t>(ceil_div(most_members, TB * CUT_WIDE_ITEMS), 256), (unsigned)n);
      GINEX_HIP(fill_async<uint32_t>(digit_counts, n * (CUT_DIGITS * CUT_BINS), 0u, st));
      hipLaunchKernelGGL(k_cut_wide<0>, grid, dim3(TB), 0, st, q, now, (int)first, digit_counts);
      hipLaunchKernelGGL(k_cut_wide<1>, grid, dim3(TB), 0, st, q, now, (int)first, digit_counts);
      hipLaunchKernelGGL(k_cut_wide<2>, grid, dim3(TB), 0, st, q, now, (int)first, digit_counts);
      hipLaunchKernelGGL(k_cut_wide<CUT_DIGITS>, grid, dim3(TB), 0, st, q, now, (int)first, digit_counts);
    }
    if (wides < count)
      hipLaunchKernelGGL(k_cut_decide, dim3((unsigned)(count - wides)), dim3(BIG), 0, st, q, now, (int)wides);
    GINEX_LAUNCH_CHECK();
    at += count;
  }
  return GINEX_OK;
}

// GINEX_TRACE=1: a line on stderr that says which way the call goes; 2: and another how it finds the lines
int trace_level() {
  const char* const env = getenv("GINEX_TRACE");
  return env && (env[0] == '1' || env[0] == '2') ? env[0] - '0' : 0;
}

// The changesets of a full cache whose state (res_id, addr of the accessed rows, rhist and, for a
// carried cache, dead_bits) is set up, from the node-sorted accesses (see stays.hpp).
// `ends`: the other buffer of the sort, `rows`: a word per distinct row.  last_head: the last row of
// C_0, null for a carried cache, whose rows are in held_bits; accessed: the superbatch's; start: the rows of the start
// state by line.
int32_t stays_run(const char* who, const Workspace& w, const uint64_t* sorted, uint64_t* ends,
                  uint64_t* rows, int64_t distinct, const uint64_t* last_head,
                  const uint32_t* held_bits, const uint32_t* accessed, const int32_t* ids,
                  const int64_t* ids_offsets, int64_t total, int32_t S, int32_t* in_ids, int32_t* out_ids,
                  int32_t* in_positions,
                  int64_t cs_capacity, int64_t* cs_offsets, int64_t* miss_count, int32_t* src_line,
                  int64_t* total_changes, int64_t* init_ready, bool carried, const int32_t* start,
                  int32_t* final_ids, Returns& back, hipStream_t st) {
  const State& state = w.st;
  const Plan& pl = w.plan;
  const size_t off_lds = sizeof(int32_t) * (S + 1);
  const bool lru = state.lru;
  uint64_t* const limits = reinterpret_cast<uint64_t*>(w.cuts);   // (there are no cuts then)
  int device = 0;
  GINEX_HIP(hipGetDevice(&device));
  MoveTurn turn(device);
  Stays q{ends, w.d_offsets, ids, w.key_hists, w.cuts, w.next_iter, pl.cand_id, limits, S,
          bits_for(state.num_nodes)};
  int64_t longest = 0;
  for (int32_t i = 0; i < S; ++i)
    longest = std::max<int64_t>(longest, ids_offsets[i + 1] - ids_offsets[i]);

  // both ends of every stay, the thresholds, the table
  // many of them through windows of positions, where the results have room in between: in the heads and the array of
  // next iterations, neither of which holds anything here (the last head was put aside), the tiles' starts in the
  // counters of the sort
  const Dealt dealt{w.heads_a, reinterpret_cast<uint16_t*>(w.hist), total, (int32_t)deal_windows(total)};
  const int64_t room = reinterpret_cast<uint64_t*>(w.next_iter + total) - w.heads_a;
  if (total >= DEAL_MIN && total <= DEAL_TOTAL_MAX && total <= room &&
      deal_start_bytes(total) <= sizeof(uint32_t) * radix_plan(total).hist_elems) {
    hipLaunchKernelGGL(k_stay_deal, dim3((unsigned)deal_tiles(total)), dim3(DEAL_THREADS), 0, st, sorted, total,
                       w.d_offsets, S, last_head, held_bits, dealt);
    collect_async(dealt, PutEnds{ends, w.d_offsets, S}, off_lds, st);
  } else {
    const int64_t windows = ceil_div(total, ENDS_WINDOW);
    const int64_t window = windows <= ENDS_WINDOWS_MAX ? ceil_div(total, windows) : total;
    for (int64_t from = 0; from < total; from += window)
      hipLaunchKernelGGL(k_stay_ends, dim3((unsigned)w.look_tiles), dim3(TB), off_lds, st, sorted, total,
                         w.d_offsets, S, last_head, held_bits, (uint32_t)from,
                         (uint32_t)std::min(total, from + window), ends);
  }
  // (and the words that the blocks of k_move_lines exchange, in an array of the planned path)
  constexpr int MOVE_STATE = 2 * MOVE_BLOCKS + 1;
  static_assert(MOVE_STATE <= PLAN_CAND_WORDS, "room for them");
  GINEX_HIP(zero_async(Zeros().add(w.key_hists, (int64_t)S * (S + 1)).add(pl.arr_cur, S + 1)
                           .add(pl.cand_dead, MOVE_STATE), st));
  hipLaunchKernelGGL(k_key_hists, dim3((unsigned)ceil_div(longest, TB * TOUCH_ITEMS), (unsigned)S),
                     dim3(TB), sizeof(uint32_t) * (S + 1), st, ends, w.d_offsets, S, w.key_hists);
  bool never = false;      // bucket "never" is cut
  std::vector<int32_t> jobs;   // of the cuts
  if (lru) {
    hipLaunchKernelGGL(k_lru_counts, dim3((unsigned)S), dim3(WAVE), 0, st, S, w.key_hists);
    // (more iterations fill the GPU with a block each)
    const bool wide = longest > LRU_WIDE && S <= WIDE_AT_ONCE;
    LruJob* const lru_jobs = wide ? reinterpret_cast<LruJob*>(pl.cand_line) : nullptr;
    hipLaunchKernelGGL(k_lru_limits, dim3((unsigned)S), dim3(BIG), 0, st, q, w.key_hists, state.cap, limits, lru_jobs);
    if (wide) {
      uint32_t* const digit_counts = reinterpret_cast<uint32_t*>(pl.arr_cand);
      const dim3 grid((unsigned)std::min<int64_t>(ceil_div(longest, TB * CUT_WIDE_ITEMS), 256), (unsigned)S);
      GINEX_HIP(fill_async<uint32_t>(digit_counts, (int64_t)S * (CUT_DIGITS * CUT_BINS), 0u, st));
      hipLaunchKernelGGL(k_lru_wide<0>, grid, dim3(TB), 0, st, q, lru_jobs, limits, digit_counts);
      hipLaunchKernelGGL(k_lru_wide<1>, grid, dim3(TB), 0, st, q, lru_jobs, limits, digit_counts);
      hipLaunchKernelGGL(k_lru_wide<2>, grid, dim3(TB), 0, st, q, lru_jobs, limits, digit_counts);
      hipLaunchKernelGGL(k_lru_wide<CUT_DIGITS>, dim3(1, (unsigned)S), dim3(TB), 0, st, q, lru_jobs, limits,
                         digit_counts);
    }
    GINEX_LAUNCH_CHECK();
  } else if (int32_t rc = stays_cuts(w, q, ids_offsets, miss_count, &never, jobs, back, st)) {
    return rc;
  }

  // hits, misses, insertions
  const dim3 mark_grid((unsigned)ceil_div(total, CUT_TILE));
  if (lru) hipLaunchKernelGGL(k_stays_mark<true>, mark_grid, dim3(TB), off_lds, st, q, total, src_line, pl.ins_bits);
  else hipLaunchKernelGGL(k_stays_mark<false>, mark_grid, dim3(TB), off_lds, st, q, total, src_line, pl.ins_bits);
  // (init_ready: null, or waiting on the device for the next copy to the host)
  auto finish = [&]() -> int32_t {
    if (init_ready) back.get(init_ready, w.d_ready, S);
    if (final_ids)
      GINEX_HIP(hipMemcpyAsync(final_ids, state.res_id, sizeof(int32_t) * state.cap,
                               hipMemcpyDeviceToDevice, st));
    GINEX_HIP(back.wait(st));
    return GINEX_OK;
  };
  // nothing is inserted: the lines are those of the start state
  auto lines_of_start = [&]() -> int32_t {
    if (src_line) {
      Step s{};
      s.ids = ids;
      s.n = total;
      s.src_line = src_line;
      hipLaunchKernelGGL((k_step_lines<64, false>), dim3((unsigned)ceil_div(total, TB * 4)), dim3(TB), 0, st, state, s);
      GINEX_LAUNCH_CHECK();
    }
    return finish();
  };
  if (distinct == total && !lru) {
    // no row is accessed twice (a superbatch of one iteration, for one), so the lists stay empty (one iteration of
    // 15 k accesses, 2 k lines carried: 457 -> 311 us per call)
    return lines_of_start();
  }
  uint32_t* const leave_start = reinterpret_cast<uint32_t*>(state.res_next);
  // both sets of bits in node order where the members of the cuts were: a quarter byte per access in an
  // array of four (padded to 256 bytes, so the last words have room in the smallest one too)
  const int64_t words = ceil_div(total, WAVE);
  uint64_t* const hit_words = reinterpret_cast<uint64_t*>(w.next_iter);
  uint64_t* const ins_words = hit_words + words;
  Never nv{};
  nv.rows = rows;
  if (!lru)
    hipLaunchKernelGGL(k_stays_links, dim3((unsigned)w.look_tiles), dim3(TB), off_lds, st, q, sorted, total,
                       w.head_tiles, last_head, held_bits, state.addr, nv, hit_words, ins_words, leave_start);
  // bucket "never"
  if (never) {
    static_assert(NEVER_COUNTS <= PLAN_CAND_MAX && NEVER_LEVELS * (STATIC_S_MAX + 1) + NEVER_PARTS <= PLAN_CAND_MAX,
                  "counters and limits sit in the candidate arrays of the planned path");
    nv.idle = carried ? state.dead_bits : nullptr;
    nv.distinct = distinct;
    nv.num_nodes = state.num_nodes;
    // parts, a power of two of ids: a few thousand rows to a part where the graph is small, so that
    // there are few parts to walk over, but never more ids than its bitmap has room for
    int64_t most = NEVER_THREADS;
    while (most > 1 && (most * S > NEVER_COUNTS || most * 4096 > distinct)) most /= 2;
    nv.shift = 5;                           // (whole words of the bitmap)
    while (nv.shift < NEVER_SHIFT && ceil_div(state.num_nodes, int64_t(1) << nv.shift) > most) ++nv.shift;
    nv.parts = (int32_t)ceil_div(state.num_nodes, int64_t(1) << nv.shift);
    // (the array of first accesses: the bits of the rows held sat in it, which were read last by k_stays_links)
    nv.counts = (int64_t)S * nv.parts <= NEVER_COUNTS ? reinterpret_cast<uint32_t*>(pl.cand_line)
                                                      : reinterpret_cast<uint32_t*>(w.first_of);
    uint32_t* const idle_counts = reinterpret_cast<uint32_t*>(pl.cand_id) + NEVER_LEVELS * (STATIC_S_MAX + 1);
    GINEX_HIP(fill_async<uint32_t>(nv.counts, (int64_t)S * nv.parts, 0u, st));
    const int64_t count_blocks = std::min<int64_t>(ceil_div(distinct, TB * 8), 2048);
    hipLaunchKernelGGL(k_never_counts, dim3((unsigned)count_blocks), dim3(TB), sizeof(uint32_t) * S, st,
                       nv, S);
    if (carried)
      hipLaunchKernelGGL(k_never_idle, dim3((unsigned)nv.parts), dim3(TB), 0, st, nv, idle_counts);
    const uint32_t* const idle_rows = carried ? idle_counts : nullptr;
    if (nv.parts <= NEVER_THREADS)
      hipLaunchKernelGGL((k_never_parts<1, 4>), dim3(1), dim3(NEVER_THREADS), 0, st, nv, S, w.cuts, idle_rows);
    else if (nv.parts <= 4 * NEVER_THREADS)
      hipLaunchKernelGGL((k_never_parts<4, 4>), dim3(1), dim3(NEVER_THREADS), 0, st, nv, S, w.cuts, idle_rows);
    else
      hipLaunchKernelGGL((k_never_parts<16, 1>), dim3(1), dim3(NEVER_THREADS), 0, st, nv, S, w.cuts, idle_rows);
    hipLaunchKernelGGL(k_never_select, dim3((unsigned)nv.parts), dim3(NEVER_THREADS), 0, st, nv, S, w.cuts);
    GINEX_LAUNCH_CHECK();
  }
  if (!lru) hipLaunchKernelGGL(k_never_lift, dim3(1), dim3(BIG), 0, st, w.cuts, S, pl.cand_id);
  hipLaunchKernelGGL(k_ins_count, dim3((unsigned)S, (unsigned)std::min<int64_t>(ceil_div(longest, 32 * TB * 8), 64)),
                     dim3(TB), 0, st, pl.ins_bits, w.d_offsets, cs_offsets, lru ? miss_count : (int64_t*)nullptr);
  hipLaunchKernelGGL(k_ins_offsets, dim3(1), dim3(BIG), 0, st, cs_offsets, S, w.d_cs_offsets);
  GINEX_LAUNCH_CHECK();
  std::vector<int64_t> host(2 * S + 1);
  back.get(host.data(), w.d_ready, host.size());
  hipLaunchKernelGGL(k_bit_tiles, dim3((unsigned)pl.ins_tile_count), dim3(TB), 0, st, pl.ins_bits,
                     pl.ins_words, pl.ins_tiles);
  GINEX_HIP(exclusive_scan_inplace<uint32_t>(pl.ins_tiles, pl.ins_tile_count + 1,
                                             pl.ins_tiles + pl.ins_tile_count + 1, st));
  GINEX_HIP(back.wait(st));
  if (init_ready) std::copy_n(host.begin(), S, init_ready);
  init_ready = nullptr;
  const int64_t* const cs = host.data() + S;
  const int64_t M = cs[S];
  *total_changes = M;
  if (M > cs_capacity)
    return fail(GINEX_ERR_CAPACITY, "%s: %lld changeset records, capacity %lld", who, (long long)M,
                (long long)cs_capacity);

  // the insertion lists, and when every line is given up again
  // (the ends are not read any more)
  uint64_t* const leave_ins = ends;
  // (the numbers of candidates are the planned path's)
  uint64_t* const ins_pairs = sizeof(int32_t) * w.max_heads >= sizeof(uint64_t) * pl.ins_words
                                  ? reinterpret_cast<uint64_t*>(pl.ins_cand) : nullptr;
  const InsIndex at_ins{ins_pairs, pl.ins_bits, pl.ins_base};
  if (M == 0) return lines_of_start();
  hipLaunchKernelGGL(k_ins_emit, dim3((unsigned)pl.ins_tile_count), dim3(TB), off_lds, st, pl.ins_bits,
                     pl.ins_words, pl.ins_tiles, ids, w.d_offsets, S, in_ids, in_positions,
                     pl.ins_base, ins_pairs, (int32_t*)nullptr);
  if (carried)
    hipLaunchKernelGGL(k_stays_idle, dim3((unsigned)ceil_div(state.cap, TB)), dim3(TB), 0, st, q,
                       state.res_id, accessed, state.cap, leave_start);
  int levels = 1;
  while ((1 << levels) <= S) ++levels;
  Moves moves{};
  if (int32_t rc = moves_shape(state, longest, device, &turn, &moves)) return rc;
  int32_t* const hand_over = moves.blocks > 0 ? src_line : nullptr;
  const dim3 walk_grid((unsigned)ceil_div(total, WALK_TILE));
  if (lru)
    hipLaunchKernelGGL(k_lru_walk, walk_grid, dim3(TB), sizeof(uint64_t) * S + off_lds, st, q, sorted, total,
                       last_head, state.addr, at_ins, leave_ins, leave_start, hand_over);
  else if (S <= NEVER_LDS_S)
    hipLaunchKernelGGL(k_stays_walk<true>, walk_grid, dim3(TB), off_lds * (1 + levels), st, q, sorted,
                       total, state.addr, hit_words, ins_words, at_ins, leave_ins,
                       leave_start, hand_over);
  else
    hipLaunchKernelGGL(k_stays_walk<false>, walk_grid, dim3(TB), off_lds, st, q, sorted, total,
                       state.addr, hit_words, ins_words, at_ins, leave_ins,
                       leave_start, hand_over);
  GINEX_LAUNCH_CHECK();

  // the lines
  auto say = [&](const char* way) {
    if (trace_level() > 1) fprintf(stderr, "[ginex] %s: lines: %s\n", who, way);
  };
  say(moves.blocks > 0 ? "all iterations together" : "a launch per iteration");
  if (moves.blocks > 0) {
    moves.words = pl.cand_dead;
    moves.gave_up = pl.cand_dead + 2 * MOVE_BLOCKS;
    moves.leave_start = leave_start;
    moves.leave_ins = leave_ins;
    moves.ids = ids;
    moves.in_ids = in_ids;
    moves.out_ids = out_ids;
    moves.src_line = src_line;
    move_lines_async(state, moves, w.d_offsets, cs_offsets, st);
    if (final_ids) final_lines_async(state, final_ids, moves.gave_up, st);
    GINEX_LAUNCH_CHECK();
    uint32_t gave_up = 1;
    back.get(&gave_up, moves.gave_up);
    GINEX_HIP(back.wait(st));
    turn.give();
    if (!gave_up) return GINEX_OK;
    say("given up, a launch per iteration");
    hipLaunchKernelGGL(k_start_lines, dim3((unsigned)ceil_div(std::max(state.cap, total), TB)), dim3(TB), 0, st, state,
                       start, total, src_line);
    GINEX_LAUNCH_CHECK();
  }
  int32_t* const leaving = reinterpret_cast<int32_t*>(ends == w.pairs_a ? w.pairs_b : w.pairs_a);   // (nor the accesses)
  const int64_t place_blocks = std::min<int64_t>(ceil_div(M + state.cap, TB * 8), 512);
  hipLaunchKernelGGL(k_leave_places, dim3((unsigned)place_blocks), dim3(TB), sizeof(uint32_t) * S, st,
                     M, state.cap, S, leave_ins, leave_start, cs_offsets, pl.arr_cur, leaving);
  GINEX_LAUNCH_CHECK();
  Step s{};
  s.words = ceil_div(state.cap, 64);
  // tiles of 512 lines while there are few of them (their counters are atomics that share cache
  // lines), of 4096 for large caches (every block adds up the counters in front of its own)
  const bool large = state.cap >= LARGE_CACHE;
  s.tile_shift = large ? 12 : 9;
  s.tiles = ceil_div(state.cap, int64_t(1) << s.tile_shift);
  // and there four counters to a 128-byte line, on which additions queue up (0.2 G/s per line;
  // 13 M lines: 29.9 -> 28.0 us per iteration), as where most iterations change many lines, as far as
  // there is room
  int64_t most = 0;
  for (int32_t t = 0; t < S; ++t) most = std::max(most, cs[t + 1] - cs[t]);
  s.cnt_shift = large || most * DENSE_SHARE > state.cap ? 3 : 0;
  while (s.cnt_shift > 0 && 3 * (s.tiles << s.cnt_shift) > state.words) --s.cnt_shift;
  const int64_t stride = s.tiles << s.cnt_shift;
  // flag words: evict_words, and the scratch bitmap over ids, which has room for them (cap is at
  // most num_nodes, and the arrays of the workspace are padded to 256 bytes); the counters sit in
  // the second scratch bitmap, one counter for 512 lines or more against one word for 32 ids
  uint64_t* flags[2] = {state.evict_words, reinterpret_cast<uint64_t*>(state.bitmap)};
  uint32_t* counts = state.bitmap_in;
  // (see DENSE_SHARE)
  auto is_dense = [&](int64_t n) {
    return n * DENSE_SHARE > state.cap || (lru && n > 0 && s.tiles <= DENSE_TILES);
  };
  GINEX_HIP(zero_async(Zeros().add(flags[0], s.words).add(flags[1], s.words).add(counts, 3 * stride), st));
  s.leaving = leaving;
  s.leave_ins = leave_ins;
  s.in_ids = in_ids;
  s.out_ids = out_ids;
  auto changes = [&](int32_t t) { return t < S ? cs[t + 1] - cs[t] : int64_t(0); };
  auto flag_blocks = [&](int32_t t, bool dense) {
    return std::min<int64_t>(ceil_div(changes(t), dense ? DENSE_ENTRIES : TB), 256);
  };
  s.next = flags[0];
  s.cnt_next = counts;
  s.next_dst = 0;
  s.next_n = cs[1];
  s.next_filled = pl.arr_cur;
  if (is_dense(cs[1]))
    hipLaunchKernelGGL(k_step_flags<true>, dim3((unsigned)flag_blocks(0, true)), dim3(TB), 0, st, s);
  else if (cs[1] > 0)
    hipLaunchKernelGGL(k_step_flags<false>, dim3((unsigned)flag_blocks(0, false)), dim3(TB), 0, st, s);
  for (int32_t t = 0; t < S; ++t) {
    s.now = flags[t & 1];
    s.next = flags[(t + 1) & 1];
    s.cnt_now = counts + (t % 3) * stride;
    s.cnt_next = counts + ((t + 1) % 3) * stride;
    s.cnt_clear = counts + ((t + 2) % 3) * stride;
    const bool dense = is_dense(std::max(changes(t), changes(t + 1)));
    const int64_t line_words = dense ? (large ? 64 : 8) : large ? 256 : 64;
    s.emit_blocks = ceil_div(s.words, line_words);
    s.flag_blocks = flag_blocks(t + 1, dense);
    s.dst = cs[t];
    s.n_change = changes(t);
    s.next_dst = cs[t + 1];
    s.next_n = changes(t + 1);
    s.next_filled = pl.arr_cur + t + 1;
    s.ids = ids + ids_offsets[t];
    s.n = ids_offsets[t + 1] - ids_offsets[t];
    s.src_line = src_line ? src_line + ids_offsets[t] : nullptr;
    const dim3 blocks((unsigned)(s.emit_blocks + s.flag_blocks + (src_line ? ceil_div(s.n, TB * 4) : 0)));
    if (blocks.x == 0) continue;
    if (dense && large) hipLaunchKernelGGL((k_step_lines<64, true>), blocks, dim3(TB), 0, st, state, s);
    else if (dense) hipLaunchKernelGGL((k_step_lines<8, true>), blocks, dim3(TB), 0, st, state, s);
    else if (large) hipLaunchKernelGGL((k_step_lines<256, false>), blocks, dim3(TB), 0, st, state, s);
    else hipLaunchKernelGGL((k_step_lines<64, false>), blocks, dim3(TB), 0, st, state, s);
  }
  GINEX_LAUNCH_CHECK();
  return finish();
}

// The tiles and buckets of a call (see fits.hpp): ids and places in ids_buffer, 6 bytes per access, the starts in
// start_buffer (*start_bytes of its start_room).  buckets = 0 where this way does not serve the shape, or where even
// buckets that are equally full are too full.  lookup: for k_fit_lookup.
Fit fit_shape(const Workspace& w, int64_t num_nodes, int64_t total, int32_t S, int64_t max_n, bool lookup,
              uint64_t* ids_buffer, uint64_t* start_buffer, size_t start_room, size_t* start_bytes) {
  Fit f{};
  f.shift = fit_shift(num_nodes);
  f.S = S;
  const int64_t buckets = ceil_div(num_nodes, int64_t(1) << f.shift), per_iteration = ceil_div(max_n, FIT_TILE);
  const int64_t tiles = S * per_iteration;
  *start_bytes = (sizeof(uint16_t) * (size_t)(tiles * (buckets + 1)) + 255) & ~size_t(255);
  if (buckets > FIT_BUCKETS || total < FIT_SHARE_MIN * tiles * buckets || fit_lines_lds(f) > FIT_LDS ||
      *start_bytes > start_room)
    return f;
  const int64_t allowed = fit_ids_allowed(total, f.shift, lookup);
  if (ceil_div(total, buckets) > allowed) return f;
  f.sampled = total >= FIT_SAMPLE_MIN && allowed < total;
  f.sample = reinterpret_cast<uint32_t*>(w.next_iter);
  f.most = reinterpret_cast<uint32_t*>(w.d_counts + 1);
  f.most_allowed = (uint32_t)(allowed * FIT_SAMPLES / total);
  f.off = w.d_offsets;
  f.ids = reinterpret_cast<uint32_t*>(ids_buffer);
  f.rank = reinterpret_cast<uint16_t*>(f.ids + total);
  f.start = reinterpret_cast<uint16_t*>(start_buffer);
  f.bad = reinterpret_cast<uint32_t*>(w.d_counts);
  f.num_nodes = num_nodes;
  f.words = w.st.words;
  // (whether a call goes this way does not depend on the tiles' width; wide ones have fewer starts)
  const bool wide = S * ceil_div(max_n, FIT_WIDE_TILE) >= FIT_WIDE_MIN && buckets >= FIT_WIDE_BUCKETS;
  f.tile = wide ? FIT_WIDE_TILE : FIT_TILE;
  f.per_iteration = (int32_t)ceil_div(max_n, f.tile);
  f.tiles = S * f.per_iteration;
  f.buckets = (int32_t)buckets;
  return f;
}

void fit_sample_async(const Fit& f, const int32_t* ids, int64_t total, hipStream_t st) {
  hipLaunchKernelGGL(k_fit_sample, dim3(FIT_SAMPLE_BLOCKS), dim3(FIT_SAMPLE_THREADS), 0, st, f, ids, total);
}
void fit_deal_async(const Fit& f, const int32_t* ids, hipStream_t st) {
  const dim3 grid((unsigned)f.per_iteration, (unsigned)f.S);
  const size_t lds = sizeof(uint32_t) * f.buckets;
  if (f.tile == FIT_WIDE_TILE)
    hipLaunchKernelGGL(k_fit_deal<FIT_WIDE_THREADS>, grid, dim3(FIT_WIDE_THREADS), lds, st, f, ids);
  else
    hipLaunchKernelGGL(k_fit_deal<FIT_THREADS>, grid, dim3(FIT_THREADS), lds, st, f, ids);
}
void fit_place_async(const Fit& f, int32_t* src_line, hipStream_t st) {
  const dim3 grid((unsigned)f.per_iteration, (unsigned)f.S);
  if (f.tile == FIT_WIDE_TILE)
    hipLaunchKernelGGL(k_fit_place<FIT_WIDE_THREADS>, grid, dim3(FIT_WIDE_THREADS), 0, st, f, src_line);
  else
    hipLaunchKernelGGL(k_fit_place<FIT_THREADS>, grid, dim3(FIT_THREADS), 0, st, f, src_line);
}
dim3 fit_grid(const Fit& f) { return dim3((unsigned)(ceil_div(f.buckets, 8) * 8)); }

// A fresh cache that holds every row (see fits.hpp): *distinct rows of the superbatch, and if they fit `cap`, the
// results; -1 where this way does not serve the shape, the ids crowd in a bucket or (not certain) too many rows are
// estimated.
int32_t fits_run(const char* who, const Workspace& w, int64_t num_nodes, const int32_t* ids, int64_t total, int32_t S,
                 int64_t max_n, int64_t cap, bool certain, int32_t* init_ids, int32_t* src_line,
                 int64_t* init_ready, int64_t* distinct, Returns& back, hipStream_t st) {
  *distinct = -1;
  size_t start_bytes;
  const size_t room = sizeof(uint64_t) * total;
  Fit f = fit_shape(w, num_nodes, total, S, max_n, false, w.pairs_a, w.pairs_b, room, &start_bytes);
  const int64_t counts = (int64_t)S * f.buckets + 1;
  if (f.buckets == 0 || start_bytes + sizeof(uint32_t) * (counts + scan_scratch_elems(counts)) > room) return GINEX_OK;
  f.counts = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(w.pairs_b) + start_bytes);
  f.list = reinterpret_cast<uint32_t*>(w.st.addr);
  f.bits = w.st.dead_bits;
  f.marked = f.most + 1;
  f.marked_allowed = 0xFFFFFFFFu;
  if (!certain) {
    while (f.mark_shift < 32 - FIT_MARK_LOG && total >> f.mark_shift >= FIT_MARKS) ++f.mark_shift;
    f.marks = f.sample + FIT_BUCKETS;
    const double ids_marked = (double)(cap + cap / 128) / (double)(1 << f.mark_shift);
    f.marked_allowed = (uint32_t)(-FIT_MARK_BITS * std::expm1(-ids_marked / FIT_MARK_BITS));
  }
  // (the words for ids out of range, the fullest bucket and the marks were cleared, and the sample)
  if (f.sampled) fit_sample_async(f, ids, total, st);
  fit_deal_async(f, ids, st);
  hipLaunchKernelGGL(k_fit_rows, fit_grid(f), dim3(FIT_LINE_THREADS), fit_rows_lds(f), st, f);
  GINEX_HIP(exclusive_scan_inplace<uint32_t>(f.counts, counts, f.counts + counts, st, FitReady{f, w.d_ready}));
  GINEX_LAUNCH_CHECK();
  std::vector<int64_t> ready(S);
  back.get(ready.data(), w.d_ready, S);
  GINEX_HIP(back.wait(st));
  *distinct = ready[S - 1];
  if (*distinct == FIT_NOT) return GINEX_OK;
  // (the other ways would use such an id as an index)
  if (*distinct == FIT_BAD)
    return fail(GINEX_ERR_INPUT, "%s: ids out of range, there are %lld nodes", who, (long long)num_nodes);
  if (*distinct > cap) return GINEX_OK;
  if (init_ready) std::copy(ready.begin(), ready.end(), init_ready);
  hipLaunchKernelGGL(k_fit_lines, fit_grid(f), dim3(FIT_LINE_THREADS), fit_lines_lds(f), st, f, init_ids,
                     src_line != nullptr);
  if (src_line) fit_place_async(f, src_line, st);
  GINEX_LAUNCH_CHECK();
  GINEX_HIP(hipStreamSynchronize(st));
  return GINEX_OK;
}

// The smallest calls, see changeset_run.
constexpr int32_t LOOP_S = 6;
constexpr int64_t LOOP_IDS = 4096, LOOP_NODES = int64_t(1) << 26;
constexpr int32_t LOOP_LRU_S = 2;
constexpr int64_t LOOP_LRU_IDS = 1 << 16, LOOP_LRU_LINES = 1 << 22;

// Both replacement policies share every kernel: a policy only decides the key an access
// leaves behind (Belady: its next accessed iteration; LRU: S-1-i, so that the least
// recently used rows hold the largest keys) and the key of the prefetched rows.
//
// The ways to the lists, in the order in which they are looked at (GINEX_TRACE=1 says which one a call took; what a
// rule costs on its either side stands at the rule):
//   1  nothing is accessed
//   2  fresh, every row fits, or is likely to: fits.hpp, no sort.  Not with GINEX_VALIDATE=1, which goes on with the
//      accesses it has sorted; where the ids crowd in few buckets, or the rows do not fit, the call goes on to the next
//   3  fresh Belady, few rows that do not fit: one workgroup, small.hpp.  Not with GINEX_STATIC_THRESHOLDS
//   4  fresh, every row fits, or there is no cache: from the sorted accesses
//   5  carried, every row fits: the planned path (all iterations together, or steps); gives way to 6 or 7 where its
//      arrays do not hold the call.  Not with GINEX_PLANNED=0 or GINEX_LIVE_SELECT=1
//   6  from the trace, stays.hpp (of many accesses through the windows of deal.hpp): up to 2 048 iterations, LRU with
//      lines for the longest of them, but not the smallest calls (GINEX_STATIC_THRESHOLDS=1: these, too)
//   7  the loop over the state (GINEX_STATIC_THRESHOLDS=0: in the place of 6)
int32_t changeset_run(const char* who, bool lru, int64_t num_nodes, const int32_t* ids,
                      const int64_t* ids_offsets, int32_t S, int64_t cap, int32_t* init_ids,
                      int64_t* init_count, int32_t* in_ids, int32_t* out_ids,
                      int32_t* in_positions, int64_t cs_capacity, int64_t* cs_offsets,
                      int64_t* miss_count, int32_t* src_line, int64_t* total_changes,
                      int64_t* init_ready, const int32_t* start_ids, int32_t* final_ids, void* ws,
                      size_t ws_bytes, void* stream, bool pinned = true, bool allow_planned = true) {
  if (!ids_offsets || !init_count || !cs_offsets || !miss_count || !total_changes || !ws)
    return fail(GINEX_ERR_ARG, "%s: a required pointer is null", who);
  if (S >= 1 && ids_offsets[0] != 0)
    return fail(GINEX_ERR_INPUT, "%s: ids_offsets[0] must be 0", who);
  int64_t max_n = 0;
  for (int32_t i = 0; S >= 1 && i < S; ++i) {
    const int64_t n = ids_offsets[i + 1] - ids_offsets[i];
    if (n < 0) return fail(GINEX_ERR_INPUT, "%s: ids_offsets not monotone at %d", who, i);
    if (n > num_nodes)
      return fail(GINEX_ERR_INPUT, "%s: iteration %d has more ids than nodes", who, i);
    if (n > max_n) max_n = n;
  }
  const int64_t total = S >= 1 ? ids_offsets[S] : 0;
  if (int32_t rc = check_shape(num_nodes, total, S, cap, who)) return rc;
  if (total > 0 && !ids) return fail(GINEX_ERR_ARG, "%s: ids is null", who);
  if (cap > 0 && !init_ids && !start_ids)
    return fail(GINEX_ERR_ARG, "%s: init_ids is null", who);
  if (start_ids && cap < 1)
    return fail(GINEX_ERR_ARG, "%s: a carried cache needs cap >= 1", who);
  if (cs_capacity < 0 || (cs_capacity > 0 && (!in_ids || !out_ids || !in_positions)))
    return fail(GINEX_ERR_ARG, "%s: bad changeset output arrays", who);
  const int64_t bound = total < num_nodes ? total : num_nodes;
  Workspace w = carve(ws, num_nodes, total, S, cap, bound);
  if (ws_bytes < w.bytes)
    return fail(GINEX_ERR_WORKSPACE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes,
                w.bytes);
  if ((uintptr_t)ws & 255) return fail(GINEX_ERR_ARG, "%s: workspace must be 256-byte aligned", who);
  hipStream_t st = (hipStream_t)stream;
  Returns back(pinned);
  State& state = w.st;
  state.lru = lru ? 1 : 0;
  // The loop only (Belady beyond 2 048 iterations): worth it where a pass over the cache lines is
  // long; GINEX_DEAD_SCATTER=0/1 overrides the choice (both ways give the same lists).
  const char* scatter_env = getenv("GINEX_DEAD_SCATTER");
  state.dead_scatter = !lru && (scatter_env ? scatter_env[0] == '1' : cap >= (int64_t(1) << 20));
  state.dead_only = 0;

  {
    Zeros z = Zeros().add(miss_count, S).add(cs_offsets, S + 1).add(w.d_counts, 2);
    if (total >= FIT_SAMPLE_MIN) z.add(w.next_iter, FIT_BUCKETS);   // (see fit_shape)
    if (S <= NearOffsets::MOST) {
      NearOffsets near;
      for (int32_t i = 0; i <= S; ++i) near.at[i] = (int32_t)ids_offsets[i];
      hipLaunchKernelGGL(k_begin, dim3(1), dim3(TB), 0, st, near, S, w.d_offsets, z);
      GINEX_LAUNCH_CHECK();
    } else {
      GINEX_HIP(hipMemcpyAsync(w.d_offsets, ids_offsets, sizeof(int64_t) * (S + 1), hipMemcpyHostToDevice, st));
      GINEX_HIP(zero_async(z, st));
    }
  }
  const bool trace = trace_level() > 0;
  auto say = [&](const char* way) {
    if (trace) fprintf(stderr, "[ginex] %s: %s\n", who, way);
  };
  *init_count = start_ids ? cap : 0;
  *total_changes = 0;
  if (init_ready)
    for (int32_t i = 0; i < S; ++i) init_ready[i] = start_ids ? cap : 0;
  if (total == 0) {
    say("nothing is accessed");
    if (start_ids && final_ids && final_ids != start_ids)
      GINEX_HIP(hipMemcpyAsync(final_ids, start_ids, sizeof(int32_t) * cap,
                               hipMemcpyDeviceToDevice, st));
    GINEX_HIP(hipStreamSynchronize(st));
    return GINEX_OK;
  }

  const char* validate_env = getenv("GINEX_VALIDATE");
  const bool validate = validate_env && validate_env[0] == '1';
  // Where every row fits, or is likely to, a way that needs no sort.  It ends when the ids were dealt where too many rows
  // are estimated (see FIT_MARKS): not tried for less than three lines to four
  // accesses, where the rows would have to be accessed less than 4/3 times on the mean not to fit, nor for few
  // accesses unless it is certain.
  int64_t rows = -1;
  const bool certain = cap >= std::min(total, num_nodes);
  if (!start_ids && cap > 0 && !validate && (certain || (4 * cap >= 3 * total && total >= FIT_GUESS_MIN))) {
    if (int32_t rc = fits_run(who, w, num_nodes, ids, total, S, max_n, cap, certain, init_ids, src_line,
                              init_ready, &rows, back, st))
      return rc;
    if (rows >= 0 && rows <= cap) {
      say("every row fits, no sort");
      *init_count = rows;
      return GINEX_OK;
    }
    if (rows >= 0) say("too many rows, to the sort");
  }

  // part 1: sort (node, position) by node, then look right
  // (the first pass reads the ids themselves and forms the pairs on the way)
  uint64_t* sorted = nullptr;
  // when validating, sort on all 32 id bits so that ids beyond num_nodes are ordered too
  GINEX_HIP(radix_sort_values_with_positions(ids, w.pairs_a, w.pairs_b, total,
                                             validate ? 64 : 32 + bits_for(num_nodes), w.hist, st,
                                             &sorted));
  if (validate) {
    unsigned long long bad[2] = {0, 0};
    GINEX_HIP(fill_async<unsigned long long>(w.d_counts, 2, 0ull, st));
    hipLaunchKernelGGL(k_validate, dim3((unsigned)ceil_div(total, TB)), dim3(TB),
                       sizeof(int32_t) * (S + 1), st, sorted, total, w.d_offsets, S, num_nodes,
                       w.d_counts);
    GINEX_LAUNCH_CHECK();
    back.get(bad, w.d_counts, 2);
    GINEX_HIP(back.wait(st));
    if (bad[0] || bad[1])
      return fail(GINEX_ERR_INPUT, "%s: %llu ids outside [0, %lld), %llu ids repeated inside an "
                  "iteration", who, bad[0], (long long)num_nodes, bad[1]);
  }
  hipLaunchKernelGGL(k_count_heads, dim3((unsigned)w.look_tiles), dim3(TB), 0, st, sorted, total,
                     w.head_tiles);
  GINEX_LAUNCH_CHECK();
  GINEX_HIP(exclusive_scan_inplace<uint32_t>(w.head_tiles, w.look_tiles + 1,
                                             w.head_tiles + w.look_tiles + 1, st));
  int64_t distinct = rows;
  if (rows < 0) {
    uint32_t distinct32 = 0;
    back.get(&distinct32, w.head_tiles + w.look_tiles);
    GINEX_HIP(back.wait(st));
    distinct = distinct32;
  }
  if (distinct > w.max_heads)
    return fail(GINEX_ERR_INPUT, "%s: %lld distinct ids among %lld nodes: ids out of range?", who,
                (long long)distinct, (long long)num_nodes);

  // the smallest calls whose rows do not fit (GINEX_STATIC_THRESHOLDS chooses one of the other ways)
  const char* static_env = getenv("GINEX_STATIC_THRESHOLDS");
  if (!start_ids && !lru && !static_env && cap > 0 && cap < distinct && distinct <= SMALL_ROWS && S <= SMALL_S &&
      total <= SMALL_IDS) {
    say("one workgroup");
    const Small small{reinterpret_cast<uint32_t*>(w.next_iter), reinterpret_cast<int32_t*>(w.heads_a),
                      reinterpret_cast<uint32_t*>(w.heads_b), w.d_offsets, (int32_t)distinct, (int32_t)cap, S,
                      init_ids, in_ids, out_ids, in_positions, cs_capacity, cs_offsets, miss_count, src_line,
                      w.d_ready, w.d_cs_offsets};
    hipLaunchKernelGGL(k_small_ranks, dim3((unsigned)w.look_tiles), dim3(TB), 0, st, sorted, total, w.head_tiles,
                       small);
    hipLaunchKernelGGL(k_small_belady, dim3(1), dim3(BIG), 0, st, small);
    GINEX_LAUNCH_CHECK();
    std::vector<int64_t> host(2 * S + 1);
    back.get(host.data(), w.d_ready, host.size());
    GINEX_HIP(back.wait(st));
    *init_count = cap;
    if (init_ready) std::copy_n(host.begin(), S, init_ready);
    *total_changes = host[2 * S];
    if (*total_changes > cs_capacity)
      return fail(GINEX_ERR_CAPACITY, "%s: %lld changeset records, capacity %lld", who, (long long)*total_changes,
                  (long long)cs_capacity);
    return GINEX_OK;
  }

  // part 2: C_0
  const size_t off_lds = sizeof(int32_t) * (S + 1);
  hipLaunchKernelGGL(k_heads_write, dim3((unsigned)w.look_tiles), dim3(TB), off_lds, st, sorted,
                     total, w.d_offsets, S, w.head_tiles, w.heads_a);
  GINEX_LAUNCH_CHECK();
  uint64_t* heads = w.heads_a;
  if (!start_ids)   // C_0: the heads in order of first access
    GINEX_HIP(radix_sort_u64(w.heads_a, w.heads_b, distinct, 32, 32 + bits_for(S), w.hist, st,
                             &heads));
  const int64_t n_init = start_ids ? cap : (distinct < cap ? distinct : cap);
  *init_count = n_init;
  if (init_ready && n_init > 0 && !start_ids) {   // every path below waits for the stream before it returns
    hipLaunchKernelGGL(k_init_ready, dim3((unsigned)ceil_div(S, TB)), dim3(TB), 0, st, heads, n_init,
                       S, w.d_ready);
    GINEX_LAUNCH_CHECK();
  } else {
    init_ready = nullptr;
  }
  // (to the host with the next copy that has to be waited for anyway)
  auto bring_ready = [&]() {
    if (init_ready) back.get(init_ready, w.d_ready, S);
  };
  if (!start_ids && (distinct <= cap || cap == 0)) {
    // everything fits (no row ever misses), or there is no cache (every row misses and
    // nothing is inserted): all changesets are empty
    say(cap == 0 ? "no cache" : "every row fits, from the sorted accesses");
    if (n_init > 0) {
      hipLaunchKernelGGL(k_copy_init, dim3((unsigned)ceil_div(n_init, TB)), dim3(TB), 0, st, heads,
                         n_init, init_ids);
      GINEX_LAUNCH_CHECK();
    }
    if (cap == 0) {
      hipLaunchKernelGGL(k_iteration_lengths, dim3((unsigned)ceil_div(S, TB)), dim3(TB), 0, st,
                         w.d_offsets, S, miss_count);
      GINEX_LAUNCH_CHECK();
      if (src_line) GINEX_HIP(fill_async<int32_t>(src_line, total, -1, st));
    } else if (src_line) {
      // every accessed row sits in the line of its rank for the whole superbatch
      hipLaunchKernelGGL(k_scatter_rank, dim3((unsigned)ceil_div(n_init, TB)), dim3(TB), 0, st,
                         heads, n_init, state.addr);
      hipLaunchKernelGGL(k_lookup_lines, dim3((unsigned)ceil_div(total, TB * 4)), dim3(TB), 0, st,
                         ids, total, state.addr, src_line);
      GINEX_LAUNCH_CHECK();
    }
    bring_ready();
    GINEX_HIP(back.wait(st));
    return GINEX_OK;
  }
  // A carried cache with room for every row of the superbatch never evicts a row that is
  // still needed: each iteration keeps all live candidates, so the threshold bucket is
  // "never" and the select runs on the dead rows.  The changesets then follow without a loop
  // over the state (the planned path; GINEX_PLANNED=0 switches it off); the loop, where it runs
  // all the same, leaves the two launches of the live select out.
  // GINEX_LIVE_SELECT=1 keeps them in, and the planned path out.  All ways give the same lists.
  const char* live_env = getenv("GINEX_LIVE_SELECT");
  const char* plan_env = getenv("GINEX_PLANNED");
  state.dead_only = start_ids && distinct <= cap && !(live_env && live_env[0] == '1');
  const bool planned = state.dead_only && allow_planned && S <= PLAN_S_MAX &&
                       !(plan_env && plan_env[0] == '0');
  // Belady, otherwise: the changesets from the trace and the start state (stays.hpp), but for more
  // iterations than the table of the stays is kept for, and for the smallest calls, which are a
  // chain of launches either way: the loop has six to an iteration, the other way some 40.
  // Carried, lines for a tenth and for eight tenths of the rows, the loop and the trace: 2 000 nodes, iterations of 300
  // accesses, two 253 and 325 us, 237 and 302, four 292 and 339, 281 and 309, six 349 and 364, 359 and 323, eight 401
  // and 393, 415 and 339; 20 000 nodes, three of 3 000 accesses 286 and 349, 298 and 318, four of 2 000 332 and 352, 337
  // and 325.  Many nodes: the loop clears two words for each; three iterations of 200 accesses, 30 M nodes 285 and 350,
  // 289 and 334, 66 M 358 and 354, 359 and 338.  GINEX_STATIC_THRESHOLDS=0/1 chooses the loop / the trace.
  // LRU (the trace's way has no cuts): 20 000 nodes, iterations of 3 000 accesses, two 226 and 240, three 276
  // and 244, six 421 and 259; 200 000 nodes, of 20 000, two 258 and 252, three 318 and 262.  And a large cache of just
  // the lines that an iteration accesses: the loop gives all of them up without a select (5 iterations of 8 M 4.2 and
  // 5.0 ms, 8 of 4 M 3.55 and 3.76; of 2 M 2.6 and 2.0; with 6 % more lines 26.9 and 5.1, 19.6 and 3.8).
  const bool by_loop =
      (lru && max_n == cap && cap >= LOOP_LRU_LINES) ||
      (num_nodes <= LOOP_NODES &&
       (lru ? S <= LOOP_LRU_S && total <= LOOP_LRU_IDS
            : S <= LOOP_S && total <= (S <= LOOP_S / 2 ? 4 * LOOP_IDS : LOOP_IDS) && distinct < total));
  const bool stays = S <= STATIC_S_MAX && (!lru || max_n <= cap) &&
                     (static_env ? static_env[0] != '0' : !by_loop);
  const bool loop = !stays;   // (the loop still is the last way out of the planned path then)
  {
    Zeros z;
    z.add(state.rhist, S + 2);
    if (loop || planned) {    // (the steps of the planned path use the fault word and the flag words)
      z.add(state.bitmap, state.words).add(state.fault, 1);
      if (state.dead_scatter) z.add(state.evict_words, w.evict_tiles * WAVE);
    }
    if (loop)
      z.add(state.dead_bits, state.words).add(state.dead_part, state.parts).add(state.ihist, S + 2)
          .add(state.sel_part, state.parts).add(state.bitmap_in, state.words)
          .add(state.sel_part_in, state.parts).add(state.pair, w.max_change);
    GINEX_HIP(zero_async(z, st));
  }
  if (loop && !lru && !planned) {   // the next accessed iteration of every access
    hipLaunchKernelGGL(k_look_right, dim3((unsigned)w.look_tiles), dim3(TB), off_lds, st, sorted,
                       total, w.d_offsets, S, w.next_iter);
    GINEX_LAUNCH_CHECK();
  }
  // the loop looks every access up in the address table, and finds repeated rows of a carried state
  // there; the other ways only read entries that were written
  const bool for_loop = loop && !planned;   // (where the planned path gives up, the loop starts afresh)
  if (for_loop) GINEX_HIP(fill_async<int32_t>(state.addr, num_nodes, -1, st));
  // a carried state without the loop: bytes per row held in the array of first accesses, behind them
  // the same as bits; the bitmap of accessed rows in the loop's scratch
  uint8_t* const held = reinterpret_cast<uint8_t*>(w.first_of);
  uint32_t* const held_bits = reinterpret_cast<uint32_t*>(held) + state.words * 8;
  uint32_t* const accessed = state.bitmap_in;
  {
    int64_t blocks = ceil_div(cap, TB * 8);
    if (blocks > 4096) blocks = 4096;
    if (start_ids) {
      unsigned long long bad = 0;
      if (for_loop) {
        GINEX_HIP(fill_async<unsigned long long>(w.d_counts, 1, 0ull, st));
        GINEX_HIP(fill_async<int32_t>(w.first_of, num_nodes, S, st));
        hipLaunchKernelGGL(k_scatter_first, dim3((unsigned)ceil_div(distinct, TB)), dim3(TB), 0, st,
                           heads, distinct, w.first_of);
        hipLaunchKernelGGL(k_init_state_resume, dim3((unsigned)blocks), dim3(TB),
                           sizeof(uint32_t) * (S + 1), st, start_ids, w.first_of, state, w.d_counts);
        // the part counts of the dead rows the start state brought along
        hipLaunchKernelGGL(k_part_count, dim3((unsigned)state.parts), dim3(TB), 0, st,
                           state.dead_bits, state.words, state.dead_part);
      } else {
        GINEX_HIP(hipMemcpyAsync(state.res_id, start_ids, sizeof(int32_t) * cap, hipMemcpyDeviceToDevice, st));
        const unsigned hold_blocks = (unsigned)ceil_div(ceil_div(cap, TB * HOLD_ITEMS), 8) * 8;
        const RadixValuesWithPositions lines{start_ids};
        const int id_bits = bits_for(num_nodes), deal_bits = std::min(8, std::max(1, id_bits - HOLD_SHIFT_MIN));
        const int shift = id_bits - deal_bits;
        const bool deals = cap >= HOLD_DEAL_MIN && cap <= total;
        uint64_t* const dealt = sorted == w.pairs_a ? w.pairs_b : w.pairs_a;
        if (deals) GINEX_HIP(radix_pass(lines, dealt, cap, 32 + shift, deal_bits, w.hist, st));
        // (shorter stretches: more lines than nodes, which is refused below)
        if (deals && shift >= HOLD_SHIFT_MIN && shift <= HOLD_SHIFT_MAX) {
          GINEX_HIP(fill_async<unsigned long long>(w.d_counts, 1, 0ull, st));
          const int share = std::min(HOLD_SHARE_MAX, shift - HOLD_SHIFT_MIN);
          const int64_t stretches = ceil_div(ceil_div(num_nodes, int64_t(1) << shift), 8) * 8;
          hipLaunchKernelGGL(k_hold_stretch, dim3((unsigned)(stretches << share)), dim3(BIG), 0, st, dealt, w.hist,
                             radix_tiles(cap, deal_bits), 1 << radix_digit(cap, deal_bits).bits, shift, share, state,
                             heads, distinct, accessed, held_bits, w.d_counts);
        } else {
          GINEX_HIP(zero_async(Zeros().add(accessed, state.words).add(reinterpret_cast<uint64_t*>(held), state.words * 4)
                                   .add(w.d_counts, 1), st));
          hipLaunchKernelGGL(k_accessed_bits, dim3((unsigned)ceil_div(distinct, TB)), dim3(TB), 0, st, heads,
                             distinct, accessed);
          if (deals)
            hipLaunchKernelGGL(k_hold<true>, dim3(hold_blocks), dim3(TB), 0, st, RadixWords{dealt}, cap,
                               num_nodes, accessed, held, state.addr);
          else
            hipLaunchKernelGGL(k_hold<false>, dim3(hold_blocks), dim3(TB), 0, st, lines, cap, num_nodes,
                               accessed, held, state.addr);
          hipLaunchKernelGGL(k_held_words, dim3((unsigned)state.parts), dim3(TB), 0, st, held, state,
                             accessed, held_bits, w.d_counts);
        }
      }
      GINEX_LAUNCH_CHECK();
      back.get(&bad, w.d_counts);
      GINEX_HIP(back.wait(st));
      if (!for_loop) bad = (unsigned long long)cap - bad;   // (rows held, so far)
      if (bad)
        return fail(GINEX_ERR_INPUT, "%s: %llu entries of start_ids are out of range or repeated",
                    who, bad);
    } else {
      hipLaunchKernelGGL(k_init_state, dim3((unsigned)blocks), dim3(TB),
                         sizeof(uint32_t) * (S + 1), st, heads, cap, init_ids, state,
                         reinterpret_cast<uint64_t*>(w.d_counts));
      GINEX_LAUNCH_CHECK();
    }
  }

  if (planned) {
    const Plan& pl = w.plan;
    GINEX_HIP(zero_async(Zeros().add(pl.ins_bits, pl.ins_words).add(pl.arr_off, S + 2)
                             .add(pl.cand_dead, PLAN_CAND_WORDS).add(pl.scalars + PLAN_FULLEST, 1), st));
    {
      const int64_t blocks = std::min(ceil_div(total, PLAN_HEADS_TILE), PLAN_HEADS_BLOCKS);
      hipLaunchKernelGGL(k_plan_heads, dim3((unsigned)blocks), dim3(BIG),
                         sizeof(int32_t) * (3 * (size_t)S + 1), st, sorted, total, w.d_offsets, S,
                         held_bits, state.addr, pl.ins_bits, (unsigned long long*)miss_count,
                         (unsigned long long*)cs_offsets);
      hipLaunchKernelGGL(k_plan_scan, dim3(1), dim3(BIG), 0, st, state, sorted, total, cs_offsets,
                         pl.scalars);
      // the id bitmap of the candidates (in the select's scratch bitmap, which is all zero
      // here) and their number, still without the host
      int64_t tail_blocks = ceil_div(total, (int64_t)TB * 16);
      tail_blocks = tail_blocks < 1 ? 1 : (tail_blocks > 1024 ? 1024 : tail_blocks);
      hipLaunchKernelGGL(k_cand_start, dim3((unsigned)tail_blocks), dim3(TB), 0, st,
                         state.dead_bits, state.words, num_nodes, pl.scalars, state.bitmap);
      hipLaunchKernelGGL(k_plan_arrivals<false>, dim3((unsigned)tail_blocks), dim3(TB), 2 * off_lds, st,
                         sorted, total, pl.scalars, held_bits, w.d_offsets, S, state.bitmap,
                         pl.cand_base, num_nodes, pl, (int32_t*)nullptr, (int32_t*)nullptr);
      hipLaunchKernelGGL(k_plan_arrival_offsets, dim3(1), dim3(BIG), 0, st, pl.arr_off,
                         pl.arr_cur, S, pl.scalars);
      GINEX_LAUNCH_CHECK();
    }
    // Every row has one line for the whole superbatch: the start state's or the one it is given.  Through
    // buckets where the table is larger than the caches (random words of 55 G/s then): the accesses are
    // sorted still in one buffer, the other and the heads have room for them
    size_t start_bytes;
    Fit fit{};
    if (src_line && total >= FIT_LOOKUP_MIN && distinct >= FIT_LOOKUP_ROWS && total * FIT_LOOKUP_NODES >= num_nodes)
      fit = fit_shape(w, num_nodes, total, S, max_n, true, sorted == w.pairs_a ? w.pairs_b : w.pairs_a, w.heads_a,
                      sizeof(uint64_t) * w.max_heads, &start_bytes);
    if (fit.buckets > 0) {
      fit.most = reinterpret_cast<uint32_t*>(pl.scalars + PLAN_FULLEST);
      if (fit.sampled) fit_sample_async(fit, ids, total, st);
    }
    int64_t sc[PLAN_SCALARS] = {};
    back.get(sc, pl.scalars, PLAN_SCALARS);
    GINEX_HIP(back.wait(st));
    const int64_t M = sc[PLAN_M], lo_id = sc[PLAN_LO_ID];
    // all iterations together where their arrays hold the call, else (or with GINEX_PLANNED=2) the
    // steps on the bitmap in global memory; neither with fewer dead rows than insertions
    // (the arrays: the candidates, at most twice the distinct rows, in the heads that are not used any more, the
    // counters in the start state's keys or the table of the stays.  The candidates are also at most twice the lines,
    // so the counters fit one of the two.)
    const int64_t parts = ceil_div(sc[PLAN_CANDS], PLAN_PART);
    const bool in_keys = S * parts <= cap;
    const bool stepped = M > 0 && lo_id >= 0 &&
                         ((plan_env && plan_env[0] == '2') || sc[PLAN_MAX_N] > PLAN_SORT_MAX ||
                          sc[PLAN_CANDS] > PLAN_CAND_MAX || sc[PLAN_CANDS] > 2 * w.max_heads ||
                          (!in_keys && parts > S + 1));
    const bool fits = M == 0 || lo_id >= 0;
    const char* const otherwise = loop ? "loop" : "from the trace, as any other cache";
    if (trace)
      fprintf(stderr, "[ginex] %s: %lld insertions, at most %lld per iteration, %lld rows dead from "
              "the start, lowest possible victim %lld of %lld ids, %lld candidates: %s\n", who,
              (long long)M, (long long)sc[PLAN_MAX_N], (long long)sc[PLAN_DEAD], (long long)lo_id,
              (long long)num_nodes, (long long)sc[PLAN_CANDS],
              !fits ? otherwise : stepped ? "stepped path" : "planned path");
    if (fits) {
      *total_changes = M;
      if (M > cs_capacity)
        return fail(GINEX_ERR_CAPACITY, "%s: %lld changeset records, capacity %lld", who,
                    (long long)M, (long long)cs_capacity);
      if (M > 0) {
        // the insertion lists
        hipLaunchKernelGGL(k_bit_tiles, dim3((unsigned)pl.ins_tile_count), dim3(TB), 0, st,
                           pl.ins_bits, pl.ins_words, pl.ins_tiles);
        GINEX_LAUNCH_CHECK();
        GINEX_HIP(exclusive_scan_inplace<uint32_t>(pl.ins_tiles, pl.ins_tile_count + 1,
                                                   pl.ins_tiles + pl.ins_tile_count + 1, st));
        hipLaunchKernelGGL(k_ins_emit, dim3((unsigned)pl.ins_tile_count), dim3(TB), off_lds, st,
                           pl.ins_bits, pl.ins_words, pl.ins_tiles, ids, w.d_offsets, S, in_ids,
                           in_positions, pl.ins_base, (uint64_t*)nullptr, pl.ins_cand);
        GINEX_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_dead_lines, dim3((unsigned)(ceil_div(cap, TB * 8) > 4096 ? 4096 : ceil_div(cap, TB * 8))),
                           dim3(TB), 0, st, state, accessed, lo_id);
        int64_t tail_blocks = ceil_div(total - sc[PLAN_TAIL], TB);
        tail_blocks = tail_blocks < 1 ? 1 : (tail_blocks > 1024 ? 1024 : tail_blocks);
        if (stepped) {
          // the rows that die, as ids grouped by iteration (in the array of the candidate numbers of
          // the insertions, which the steps do not need)
          int32_t* const arr_ids = pl.ins_cand;
          hipLaunchKernelGGL(k_plan_arrivals<true>, dim3((unsigned)tail_blocks), dim3(TB),
                             2 * off_lds, st, sorted, total, pl.scalars, held_bits, w.d_offsets, S,
                             state.bitmap, pl.cand_base, num_nodes, pl, (int32_t*)nullptr, arr_ids);
          GINEX_LAUNCH_CHECK();
          std::vector<int64_t> cs(S + 1);
          std::vector<uint32_t> arr(S + 2);
          back.get(cs.data(), cs_offsets, S + 1);
          back.get(arr.data(), pl.arr_off, S + 1);
          GINEX_HIP(back.wait(st));
          arr[S + 1] = arr[S];
          if (!state.dead_scatter)
            GINEX_HIP(fill_async<uint64_t>(state.evict_words, w.evict_tiles * WAVE, 0ull, st));
          const int64_t evict_blocks = ceil_div(w.evict_tiles, TB / WAVE);
          int64_t scatter_blocks = ceil_div(state.words, TB);
          scatter_blocks = scatter_blocks > 256 ? 256 : scatter_blocks;
          auto arrive_blocks = [](uint32_t count) {
            const int64_t b = ceil_div((int64_t)count, TB);
            return (unsigned)(b < 1 ? 1 : (b > 64 ? 64 : b));
          };
          if (arr[1] > arr[0])
            hipLaunchKernelGGL(k_step_arrive, dim3(arrive_blocks(arr[1] - arr[0])), dim3(TB), 0, st,
                               state, arr_ids, arr[0], arr[1]);
          for (int32_t i = 0; i < S; ++i) {
            const int64_t n = cs[i + 1] - cs[i];
            const uint32_t a0 = arr[i + 1], a1 = i + 1 < S ? arr[i + 2] : arr[i + 1];
            if (n > 0) {
              hipLaunchKernelGGL(k_step_find, dim3(1), dim3(BIG), 0, st, state, n, w.evict_tiles);
              hipLaunchKernelGGL(k_step_scatter, dim3((unsigned)scatter_blocks), dim3(TB), 0, st,
                                 state);
              hipLaunchKernelGGL(k_step_emit,
                                 dim3((unsigned)evict_blocks + (a1 > a0 ? arrive_blocks(a1 - a0) : 0u)),
                                 dim3(TB), 0, st, state, w.evict_tiles, evict_blocks, cs[i], in_ids,
                                 out_ids, arr_ids, a0, a1);
            } else if (a1 > a0) {
              hipLaunchKernelGGL(k_step_arrive, dim3(arrive_blocks(a1 - a0)), dim3(TB), 0, st, state,
                                 arr_ids, a0, a1);
            }
          }
          GINEX_LAUNCH_CHECK();
          // (a step that met fewer dead rows than insertions leaves its mark in the word the
          // copy below brings over beside the planned path's)
          hipLaunchKernelGGL(k_step_verdict, dim3(1), dim3(1), 0, st, state.fault, pl.scalars);
          GINEX_LAUNCH_CHECK();
        } else {
          // the candidates numbered in id order
          const char* const stop = getenv("GINEX_PLAN_STOP");
          const Victims victims{reinterpret_cast<int32_t*>(w.heads_b),
                                in_keys ? reinterpret_cast<uint32_t*>(state.res_next) : w.key_hists,
                                pl.arr_cand, state.res_next, pl.arr_cur, (int32_t)parts, S, stop ? atoi(stop) : -1};
          const int64_t lo_word = lo_id >> 5;
          const int64_t nwords = state.words - lo_word;
          const int64_t ctiles = ceil_div(nwords, TB);
          hipLaunchKernelGGL(k_bit_tiles, dim3((unsigned)ctiles), dim3(TB), 0, st,
                             state.bitmap + lo_word, nwords, pl.cand_tiles);
          GINEX_LAUNCH_CHECK();
          GINEX_HIP(exclusive_scan_inplace<uint32_t>(pl.cand_tiles, ctiles + 1,
                                                     pl.cand_tiles + ctiles + 1, st));
          hipLaunchKernelGGL(k_cand_emit, dim3((unsigned)ctiles), dim3(TB), 0, st, state.bitmap,
                             state.dead_bits, lo_word, nwords, pl.cand_tiles, state.addr, pl, victims.when, S);
          hipLaunchKernelGGL(k_plan_arrivals<true>, dim3((unsigned)tail_blocks), dim3(TB), 2 * off_lds, st,
                             sorted, total, pl.scalars, held_bits, w.d_offsets, S, state.bitmap,
                             pl.cand_base, num_nodes, pl, victims.when, (int32_t*)nullptr);
          if (parts > 1)
            hipLaunchKernelGGL(k_plan_counts, dim3((unsigned)S), dim3(TB), 0, st, pl, victims, sc[PLAN_CANDS]);
          hipLaunchKernelGGL(k_plan_victims, dim3((unsigned)parts), dim3(WAVE), 0, st, pl, victims, ctiles,
                             cs_offsets);
          hipLaunchKernelGGL(k_plan_sort, dim3((unsigned)S), dim3(BIG), 0, st, pl, victims, cs_offsets);
          if (S >= 4)   // (iteration 0 evicts no row it inserted, the last one inserts none: the third of three waits for none)
            hipLaunchKernelGGL(k_plan_chain, dim3(1), dim3(BIG), 0, st, pl, victims, cs_offsets);
          hipLaunchKernelGGL(k_plan_pairs, dim3((unsigned)S), dim3(BIG), 0, st, state, pl, victims, cs_offsets,
                             in_ids, out_ids);
          GINEX_LAUNCH_CHECK();
        }
      }
      if (src_line) {
        if (fit.buckets > 0 && sc[PLAN_FULLEST] <= (int64_t)fit.most_allowed) {
          say("lines by bucket");
          fit.bits = accessed;
          fit_deal_async(fit, ids, st);
          hipLaunchKernelGGL(k_fit_lookup, fit_grid(fit), dim3(FIT_LINE_THREADS), fit_rows_lds(fit), st, fit,
                             state.addr);
          fit_place_async(fit, src_line, st);
        } else {
          hipLaunchKernelGGL(k_lookup_lines, dim3((unsigned)ceil_div(total, TB * 4)), dim3(TB), 0, st,
                             ids, total, state.addr, src_line);
        }
        if (M > 0)
          hipLaunchKernelGGL(k_ins_lines, dim3((unsigned)pl.ins_tile_count), dim3(TB), 0, st,
                             pl.ins_bits, pl.ins_words, src_line);
        GINEX_LAUNCH_CHECK();
      }
      if (final_ids) final_lines_async(state, final_ids, pl.scalars + PLAN_FAILED, st);
      GINEX_LAUNCH_CHECK();
      int64_t failed[2] = {0, 0};
      back.get(failed, pl.scalars + PLAN_FAILED, 2);
      GINEX_HIP(back.wait(st));
      if (!failed[0]) return GINEX_OK;
      if (trace)
        fprintf(stderr, "[ginex] %s: the planned path gave up (reason %lld, iteration %lld): %s\n", who,
                (long long)failed[0], (long long)failed[1], otherwise);
      // it gave up, possibly after it had changed the state: start over, without it
      return changeset_run(who, lru, num_nodes, ids, ids_offsets, S, cap, init_ids, init_count,
                           in_ids, out_ids, in_positions, cs_capacity, cs_offsets, miss_count,
                           src_line, total_changes, init_ready, start_ids, final_ids, ws, ws_bytes,
                           stream, pinned, false);
    }
    // not for this path
    if (loop)
      return changeset_run(who, lru, num_nodes, ids, ids_offsets, S, cap, init_ids, init_count,
                           in_ids, out_ids, in_positions, cs_capacity, cs_offsets, miss_count,
                           src_line, total_changes, init_ready, start_ids, final_ids, ws, ws_bytes,
                           stream, pinned, false);
    GINEX_HIP(fill_async<int64_t>(cs_offsets, S + 1, 0, st));
  }

  if (stays) {
    if (start_ids) {
      const int64_t hist_blocks = std::min<int64_t>(ceil_div(distinct, TB * 16), 1024);
      hipLaunchKernelGGL(k_held_hist, dim3((unsigned)hist_blocks), dim3(TB), sizeof(uint32_t) * S, st,
                         heads, distinct, held_bits, state);
      GINEX_LAUNCH_CHECK();
    }
    say("from the trace");
    uint64_t* const ends = sorted == w.pairs_a ? w.pairs_b : w.pairs_a;
    uint64_t* const rows = heads == w.heads_a ? w.heads_b : w.heads_a;
    return stays_run(who, w, sorted, ends, rows, distinct, start_ids ? nullptr : reinterpret_cast<uint64_t*>(w.d_counts),
                     held_bits, accessed, ids, ids_offsets, total, S, in_ids, out_ids, in_positions,
                     cs_capacity, cs_offsets, miss_count,
                     src_line, total_changes, init_ready, start_ids != nullptr, start_ids ? start_ids : init_ids,
                     final_ids, back, st);
  }

  // part 3: the recurrence, with no host round trip between iterations
  say("loop");
  const size_t touch_lds = sizeof(uint32_t) * 2 * (S + 1);
  Outputs outs{in_ids, out_ids, in_positions, cs_capacity, cs_offsets, miss_count};
  {
    const int64_t res_blocks = ceil_div(cap, TB * MARK_ITEMS);
    // waves per tile of lines in k_emit_pair (one where a wave takes the flags of its tile back)
    const int32_t split = state.dead_scatter || w.evict_tiles > 256 ? 1 : 16;
    const int64_t evict_blocks = ceil_div(w.evict_tiles * split, TB / WAVE);
    for (int32_t i = 0; i < S; ++i) {
      Iter it;
      const int64_t lo = ids_offsets[i];
      it.ids = ids + lo;
      it.next = w.next_iter + lo;
      it.n = ids_offsets[i + 1] - lo;
      it.i = i;
      it.key = lru ? S - 1 - i : -1;
      it.lo_bin = lru ? S - 1 - i : i + 1;
      it.src_line = src_line ? src_line + lo : nullptr;
      if (it.n > 0) {
        hipLaunchKernelGGL(k_touch, dim3((unsigned)ceil_div(it.n, TB * TOUCH_ITEMS)), dim3(TB),
                           touch_lds, st, state, it, (unsigned long long*)(miss_count + i));
        GINEX_LAUNCH_CHECK();
      }
      hipLaunchKernelGGL(k_threshold, dim3(1), dim3(BIG), 0, st, state, i, it.lo_bin, outs,
                         w.evict_tiles);
      GINEX_LAUNCH_CHECK();
      if (it.n == 0) continue;  // nothing missed, nothing changes
      const int64_t in_tiles = ceil_div(it.n, (int64_t)TB * IN_ITEMS);
      if (!state.dead_only) {
        hipLaunchKernelGGL(k_mark, dim3((unsigned)(res_blocks + ceil_div(it.n, TB * MARK_ITEMS))),
                           dim3(TB), 0, st, state, it, res_blocks);
        hipLaunchKernelGGL(k_find, dim3(1), dim3(BIG), 0, st, state);
        GINEX_LAUNCH_CHECK();
      }
      hipLaunchKernelGGL(k_flags, dim3((unsigned)(w.evict_tiles + in_tiles + 1)), dim3(TB), 0,
                         st, state, it, w.evict_tiles, in_tiles);
      hipLaunchKernelGGL(k_emit_pair, dim3((unsigned)(evict_blocks + in_tiles)), dim3(TB), 0, st,
                         state, it, outs, w.evict_tiles, evict_blocks, split);
      GINEX_LAUNCH_CHECK();
    }
  }
  if (start_ids && final_ids)
    GINEX_HIP(hipMemcpyAsync(final_ids, state.res_id, sizeof(int32_t) * cap,
                             hipMemcpyDeviceToDevice, st));
  back.get(total_changes, cs_offsets + S);
  bring_ready();
  int32_t fault = 0;
  back.get(&fault, state.fault);
  GINEX_HIP(back.wait(st));
  if (fault)
    return fail(GINEX_ERR_INPUT, "%s: an iteration needed a select among live rows although all "
                "%lld rows of the superbatch fit the cache of %lld lines: ids repeated inside an "
                "iteration?", who, (long long)distinct, (long long)cap);
  if (*total_changes > cs_capacity)
    return fail(GINEX_ERR_CAPACITY, "%s: %lld changeset records, capacity %lld", who,
                (long long)*total_changes, (long long)cs_capacity);
  return GINEX_OK;
}

}  // namespace
}  // namespace ginex

extern "C" int32_t ginex_changeset(int64_t num_nodes, const int32_t* ids,
                                   const int64_t* ids_offsets, int32_t S, int64_t cap,
                                   int32_t* init_ids, int64_t* init_count, int32_t* in_ids,
                                   int32_t* out_ids, int32_t* in_positions, int64_t cs_capacity,
                                   int64_t* cs_offsets, int64_t* miss_count, int32_t* src_line,
                                   int64_t* total_changes, int64_t* init_ready, void* ws,
                                   size_t ws_bytes, void* stream) {
  return changeset_run("ginex_changeset", false, num_nodes, ids, ids_offsets, S, cap, init_ids,
                       init_count, in_ids, out_ids, in_positions, cs_capacity, cs_offsets,
                       miss_count, src_line, total_changes, init_ready, nullptr, nullptr, ws,
                       ws_bytes, stream);
}

extern "C" int32_t ginex_changeset_resume(int64_t num_nodes, const int32_t* ids,
                                          const int64_t* ids_offsets, int32_t S, int64_t cap,
                                          const int32_t* start_ids, int32_t* final_ids,
                                          int32_t* in_ids, int32_t* out_ids,
                                          int32_t* in_positions, int64_t cs_capacity,
                                          int64_t* cs_offsets, int64_t* miss_count,
                                          int32_t* src_line, int64_t* total_changes, void* ws,
                                          size_t ws_bytes, void* stream) {
  if (!start_ids)
    return fail(GINEX_ERR_ARG, "ginex_changeset_resume: start_ids is null");
  int64_t init_count = 0;
  return changeset_run("ginex_changeset_resume", false, num_nodes, ids, ids_offsets, S, cap,
                       nullptr, &init_count, in_ids, out_ids, in_positions, cs_capacity,
                       cs_offsets, miss_count, src_line, total_changes, nullptr, start_ids,
                       final_ids, ws, ws_bytes, stream);
}

extern "C" int32_t ginex_changeset_lru(int64_t num_nodes, const int32_t* ids,
                                       const int64_t* ids_offsets, int32_t S, int64_t cap,
                                       int32_t* init_ids, int64_t* init_count, int32_t* in_ids,
                                       int32_t* out_ids, int32_t* in_positions,
                                       int64_t cs_capacity, int64_t* cs_offsets,
                                       int64_t* miss_count, int32_t* src_line,
                                       int64_t* total_changes, int64_t* init_ready, void* ws,
                                       size_t ws_bytes, void* stream) {
  return changeset_run("ginex_changeset_lru", true, num_nodes, ids, ids_offsets, S, cap, init_ids,
                       init_count, in_ids, out_ids, in_positions, cs_capacity, cs_offsets,
                       miss_count, src_line, total_changes, init_ready, nullptr, nullptr, ws,
                       ws_bytes, stream);
}

// ---- the variant that allocates nothing ------------------------------------------------
//
// The workspace of ginex_changeset_noalloc is a static device array.  Every GPU the library
// runs on holds its own copy at its own address until the process ends; in host code the
// array's name is only a stand-in for the symbol, so the device address is looked up once per
// device (with that device current) and that pointer is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[GINEX_NOALLOC_SCRATCH_BYTES];

namespace ginex {
namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};

int32_t scratch_for_current_device(const char* who, void** out) {
  int device = -1;
  GINEX_HIP(hipGetDevice(&device));
  if (device < 0 || device >= MAX_DEVICES)
    return fail(GINEX_ERR_HIP, "%s: device index %d outside [0, %d)", who, device, MAX_DEVICES);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    void* ptr = nullptr;
    GINEX_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(GINEX_ERR_HIP, "%s: the scratch array has no device address", who);
    g_scratch_ptr[device] = ptr;
  }
  *out = g_scratch_ptr[device];
  return GINEX_OK;
}

}  // namespace
}  // namespace ginex

extern "C" int32_t ginex_changeset_noalloc(int64_t num_nodes, const int32_t* ids,
                                           const int64_t* ids_offsets, int32_t S, int64_t cap,
                                           int32_t* init_ids, int64_t* init_count,
                                           int32_t* in_ids, int32_t* out_ids,
                                           int32_t* in_positions, int64_t cs_capacity,
                                           int64_t* cs_offsets, int64_t* miss_count,
                                           int32_t* src_line, int64_t* total_changes,
                                           int64_t* init_ready, void* stream) {
  const char* who = "ginex_changeset_noalloc";
  if (!ids_offsets) return fail(GINEX_ERR_ARG, "%s: ids_offsets is null", who);
  const int64_t total = S >= 1 ? ids_offsets[S] : 0;
  if (int32_t rc = check_shape(num_nodes, total, S, cap, who)) return rc;
  const int64_t bound = total < num_nodes ? total : num_nodes;
  const size_t need = carve(nullptr, num_nodes, total, S, cap, bound).bytes;
  if (need > (size_t)GINEX_NOALLOC_SCRATCH_BYTES)
    return fail(GINEX_ERR_WORKSPACE,
                "%s: this shape (num_nodes=%lld, %lld ids, S=%d, cap=%lld) needs %zu bytes of "
                "scratch, the built-in array holds %zu: use ginex_changeset with a workspace", who,
                (long long)num_nodes, (long long)total, S, (long long)cap, need,
                (size_t)GINEX_NOALLOC_SCRATCH_BYTES);
  void* ws = nullptr;
  if (int32_t rc = scratch_for_current_device(who, &ws)) return rc;
  return changeset_run(who, false, num_nodes, ids, ids_offsets, S, cap, init_ids, init_count,
                       in_ids, out_ids, in_positions, cs_capacity, cs_offsets, miss_count,
                       src_line, total_changes, init_ready, nullptr, nullptr, ws,
                       (size_t)GINEX_NOALLOC_SCRATCH_BYTES, stream, false);   // (no pinned block either)
}
