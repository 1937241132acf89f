// A fresh cache that holds every row of the superbatch, without a sort.  Included by changeset.hip only.
//
// Nothing is ever missed then: C_0 is all distinct rows by (first access, id), and every access finds its row in
// the line of that rank.  Which iteration accesses a row first and what its rank is takes no order among the
// accesses of a row, so the ids are only dealt to buckets, 2^shift neighbouring ids each, small enough for a bitmap
// and the lines of a bucket's rows in LDS:
//   k_fit_sample how full the fullest bucket is, from some of the accesses: where the ids crowd, not this way
//   k_fit_deal   a block per tile of the accesses of an iteration: sorts them by bucket in LDS, writes ids
//                and their places in the tile in that order, and the start of every bucket inside the tile
//   k_fit_rows   a block per bucket: the bits of its ids, then the first iteration of every row (the smallest), then
//                its rank among the bucket's rows of that iteration
//   (scan of the numbers of new rows by iteration, then bucket: the rank of each of these lists' pieces; FitReady)
//   k_fit_lines  a block per bucket: line of every row into LDS, C_0; then of every access, in the tiles' order
//   k_fit_place  a block per tile: the lines back in the order of the accesses
// A carried cache that holds every row takes its lines the same way, with k_fit_lookup in the place of the two.
// Ids in order (a bucket's share lies in one tile of every iteration then, some hundred ids long) and ids that crowd
// in few buckets make long shares; they go to whole waves, with several reads in flight, and lanes that meet in a
// bucket count together in k_fit_deal.  In order: 24 M accesses, 339 268 nodes, 143 iterations 2 714 -> 699 us a call
// (701 through the sorted accesses), 40 M on 5.1 M nodes 4 164 -> 1 540 (1 707), 72 560 on 49 M nodes in 2
// iterations 1 772 -> 365; in no order, 10 M on 11 M nodes, 303 and 303.
// 33 M accesses, 9 M rows of 111 M nodes, 200 iterations: k_fit_sample 8, k_fit_deal 106 us (with the marks of the guess; 78
// without), k_fit_rows 197 and k_fit_lines 157 (3.7 M shares of ten ids, a line or two each in three arrays), k_fit_place 57; 631
// a call.  Through the sorted accesses 2 004: four radix passes 0.72 ms, heads 0.23, the rows' lines
// scattered to a table over all nodes and looked up there for every access 0.82 (random words).
// (A wave per bucket that takes the iterations one after the other, without a table of first iterations: 626 us for
// k_fit_rows, 83 000 vector instructions in a chain of 6 per CU.)
#pragma once

// An id to a bucket of a tile on the mean, below which nearly all of the work is looking at empty shares.  No lower
// limit on the accesses otherwise (2 iterations of 500: 206 -> 160 us, 8 of 4 000 on 16 384 nodes 204 -> 178).
constexpr int64_t FIT_SHARE_MIN = 1;
constexpr int64_t FIT_GUESS_MIN = 1 << 20;             // see changeset_run
// k_fit_lookup (33 M accesses, 9 M rows of 111 M nodes: 78 + 234 + 57 us against 626 for a random word per access):
// accesses, nodes to an access, beyond which few entries of a line of the table are used (carried caches,
// calls in all: 10 M nodes, 1 M accesses 903 -> 889 us, 8.4 M 1 746 -> 1 672; 100 M nodes, 2 M 892 and 917, 8.4 M
// 2 018 and 2 013, 17 M 5 427 -> 5 382), and rows, whose entries are more than an L2 holds (in no order 2.1 M rows,
// 40 M accesses 2 509 -> 2 356, 0.8 M, 7 M 2 752 and 2 740, 0.2 M, 11 M 573 and 581; ids in order, whose entries lie side by
// side: 5.1 M rows, 40 M 6 018 and 6 125, 1.1 M neighbours among 2.8 M nodes, 27 M 3 650 and 3 945, 0.3 M, 24 M 837
// and 1 010).
constexpr int64_t FIT_LOOKUP_MIN = 1 << 20, FIT_LOOKUP_NODES = 8, FIT_LOOKUP_ROWS = 1 << 21;

// A tile's accesses.  Wide tiles make half the shares of twice the length, and a share is a line of ids, one of places and one
// of starts however few it holds: 33 M accesses in 1 695 buckets, shares of 4.9 and 9.8, k_fit_rows 245 -> 197 us,
// k_fit_lines 196 -> 157, k_fit_lookup 281 -> 234 (the calls 714 -> 631 and 2 479 -> 2 436); 256 x 150 000 on 60 M nodes 726 ->
// 615, 512 x 30 000 405 -> 359, 40 x 400 000 on 20 M 312 -> 298.  Fewer buckets have shares that fill the lanes already
// (1 M nodes, 489 buckets, 64 x 120 000 184 and 179 us, 300 x 17 000 173 and 186), and fewer than two wide tiles to a CU
// leave CUs without work.
constexpr int FIT_THREADS = 512, FIT_WIDE_THREADS = 1024;
constexpr int FIT_ITEMS = 16;
constexpr int FIT_TILE = FIT_THREADS * FIT_ITEMS, FIT_WIDE_TILE = FIT_WIDE_THREADS * FIT_ITEMS;
constexpr int64_t FIT_WIDE_MIN = 512, FIT_WIDE_BUCKETS = 1024;   // wide tiles and buckets from which they are taken
constexpr int FIT_SHIFT_MIN = 11, FIT_SHIFT_MAX = 16;  // ids of a bucket: ranks among them have 16 bits
constexpr int FIT_BUCKETS = 4096;                      // at most, 2^28 nodes
constexpr int FIT_LINE_THREADS = 1024;
constexpr int FIT_ROWS = 7168;                         // rows of a bucket in LDS at a time (above: 5 300)
constexpr int FIT_SHARES = 2048;                       // tiles whose shares are laid out at a time
constexpr int FIT_SHARE_LANES = 8, FIT_SHARE_ITEMS = 4;
constexpr int FIT_TOGETHER = 8;                        // lanes of a wave, see k_fit_deal
constexpr int FIT_LONG_SHARE = 128;                    // what a share has beyond this goes to a whole wave

// How full the fullest bucket may be.  One workgroup takes it, so its ids follow one another where the others'
// are taken side by side: ids that crowd (in order of degree, or of a part of the graph) or few buckets make one
// workgroup the whole call (all among the 354 000 lowest of 111 M ids, 35 M accesses: 61 ms, 1.4 through the sorted
// accesses).  The measure is ids of the bucket times passes over them, one for its bits and two for every FIT_ROWS
// rows.  Calls in order and not, 62 720 to 40 M accesses on 2 027 to 98 M nodes: up to FIT_CHAIN + accesses / 32 never
// slower than through the sorted accesses (0.4 to 1.0 times), from there to twice that 0.9 to 1.4 times, further up to 11
// times.  k_fit_lookup: against a random word per access, with one pass for every FIT_ROWS rows; up to 25 000 + accesses /
// 128 0.93 to 1.0 times, from 300 000 + accesses / 32 on 1.04 to 1.4 times.
constexpr int64_t FIT_CHAIN = 250'000, FIT_CHAIN_SHARE = 32, FIT_LOOKUP_CHAIN = 25'000, FIT_LOOKUP_SHARE = 128;
// A sample of the accesses says so before anything else is done, where that many accesses could crowd too much and are
// not so few that the gain is gone (some 6 us).
constexpr int64_t FIT_SAMPLE_MIN = 1 << 15;
constexpr int FIT_SAMPLE_BLOCKS = 64, FIT_SAMPLE_THREADS = 512;
constexpr int64_t FIT_SAMPLES = FIT_SAMPLE_BLOCKS * FIT_SAMPLE_THREADS;

// Where it is a guess that the rows fit, their number is estimated while the ids are dealt: ids with FIT_MARKS / 2 to
// FIT_MARKS accesses among them, chosen by a hash, set a bit each in FIT_MARK_BITS bits, by other bits of the hash.  From the
// bits set follows how many of these ids there are (-m ln(1 - b / m) of b set among m bits), within 0.4 % or so: up to
// 1 / 128 more rows than lines are let through, so that a cache of just as many is (8 M accesses 743 -> 256 us a call).
// Too small a cache, to sort and without a guess: 33 M accesses 5 504 us, 5 697 with this estimate, 6 096 where the rows
// are known after k_fit_rows only; 8 M 1 219, 1 299 and 1 318; 1.3 M 548, 604 and 590.
constexpr int64_t FIT_MARKS = 1 << 18;
constexpr int FIT_MARK_LOG = 21, FIT_MARK_BITS = 1 << FIT_MARK_LOG;

constexpr uint32_t FIT_DONE = 0x80000000u;             // a line in the place of an id (both are below 2^31)

struct Fit {
  const int64_t* off;      // [S + 1]
  uint32_t* ids;           // [total] the ids of a tile by bucket, at the tile's own place; later their lines
  uint16_t* rank;          // [total] their places in the tile
  uint16_t* start;         // [tiles][buckets + 1] start of every bucket inside the tile
  uint32_t* counts;        // [S][buckets] new rows, later the sum of all in front; and one more
  uint32_t* list;          // [buckets][2^shift] of a row, in id order: first iteration << 16 | rank in it and the bucket
  uint32_t* bits;          // [words] rows accessed, by id
  uint32_t* bad;           // set where an id is out of range
  int64_t num_nodes, words;
  int32_t S, tile, per_iteration, tiles;   // accesses of a tile, tiles of an iteration, of all
  int32_t buckets, shift;
  uint32_t* sample;        // [buckets] sampled ids, zero before
  uint32_t* most;          // the fullest bucket's, zero before
  uint32_t most_allowed;   // beyond: not this way
  bool sampled;
  uint32_t* marks;         // [FIT_MARK_BITS / 32] null: certain that the rows fit
  uint32_t* marked;        // bits set, zero before
  uint32_t marked_allowed;
  int32_t mark_shift;      // an id of 2^mark_shift is marked
  // known when the ids are dealt
  __device__ __forceinline__ bool serves() const { return *most <= most_allowed && *marked <= marked_allowed; }
};

// Passes over a bucket of that many ids (lines: k_fit_lookup's).
__host__ __device__ __forceinline__ int64_t fit_chain(int64_t ids, int32_t shift, bool lookup) {
  const int64_t rows = ids < (int64_t(1) << shift) ? ids : int64_t(1) << shift, slices = (rows + FIT_ROWS - 1) / FIT_ROWS;
  return lookup ? ids * slices : ids * (1 + 2 * slices);
}
inline int64_t fit_chain_allowed(int64_t total, bool lookup) {
  return lookup ? FIT_LOOKUP_CHAIN + total / FIT_LOOKUP_SHARE : FIT_CHAIN + total / FIT_CHAIN_SHARE;
}
// The most ids that a bucket may have.
inline int64_t fit_ids_allowed(int64_t total, int32_t shift, bool lookup) {
  int64_t lo = 0, hi = total;
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) / 2;
    if (fit_chain(mid, shift, lookup) <= fit_chain_allowed(total, lookup)) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The bit of an id's hash inside its word of the marks.
__device__ __forceinline__ uint32_t fit_mark(uint32_t h) { return h >> (32 - FIT_MARK_LOG) & 31u; }

// How many of FIT_SAMPLES accesses fall into the fullest bucket.
__global__ __launch_bounds__(FIT_SAMPLE_THREADS) void k_fit_sample(Fit f, const int32_t* __restrict__ ids, int64_t total) {
  __shared__ uint32_t s_count[FIT_BUCKETS];
  __shared__ uint32_t s_most;
  const int64_t me = (int64_t)blockIdx.x * FIT_SAMPLE_THREADS + threadIdx.x;
  const uint32_t q = (uint32_t)ids[me * total / FIT_SAMPLES] >> f.shift;
  if (f.marks)
    for (int64_t w = me; w < FIT_MARK_BITS / 32; w += FIT_SAMPLES) f.marks[w] = 0;
  for (int b = threadIdx.x; b < f.buckets; b += FIT_SAMPLE_THREADS) s_count[b] = 0;
  if (threadIdx.x == 0) s_most = 0;
  __syncthreads();
  atomicAdd(&s_count[q < (uint32_t)f.buckets ? q : f.buckets - 1], 1u);
  __syncthreads();
  constexpr int PER = FIT_BUCKETS / FIT_SAMPLE_THREADS;
  uint32_t c[PER], most = 0;                         // (all additions on their way together)
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int b = k * FIT_SAMPLE_THREADS + threadIdx.x;
    c[k] = b < f.buckets ? s_count[b] : 0u;
    if (c[k]) c[k] += atomicAdd(&f.sample[b], c[k]);
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) most = c[k] > most ? c[k] : most;
  if (most) atomicMax(&s_most, most);
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(f.most, s_most);
}

inline int32_t fit_shift(int64_t num_nodes) {
  int32_t shift = FIT_SHIFT_MIN;
  while (shift < FIT_SHIFT_MAX && ceil_div(num_nodes, int64_t(1) << shift) > FIT_BUCKETS / 2) ++shift;
  return shift;
}

// neighbouring buckets on one XCD (blocks go to the eight XCDs in turn), as their shares share cache lines
__device__ __forceinline__ int32_t fit_bucket() { return blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8; }

// (the places wait in registers until the ids have left LDS, so that two blocks of wide tiles, which is all waves of
// a CU, have room side by side: 153 -> 106 us for 33 M accesses, the narrow ones 108 -> 93)
template <int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS / 128))) void k_fit_deal(
    Fit f, const int32_t* __restrict__ ids) {
  constexpr int TILE = THREADS * FIT_ITEMS;
  extern __shared__ uint32_t s_count[];              // [buckets]
  __shared__ uint32_t s_id[TILE];                    // then the places
  uint16_t* const s_rank = reinterpret_cast<uint16_t*>(s_id);
  __shared__ uint32_t smem[THREADS / WAVE + 1];
  if (*f.most > f.most_allowed) return;              // (nothing writes it while this runs)
  __shared__ uint32_t s_new;
  if (threadIdx.x == 0) s_new = 0;
  const int64_t pos = f.off[blockIdx.y] + (int64_t)blockIdx.x * TILE, left = f.off[blockIdx.y + 1] - pos;
  const int32_t n = left < 0 ? 0 : left < TILE ? (int32_t)left : TILE;
  for (int q = threadIdx.x; q < f.buckets; q += THREADS) s_count[q] = 0;
  __syncthreads();
  uint32_t v[FIT_ITEMS], at[FIT_ITEMS];              // at: bucket << 16 | place among the tile's ids of the bucket
#pragma unroll
  for (int k = 0; k < FIT_ITEMS; ++k) {
    const int32_t x = k * THREADS + threadIdx.x;
    v[k] = x < n ? (uint32_t)ids[pos + x] : 0u;
  }
  if (f.marks) {
    uint32_t old[FIT_ITEMS], fresh = 0;              // (all on their way together)
#pragma unroll
    for (int k = 0; k < FIT_ITEMS; ++k) {
      const uint32_t h = hash_mix(v[k]);
      old[k] = 0xFFFFFFFFu;
      if (k * THREADS + (int32_t)threadIdx.x < n && (h & ((1u << f.mark_shift) - 1u)) == 0)
        old[k] = atomicOr(&f.marks[h >> (32 - FIT_MARK_LOG + 5)], 1u << fit_mark(h));
    }
#pragma unroll
    for (int k = 0; k < FIT_ITEMS; ++k) fresh += !(old[k] >> fit_mark(hash_mix(v[k])) & 1u);
    if (fresh) atomicAdd(&s_new, fresh);
  }
  // Lanes of one bucket count together where a wave has many of them (ids in order, or few buckets): their additions
  // to its counter would follow one another.
  const int lane = lane_id();
  bool together = false;
#pragma unroll
  for (int k = 0; k < FIT_ITEMS; ++k) {
    const bool valid = k * THREADS + (int32_t)threadIdx.x < n;
    uint32_t q = v[k] >> f.shift;
    if (valid && v[k] >= (uint64_t)f.num_nodes) *f.bad = 1;
    if (q >= (uint32_t)f.buckets) q = f.buckets - 1;   // (stays inside the arrays)
    uint64_t left = __ballot(valid);
    if (k == 0) together = __popcll(__ballot(q == __shfl(q, 0)) & left) >= FIT_TOGETHER;
    while (together && left) {
      const int first = __ffsll((unsigned long long)left) - 1;
      const uint32_t q0 = __shfl(q, first);
      const uint64_t same = __ballot(q == q0) & left;
      if (__popcll(same) < FIT_TOGETHER) break;
      uint32_t base = 0;
      if (lane == first) base = atomicAdd(&s_count[q0], (uint32_t)__popcll(same));
      base = __shfl(base, first);
      if (same >> lane & 1) at[k] = q0 << 16 | (base + (uint32_t)__popcll(same & ((1ull << lane) - 1)));
      left &= ~same;
    }
    if (left >> lane & 1) at[k] = q << 16 | atomicAdd(&s_count[q], 1u);
  }
  __syncthreads();
  // (buckets are at most eight to a thread)
  const int32_t per = (f.buckets + THREADS - 1) / THREADS, q0 = threadIdx.x * per;
  uint32_t mine = 0;
  for (int32_t q = q0; q < q0 + per && q < f.buckets; ++q) mine += s_count[q];
  uint32_t total;
  uint32_t run = block_exclusive_scan<uint32_t, THREADS>(mine, smem, total);
  uint16_t* const start = f.start + ((int64_t)blockIdx.y * f.per_iteration + blockIdx.x) * (f.buckets + 1);
  for (int32_t q = q0; q < q0 + per && q < f.buckets; ++q) {
    const uint32_t c = s_count[q];
    s_count[q] = run;
    run += c;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < f.buckets; q += THREADS) start[q] = (uint16_t)s_count[q];
  if (threadIdx.x == 0) {
    start[f.buckets] = (uint16_t)total;
    if (s_new) atomicAdd(f.marked, s_new);
  }
#pragma unroll
  for (int k = 0; k < FIT_ITEMS; ++k) {
    if (k * THREADS + (int32_t)threadIdx.x >= n) continue;
    at[k] = s_count[at[k] >> 16] + (at[k] & 0xFFFFu);
    s_id[at[k]] = v[k];
  }
  __syncthreads();
  for (int32_t x = threadIdx.x; x < n; x += THREADS) f.ids[pos + x] = s_id[x];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < FIT_ITEMS; ++k)
    if (k * THREADS + (int32_t)threadIdx.x < n) s_rank[at[k]] = (uint16_t)(k * THREADS + threadIdx.x);
  __syncthreads();
  for (int32_t x = threadIdx.x; x < n; x += THREADS) f.rank[pos + x] = s_rank[x];
}

// What the two kernels that take a bucket each have in LDS.
struct FitLds {
  uint32_t* bits;            // [words of the bucket] its rows
  uint32_t* row;             // [FIT_ROWS] of a row, by its rank in the bucket: first iteration, or line
  uint32_t* at;              // [FIT_SHARES] a tile's share: its place among all accesses ...
  uint32_t* share;           // [FIT_SHARES] ... entries | iteration << 16
  uint16_t* base;            // [words] rows in front of the word (a bucket has at most 2^16)
  uint32_t* rest;
};
__device__ __forceinline__ FitLds fit_lds(uint32_t* lds, const Fit& f) {
  const int32_t words = 1 << (f.shift - 5);
  uint32_t* const row = lds + words;
  uint32_t* const at = row + FIT_ROWS;
  uint32_t* const base = at + 2 * FIT_SHARES;
  return {lds, row, at, at + FIT_SHARES, reinterpret_cast<uint16_t*>(base), base + words / 2};
}
__device__ __forceinline__ uint32_t fit_rank(const FitLds& l, uint32_t v) {
  return l.base[v >> 5] + __popc(l.bits[v >> 5] & ((1u << (v & 31)) - 1u));
}

// fn(place among all accesses, what is there, iteration) for the bucket's share of every tile, by the block: a share
// (five ids on the mean where there are most buckets) to a group of lanes.
template <typename Fn>
__device__ __forceinline__ void fit_shares(const Fit& f, int32_t q, const FitLds& l, const Fn& fn) {
  constexpr int GROUPS = FIT_LINE_THREADS / FIT_SHARE_LANES, WAVES = FIT_LINE_THREADS / WAVE;
  constexpr int PER_WAVE = WAVE / FIT_SHARE_LANES;
  static_assert(FIT_SHARES == 2 * FIT_LINE_THREADS, "two tiles to a thread");
  const int32_t lane = lane_id(), wave = threadIdx.x / WAVE, sub = lane % FIT_SHARE_LANES, group = lane / FIT_SHARE_LANES;
  // few tiles: neighbouring ones to different waves, and those at the same place of the iterations, too
  const bool few = f.tiles <= GROUPS;
  const int32_t first = few ? group * WAVES + ((wave - 3 * group) & (WAVES - 1)) : group;
  // entries e, e + step, ... of the share at p, below `end`
  auto several = [&](uint32_t p, int32_t e, int32_t end, int32_t step, int32_t i) {
    uint32_t id[FIT_SHARE_ITEMS];
#pragma unroll
    for (int k = 0; k < FIT_SHARE_ITEMS; ++k)
      if (e + k * step < end) id[k] = f.ids[p + e + k * step];
#pragma unroll
    for (int k = 0; k < FIT_SHARE_ITEMS; ++k)
      if (e + k * step < end) fn(p + e + k * step, id[k], i);
  };
  uint32_t at[2], share[2];
  auto request = [&](int32_t t0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int32_t t = t0 + h * FIT_LINE_THREADS + threadIdx.x;
      at[h] = share[h] = 0;
      if (t >= f.tiles) continue;
      const uint16_t* start = f.start + (int64_t)t * (f.buckets + 1) + q;
      const uint32_t lo = start[0], hi = start[1];
      const int32_t i = t / f.per_iteration;
      at[h] = (uint32_t)f.off[i] + (uint32_t)((t - i * f.per_iteration) * f.tile) + lo;
      share[h] = (hi - lo) | (uint32_t)i << 16;
    }
  };
  request(0);
  for (int32_t t0 = 0; t0 < f.tiles; t0 += FIT_SHARES) {
    const int32_t n = f.tiles - t0 < FIT_SHARES ? f.tiles - t0 : FIT_SHARES;
    __syncthreads();                                 // what the calls need is there, the shares are free
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      l.at[h * FIT_LINE_THREADS + threadIdx.x] = at[h];
      l.share[h * FIT_LINE_THREADS + threadIdx.x] = share[h];
    }
    __syncthreads();
    request(t0 + FIT_SHARES);
    // (whole waves; behind the last tile there are empty shares)
    for (int32_t g0 = few ? 0 : wave * PER_WAVE; g0 < n; g0 += GROUPS * FIT_SHARE_ITEMS) {
      const int32_t g = g0 + first;
      uint32_t id[FIT_SHARE_ITEMS], id2[FIT_SHARE_ITEMS], p[FIT_SHARE_ITEMS], sh[FIT_SHARE_ITEMS];
      bool longer = false;
#pragma unroll
      for (int k = 0; k < FIT_SHARE_ITEMS; ++k) {    // (FIT_SHARES is a multiple of the groups' stride)
        p[k] = l.at[g + k * GROUPS] + sub;
        sh[k] = l.share[g + k * GROUPS];
        const int32_t entries = sh[k] & 0xFFFFu;
        if (sub < entries) id[k] = f.ids[p[k]];
        if (sub + FIT_SHARE_LANES < entries) id2[k] = f.ids[p[k] + FIT_SHARE_LANES];
        longer |= entries > 2 * FIT_SHARE_LANES;
      }
#pragma unroll
      for (int k = 0; k < FIT_SHARE_ITEMS; ++k) {
        const int32_t entries = sh[k] & 0xFFFFu, i = sh[k] >> 16;
        if (sub < entries) fn(p[k], id[k], i);
        if (sub + FIT_SHARE_LANES < entries) fn(p[k] + FIT_SHARE_LANES, id2[k], i);
      }
      if (!__any(longer)) continue;
#pragma unroll 1
      for (int k = 0; k < FIT_SHARE_ITEMS; ++k) {
        const uint32_t at = l.at[g + k * GROUPS], share = l.share[g + k * GROUPS];
        const int32_t entries = share & 0xFFFFu, near = entries < FIT_LONG_SHARE ? entries : FIT_LONG_SHARE;
        for (int32_t e = 2 * FIT_SHARE_LANES + sub; e < near; e += FIT_SHARE_LANES * FIT_SHARE_ITEMS)
          several(at, e, near, FIT_SHARE_LANES, share >> 16);
        for (uint64_t left = __ballot(sub == 0 && entries > FIT_LONG_SHARE); left; left &= left - 1) {
          const int from = __ffsll((unsigned long long)left) - 1;
          const uint32_t at2 = __shfl(at, from), share2 = __shfl(share, from);
          const int32_t end = share2 & 0xFFFFu;
          for (int32_t e = FIT_LONG_SHARE + lane; e < end; e += WAVE * FIT_SHARE_ITEMS) several(at2, e, end, WAVE, share2 >> 16);
        }
      }
    }
  }
  __syncthreads();
}
static_assert(FIT_SHARES % (FIT_LINE_THREADS / FIT_SHARE_LANES * FIT_SHARE_ITEMS) == 0, "whole rounds");

// The rows in front of every word, from s_bits; returns their number.
__device__ __forceinline__ uint32_t fit_bases(const Fit& f, const FitLds& l, uint32_t* smem) {
  static_assert((1 << (FIT_SHIFT_MAX - 5)) <= 2 * FIT_LINE_THREADS, "two words to a thread");
  const int32_t w = 2 * threadIdx.x, words = 1 << (f.shift - 5);
  const uint32_t a = w < words ? __popc(l.bits[w]) : 0u, b = w < words ? __popc(l.bits[w + 1]) : 0u;
  uint32_t total;
  const uint32_t at = block_exclusive_scan<uint32_t, FIT_LINE_THREADS>(a + b, smem, total);
  if (w < words) {
    l.base[w] = (uint16_t)at;
    l.base[w + 1] = (uint16_t)(at + a);
  }
  return total;
}

// Where a wave's counters of k_fit_rows sit: 16 bits per iteration, in the room of the shares, so fewer waves rank where
// there are many iterations.
__host__ __device__ __forceinline__ int32_t fit_rank_waves(int32_t S) {
  const int32_t waves = 2 * FIT_SHARES * 2 / S;
  return waves < FIT_LINE_THREADS / WAVE ? waves : FIT_LINE_THREADS / WAVE;
}

__global__ __launch_bounds__(FIT_LINE_THREADS) __attribute__((amdgpu_waves_per_eu(8))) void k_fit_rows(Fit f) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t smem[FIT_LINE_THREADS / WAVE + 1];
  const int32_t q = fit_bucket();
  if (q >= f.buckets) return;
  if (!f.serves()) return;
  const FitLds l = fit_lds(lds, f);
  const int32_t words = 1 << (f.shift - 5);
  const uint32_t mask = (1u << f.shift) - 1u;
  for (int32_t w = threadIdx.x; w < words; w += FIT_LINE_THREADS) l.bits[w] = 0;
  if (q == 0 && threadIdx.x == 0) f.counts[(int64_t)f.S * f.buckets] = 0;
  fit_shares(f, q, l, [&](uint32_t, uint32_t id, int32_t) {
    const uint32_t v = id & mask;
    atomicOr(&l.bits[v >> 5], 1u << (v & 31));
  });
  const int64_t word0 = ((int64_t)q << f.shift) >> 5;
  for (int32_t w = threadIdx.x; w < words; w += FIT_LINE_THREADS) {
    if (word0 + w < f.words) f.bits[word0 + w] = l.bits[w];
    else l.bits[w] = 0;                              // (an id out of range)
  }
  __syncthreads();
  const uint32_t rows = fit_bases(f, l, smem);
  uint32_t* const seen = f.counts + q;               // rows of an iteration, in the slices so far: at seen[i * buckets]
  for (int32_t i = threadIdx.x; i < f.S; i += FIT_LINE_THREADS) seen[(int64_t)i * f.buckets] = 0;
  uint16_t* const s_count = reinterpret_cast<uint16_t*>(l.at);   // [waves][S]
  const int32_t waves = fit_rank_waves(f.S), wave = threadIdx.x / WAVE, lane = lane_id();
  const int32_t bits = 32 - __clz(f.S);
  for (uint32_t from = 0; from < rows; from += FIT_ROWS) {   // more rows than fit LDS: in slices by id
    const int32_t n = rows - from < FIT_ROWS ? (int32_t)(rows - from) : FIT_ROWS;
    for (int32_t r = threadIdx.x; r < n; r += FIT_LINE_THREADS) l.row[r] = 0xFFFFFFFFu;
    fit_shares(f, q, l, [&](uint32_t, uint32_t id, int32_t i) {
      const uint32_t r = fit_rank(l, id & mask) - from;      // (wraps below)
      if (r < (uint32_t)n && l.row[r] > (uint32_t)i) atomicMin(&l.row[r], (uint32_t)i);
    });
    // every row's rank among the rows of its first iteration: a wave takes a stretch of rows, twice, for
    // the iterations' numbers in it and, with those of the stretches in front, for the ranks
    for (int32_t x = threadIdx.x; x < waves * f.S; x += FIT_LINE_THREADS) s_count[x] = 0;
    __syncthreads();
    const int32_t stretch = ((n + waves - 1) / waves + WAVE - 1) / WAVE * WAVE;
    uint16_t* const mine = s_count + wave * f.S;
    for (int pass = 0; pass < 2; ++pass) {
      if (wave < waves)
        for (int32_t r0 = wave * stretch; r0 < (wave + 1) * stretch && r0 < n; r0 += WAVE) {
          const int32_t r = r0 + lane;
          const uint32_t i = r < n ? l.row[r] : 0u;
          uint64_t peers = __ballot(r < n);
          for (int b = 0; b < bits; ++b) {
            const uint64_t m = __ballot((i >> b) & 1);
            peers &= (i >> b) & 1 ? m : ~m;
          }
          if (r < n) {
            const uint32_t before = __popcll(peers & ((1ull << lane) - 1));
            const uint32_t rank = mine[i] + before;  // (read by all lanes before the last of them writes)
            if (before + 1 == (uint32_t)__popcll(peers)) mine[i] = (uint16_t)(rank + 1);
            if (pass) f.list[((int64_t)q << f.shift) + from + r] = i << 16 | rank;
          }
        }
      __syncthreads();
      if (pass) continue;
      for (int32_t i = threadIdx.x; i < f.S; i += FIT_LINE_THREADS) {
        uint32_t run = seen[(int64_t)i * f.buckets];
        for (int32_t w = 0; w < waves; ++w) {
          const uint32_t c = s_count[w * f.S + i];
          s_count[w * f.S + i] = (uint16_t)run;
          run += c;
        }
        seen[(int64_t)i * f.buckets] = run;
      }
      __syncthreads();
    }
  }
}

// ready[i] = rows first accessed in iterations 0..i, FIT_BAD: an id was out of range, FIT_NOT: a bucket is too
// full, or there are too many rows
constexpr int64_t FIT_BAD = -1, FIT_NOT = -2;
struct FitReady {          // with the scan of the counts: the last of an iteration is what all up to it have
  Fit f;
  int64_t* ready;
  __device__ __forceinline__ void operator()(int64_t base, const uint32_t (&v)[SCAN_ITEMS], int64_t n) const {
    int64_t i = (base + f.buckets - 1) / f.buckets, at = i * f.buckets;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
      if (base + k != at || at >= n) continue;
      if (i > 0) ready[i - 1] = *f.bad ? FIT_BAD : !f.serves() ? FIT_NOT : (int64_t)v[k];
      ++i;
      at += f.buckets;
    }
  }
};

constexpr size_t FIT_LDS = 65000;                    // at most (k_fit_lines; iterations: up to some 1 900)
inline size_t fit_rows_lds(const Fit& f) {
  return 6 * ((size_t)1 << (f.shift - 5)) + sizeof(uint32_t) * (FIT_ROWS + 2 * FIT_SHARES);
}
inline size_t fit_lines_lds(const Fit& f) { return fit_rows_lds(f) + sizeof(uint32_t) * f.S; }

// with_lines: C_0 alone, or every access's line, too
__global__ __launch_bounds__(FIT_LINE_THREADS) __attribute__((amdgpu_waves_per_eu(8))) void k_fit_lines(
    Fit f, int32_t* __restrict__ init_ids, bool with_lines) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t smem[FIT_LINE_THREADS / WAVE + 1];
  const int32_t q = fit_bucket();
  if (q >= f.buckets) return;
  const FitLds l = fit_lds(lds, f);
  uint32_t* const s_first = l.rest;                  // [S] line of the bucket's first row of the iteration
  const int32_t words = 1 << (f.shift - 5);
  const uint32_t mask = (1u << f.shift) - 1u;
  const int64_t word0 = ((int64_t)q << f.shift) >> 5;
  for (int32_t w = threadIdx.x; w < words; w += FIT_LINE_THREADS) l.bits[w] = word0 + w < f.words ? f.bits[word0 + w] : 0u;
  for (int32_t i = threadIdx.x; i < f.S; i += FIT_LINE_THREADS) s_first[i] = f.counts[(int64_t)i * f.buckets + q];
  __syncthreads();
  const uint32_t rows = fit_bases(f, l, smem);
  const uint32_t* const list = f.list + ((int64_t)q << f.shift);
  for (uint32_t from = 0; from < rows; from += FIT_ROWS) {   // more rows than fit LDS: in slices by id
    const uint32_t n = rows - from < FIT_ROWS ? rows - from : FIT_ROWS;
    for (uint32_t r = threadIdx.x; r < n; r += FIT_LINE_THREADS) {
      const uint32_t row = list[from + r];
      l.row[r] = s_first[row >> 16] + (row & 0xFFFFu);
    }
    __syncthreads();
    for (int32_t w = threadIdx.x; w < words; w += FIT_LINE_THREADS) {
      uint32_t r = l.base[w] - from;                 // (wraps below)
      for (uint32_t left = l.bits[w]; left; left &= left - 1, ++r)
        if (r < n) init_ids[l.row[r]] = (int32_t)(((uint32_t)q << f.shift) + (uint32_t)(w * 32 + __ffs(left) - 1));
    }
    if (with_lines)                                  // (a line in the place of an id: not an id of a later slice)
      fit_shares(f, q, l, [&](uint32_t at, uint32_t id, int32_t) {
        const uint32_t r = fit_rank(l, id & mask) - from;
        if (r < n && !(id & FIT_DONE)) f.ids[at] = l.row[r] | FIT_DONE;
      });
    __syncthreads();
  }
}

// The lines of the accesses from a table over all nodes, for rows that keep one line (f.bits: rows accessed): the
// bucket's entries go to LDS in id order, not one random word per access.
__global__ __launch_bounds__(FIT_LINE_THREADS) __attribute__((amdgpu_waves_per_eu(8))) void k_fit_lookup(
    Fit f, const int32_t* __restrict__ addr) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t smem[FIT_LINE_THREADS / WAVE + 1];
  const int32_t q = fit_bucket();
  if (q >= f.buckets) return;
  const FitLds l = fit_lds(lds, f);
  const int32_t words = 1 << (f.shift - 5);
  const uint32_t mask = (1u << f.shift) - 1u;
  const int64_t word0 = ((int64_t)q << f.shift) >> 5;
  for (int32_t w = threadIdx.x; w < words; w += FIT_LINE_THREADS) l.bits[w] = word0 + w < f.words ? f.bits[word0 + w] : 0u;
  __syncthreads();
  const uint32_t rows = fit_bases(f, l, smem);
  __syncthreads();
  for (uint32_t from = 0; from < rows; from += FIT_ROWS) {   // more rows than fit LDS: in slices by id
    const uint32_t n = rows - from < FIT_ROWS ? rows - from : FIT_ROWS;
    // the rows' ids first, so that neighbours read neighbouring entries, several at a time
    for (int32_t w = threadIdx.x; w < words; w += FIT_LINE_THREADS) {
      uint32_t r = l.base[w] - from;                 // (wraps below)
      for (uint32_t left = l.bits[w]; left; left &= left - 1, ++r)
        if (r < n) l.row[r] = (uint32_t)(w * 32 + __ffs(left) - 1);
    }
    __syncthreads();
    const int32_t* const entries = addr + ((int64_t)q << f.shift);
    uint32_t line[FIT_ROWS / FIT_LINE_THREADS];
#pragma unroll
    for (int k = 0; k < FIT_ROWS / FIT_LINE_THREADS; ++k)
      if (k * FIT_LINE_THREADS + threadIdx.x < n) line[k] = (uint32_t)entries[l.row[k * FIT_LINE_THREADS + threadIdx.x]];
#pragma unroll
    for (int k = 0; k < FIT_ROWS / FIT_LINE_THREADS; ++k)
      if (k * FIT_LINE_THREADS + threadIdx.x < n) l.row[k * FIT_LINE_THREADS + threadIdx.x] = line[k];
    fit_shares(f, q, l, [&](uint32_t at, uint32_t id, int32_t) {
      const uint32_t r = fit_rank(l, id & mask) - from;
      if (r < n && !(id & FIT_DONE)) f.ids[at] = l.row[r] | FIT_DONE;
    });
  }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_fit_place(Fit f, int32_t* __restrict__ src_line) {
  constexpr int TILE = THREADS * FIT_ITEMS;
  __shared__ uint32_t s_line[TILE];
  const int64_t pos = f.off[blockIdx.y] + (int64_t)blockIdx.x * TILE, left = f.off[blockIdx.y + 1] - pos;
  const int32_t n = left < 0 ? 0 : left < TILE ? (int32_t)left : TILE;
  uint32_t line[FIT_ITEMS], rank[FIT_ITEMS];
#pragma unroll
  for (int k = 0; k < FIT_ITEMS; ++k) {
    const int32_t x = k * THREADS + threadIdx.x;
    if (x < n) {
      line[k] = f.ids[pos + x];
      rank[k] = f.rank[pos + x];
    }
  }
#pragma unroll
  for (int k = 0; k < FIT_ITEMS; ++k)
    if (k * THREADS + (int32_t)threadIdx.x < n)
      s_line[rank[k]] = line[k] == 0xFFFFFFFFu ? line[k] : line[k] & ~FIT_DONE;   // (-1: no line; lines are below 2^31 - 1)
  __syncthreads();
  for (int32_t x = threadIdx.x; x < n; x += THREADS) src_line[pos + x] = (int32_t)s_line[x];
}
