// The evicted rows and their lines on the planned path, without a step per iteration.  Included by changeset.hip only.
//
// Every iteration gives up the n_t dead residents with the largest ids, and which rows die when is known.  So of the
// candidates from number x on, those waiting at the end of iteration t are
//   B_x(t) = max(0, B_x(t - 1) + arrivals_x(t) - n_t),
// whatever the candidates below x are, and the difference of B_x and the next part's says how many an iteration takes
// from one part of PLAN_PART candidates.  The maxima and sums of the iterations are a scan (the steps x -> max(x + c, d)
// compose), and with its numbers known a part is a matter of one wave: k_plan_counts, k_plan_victims.
//
// The lines.  A row has one line, so a victim's is known unless the row was inserted in this call.  k_plan_sort orders
// the known ones of each iteration.  Only where an iteration evicts rows with a line to come and inserts rows that
// are evicted again do iterations wait for each other: k_plan_chain, one workgroup, finds those rows' lines.  k_plan_pairs
// then pairs all evictions of all iterations with the insertions.
//
// 200 iterations of 338 evictions each, 101 000 candidates: one workgroup that went through the iterations, selection,
// ranks and pairing each behind the other's barriers, took 1 318 us (the call 3 920); now k_plan_counts 6, k_plan_victims
// 47 (for the uppermost parts a step of 0.2 us per iteration), k_plan_sort 8, k_plan_chain 87 (two reads and some six
// barriers for each of the iterations that wait), k_plan_pairs 8 (the call 2 805).  The smallest calls have two to four
// launches more, 5 to 10 of 280 us, more than a hundred iterations gain whatever else they hold (256 of 1 000 accesses
// 1 160 -> 580).
#pragma once

constexpr int PLAN_PART = 1024;                        // candidates of a wave
constexpr int PLAN_PARTS = PLAN_CAND_MAX / PLAN_PART;  // at most
constexpr int PLAN_PER_LANE = PLAN_PART / WAVE;
constexpr int PLAN_EPT = PLAN_SORT_MAX / BIG;          // evictions of a thread
constexpr int32_t PLAN_NEW = int32_t(1) << 30;         // flag of a candidate whose line comes with its insertion
static_assert(PLAN_CAND_MAX < PLAN_NEW, "a flag beside the number");

struct Victims {
  int32_t* when;        // [candidates] iteration in which a candidate dies (S: none), then the one that evicts it
  uint32_t* counts;     // [S * parts] rows of this part or above that die in an iteration; unused for one part
  int32_t* list;        // [evictions] candidates by iteration; after k_plan_sort those with known lines first, by line
  int32_t* lines;       // [evictions] the lines of those
  uint32_t* fresh;      // [S] evictions of rows inserted in this call; bit 31: an inserted row is evicted again
  int32_t parts, S;
  int32_t stop;         // iteration in which k_plan_pairs gives up whatever it reads; -1: none
};
constexpr uint32_t PLAN_CHAINED = 1u << 31;

// A block per iteration: its rows that die, by part, summed up from the last part down.
__global__ __launch_bounds__(TB) void k_plan_counts(Plan pl, Victims q, int64_t n_cand) {
  static_assert(PLAN_PARTS == 2 * TB, "two parts to a thread");
  __shared__ uint32_t s_part[PLAN_PARTS];
  __shared__ uint32_t smem[TB / WAVE + 1];
  const int32_t t = blockIdx.x;
  for (int x = threadIdx.x; x < PLAN_PARTS; x += TB) s_part[x] = 0;
  __syncthreads();
  for (uint32_t a = pl.arr_off[t] + threadIdx.x; a < pl.arr_off[t + 1]; a += TB) {
    const int32_t c = pl.arr_cand[a];
    atomicAdd(&s_part[c / PLAN_PART], 1u);
  }
  if (t == 0)           // and those that are dead from the start
    for (int64_t w = threadIdx.x; w < (n_cand + 31) / 32; w += TB)
      if (const uint32_t dead = pl.cand_dead[w]) atomicAdd(&s_part[w / (PLAN_PART / 32)], (uint32_t)__popc(dead));
  __syncthreads();
  const int upper = PLAN_PARTS - 1 - 2 * (int)threadIdx.x;
  const uint32_t c1 = s_part[upper], c0 = s_part[upper - 1];
  uint32_t total;
  const uint32_t above = block_exclusive_scan<uint32_t, TB>(c1 + c0, smem, total);
  uint32_t* const row = q.counts + (int64_t)t * q.parts;
  if (upper < q.parts) row[upper] = above + c1;
  if (upper - 1 < q.parts) row[upper - 1] = above + c1 + c0;
}

// The rows served in iterations t0 .. t0 + 63, one to a lane, from a queue that `waiting` rows stood in before them.
__device__ __forceinline__ int32_t queue_serves(int32_t arrive, int32_t most, int32_t& waiting) {
  int32_t c = arrive - most, d = 0;         // the steps x -> max(x + c, d) of the lanes up to this one
#pragma unroll
  for (int k = 1; k < WAVE; k <<= 1) {
    const int32_t pc = __shfl_up(c, k, WAVE), pd = __shfl_up(d, k, WAVE);
    if (lane_id() >= k) {
      d = pd + c > d ? pd + c : d;
      c += pc;
    }
  }
  const int32_t after = waiting + c > d ? waiting + c : d;
  int32_t before = __shfl_up(after, 1, WAVE);
  if (lane_id() == 0) before = waiting;
  waiting = of_lane(after, WAVE - 1);
  return before + arrive - after;
}

// A wave per part of the candidates: how many of them each iteration takes, and which.
__global__ __launch_bounds__(WAVE) void k_plan_victims(Plan pl, Victims q, int64_t n_cand_tiles,
                                                       const int64_t* __restrict__ cs_offsets) {
  const int32_t S = q.S, part = blockIdx.x, lane = lane_id();
  const int64_t n_cand = pl.cand_tiles[n_cand_tiles];
  const int64_t c0 = (int64_t)part * PLAN_PART + lane * PLAN_PER_LANE;
  int32_t dies[PLAN_PER_LANE];
  uint32_t fresh = 0, gone = 0;
#pragma unroll
  for (int e = 0; e < PLAN_PER_LANE; ++e) {
    const bool is = c0 + e < n_cand;
    dies[e] = is ? q.when[c0 + e] : S;
    fresh |= (is && pl.cand_line[c0 + e] < 0 ? 1u : 0u) << e;
  }
  int32_t waiting = 0, waiting_above = 0;
  bool failed = false;
  for (int32_t t0 = 0; t0 < S; t0 += WAVE) {
    const int32_t t = t0 + lane;
    const int32_t first = t < S ? (int32_t)cs_offsets[t] : 0;
    const int32_t most = t < S ? (int32_t)cs_offsets[t + 1] - first : 0;
    int32_t arrive = 0, arrive_above = 0;
    if (q.parts == 1) {                               // uniform
      if (t < S) arrive = (int32_t)(pl.arr_off[t + 1] - pl.arr_off[t]) + (t == 0 ? (int32_t)pl.scalars[PLAN_M] : 0);
    } else if (t < S) {
      const uint32_t* const row = q.counts + (int64_t)t * q.parts + part;
      arrive = (int32_t)row[0];
      if (part + 1 < q.parts) arrive_above = (int32_t)row[1];
    }
    const int32_t served = queue_serves(arrive, most, waiting);
    const int32_t served_above = queue_serves(arrive_above, most, waiting_above);
    const int32_t mine = served - served_above;
    if (part == 0 && served != most) failed = true;   // cannot happen: the dead rows are enough
    uint64_t todo = __ballot(mine > 0);
    while (todo) {                                    // uniform
      const int j = __ffsll((unsigned long long)todo) - 1;
      todo &= todo - 1;
      const int32_t now = t0 + j, n = of_lane(mine, j), at = of_lane(first + served_above, j);
      uint32_t dead = 0;
#pragma unroll
      for (int e = 0; e < PLAN_PER_LANE; ++e) dead |= (dies[e] <= now ? 1u : 0u) << e;
      dead &= ~gone;
      const int32_t have = __popc(dead);
      const int32_t upto = wave_inclusive_scan(have);
      const int32_t all = of_lane(upto, WAVE - 1), above = all - upto;
      if (all < n) failed = true;                     // cannot happen
      const int32_t take = n - above < have ? n - above : have;
      for (int32_t k = 0; k < take; ++k) {            // the uppermost of the lane's
        const int e = 31 - __clz(dead);
        dead ^= 1u << e;
        gone |= 1u << e;
        q.list[at + above + k] = (int32_t)(c0 + e) | (fresh >> e & 1u ? PLAN_NEW : 0);
        q.when[c0 + e] = now;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < PLAN_PER_LANE; ++e)
    if (c0 + e < n_cand && !(gone >> e & 1u)) q.when[c0 + e] = S;
  if (failed) pl.scalars[PLAN_FAILED] = 1;
}

// Exclusive prefix of v over the BIG threads of the block, and the block total, with a single
// barrier: every thread adds up the totals of the waves in front of its own.  `slots` (one
// per wave) must not be rewritten before a later barrier.
__device__ __forceinline__ uint32_t block_prefix_one_barrier(uint32_t v, uint32_t* slots,
                                                             uint32_t& total) {
  const uint32_t inc = wave_inclusive_scan(v);
  const int w = threadIdx.x / WAVE;
  if (lane_id() == WAVE - 1) slots[w] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < BIG / WAVE; ++q) {
    const uint32_t t = slots[q];
    all += t;
    if (q < w) before += t;
  }
  total = all;
  return before + inc - v;
}

struct RankShared {
  int32_t a[PLAN_SORT_MAX], b[PLAN_SORT_MAX];
  uint32_t slots_a[BIG / WAVE], slots_b[BIG / WAVE];
  int32_t lo[BIG / WAVE], hi[BIG / WAVE];
};

// The rank of each of n different lines among them, up to PLAN_EPT to a thread (-1: none).  All threads of a block of BIG;
// `sh` is free before and, after a barrier of the caller, behind it.
__device__ __forceinline__ void rank_lines(RankShared& sh, int32_t n, const int32_t (&line)[PLAN_EPT],
                                           int32_t (&rank)[PLAN_EPT]) {
  static_assert(BIG + PLAN_SORT_MAX / 2 <= PLAN_SORT_MAX && 2 * BIG <= PLAN_SORT_MAX,
                "the fine buckets and the coarse buckets' records fit the two arrays");
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) rank[e] = 0;
  if (n <= 1) return;                               // uniform
  if (n <= PLAN_RANK_DIRECT) {                      // uniform: every thread counts over all lines
    if (threadIdx.x == 0) sh.slots_a[0] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e)
      if (line[e] >= 0) sh.b[atomicAdd(&sh.slots_a[0], 1u)] = line[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      if (line[e] < 0) continue;
      int32_t r = 0;
      for (int32_t q = 0; q < n; ++q) r += sh.b[q] < line[e];
      rank[e] = r;
    }
    return;
  }
  // Many: the lines are dealt to buckets that grow with the line, a scan of the bucket sizes gives the number of
  // lines in the buckets below, and a line is compared with the members of its own bucket only.  The
  // evicted lines crowd where rows come and go, so buckets of equal width over their range would leave most
  // of them in a few: BIG coarse buckets of equal width are counted first, and a coarse bucket with m
  // members is cut into about m/4 fine ones (a power of two, at most one per line), fewer than BIG + n/2 in
  // all.  a: the fine counters; b: the coarse counts, then first fine bucket and cut of every coarse bucket, then the
  // lines by fine bucket.
  int32_t range_lo = INT32_MAX, range_hi = 0;
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e)
    if (line[e] >= 0) {
      range_lo = line[e] < range_lo ? line[e] : range_lo;
      range_hi = line[e] > range_hi ? line[e] : range_hi;
    }
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) {
    const int32_t olo = __shfl_xor(range_lo, d, WAVE), ohi = __shfl_xor(range_hi, d, WAVE);
    range_lo = olo < range_lo ? olo : range_lo;
    range_hi = ohi > range_hi ? ohi : range_hi;
  }
  if (lane_id() == 0) {
    sh.lo[threadIdx.x / WAVE] = range_lo;
    sh.hi[threadIdx.x / WAVE] = range_hi;
  }
  sh.b[threadIdx.x] = 0;
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) sh.a[threadIdx.x + e * BIG] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < BIG / WAVE; ++q) {
    range_lo = sh.lo[q] < range_lo ? sh.lo[q] : range_lo;
    range_hi = sh.hi[q] > range_hi ? sh.hi[q] : range_hi;
  }
  int coarse_shift = 0;                             // (line - range_lo) >> coarse_shift < BIG
  while (((range_hi - range_lo) >> coarse_shift) >= BIG) ++coarse_shift;
  int32_t coarse[PLAN_EPT], bucket[PLAN_EPT], slot[PLAN_EPT];
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    coarse[e] = bucket[e] = slot[e] = 0;
    if (line[e] < 0) continue;
    coarse[e] = (line[e] - range_lo) >> coarse_shift;
    atomicAdd(&sh.b[coarse[e]], 1);
  }
  __syncthreads();
  {
    const uint32_t members = (uint32_t)sh.b[threadIdx.x];
    int cut = 0;                                    // the coarse bucket becomes 1 << cut fine ones
    while ((4u << cut) < members && cut < coarse_shift) ++cut;
    uint32_t fine_total;
    const uint32_t fine_first = block_prefix_one_barrier(1u << cut, sh.slots_a, fine_total);
    sh.b[threadIdx.x] = (int32_t)fine_first;        // (only this thread read the entry)
    sh.b[BIG + threadIdx.x] = cut;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    if (line[e] < 0) continue;
    const int cut = sh.b[BIG + coarse[e]];
    const int32_t within = (line[e] - range_lo) & ((1 << coarse_shift) - 1);
    bucket[e] = sh.b[coarse[e]] + (within >> (coarse_shift - cut));
    slot[e] = atomicAdd(&sh.a[bucket[e]], 1);
  }
  __syncthreads();
  {
    uint32_t count[PLAN_EPT], sum = 0;
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      count[e] = (uint32_t)sh.a[threadIdx.x * PLAN_EPT + e];
      sum += count[e];
    }
    uint32_t all;
    uint32_t run = block_prefix_one_barrier(sum, sh.slots_b, all);
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      sh.a[threadIdx.x * PLAN_EPT + e] = (int32_t)run;
      run += count[e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e)
    if (line[e] >= 0) sh.b[sh.a[bucket[e]] + slot[e]] = line[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    if (line[e] < 0) continue;
    const int32_t first = sh.a[bucket[e]];
    const int32_t end = bucket[e] + 1 < PLAN_SORT_MAX ? sh.a[bucket[e] + 1] : n;
    int32_t r = first;
    for (int32_t q = first; q < end; ++q) r += sh.b[q] < line[e];
    rank[e] = r;
  }
}

// how many of n ascending values are below x
__device__ __forceinline__ int32_t how_many_below(const int32_t* sorted, int32_t n, int32_t x) {
  int32_t lo = 0, hi = n;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (sorted[mid] < x) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// A block per iteration: its victims with known lines in the order of these, in front of the others.  An inserted
// row's number is kept (Plan::ins_cand) where the row is evicted again only, and if all lines are known it gets its own here.
__global__ __launch_bounds__(BIG) void k_plan_sort(Plan pl, Victims q, const int64_t* __restrict__ cs_offsets) {
  __shared__ RankShared sh;
  __shared__ int32_t s_fresh, s_chained;
  const int32_t t = blockIdx.x, first = (int32_t)cs_offsets[t], n = (int32_t)cs_offsets[t + 1] - first;
  if (n == 0 || pl.scalars[PLAN_FAILED]) {          // uniform
    if (threadIdx.x == 0) q.fresh[t] = 0;
    return;
  }
  if (threadIdx.x == 0) s_fresh = s_chained = 0;
  __syncthreads();
  int32_t cand[PLAN_EPT], line[PLAN_EPT], rank[PLAN_EPT], slot[PLAN_EPT];
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    const int32_t k = threadIdx.x + e * BIG;
    cand[e] = k < n ? q.list[first + k] : -1;
    line[e] = slot[e] = -1;
    if (cand[e] >= 0 && !(cand[e] & PLAN_NEW)) line[e] = pl.cand_line[cand[e]];
    if (cand[e] >= 0 && (cand[e] & PLAN_NEW)) slot[e] = atomicAdd(&s_fresh, 1);
    int32_t again = k < n ? pl.ins_cand[first + k] : -1;
    if (again >= 0) {
      if (q.when[again] < q.S) s_chained = 1;
      else pl.ins_cand[first + k] = -1;
    }
  }
  __syncthreads();
  const int32_t fresh = s_fresh, known = n - fresh;
  rank_lines(sh, known, line, rank);
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    if (slot[e] >= 0) q.list[first + known + slot[e]] = cand[e] & ~PLAN_NEW;
    if (line[e] < 0) continue;
    q.list[first + rank[e]] = cand[e];
    q.lines[first + rank[e]] = line[e];
    if (!s_chained || fresh) continue;              // uniform
    const int32_t again = pl.ins_cand[first + rank[e]];
    if (again >= 0 && q.when[again] < q.S) pl.cand_line[again] = line[e];
  }
  if (threadIdx.x == 0) q.fresh[t] = (uint32_t)fresh | (s_chained ? PLAN_CHAINED : 0u);
}

// One block: the lines of inserted rows that are evicted again, iteration by iteration where one waits for another.
// What an iteration reads besides the lines that come is asked for an iteration ahead.
__global__ __launch_bounds__(BIG) void k_plan_chain(Plan pl, Victims q, const int64_t* __restrict__ cs_offsets) {
  __shared__ RankShared sh;
  __shared__ int32_t s_known[PLAN_SORT_MAX];        // known lines of the iteration, ascending
  __shared__ int32_t s_come[PLAN_SORT_MAX], s_at[PLAN_SORT_MAX];   // the others, ascending, and their ranks among all
  __shared__ uint16_t s_todo[PLAN_S_MAX];
  __shared__ int32_t s_count, s_failed;
  if (pl.scalars[PLAN_FAILED]) return;              // uniform
  // the iterations with both, in order
  if (threadIdx.x == 0) s_count = s_failed = 0;
  __syncthreads();
  for (int32_t t0 = 0; t0 < q.S; t0 += BIG) {
    const int32_t t = t0 + threadIdx.x;
    const uint32_t w = t < q.S ? q.fresh[t] : 0u;
    const bool todo = (w & PLAN_CHAINED) && (w & ~PLAN_CHAINED);
    uint32_t total;
    const uint32_t before = block_prefix_one_barrier(todo ? 1u : 0u, sh.slots_a, total);
    if (todo) s_todo[s_count + before] = (uint16_t)t;
    __syncthreads();
    if (threadIdx.x == 0) s_count += (int32_t)total;
    __syncthreads();
  }
  const int32_t count = s_count;
  int32_t next_cand[PLAN_EPT], next_known[PLAN_EPT], next_again[PLAN_EPT];
  int32_t next_first = 0, next_n = 0, next_fresh = 0;
  auto ask = [&](int32_t x) {
    const int32_t t = s_todo[x];
    next_first = (int32_t)cs_offsets[t];
    next_n = (int32_t)cs_offsets[t + 1] - next_first;
    next_fresh = (int32_t)(q.fresh[t] & ~PLAN_CHAINED);
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      const int32_t k = threadIdx.x + e * BIG;
      next_known[e] = k < next_n - next_fresh ? q.lines[next_first + k] : -1;
      next_cand[e] = k < next_fresh ? q.list[next_first + next_n - next_fresh + k] : -1;
      next_again[e] = k < next_n ? pl.ins_cand[next_first + k] : -1;
    }
  };
  if (count > 0) ask(0);
  for (int32_t x = 0; x < count; ++x) {
    const int32_t fresh = next_fresh, known = next_n - next_fresh;
    int32_t line[PLAN_EPT], again[PLAN_EPT], rank[PLAN_EPT];
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      const int32_t k = threadIdx.x + e * BIG;
      line[e] = -1;
      if (next_cand[e] >= 0 && (line[e] = pl.cand_line[next_cand[e]]) < 0) s_failed = s_todo[x] + 1;   // cannot happen
      again[e] = next_again[e];
      if (next_known[e] >= 0) s_known[k] = next_known[e];
    }
    if (x + 1 < count) ask(x + 1);
    __syncthreads();
    if (s_failed) break;                            // uniform
    rank_lines(sh, fresh, line, rank);
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      if (line[e] < 0) continue;
      s_come[rank[e]] = line[e];
      s_at[rank[e]] = rank[e] + how_many_below(s_known, known, line[e]);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      if (again[e] < 0) continue;
      const int32_t k = threadIdx.x + e * BIG;
      const int32_t j = how_many_below(s_at, fresh, k);
      pl.cand_line[again[e]] = j < fresh && s_at[j] == k ? s_come[j] : s_known[k - j];
    }
    __syncthreads();                                // also makes these visible to the block's later reads
  }
  if (threadIdx.x == 0 && s_failed) {
    pl.scalars[PLAN_FAILED] = 2;
    pl.scalars[PLAN_WHERE] = s_failed - 1;
  }
}

// A block per iteration: its evictions in line order, and the insertions that take the lines.
__global__ __launch_bounds__(BIG) void k_plan_pairs(State st, Plan pl, Victims q,
                                                    const int64_t* __restrict__ cs_offsets,
                                                    const int32_t* __restrict__ in_ids,
                                                    int32_t* __restrict__ out_ids) {
  __shared__ RankShared sh;
  __shared__ int32_t s_known[PLAN_SORT_MAX], s_come[PLAN_SORT_MAX];
  __shared__ int32_t s_given_up, s_failed;
  const int32_t t = blockIdx.x, first = (int32_t)cs_offsets[t], n = (int32_t)cs_offsets[t + 1] - first;
  // (read once: other blocks of this launch may set it, and threads that read different values would part at a barrier)
  if (threadIdx.x == 0) {
    s_given_up = pl.scalars[PLAN_FAILED] != 0;
    s_failed = 0;
  }
  __syncthreads();
  if (n == 0 || s_given_up) return;                 // uniform
  if (t == q.stop) {
    if (threadIdx.x == 0) {
      pl.scalars[PLAN_FAILED] = 3;
      pl.scalars[PLAN_WHERE] = t;
    }
    return;
  }
  const int32_t fresh = (int32_t)(q.fresh[t] & ~PLAN_CHAINED), known = n - fresh;
  int32_t cand[PLAN_EPT], line[PLAN_EPT], rank[PLAN_EPT];
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    const int32_t k = threadIdx.x + e * BIG;
    cand[e] = k < n ? q.list[first + k] : -1;
    line[e] = k < known ? q.lines[first + k] : -1;
    rank[e] = k;
  }
  if (fresh > 0) {                                  // uniform
    int32_t come[PLAN_EPT], among[PLAN_EPT];
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      const int32_t k = threadIdx.x + e * BIG;
      come[e] = k >= known && k < n ? pl.cand_line[cand[e]] : -1;
      if (k >= known && k < n && come[e] < 0) s_failed = 1;   // cannot happen
      if (line[e] >= 0) s_known[k] = line[e];
    }
    __syncthreads();
    if (s_failed) {                                 // uniform
      if (threadIdx.x == 0) {
        pl.scalars[PLAN_FAILED] = 2;
        pl.scalars[PLAN_WHERE] = t;
      }
      return;
    }
    rank_lines(sh, fresh, come, among);
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e)
      if (come[e] >= 0) s_come[among[e]] = come[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PLAN_EPT; ++e) {
      if (come[e] >= 0) {
        line[e] = come[e];
        rank[e] = among[e] + how_many_below(s_known, known, come[e]);
      } else if (line[e] >= 0) {
        rank[e] += how_many_below(s_come, fresh, line[e]);
      }
    }
  }
  int32_t comes[PLAN_EPT], goes[PLAN_EPT], again[PLAN_EPT];
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    const bool is = cand[e] >= 0;
    comes[e] = is ? in_ids[first + rank[e]] : 0;
    again[e] = is ? pl.ins_cand[first + rank[e]] : 0;
    goes[e] = is ? pl.cand_id[cand[e]] : 0;
  }
#pragma unroll
  for (int e = 0; e < PLAN_EPT; ++e) {
    if (cand[e] < 0) continue;
    out_ids[first + rank[e]] = goes[e];
    st.addr[comes[e]] = line[e];
    if (again[e] < 0) st.res_id[line[e]] = comes[e];   // (a line that is given up again: by the last to take it)
  }
}
