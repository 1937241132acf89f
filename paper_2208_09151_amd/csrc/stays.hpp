// Belady changesets from the trace alone (Ginex Section 3.4), for a cache that is smaller than
// the distinct rows of the superbatch.  Included by changeset.hip only.
//
// A stay is the time between two accesses of a row, from iteration i to iteration j (j = S: the
// row is not accessed again; i = "start": the row is in the start state).  During its stay the
// row's key is j.  k_static_roll knows, before anything is simulated, the threshold bucket j*_t
// of every iteration t and how many rows it drops from that bucket (rem_t), so
//   * a stay ends at the first t in [i, j) with j*_t < j, whatever the cache holds,
//   * only where j*_t = j and rem_t > 0 the row is in the bucket that is cut, and there its
//     class (incoming rows go first) and its id decide.
// A table over (j, i) holds both the first t with j*_t < j and the first cut of bucket j from i on;
// a cut is three words (kind, id limit T, nothing else).  Cuts of different iterations depend on
// each other only through the accesses of iteration t itself (which of them hit: cuts of bucket
// t) and through earlier cuts of the same bucket, so they are decided in a few levels of
// independent cuts instead of one after the other.  The cuts of bucket "never" (j* = S, most of the
// last iterations) decide no hit and no insertion; they follow after the others, see below.
// With all cuts decided, hits, misses, insertions and the iteration that evicts every row
// follow for all accesses at once, and the only thing left that is sequential is which line
// an inserted row gets: lines.hpp.
// Before, an iteration was four launches that passed over its accesses and over all lines.
//
// LRU goes the same way with other thresholds, see "LRU" below.
//
// 200 iterations of 163 840 accesses, 111 M nodes, every iteration evicts: that loop 200 x 41 us, and
// 0.83 ms to look right.  Here: k_stay_ends 0.49 ms (scattered words), k_key_hists 0.05,
// k_static_roll 0.13, 17 levels of k_cut_members + k_cut_decide 0.023 + 0.010 each (two chains of
// dependent reads), k_stays_mark 0.14 (random words of the table, L2), k_stays_links 0.28 (one random
// word per pair, 117 G/s), bucket "never" 0.11, k_stays_walk 0.43, k_ins_emit 0.05, k_move_lines 0.83.
#pragma once

constexpr int STATIC_S_MAX = 2048;      // iterations up to which the (S + 1) x S table is kept
enum { CUT_NONE = 0,      // nothing is dropped from bucket j*
       CUT_IN_SOME = 1,   // incoming rows of the bucket with an id above T
       CUT_IN_ALL = 2,    // all incoming rows of the bucket
       CUT_RES = 3 };     // all incoming rows, and residents of the bucket with an id above T

struct Cut {              // one per iteration
  int32_t jstar;          // threshold bucket, S + 1: the iteration drops nothing
  int32_t rem;            // rows to drop from it
  int32_t kind;           // CUT_*
  int32_t T;              // (until it is decided: the bucket's members, as the thresholds have them)
  uint32_t n_res, n_in;   // members of the bucket by class, while the cut is decided;
                          // bucket "never": the part of the ids that is cut, rows that stay in it
};

// The ends of an access's two stays in one word: where and when the row was accessed before, when
// it is accessed next.  Bit 63: the cut of this access's own iteration dropped it.
constexpr uint32_t FROM_START = 0xFFFEu;    // no earlier access, but the start state holds the row
constexpr uint32_t NO_STAY = 0xFFFFu;       // no earlier access: a miss
constexpr uint64_t BYPASSED = 1ull << 63;
constexpr uint32_t NO_CUT = 0xFFFFu;        // in the table: no cut ahead

__device__ __forceinline__ uint32_t stay_prev_pos(uint64_t w) { return (uint32_t)w; }
__device__ __forceinline__ uint32_t stay_prev(uint64_t w) { return (uint32_t)(w >> 32) & 0xFFFFu; }
__device__ __forceinline__ int32_t stay_next(uint64_t w) { return (int32_t)(w >> 48) & 0x7FFF; }

struct Stays {
  uint64_t* ends;          // [total] see above (free once the insertions are marked)
  const int64_t* off;      // [S + 1]
  const int32_t* ids;      // [total]
  const uint32_t* table;   // [(S + 1) * S]
  Cut* cuts;               // [S]
  int32_t* members;        // [total] members of the buckets that are being cut, bucket j at off[j]
  const int32_t* never;    // [NEVER_LEVELS * (S + 1)] see k_never_lift
  const uint64_t* limits;  // [S] LRU, see below
  int32_t S, id_bits;      // ids are below 2^id_bits
};

// Is the row of a run head (first access of its row, in iteration `first`) in the start state?
// Fresh superbatch: C_0 is the `cap` smallest (first access, id), the last of them *last_head.
// Carried cache: the bitmap of the rows it holds says.
__device__ __forceinline__ bool in_start_state(uint32_t v, int32_t first, const uint64_t* last_head,
                                               const uint32_t* held) {
  return last_head ? (((uint64_t)(uint32_t)first << 32) | v) <= *last_head : held[v >> 5] >> (v & 31) & 1u;
}

// One pass over the node-sorted pairs: the ends of every access's stays, written at its position
// (one scattered word per access; bound by that store).  A wave takes LOOK_ITEMS * 64 consecutive pairs
// and passes positions and iterations on to the neighbours, so that each is read and searched once.
// For up to 2^26 accesses, or where the results have no room between two kernels (see deal.hpp).
// Scattered words are collected in the 256 MB memory-side cache as long as the window of positions
// [from, to) that a launch writes fits there (33 M accesses: 0.50 ms, 66 G words/s); beyond it they go
// to memory one by one (154 M: 6.1 ms, 25 G/s).  So one launch per ENDS_WINDOW positions, each reading
// all pairs: 154 M in 4.5 ms (windows of 80 M: 5.3, of 20 M: 4.6, of 10 M: 8.1).  That reading grows with
// the square of the accesses, so beyond ENDS_WINDOWS_MAX windows there is one (290 M: 9 windows 11.8 ms,
// one 12.7; 600 M: 18 windows 36.1, one 27.3; 1 000 M: 30 windows 85.2, one 46.4).
constexpr int64_t ENDS_WINDOW = int64_t(1) << 25;
constexpr int64_t ENDS_WINDOWS_MAX = 9;
__global__ __launch_bounds__(TB) void k_stay_ends(const uint64_t* __restrict__ sorted, int64_t n,
                                                  const int64_t* __restrict__ off, int32_t S,
                                                  const uint64_t* __restrict__ last_head,
                                                  const uint32_t* __restrict__ held, uint32_t from,
                                                  uint32_t to, uint64_t* __restrict__ ends) {
  extern __shared__ int32_t lds_off[];
  load_offsets(lds_off, off, S);
  const int lane = lane_id();
  const int64_t base = (int64_t)blockIdx.x * LOOK_TILE + (threadIdx.x / WAVE) * (WAVE * LOOK_ITEMS);
  if (base >= n) return;                           // uniform over the wave
  // behind n: an id that no access has; chunk LOOK_ITEMS holds the pair behind the stretch
  uint64_t cur[LOOK_ITEMS + 1];
#pragma unroll
  for (int k = 0; k <= LOOK_ITEMS; ++k) {
    const int64_t x = base + k * WAVE + (k < LOOK_ITEMS ? lane : 0);
    cur[k] = x < n ? sorted[x] : ~0ull;
  }
  uint64_t before = base > 0 ? sorted[base - 1] : ~0ull;
  int32_t it[LOOK_ITEMS + 1];
#pragma unroll
  for (int k = 0; k <= LOOK_ITEMS; ++k)
    it[k] = (cur[k] >> 32) != 0xFFFFFFFFull ? iter_of(lds_off, S, (int32_t)(uint32_t)cur[k]) : S;
  int32_t before_it = (before >> 32) != 0xFFFFFFFFull ? iter_of(lds_off, S, (int32_t)(uint32_t)before) : S;
#pragma unroll
  for (int k = 0; k < LOOK_ITEMS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    uint32_t lv = from_left(v), lp = from_left(p), rv = from_right(v);
    int32_t li = from_left(it[k]), ri = from_right(it[k]);
    const uint32_t ov = of_lane((uint32_t)(cur[k + 1] >> 32), 0);
    const int32_t oi = of_lane(it[k + 1], 0);
    if (lane == 0) {
      lv = (uint32_t)(before >> 32);
      lp = (uint32_t)before;
      li = before_it;
    }
    if (lane == WAVE - 1) {
      rv = ov;
      ri = oi;
    }
    before = of_lane(cur[k], WAVE - 1);
    before_it = of_lane(it[k], WAVE - 1);
    if (base + k * WAVE + lane >= n || p < from || p >= to) continue;
    uint32_t prev_pos = 0, prev = NO_STAY;
    if (lv == v) {
      prev_pos = lp;
      prev = (uint32_t)li;
    } else if (in_start_state(v, it[k], last_head, held)) {
      prev = FROM_START;
    }
    const uint32_t next = rv == v ? (uint32_t)ri : (uint32_t)S;
    ends[p] = ((uint64_t)next << 48) | ((uint64_t)prev << 32) | prev_pos;
  }
}

// The same dealt by windows of positions (see deal.hpp): place in the window, next (12 bits: S is at most 2 048),
// previous access (its position + 2, or one of the two below).  The iteration of the previous access is
// searched anew when the word is put to its place.
constexpr uint32_t DEAL_NO_STAY = 0, DEAL_FROM_START = 1;

__global__ __launch_bounds__(DEAL_THREADS) void k_stay_deal(const uint64_t* __restrict__ sorted, int64_t n,
                                                            const int64_t* __restrict__ off, int32_t S,
                                                            const uint64_t* __restrict__ last_head,
                                                            const uint32_t* __restrict__ held, Dealt d) {
  __shared__ DealShared sh;
  __shared__ int32_t lds_off[STATIC_S_MAX + 1];
  __shared__ uint16_t s_coarse[IterFinder::COARSE + 1];
  deal_clear(d, sh);
  const IterFinder find = iter_finder(lds_off, s_coarse, off, S);
  const int lane = lane_id();
  const int64_t base = (int64_t)blockIdx.x * DEAL_TILE + (threadIdx.x / WAVE) * (WAVE * DEAL_ITEMS);
  uint64_t cur[DEAL_ITEMS + 1];                    // as in k_stay_ends
#pragma unroll
  for (int k = 0; k <= DEAL_ITEMS; ++k) {
    const int64_t x = base + k * WAVE + (k < DEAL_ITEMS ? lane : 0);
    cur[k] = x < n ? sorted[x] : ~0ull;
  }
  uint64_t before = base > 0 && base - 1 < n ? sorted[base - 1] : ~0ull;
  auto iteration = [&](uint64_t pair) { return (pair >> 32) != 0xFFFFFFFFull ? find((uint32_t)pair) : S; };
  uint32_t at[DEAL_ITEMS];
  uint64_t word[DEAL_ITEMS];
  int32_t it = iteration(cur[0]);
#pragma unroll
  for (int k = 0; k < DEAL_ITEMS; ++k) {
    const int32_t it_next = iteration(cur[k + 1]);
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    const bool valid = base + k * WAVE + lane < n;
    uint32_t lv = from_left(v), lp = from_left(p), rv = from_right(v);
    int32_t ri = from_right(it);
    const uint32_t ov = of_lane((uint32_t)(cur[k + 1] >> 32), 0);
    const int32_t oi = of_lane(it_next, 0);
    if (lane == 0) {
      lv = (uint32_t)(before >> 32);
      lp = (uint32_t)before;
    }
    if (lane == WAVE - 1) {
      rv = ov;
      ri = oi;
    }
    before = of_lane(cur[k], WAVE - 1);
    uint32_t prev = DEAL_NO_STAY;
    if (lv == v) prev = lp + 2;
    else if (valid && in_start_state(v, it, last_head, held)) prev = DEAL_FROM_START;
    const uint32_t next = rv == v ? (uint32_t)ri : (uint32_t)S;
    word[k] = (uint64_t)(p & ((1u << WINDOW_SHIFT) - 1u)) << 44 | (uint64_t)next << 32 | prev;
    at[k] = valid ? deal_place(sh, p) : NOT_DEALT;
    it = it_next;
  }
  deal_out(d, sh, word, at);
}

struct PutEnds {
  uint64_t* ends;
  const int64_t* off;
  int32_t S;
  __device__ __forceinline__ void operator()(int64_t first, uint64_t word, const IterFinder& iteration) const {
    const uint32_t code = (uint32_t)word;
    uint32_t prev_pos = 0, prev = code == DEAL_NO_STAY ? NO_STAY : FROM_START;
    if (code > DEAL_FROM_START) {
      prev_pos = code - 2;
      prev = (uint32_t)iteration(prev_pos);
    }
    ends[first + (int64_t)(word >> 44)] = ((word >> 32 & 0xFFFu) << 48) | ((uint64_t)prev << 32) | prev_pos;
  }
};

// table[j][s], for a stay that ends at j and is followed from iteration s on: low half the first
// t in [s, j) with j*_t < j (j if there is none), high half the first cut of bucket j in front of
// that (NO_CUT).  One thread per j walks backwards; s >= j reads "reaches j".
__global__ __launch_bounds__(WAVE) void k_stay_table(const Cut* __restrict__ cuts, int32_t S,
                                                     uint32_t* __restrict__ table) {
  extern __shared__ int32_t lds_js[];    // [S] j*, with the sign bit where nothing is cut
  for (int t = threadIdx.x; t < S; t += WAVE)
    lds_js[t] = cuts[t].rem > 0 ? cuts[t].jstar : ~cuts[t].jstar;
  __syncthreads();
  const int32_t j = blockIdx.x * WAVE + threadIdx.x;
  if (j > S) return;
  uint32_t end = (uint32_t)j, cut = NO_CUT;
  for (int32_t t = S - 1; t >= 0; --t) {
    if (t < j) {
      const int32_t raw = lds_js[t];
      const int32_t jstar = raw < 0 ? ~raw : raw;
      if (jstar < j) {
        end = (uint32_t)t;
        cut = NO_CUT;
      } else if (raw == j) {
        cut = (uint32_t)t;
      }
    }
    table[(int64_t)j * S + t] = (cut << 16) | end;
  }
}

// The iteration that drops row v during its stay [i, j), j if none does; cuts from `limit` on are
// not looked at (they may not have been decided yet).  own: the access that began the stay, as a
// word of `ends` (its BYPASSED bit is read only if the cut of its own iteration is in bucket j).  w: the
// table's word for them.
__device__ __forceinline__ uint32_t stay_word(const Stays& q, uint32_t i, int32_t j) {
  return q.table[(int64_t)j * q.S + (i >= FROM_START ? 0u : i)];
}
__device__ __forceinline__ int32_t stay_end(const Stays& q, uint32_t w, uint32_t i, int32_t j, uint32_t v,
                                            const uint64_t* own, int32_t limit) {
  const uint32_t* row = q.table + (int64_t)j * q.S;
  uint32_t t = w >> 16;
  while (t != NO_CUT && (int32_t)t < limit) {
    const Cut c = q.cuts[t];
    if (c.kind == CUT_RES && (int32_t)v > c.T) return (int32_t)t;
    if (t == i && own && (*own & BYPASSED)) return (int32_t)t;
    if ((int32_t)t + 1 >= j) break;
    t = row[t + 1] >> 16;
  }
  return (int32_t)(w & 0xFFFFu);
}

__device__ __forceinline__ int32_t stay_end(const Stays& q, uint32_t i, int32_t j, uint32_t v,
                                            const uint64_t* own, int32_t limit) {
  return stay_end(q, stay_word(q, i, j), i, j, v, own, limit);
}

// Rows that are never accessed again sit in the bucket that most of the last iterations cut, so
// their stays would meet cut after cut (108 of 200 iterations for a cache that holds two fifths of the
// rows).  never[0][t]: ids above it leave that bucket in iteration t (-1: all of them);
// never[k][t]: the smallest of 2^k entries from t on, so that the first iteration that drops a row is
// found in NEVER_LEVELS steps (15.0 -> 3.5 ms for k_stays_walk on 154 M accesses).
constexpr int NEVER_LEVELS = 12;   // 2^12 > STATIC_S_MAX

__global__ __launch_bounds__(BIG) void k_never_lift(const Cut* __restrict__ cuts, int32_t S,
                                                    int32_t* __restrict__ never) {
  for (int32_t t = threadIdx.x; t <= S; t += BIG) {
    int32_t T = -1;                 // t = S: the end of the superbatch stops every search
    if (t < S) {
      const Cut c = cuts[t];
      T = c.jstar < S ? -1 : c.jstar == S && c.kind == CUT_RES ? c.T : INT32_MAX;
    }
    never[t] = T;
  }
  for (int k = 1; k < NEVER_LEVELS; ++k) {
    __syncthreads();
    const int32_t* below = never + (int64_t)(k - 1) * (S + 1);
    for (int32_t t = threadIdx.x; t <= S; t += BIG) {
      const int32_t u = t + (1 << (k - 1));
      const int32_t a = below[t], b = below[u < S ? u : S];
      never[(int64_t)k * (S + 1) + t] = a < b ? a : b;
    }
  }
}

// The iteration that drops row v, resident and never accessed again from iteration i on; S if none.
// `never`: the array, or a copy of it in LDS; levels: as many as S needs.
__device__ __forceinline__ int32_t never_end(const int32_t* never, int32_t S, int levels, int32_t i, uint32_t v) {
  int32_t t = i;
  for (int k = levels - 1; k >= 0; --k)
    if (t + (1 << k) <= S && never[k * (S + 1) + t] >= (int32_t)v) t += 1 << k;
  return t;
}

__device__ __forceinline__ int never_levels(int32_t S) { return 32 - __clz(S); }   // 2^levels > S

// Does the access with these ends (iteration j, row v; w as above) hit?
__device__ __forceinline__ bool stay_hits(const Stays& q, uint32_t w, uint64_t ends, int32_t j, uint32_t v) {
  const uint32_t prev = stay_prev(ends);
  if (prev == NO_STAY) return false;
  return stay_end(q, w, prev, j, v, prev == FROM_START ? nullptr : &q.ends[stay_prev_pos(ends)], j) == j;
}

// Is a miss of an iteration with cut c, next accessed in iteration `next`, inserted?  (One that is never
// accessed again is not: where bucket "never" is cut, the iteration drops as many rows as it has
// misses, incoming rows of the bucket first.)
__device__ __forceinline__ bool stay_inserts(const Stays& q, const Cut& c, int32_t next, uint32_t v) {
  return next < c.jstar ? next < q.S
                        : next == c.jstar && next < q.S &&
                              (c.kind == CUT_NONE || (c.kind == CUT_IN_SOME && (int32_t)v <= c.T));
}

// ---- the cuts -----------------------------------------------------------------------------------

constexpr int CUT_ITEMS = 8;
constexpr int CUT_TILE = TB * CUT_ITEMS;

// The iterations of a level's cuts: in the launch's arguments as far as they have room (a copy to the device is a
// launch's time and a wait), else in memory.
struct Jobs {
  static constexpr int MOST = 96;
  const int32_t* far;                  // null: near
  int16_t near[MOST];                  // (iterations are at most STATIC_S_MAX)
  __device__ __forceinline__ int32_t operator[](int k) const { return far ? far[k] : near[k]; }
};

// Members of the buckets of a level's cuts (blockIdx.y = cut, jobs[] its iteration): the accesses of
// iteration j whose row is resident since before t (class resident), and the accesses of
// iteration t with key j (resident if they hit, else incoming).  Both lists are kept, residents as
// ids from the front of bucket j's region, incoming rows as positions from its end.
__global__ __launch_bounds__(TB) void k_cut_members(Stays q, Jobs jobs) {
  __shared__ uint32_t smem[TB / WAVE + 1];
  __shared__ uint32_t s_at[2];
  const int32_t t = jobs[blockIdx.y];
  Cut* cut = &q.cuts[t];
  const int32_t j = cut->jstar;
  const int64_t base = (int64_t)blockIdx.x * CUT_TILE;
  const int64_t jo = q.off[j], nj = q.off[j + 1] - jo, to = q.off[t], nt = q.off[t + 1] - to;
  if (base >= nj + nt) return;                    // uniform
  uint64_t w[CUT_ITEMS];
  uint32_t v[CUT_ITEMS], kind[CUT_ITEMS];         // kind 1: resident, 2: incoming
  uint32_t n_res = 0, n_in = 0;
#pragma unroll
  for (int k = 0; k < CUT_ITEMS; ++k) {
    int64_t x = base + k * TB + threadIdx.x;
    x = x < nj + nt ? x : base;
    const int64_t p = x < nj ? jo + x : to + (x - nj);
    w[k] = q.ends[p];
    v[k] = (uint32_t)q.ids[p];
  }
#pragma unroll
  for (int k = 0; k < CUT_ITEMS; ++k) {
    const int64_t x = base + k * TB + threadIdx.x;
    kind[k] = 0;
    if (x >= nj + nt) continue;
    if (x < nj) {                                 // an access that ends a stay with key j
      const uint32_t prev = stay_prev(w[k]);
      if (prev == NO_STAY || (prev != FROM_START && (int32_t)prev >= t)) continue;
      const int32_t end = stay_end(q, prev, j, v[k],
                                   prev == FROM_START ? nullptr : &q.ends[stay_prev_pos(w[k])], t);
      kind[k] = end >= t ? 1u : 0u;
    } else if (stay_next(w[k]) == j) {            // an access of iteration t that begins one
      kind[k] = stay_hits(q, stay_word(q, stay_prev(w[k]), t), w[k], t, v[k]) ? 1u : 2u;
      if (kind[k] == 2) v[k] = (uint32_t)(to + (x - nj));
    }
    n_res += kind[k] == 1;
    n_in += kind[k] == 2;
  }
  // one reservation per block and class
  uint32_t tot_res, tot_in;
  uint32_t at_res = block_exclusive_scan<uint32_t, TB>(n_res, smem, tot_res);
  uint32_t at_in = block_exclusive_scan<uint32_t, TB>(n_in, smem, tot_in);
  if (threadIdx.x == 0) {
    s_at[0] = tot_res ? atomicAdd(&cut->n_res, tot_res) : 0u;
    s_at[1] = tot_in ? atomicAdd(&cut->n_in, tot_in) : 0u;
  }
  __syncthreads();
  at_res += s_at[0];
  at_in += s_at[1];
  // (distinct ids inside an iteration give at most nj members; the bound keeps repeated ones
  // inside the region as well)
#pragma unroll
  for (int k = 0; k < CUT_ITEMS; ++k) {
    if (kind[k] == 1) {
      if (at_res < nj) q.members[jo + at_res] = (int32_t)v[k];
      ++at_res;
    } else if (kind[k] == 2) {
      if (at_in < nj) q.members[jo + nj - 1 - at_in] = (int32_t)v[k];
      ++at_in;
    }
  }
}

// One block of NT threads: the keep-th smallest (1-based) of the ids id(x), 0 <= x < n; entries with bit
// 31 set do not count.  Radix select from the top, over the `bits` bits that ids have here, at most 11 to a
// pass and the same number in each.  0 < keep <= ids that count.
// (Always 11 + 10 + 10 bits, the first pass over a million ids added everything to one counter: 76 000 entries
// of two words 71 us, 32 this way, either with four reads in flight to a thread.)
// ITEMS: reads in flight; one where a thread has few (with four, 17 selects of some 5 000 members took 14 us more).
constexpr int KTH_BINS = 2048;

template <int NT, int ITEMS, typename Id>
__device__ int32_t p_kth_smallest_id(int64_t n, int64_t keep, int bits, Id id) {
  __shared__ uint32_t s_hist[KTH_BINS];
  __shared__ uint32_t s_scan[NT / WAVE + 1];
  __shared__ uint32_t s_pick, s_below;
  uint32_t prefix = 0;
  uint32_t left = (uint32_t)keep;
  int shift = bits;
  for (int passes = (bits + 10) / 11; passes > 0; --passes) {
    const int width = (shift + passes - 1) / passes, bins = 1 << width;
    const int above = shift;               // the bits from here up are known
    shift -= width;
    for (int b = threadIdx.x; b < bins; b += NT) s_hist[b] = 0;
    if (threadIdx.x == 0) s_pick = s_below = 0;
    __syncthreads();
    for (int64_t x0 = threadIdx.x; x0 < n; x0 += NT * ITEMS) {
      uint32_t v[ITEMS];
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) v[k] = id(x0 + k * NT < n ? x0 + k * NT : x0);
#pragma unroll
      for (int k = 0; k < ITEMS; ++k)
        if (x0 + k * NT < n && !(v[k] >> 31) && (v[k] >> above) == prefix)
          atomicAdd(&s_hist[(v[k] >> shift) & (uint32_t)(bins - 1)], 1u);
    }
    __syncthreads();
    constexpr int PER = KTH_BINS / NT;
    uint32_t mine = 0;
    for (int b = threadIdx.x * PER; b < (int)(threadIdx.x + 1) * PER && b < bins; ++b) mine += s_hist[b];
    uint32_t total;
    uint32_t run = block_exclusive_scan<uint32_t, NT>(mine, s_scan, total);
    for (int b = threadIdx.x * PER; b < (int)(threadIdx.x + 1) * PER && b < bins; ++b) {
      const uint32_t c = s_hist[b];
      if (run < left && run + c >= left) {
        s_pick = (uint32_t)b;
        s_below = run;
      }
      run += c;
    }
    __syncthreads();
    prefix = (prefix << width) | s_pick;
    left -= s_below;
    __syncthreads();
  }
  return (int32_t)prefix;
}

// What a cut drops, from the members found: all incoming rows that leave their class no member to
// choose from, or of `n` members of the class that is cut all but the `keep` smallest ids.
struct CutChoice {
  int32_t kind;
  int64_t n, keep;         // keep 0: no choice
};

__device__ __forceinline__ CutChoice cut_choice(const Cut& c, int64_t room) {
  const int64_t R = c.n_res < room ? c.n_res : room, I = c.n_in < room ? c.n_in : room;
  if (c.rem < I) return {CUT_IN_SOME, I, I - c.rem};
  if (c.rem == I) return {CUT_IN_ALL, I, 0};
  const int64_t keep = R - (c.rem - I);   // (positive: a bucket that goes whole is not the threshold bucket)
  return {CUT_RES, R, keep > 0 ? keep : 0};
}

// Member x of the class that is cut; `region`, `room`: of its bucket.
__device__ __forceinline__ uint32_t cut_member(const Stays& q, int32_t kind, int64_t region, int64_t room, int64_t x) {
  return kind == CUT_IN_SOME ? (uint32_t)q.ids[q.members[region + room - 1 - x]] : (uint32_t)q.members[region + x];
}

// incoming rows that are dropped: the accesses that end their stays look for this mark
// (threads x0, x0 + step, ...)
__device__ __forceinline__ void cut_mark(const Stays& q, const Cut& c, int32_t kind, int32_t T, int64_t region,
                                         int64_t room, int64_t x0, int64_t step) {
  const int64_t I = c.n_in < room ? c.n_in : room;
  for (int64_t x = x0; x < I; x += step) {
    const int32_t p = q.members[region + room - 1 - x];
    if (kind != CUT_IN_SOME || q.ids[p] > T) q.ends[p] |= BYPASSED;
  }
}

// One block per cut of the level: which class is cut and where.
__global__ __launch_bounds__(BIG) void k_cut_decide(Stays q, Jobs jobs, int first) {
  Cut* cut = &q.cuts[jobs[first + blockIdx.x]];
  const Cut c = *cut;
  const int64_t region = q.off[c.jstar], room = q.off[c.jstar + 1] - region;
  const CutChoice ch = cut_choice(c, room);
  int32_t T = -1;
  if (ch.keep > 0)
    T = p_kth_smallest_id<BIG, 1>(ch.n, ch.keep, q.id_bits, [&](int64_t x) { return cut_member(q, ch.kind, region, room, x); });
  cut_mark(q, c, ch.kind, T, region, room, threadIdx.x, BIG);
  __syncthreads();   // every thread has read the cut
  if (threadIdx.x == 0) {
    cut->kind = ch.kind;
    cut->T = T;
  }
}

// The same for buckets of more than CUT_WIDE members, by many blocks (blockIdx.y = cut): a launch per
// digit of the ids, which finds the digits before it from the counts its predecessors left, and one that
// marks.  One block takes about 0.48 us per 1 000 members (1.2 M: 560 us), these launches 24 us for 70 000 and
// 30 for 1.2 M.  (The members follow from the thresholds.  By the length of the bucket's iteration
// instead, 17 levels of cuts of few members took 15 us more each.)
constexpr int64_t CUT_WIDE = 3 << 14;
constexpr int CUT_DIGITS = 3, CUT_BINS = 2048;         // 11 + 10 + 10 bits
constexpr int CUT_WIDE_ITEMS = 8;

// The digits above DIGIT of the keep-th smallest id, from their counts (keep > 0; the whole block).
template <int DIGIT>
__device__ __forceinline__ uint32_t wide_digits(const uint32_t* __restrict__ counts, uint32_t keep) {
  __shared__ uint32_t smem[TB / WAVE + 1];
  __shared__ uint32_t s_pick, s_below;
  uint32_t prefix = 0, left = keep;
#pragma unroll
  for (int d = 0; d < DIGIT; ++d) {
    constexpr int PER = CUT_BINS / TB;
    uint32_t mine[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      mine[k] = counts[d * CUT_BINS + threadIdx.x * PER + k];
      sum += mine[k];
    }
    if (threadIdx.x == 0) s_pick = s_below = 0;
    uint32_t total;
    uint32_t run = block_exclusive_scan<uint32_t, TB>(sum, smem, total);   // (barriers inside)
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (run < left && run + mine[k] >= left) {
        s_pick = (uint32_t)(threadIdx.x * PER + k);
        s_below = run;
      }
      run += mine[k];
    }
    __syncthreads();
    prefix = (prefix << (d ? 10 : 11)) | s_pick;
    left -= s_below;
    __syncthreads();
  }
  return prefix;
}

// Counts of digit DIGIT of the ids id(x), 0 <= x < n, whose digits above it are `prefix`, by the blocks of a column;
// ids with bit 31 set do not count.
template <int DIGIT, typename Id>
__device__ __forceinline__ void wide_counts(uint32_t* __restrict__ counts, int64_t n, uint32_t prefix, Id id) {
  __shared__ uint32_t s_hist[CUT_BINS];
  constexpr int SHIFT = DIGIT == 0 ? 20 : DIGIT == 1 ? 10 : 0, BITS = DIGIT == 0 ? 11 : 10;
  const int64_t first = (int64_t)blockIdx.x * (TB * CUT_WIDE_ITEMS);
  if (first >= n) return;                              // uniform
  for (int b = threadIdx.x; b < CUT_BINS; b += TB) s_hist[b] = 0;
  __syncthreads();
  for (int64_t x0 = first + threadIdx.x; x0 < n; x0 += (int64_t)gridDim.x * (TB * CUT_WIDE_ITEMS)) {
    uint32_t v[CUT_WIDE_ITEMS];
#pragma unroll
    for (int k = 0; k < CUT_WIDE_ITEMS; ++k) v[k] = id(x0 + k * TB < n ? x0 + k * TB : x0);
#pragma unroll
    for (int k = 0; k < CUT_WIDE_ITEMS; ++k)
      if (x0 + k * TB < n && !(v[k] >> 31) && (DIGIT == 0 || v[k] >> (SHIFT + BITS) == prefix))
        atomicAdd(&s_hist[(v[k] >> SHIFT) & ((1u << BITS) - 1u)], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < CUT_BINS; b += TB)
    if (s_hist[b]) atomicAdd(&counts[DIGIT * CUT_BINS + b], s_hist[b]);
}

template <int DIGIT>   // CUT_DIGITS: all are known
__global__ __launch_bounds__(TB) void k_cut_wide(Stays q, Jobs jobs, int first,
                                                 uint32_t* __restrict__ hists) {
  Cut* cut = &q.cuts[jobs[first + blockIdx.y]];
  const Cut c = *cut;                                  // (kind and T are not used: the last launch writes them)
  const int64_t region = q.off[c.jstar], room = q.off[c.jstar + 1] - region;
  const CutChoice ch = cut_choice(c, room);
  uint32_t* const counts = hists + (int64_t)blockIdx.y * (CUT_DIGITS * CUT_BINS);
  const uint32_t prefix = ch.keep > 0 ? wide_digits<DIGIT>(counts, (uint32_t)ch.keep) : 0u;   // uniform
  if constexpr (DIGIT == CUT_DIGITS) {
    const int32_t T = ch.keep > 0 ? (int32_t)prefix : -1;
    cut_mark(q, c, ch.kind, T, region, room, (int64_t)blockIdx.x * TB + threadIdx.x, (int64_t)gridDim.x * TB);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      cut->kind = ch.kind;
      cut->T = T;
    }
  } else if (ch.keep > 0) {
    wide_counts<DIGIT>(counts, ch.n, prefix, [&](int64_t x) { return cut_member(q, ch.kind, region, room, x); });
  }
}

// ---- LRU ----------------------------------------------------------------------------------------------
//
// After iteration i the cache holds the `cap` rows that were accessed last, among those of one
// iteration the ones with the smaller ids, as long as no iteration accesses more rows than the cache has lines
// (then incoming rows of the running iteration would be dropped as well, before those that hit): what an
// iteration drops are the last rows of that order, and a row only falls back in it until it is accessed again.  So
// (last access, id) of the last row that stays, limits[i], says for every row whether it is there. Rows of C_0 that
// are still to be accessed for the first time never go: C_0 is the first `cap` rows of the superbatch, so
// nothing is missed before all of them were accessed.  limits[i] follows from how many rows accessed in
// iteration t are accessed next after i, for all t <= i (sums over the histograms that Belady's thresholds
// come from), and a select among the accesses of the one iteration that the limit falls into: all
// iterations side by side.  A hit is an access whose row is not below the limit of the iteration before,
// every miss is inserted, and the iteration that evicts a row is found by bisection.
// 20 iterations of 76 000 accesses, 104 857 lines: the loop over the state, six launches an iteration, 1 263 us
// a call, this way 449 (k_move_lines 76, k_lru_limits 31, k_lru_walk 21, k_stays_mark 8; the sort 90); 100 of 100 000
// on 30 M nodes, 0.85 M lines: 15.5 ms and 2.2.

// The place of a row in the order, larger: stays longer.
__device__ __forceinline__ uint64_t lru_key(uint32_t iteration, uint32_t v) {
  return (uint64_t)iteration << 32 | (0x7FFFFFFFu - v);
}

// The iteration from i on that drops a row with this key, S if none.
__device__ __forceinline__ int32_t lru_end(const uint64_t* limits, int32_t S, int32_t i, uint64_t key) {
  int32_t lo = i, hi = S;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (limits[mid] > key) hi = mid; else lo = mid + 1;
  }
  return lo;
}

// hists[t][i] <- accesses of iteration t whose row is accessed next after iteration i.  A wave per t.
__global__ __launch_bounds__(WAVE) void k_lru_counts(int32_t S, uint32_t* __restrict__ hists) {
  uint32_t* row = hists + (int64_t)blockIdx.x * (S + 1);
  const int lane = lane_id();
  uint32_t behind = 0;
  for (int32_t r0 = 0; r0 <= S; r0 += WAVE) {      // from the right
    const int32_t j = S - r0 - lane;
    const uint32_t c = j >= 0 ? row[j] : 0u;
    const uint32_t incl = wave_inclusive_scan(c);
    if (j >= 0) row[j] = behind + incl - c;
    behind += of_lane(incl, WAVE - 1);
  }
}

// Of an iteration's limit: the iteration t whose rows are the last to stay, and how many of them do.
struct LruJob {
  int32_t t, keep;         // keep 0: the limit is known
};

// What a row of iteration t counts as in the select for iteration i: its id, if it is accessed next after i.
__device__ __forceinline__ uint32_t lru_member(const Stays& q, int64_t p, int32_t i) {
  const uint32_t v = (uint32_t)q.ids[p];               // (both reads at once)
  return stay_next(q.ends[p]) > i ? v : 0x80000000u;
}

// A block per iteration: the iteration whose rows are the last to stay, and which of them do.  jobs: null, or where
// selects among more than LRU_WIDE accesses are left to k_lru_wide: one block takes 0.55 us per 1 000 accesses (3
// iterations of 4 M, nine tenths of the rows held: 2.15 ms of a call of 3.55, now 1.39), those five launches some
// 50 us (20 iterations of 76 000: 32 us by a block each, 26 and the launches this way).
constexpr int64_t LRU_WIDE = 1 << 17;
__global__ __launch_bounds__(BIG) void k_lru_limits(Stays q, const uint32_t* __restrict__ counts, int64_t cap,
                                                    uint64_t* __restrict__ limits, LruJob* __restrict__ jobs) {
  __shared__ int64_t smem[BIG / WAVE + 1];
  __shared__ int32_t s_t;
  __shared__ int64_t s_keep;
  const int32_t i = blockIdx.x;
  if (threadIdx.x == 0) s_t = -1;
  int64_t before = 0;
  for (int32_t r0 = 0; r0 <= i && before <= cap; r0 += BIG) {   // uniform; from iteration i downwards
    const int32_t t = i - r0 - (int32_t)threadIdx.x;
    const int64_t c = t >= 0 ? counts[(int64_t)t * (q.S + 1) + i] : 0;
    int64_t total;
    const int64_t ahead = before + block_exclusive_scan<int64_t, BIG>(c, smem, total);
    if (ahead <= cap && ahead + c > cap) {         // (one thread at most)
      s_t = t;
      s_keep = cap - ahead;
    }
    before += total;
    __syncthreads();
  }
  const int32_t t = s_t;
  if (t < 0 || s_keep == 0) {                      // uniform: nothing has to go, or all rows of t
    if (threadIdx.x == 0) {
      limits[i] = (uint64_t)(t + 1) << 32;
      if (jobs) jobs[i] = {t, 0};
    }
    return;
  }
  const int64_t to = q.off[t], n = q.off[t + 1] - to;
  if (jobs && n > LRU_WIDE) {                      // uniform
    if (threadIdx.x == 0) jobs[i] = {t, (int32_t)s_keep};
    return;
  }
  const int32_t T = p_kth_smallest_id<BIG, 4>(n, s_keep, q.id_bits, [&](int64_t x) { return lru_member(q, to + x, i); });
  if (threadIdx.x == 0) {
    limits[i] = lru_key((uint32_t)t, (uint32_t)T);
    if (jobs) jobs[i] = {t, 0};
  }
}

// The selects left, by many blocks (blockIdx.y = iteration), digit by digit as k_cut_wide.
template <int DIGIT>   // CUT_DIGITS: all are known
__global__ __launch_bounds__(TB) void k_lru_wide(Stays q, const LruJob* __restrict__ jobs,
                                                 uint64_t* __restrict__ limits, uint32_t* __restrict__ hists) {
  const int32_t i = blockIdx.y;
  const LruJob job = jobs[i];
  if (job.keep == 0) return;                       // uniform
  uint32_t* const counts = hists + (int64_t)i * (CUT_DIGITS * CUT_BINS);
  const uint32_t prefix = wide_digits<DIGIT>(counts, (uint32_t)job.keep);
  if constexpr (DIGIT == CUT_DIGITS) {
    if (threadIdx.x == 0) limits[i] = lru_key((uint32_t)job.t, prefix);
  } else {
    const int64_t to = q.off[job.t];
    wide_counts<DIGIT>(counts, q.off[job.t + 1] - to, prefix, [&](int64_t x) { return lru_member(q, to + x, i); });
  }
}

// ---- the lists and the evicting iterations ----------------------------------------------------------

// In the place of an access's line until it is known.  No line has this number: there are at most INT32_MAX.
constexpr int32_t LOOK_UP = INT32_MAX;   // a hit
constexpr int32_t HANDED_OVER = -2;      // a hit whose line comes with the row's insertion, in the iteration before it

// Every access: hit or miss (src_line: LOOK_UP / -1, the lines follow), and whether a miss is an insertion
// (bit p of ins_bits).  A miss that is never accessed again is none: where
// bucket "never" is the one that is cut, the iteration drops as many rows as it has misses, incoming
// rows of the bucket first.
template <bool LRU>
__global__ __launch_bounds__(TB) void k_stays_mark(Stays q, int64_t n, int32_t* __restrict__ src_line,
                                                   uint32_t* __restrict__ ins_bits) {
  extern __shared__ int32_t lds_off[];
  load_offsets(lds_off, q.off, q.S);
  const int64_t base = (int64_t)blockIdx.x * CUT_TILE;
  const int32_t i0 = iter_of(lds_off, q.S, (int32_t)base);   // of the tile's first access; advanced below
  // what every access has to read is asked for first, level by level; only where a cut decides is there more
  // (one access after the other: 192 us for 33 M accesses, 141 this way, 4 TB/s)
  uint64_t w[CUT_ITEMS];
  uint32_t v[CUT_ITEMS], e[CUT_ITEMS];
#pragma unroll
  for (int k = 0; k < CUT_ITEMS; ++k) {
    const int64_t p = base + k * TB + threadIdx.x;
    w[k] = q.ends[p < n ? p : base];
    v[k] = (uint32_t)q.ids[p < n ? p : base];
  }
  if (!LRU) {
    int32_t i = i0;
#pragma unroll
    for (int k = 0; k < CUT_ITEMS; ++k) {
      const int64_t p = base + k * TB + threadIdx.x;
      while (i + 1 < q.S && lds_off[i + 1] <= (int32_t)p) ++i;
      e[k] = stay_word(q, stay_prev(w[k]), i);
    }
  }
  int32_t i = i0;
  Cut c{};
  uint64_t limit = 0;                              // of the iteration in front (an earlier one accessed the row)
  if (LRU) limit = q.limits[i > 0 ? i - 1 : 0];
  else c = q.cuts[i];
#pragma unroll
  for (int k = 0; k < CUT_ITEMS; ++k) {
    const int64_t p = base + k * TB + threadIdx.x;
    bool inserted = false, hit = false;
    if (p < n) {
      const int32_t before = i;
      while (i + 1 < q.S && lds_off[i + 1] <= (int32_t)p) ++i;
      if (i != before) {
        if (LRU) limit = q.limits[i - 1];
        else c = q.cuts[i];
      }
      const uint32_t prev = stay_prev(w[k]);
      if (LRU) {
        hit = prev == FROM_START;
        if (prev < FROM_START)
          hit = prev == (uint32_t)(limit >> 32) ? lru_key(prev, v[k]) >= limit : prev > (uint32_t)(limit >> 32);
        inserted = !hit;
      } else {
        if (prev != NO_STAY)
          hit = (e[k] >> 16) == NO_CUT ? (int32_t)(e[k] & 0xFFFFu) == i : stay_hits(q, e[k], w[k], i, v[k]);
        if (!hit) inserted = stay_inserts(q, c, stay_next(w[k]), v[k]);
      }
      if (src_line) src_line[p] = hit ? LOOK_UP : -1;
    }
    const uint64_t m = __ballot(inserted);
    const int64_t first = base + k * TB + (threadIdx.x & ~(WAVE - 1));
    if (lane_id() == 0 && first < n) ins_bits[first >> 5] = (uint32_t)m;
    if (lane_id() == 32 && first + 32 < n) ins_bits[(first >> 5) + 1] = (uint32_t)(m >> 32);
  }
}

// ---- the cuts of bucket "never" ---------------------------------------------------------------------
//
// The rows of the bucket are those whose last access hit (from that iteration on) and the
// start-state rows the superbatch never accesses.  Iteration t, if it cuts the bucket, keeps the
// keep_t of them with the smallest ids (keep_t is known from the thresholds), so one cut follows from
// the one before.  The ids are divided into parts; how many rows each part holds
// after every cut needs no ids: the parts below the one that is cut keep all, the parts above lose
// all.  One block walks the iterations over the parts' counts (k_never_parts: 0.24 us per iteration), and
// what id the cut falls on is then found for all parts side by side (k_never_select).  Setting bits,
// counting, finding and clearing on one bitmap over all ids, cut after cut, took 43 us per cut.
//
// A part spans at most 2^NEVER_SHIFT ids, whatever the superbatch accesses and whatever the cache
// carries, so that the rows it still holds are a bitmap in LDS: the block of a part takes the
// idle rows in once, reads the part's accessed rows once per cut and adds those that arrived since the cut
// before.  (Looking up every id of a part for every cut, three times, with parts as wide as the
// superbatch was small: a carried cache of 12 000 lines, 20 iterations of 10 000 accesses to 25 000 rows of
// 60 M nodes took 11.4 ms; 1.1 ms this way, 1.7 through the loop over the state.)
constexpr int NEVER_THREADS = 1024;
constexpr int NEVER_SHIFT = 17;
constexpr int NEVER_WORDS = 1 << (NEVER_SHIFT - 5);    // 16 KB
constexpr int NEVER_PARTS = 1 << (31 - NEVER_SHIFT);   // at most
// [S x parts] counters up to here sit in an array of the candidates that stays_run does not use.  More of
// them take more than 2^25 ids (S is at most 2 048), and are then fewer than the words of the array of
// first accesses.
constexpr int64_t NEVER_COUNTS = int64_t(1) << 19;

struct Never {
  uint64_t* rows;          // [distinct] id << 32 | iteration of its last access, if that hits (else NOT_HERE), by id
  uint32_t* counts;        // [S * parts] rows that arrive in an iteration, by part
  const uint32_t* idle;    // bitmap over ids: start-state rows without an access; null: a fresh superbatch
  int64_t distinct, num_nodes;
  int32_t parts, shift;    // part of an id = id >> shift
};
constexpr uint32_t NOT_HERE = 0xFFFFFFFFu;

// counts[i][part], a block per stretch of rows (by id).  A stretch that meets up to NEVER_ROUNDS parts
// counts per iteration in LDS and hands over where the part changes; rows that are
// thinner than that are added one by one (each part has few of them, so no counter sees many).
constexpr int NEVER_ROUNDS = 4;
__global__ __launch_bounds__(TB) void k_never_counts(Never nv, int32_t S) {
  extern __shared__ uint32_t s_cnt[];     // [S]
  const int64_t per = (((nv.distinct + gridDim.x - 1) / gridDim.x + TB - 1) / TB) * TB;
  const int64_t first = (int64_t)blockIdx.x * per;
  const int64_t last = first + per < nv.distinct ? first + per : nv.distinct;
  if (first >= last) return;
  int32_t part = (int32_t)((nv.rows[first] >> 32) >> nv.shift);
  const int32_t last_part = (int32_t)((nv.rows[last - 1] >> 32) >> nv.shift);
  if (last_part - part >= NEVER_ROUNDS) {  // uniform
    for (int64_t x = first + threadIdx.x; x < last; x += TB) {
      const uint64_t row = nv.rows[x];
      const uint32_t i = (uint32_t)row;
      if (i != NOT_HERE) atomicAdd(&nv.counts[(int64_t)i * nv.parts + (int32_t)((row >> 32) >> nv.shift)], 1u);
    }
    return;
  }
  for (int i = threadIdx.x; i < S; i += TB) s_cnt[i] = 0;
  __syncthreads();
  int64_t from = first;
  while (true) {                          // uniform: one round per part of the stretch
    int64_t lo = from, hi = last;         // the first row behind the part
    if (part == last_part) lo = last;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if ((int32_t)((nv.rows[mid] >> 32) >> nv.shift) <= part) lo = mid + 1; else hi = mid;
    }
    for (int64_t x = from + threadIdx.x; x < lo; x += TB) {
      const uint32_t i = (uint32_t)nv.rows[x];
      if (i != NOT_HERE) atomicAdd(&s_cnt[i], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < S; i += TB)
      if (s_cnt[i]) {
        atomicAdd(&nv.counts[(int64_t)i * nv.parts + part], s_cnt[i]);
        s_cnt[i] = 0;
      }
    __syncthreads();
    if (lo >= last) break;
    from = lo;
    part = (int32_t)((nv.rows[from] >> 32) >> nv.shift);
  }
}

// start-state rows without an access, per part (blockIdx.x = part)
__global__ __launch_bounds__(TB) void k_never_idle(Never nv, uint32_t* __restrict__ idle_counts) {
  __shared__ uint32_t red[TB / WAVE];
  const int64_t lo = (int64_t)blockIdx.x << nv.shift, hi = lo + (int64_t(1) << nv.shift);
  uint32_t cnt = 0;                       // (parts are whole words)
  for (int64_t w = (lo >> 5) + threadIdx.x; w < hi >> 5 && w * 32 < nv.num_nodes; w += TB)
    cnt += __popc(nv.idle[w]);
  const uint32_t total = block_sum_u32(cnt, red);
  if (threadIdx.x == 0) idle_counts[blockIdx.x] = total;
}

// One block, PER neighbouring parts to a thread: which part every cut falls into and how many of its
// rows stay.  Arrivals and thresholds are requested AHEAD iterations early.
template <int PER, int AHEAD>
__global__ __launch_bounds__(NEVER_THREADS) void k_never_parts(Never nv, int32_t S, Cut* __restrict__ cuts,
                                                               const uint32_t* __restrict__ idle_counts) {
  __shared__ uint32_t slots[2][NEVER_THREADS / WAVE];
  int set = 0;                            // the two sets of slots take turns: one barrier per cut
  const int32_t me = threadIdx.x, first = me * PER;
  uint32_t have[PER], arrive[AHEAD][PER];
  Cut cut[AHEAD];
  auto request = [&](int a, int32_t t) {
#pragma unroll
    for (int p = 0; p < PER; ++p)
      arrive[a][p] = first + p < nv.parts ? nv.counts[(int64_t)t * nv.parts + first + p] : 0u;
    cut[a] = cuts[t];
  };
#pragma unroll
  for (int p = 0; p < PER; ++p) have[p] = idle_counts && first + p < nv.parts ? idle_counts[first + p] : 0u;
#pragma unroll
  for (int a = 0; a < AHEAD; ++a)
    if (a < S) request(a, a);
  for (int32_t t0 = 0; t0 < S; t0 += AHEAD) {
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) {
      const int32_t t = t0 + a;
      if (t >= S) break;                  // uniform
      const Cut c = cut[a];
      uint32_t mine = 0;
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        have[p] = c.jstar < S ? 0u : have[p] + arrive[a][p];
        mine += have[p];
      }
      if (t + AHEAD < S) request(a, t + AHEAD);
      if (c.jstar != S) continue;         // uniform
      const uint32_t keep = c.n_res;      // (left there by k_static_roll)
      uint32_t inc = wave_inclusive_scan(mine);
      if (lane_id() == WAVE - 1) slots[set][me / WAVE] = inc;
      __syncthreads();
      uint32_t before = inc - mine, total = 0;
#pragma unroll
      for (int w = 0; w < NEVER_THREADS / WAVE; ++w) {
        const uint32_t s = slots[set][w];
        if (w < me / WAVE) before += s;
        total += s;
      }
      set ^= 1;
      if (keep >= total) {                // no resident goes
        if (me == 0) {
          cuts[t].kind = CUT_IN_ALL;
          cuts[t].n_res = (uint32_t)nv.parts;
        }
        continue;                         // uniform
      }
#pragma unroll
      for (int p = 0; p < PER; ++p) {
        const uint32_t held = have[p];
        if (before < keep && before + held >= keep) {
          cuts[t].kind = CUT_RES;
          cuts[t].n_res = (uint32_t)(first + p);
          cuts[t].n_in = keep - before;
          // the whole part stays: no look at its rows
          cuts[t].T = keep == before + held ? (int32_t)((((int64_t)(first + p) + 1) << nv.shift) - 1) : -1;
        }
        if (before >= keep) have[p] = 0;
        else if (before + held > keep) have[p] = keep - before;
        before += held;
      }
    }
  }
}

// A block per part: the ids of the cuts that fall into it, in order.  `bits` holds the part's rows
// as they stand after the cut before; a cut costs one read of the part's accessed rows (bound by
// that, by one workgroup: 200 iterations whose 100 000 rows are all neighbours, in one or two of 848 parts,
// 37 us for all their cuts; spread over the parts 4 us).
__global__ __launch_bounds__(NEVER_THREADS) void k_never_select(Never nv, int32_t S, Cut* __restrict__ cuts) {
  constexpr int WORDS = NEVER_WORDS / NEVER_THREADS, READS = 4;
  __shared__ uint32_t bits[NEVER_WORDS];
  __shared__ uint32_t smem[NEVER_THREADS / WAVE + 1];
  __shared__ int32_t s_next, s_emptied, s_T;
  const int32_t part = blockIdx.x;
  const int64_t first_word = ((int64_t)part << nv.shift) >> 5, words = (nv.num_nodes + 31) >> 5;
  int64_t from = 0, to = -1;              // the part's rows, found with its first cut
  int32_t done = -1;                      // the cut before
  while (true) {
    if (threadIdx.x == 0) {
      s_next = S;
      s_emptied = s_T = -1;
    }
    __syncthreads();
    for (int32_t t = done + 1 + threadIdx.x; t < S; t += NEVER_THREADS)
      if (cuts[t].jstar == S && cuts[t].kind == CUT_RES && cuts[t].n_res == (uint32_t)part && cuts[t].T < 0)
        atomicMin(&s_next, t);
    __syncthreads();
    const int32_t t = s_next;
    if (t >= S) return;                   // uniform
    // the last iteration since the cut before that emptied the part
    for (int32_t e = done + 1 + threadIdx.x; e < t; e += NEVER_THREADS) {
      const Cut c = cuts[e];
      if (c.jstar < S || (c.jstar == S && c.kind == CUT_RES && c.n_res < (uint32_t)part)) atomicMax(&s_emptied, e);
    }
    const bool fresh = to < 0;            // uniform
    if (fresh) {
      const uint64_t lo_id = (uint64_t)part << nv.shift, hi_id = lo_id + (1ull << nv.shift);
      int64_t a = 0, b = nv.distinct;
      while (a < b) {
        const int64_t mid = (a + b) >> 1;
        if ((nv.rows[mid] >> 32) < lo_id) a = mid + 1; else b = mid;
      }
      from = a;
      b = nv.distinct;
      while (a < b) {
        const int64_t mid = (a + b) >> 1;
        if ((nv.rows[mid] >> 32) < hi_id) a = mid + 1; else b = mid;
      }
      to = a;
    }
    __syncthreads();
    const int32_t emptied = s_emptied, after = emptied > done ? emptied : done;   // rows that arrived after it
    if (fresh || emptied > done)
      for (int w = threadIdx.x; w < NEVER_WORDS; w += NEVER_THREADS)
        bits[w] = nv.idle && emptied < 0 && w < 1 << (nv.shift - 5) && first_word + w < words
                      ? nv.idle[first_word + w] : 0u;
    __syncthreads();
    for (int64_t x0 = from + threadIdx.x; x0 < to; x0 += READS * NEVER_THREADS) {
      uint64_t row[READS];
#pragma unroll
      for (int k = 0; k < READS; ++k)
        row[k] = nv.rows[x0 + k * NEVER_THREADS < to ? x0 + k * NEVER_THREADS : from];
#pragma unroll
      for (int k = 0; k < READS; ++k) {
        const int32_t i = (int32_t)(uint32_t)row[k];   // (NOT_HERE: -1)
        const uint32_t v = (uint32_t)(row[k] >> 32) & ((1u << nv.shift) - 1u);
        if (x0 + k * NEVER_THREADS < to && i > after && i <= t) atomicOr(&bits[v >> 5], 1u << (v & 31));
      }
    }
    __syncthreads();
    // the row that stays last, WORDS neighbouring words to a thread; the rows above it go
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) mine += __popc(bits[threadIdx.x * WORDS + k]);
    uint32_t total;
    uint32_t before = block_exclusive_scan<uint32_t, NEVER_THREADS>(mine, smem, total);
    const uint32_t keep = cuts[t].n_in;   // at least one, at most `total`
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
      const int w = threadIdx.x * WORDS + k;
      const uint32_t word = bits[w], held = __popc(word);
      if (before >= keep) {
        bits[w] = 0;
      } else if (before + held >= keep) {
        uint32_t rest = word;
        for (uint32_t skip = keep - before; skip > 1; --skip) rest &= rest - 1;
        const int bit = __ffs(rest) - 1;
        bits[w] = word & (uint32_t)((2ull << bit) - 1ull);
        s_T = (int32_t)(((int64_t)part << nv.shift) + w * 32 + bit);
      }
      before += held;
    }
    __syncthreads();
    if (threadIdx.x == 0) cuts[t].T = s_T;
    done = t;
  }
}

// ---- one pass in node order: what every access's stay comes to ------------------------------------------
//
// A wave takes LINK_CHUNKS * 64 consecutive pairs, a block one tile of LOOK_TILE.  In node order the ends
// of a stay are neighbours, so hits and insertions follow from the table (which stays in L2) without a
// look at any per-access array; both are kept as bits in node order, word x / 64 for pair x.  (Reading
// them as bits by position instead costs a random 128-byte line each: 0.3 ms per 33 M accesses.)
// Written on the way: the row that ends a run and whether that access hit, for bucket "never", and
// the iteration that evicts a start-state row that is gone before its first access.
constexpr int LINK_CHUNKS = 8;
static_assert(LINK_CHUNKS * TB == LOOK_TILE, "a block works on one tile of the run heads");

__global__ __launch_bounds__(TB) void k_stays_links(Stays q, const uint64_t* __restrict__ sorted, int64_t n,
                                                    const uint32_t* __restrict__ head_bases,
                                                    const uint64_t* __restrict__ last_head,
                                                    const uint32_t* __restrict__ held,
                                                    const int32_t* __restrict__ addr, Never nv,
                                                    uint64_t* __restrict__ hit_words,
                                                    uint64_t* __restrict__ ins_words,
                                                    uint32_t* __restrict__ leave_start) {
  extern __shared__ int32_t lds_off[];
  __shared__ uint32_t s_heads[TB / WAVE];
  __shared__ uint16_t s_coarse[IterFinder::COARSE + 1];
  const IterFinder iteration = iter_finder(lds_off, s_coarse, q.off, q.S);
  const int lane = lane_id(), wave = threadIdx.x / WAVE;
  const int64_t base = (int64_t)blockIdx.x * LOOK_TILE + wave * (WAVE * LINK_CHUNKS);
  const int32_t start_end = last_head ? lds_off[(int32_t)(*last_head >> 32) + 1] : INT32_MAX;
  // behind n: an id that no access has
  uint64_t cur[LINK_CHUNKS + 1];
#pragma unroll
  for (int k = 0; k <= LINK_CHUNKS; ++k) {
    const int64_t x = base + k * WAVE + (k < LINK_CHUNKS ? lane : 0);
    cur[k] = x < n ? sorted[x] : ~0ull;
  }
  const uint64_t left = base > 0 && base - 1 < n ? sorted[base - 1] : ~0ull;
  int32_t it[LINK_CHUNKS + 1];
#pragma unroll
  for (int k = 0; k <= LINK_CHUNKS; ++k)
    it[k] = (cur[k] >> 32) != 0xFFFFFFFFull ? iteration((uint32_t)cur[k]) : q.S;
  // the next access of every pair's row, and whether the stay reaches it
  int32_t next[LINK_CHUNKS];
  uint32_t word[LINK_CHUNKS], more = 0, reach = 0, head = 0;      // bit k: chunk k
#pragma unroll
  for (int k = 0; k < LINK_CHUNKS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32);
    uint32_t rv = from_right(v), lv = from_left(v);
    int32_t rj = from_right(it[k]);
    const uint32_t ov = of_lane((uint32_t)(cur[k + 1] >> 32), 0);
    const int32_t oj = of_lane(it[k + 1], 0);
    const uint32_t bv = k > 0 ? of_lane((uint32_t)(cur[k > 0 ? k - 1 : 0] >> 32), WAVE - 1) : (uint32_t)(left >> 32);
    if (lane == WAVE - 1) {
      rv = ov;
      rj = oj;
    }
    if (lane == 0) lv = bv;
    const bool valid = v != 0xFFFFFFFFu;
    more |= (valid && rv == v ? 1u : 0u) << k;
    head |= (valid && lv != v ? 1u : 0u) << k;
    next[k] = rv == v ? rj : q.S;
    word[k] = valid && rv == v ? q.table[(int64_t)rj * q.S + it[k]] : 0u;
  }
#pragma unroll
  for (int k = 0; k < LINK_CHUNKS; ++k)
    if (more >> k & 1u) {
      const bool r = (word[k] >> 16) == NO_CUT
                         ? (int32_t)(word[k] & 0xFFFFu) == next[k]
                         : stay_end(q, (uint32_t)it[k], next[k], (uint32_t)(cur[k] >> 32),
                                    &q.ends[(uint32_t)cur[k]], next[k]) == next[k];
      reach |= (r ? 1u : 0u) << k;
    }
  // the pair in front of the wave's stretch
  bool left_reaches = false;
  if ((left >> 32) != 0xFFFFFFFFull && (uint32_t)(left >> 32) == of_lane((uint32_t)(cur[0] >> 32), 0)) {
    const int32_t j = of_lane(it[0], 0);
    left_reaches = stay_end(q, (uint32_t)iteration((uint32_t)left), j,
                            (uint32_t)(left >> 32), &q.ends[(uint32_t)left], j) == j;
  }
  uint32_t hit = 0, heads = 0;
#pragma unroll
  for (int k = 0; k < LINK_CHUNKS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    bool reached = from_left(reach) >> k & 1u;
    const bool other = k > 0 ? of_lane(reach, WAVE - 1) >> (k > 0 ? k - 1 : 0) & 1u : left_reaches;
    if (lane == 0) reached = other;
    bool h = reached;
    if (head >> k & 1u) {
      h = false;
      if ((int32_t)p < start_end && in_start_state(v, it[k], last_head, held)) {
        const int32_t e = stay_end(q, FROM_START, it[k], v, nullptr, it[k]);
        h = e == it[k];
        if (!h) leave_start[addr[v]] = (uint32_t)e;
      }
    }
    const bool valid = v != 0xFFFFFFFFu;
    hit |= (valid && h ? 1u : 0u) << k;
    bool in = false;
    if (valid && !h && (more >> k & 1u)) in = stay_inserts(q, q.cuts[it[k]], next[k], v);
    const uint64_t hw = __ballot(valid && h), iw = __ballot(in);
    const int64_t x = base + k * WAVE;
    if (lane == 0 && x < n) {
      hit_words[x / WAVE] = hw;
      ins_words[x / WAVE] = iw;
    }
    heads += __popcll(__ballot(head >> k & 1u));
  }
  // the last accesses, at the rank of their run
  if (lane == 0) s_heads[wave] = heads;
  __syncthreads();
  int64_t r = head_bases[blockIdx.x];
  for (int w = 0; w < wave; ++w) r += s_heads[w];
#pragma unroll
  for (int k = 0; k < LINK_CHUNKS; ++k) {
    const uint64_t hm = __ballot(head >> k & 1u);
    const bool last = (cur[k] >> 32) != 0xFFFFFFFFull && !(more >> k & 1u);
    const uint64_t upto = lane == WAVE - 1 ? ~0ull : (2ull << lane) - 1ull;
    if (last) nv.rows[r + __popcll(hm & upto) - 1] =
        (cur[k] & 0xFFFFFFFF00000000ull) | (hit >> k & 1u ? (uint32_t)it[k] : NOT_HERE);
    r += __popcll(hm);
  }
}

// insertions of iteration i = set bits of its positions (blockIdx.x = i, by the blocks of the column, added to
// zeros); miss_count: where all misses are inserted
__global__ __launch_bounds__(TB) void k_ins_count(const uint32_t* __restrict__ ins_bits,
                                                  const int64_t* __restrict__ off,
                                                  int64_t* __restrict__ cs_offsets,
                                                  int64_t* __restrict__ miss_count) {
  __shared__ uint32_t red[TB / WAVE];
  const int64_t lo = off[blockIdx.x], hi = off[blockIdx.x + 1];
  uint32_t cnt = 0;
  if (hi > lo)
    for (int64_t w = (lo >> 5) + blockIdx.y * TB + threadIdx.x; w <= (hi - 1) >> 5; w += (int64_t)gridDim.y * TB) {
      uint32_t word = ins_bits[w];
      if (w == lo >> 5) word &= ~((1u << (lo & 31)) - 1u);
      if (w == (hi - 1) >> 5 && (hi & 31)) word &= (1u << (hi & 31)) - 1u;
      cnt += __popc(word);
    }
  const uint32_t total = block_sum_u32(cnt, red);
  if (threadIdx.x == 0 && total) {
    atomicAdd((unsigned long long*)&cs_offsets[blockIdx.x + 1], (unsigned long long)total);
    if (miss_count) atomicAdd((unsigned long long*)&miss_count[blockIdx.x], (unsigned long long)total);
  }
}

// cs_offsets[1 .. S] <- inclusive sums, and the same for the host
__global__ __launch_bounds__(BIG) void k_ins_offsets(int64_t* __restrict__ cs_offsets, int32_t S,
                                                     int64_t* __restrict__ copy) {
  __shared__ int64_t smem[BIG / WAVE + 1];
  const int32_t per = (S + BIG - 1) / BIG, j0 = threadIdx.x * per;
  int64_t mine = 0;
  for (int32_t j = j0; j < j0 + per && j < S; ++j) mine += cs_offsets[j + 1];
  int64_t total;
  int64_t run = block_exclusive_scan<int64_t, BIG>(mine, smem, total);
  for (int32_t j = j0; j < j0 + per && j < S; ++j) {
    run += cs_offsets[j + 1];
    cs_offsets[j + 1] = run;
    copy[j + 1] = run;
  }
  if (threadIdx.x == 0) copy[0] = 0;
}

// What becomes of the line of an inserted row (or of a start-state row): the iteration that evicts
// it, LEAVES_NEXT if that is the one after its insertion, STAYS if none does.
constexpr uint32_t STAYS = 0xFFFFFFFFu;
constexpr uint32_t LEAVES_NEXT = 0xFFFFFFFEu;

// The record of an insertion: that, and the position of the row's next access where this is a hit of the iteration
// after the insertion and marked HANDED_OVER (see k_move_lines).
constexpr uint32_t NO_POSITION = 0xFFFFFFFFu;
__device__ __forceinline__ uint64_t ins_record(uint32_t leaves, uint32_t next_position) {
  return (uint64_t)next_position << 32 | leaves;
}

// The insertions' bits and the number of them in front of each word: side by side where the workspace has room (one
// random word per insertion instead of two), else in two arrays.
struct InsIndex {
  const uint64_t* pairs;   // [words] bits | in front << 32, or null
  const uint32_t *bits, *base;
  __device__ __forceinline__ uint64_t word(uint32_t p) const {
    return pairs ? pairs[p >> 5] : (uint64_t)base[p >> 5] << 32 | bits[p >> 5];
  }
  // The insertion at position p, from its word.
  static __device__ __forceinline__ uint32_t index(uint64_t word, uint32_t p) {
    return (uint32_t)(word >> 32) + __popc((uint32_t)word & ((1u << (p & 31)) - 1u));
  }
};

// The second pass in node order: for every insertion, and for the first access of every start-state row
// that hits, the iteration that evicts the row.  A resident access is linked to its right neighbour if
// that is a hit of the same row; the first stay that does not reach a hit gives the iteration for
// all accesses linked to it, and only for those stays it is looked up.  A wave takes a stretch of
// WALK_CHUNKS * 64 accesses; the words of hits and one shuffle serve 64 of them, from right to left,
// and what no stay of a chunk settles comes from the chunk to its right (for the last chunk: from
// behind the stretch, at most S accesses of one row).  Following the links access by access instead
// (one thread per insertion) took 3.3 ms for 33 M accesses of 8.8 M rows and 32 ms for 154 M accesses
// of rows that mostly stay, waves waiting for their longest row.
constexpr int WALK_CHUNKS = 8;
constexpr int64_t WALK_TILE = (int64_t)TB * WALK_CHUNKS;

// The iteration that ends a resident's stay from iteration i on, which does not reach a hit (right: the
// position of the row's next access, if there is one), as a record.
__device__ __forceinline__ uint32_t walk_leaves(const Stays& q, const IterFinder& iteration, const int32_t* never,
                                                uint32_t v, int32_t i, bool more, uint32_t right) {
  const int32_t e = more ? stay_end(q, (uint32_t)i, iteration(right), v, nullptr, q.S)
                         : never_end(never, q.S, never_levels(q.S), i, v);
  return e < q.S ? (uint32_t)e : STAYS;
}

// NEVER_LDS: the limits of bucket "never" in LDS (their random reads are what a wave waits for most),
// while that leaves room for eight blocks per CU.
constexpr int32_t NEVER_LDS_S = 400;

// (five waves per SIMD: 96 registers; with one more, which the compiler takes or not as other code in
// the file changes, four, and 466 us instead of 401 for 33 M accesses)
template <bool NEVER_LDS>
__global__ __launch_bounds__(TB) __attribute__((amdgpu_waves_per_eu(5))) void k_stays_walk(
    Stays q, const uint64_t* __restrict__ sorted, int64_t n, const int32_t* __restrict__ addr,
                                                   const uint64_t* __restrict__ hit_words,
                                                   const uint64_t* __restrict__ ins_words,
                                                   InsIndex at_ins, uint64_t* __restrict__ leave_ins,
                                                   uint32_t* __restrict__ leave_start,
                                                   int32_t* __restrict__ hand_over) {
  extern __shared__ int32_t lds_off[];    // offsets [S + 1], limits [levels * (S + 1)]
  const int32_t* never = q.never;
  if (NEVER_LDS) {
    int32_t* mine = lds_off + q.S + 1;
    for (int x = threadIdx.x; x < never_levels(q.S) * (q.S + 1); x += TB) mine[x] = q.never[x];
    never = mine;
  }
  __shared__ uint16_t s_coarse[IterFinder::COARSE + 1];
  const IterFinder iteration = iter_finder(lds_off, s_coarse, q.off, q.S);
  const int lane = lane_id();
  const int64_t base = ((int64_t)blockIdx.x * (TB / WAVE) + threadIdx.x / WAVE) * (WAVE * WALK_CHUNKS);
  if (base >= n) return;                           // uniform over the wave
  const int64_t words = (n + WAVE - 1) / WAVE;
  uint64_t cur[WALK_CHUNKS + 1], hit[WALK_CHUNKS + 1], ins[WALK_CHUNKS];
#pragma unroll
  for (int k = 0; k <= WALK_CHUNKS; ++k) {
    const int64_t x = base + k * WAVE + (k < WALK_CHUNKS ? lane : 0), w = base / WAVE + k;
    cur[k] = x < n ? sorted[x] : ~0ull;            // behind n: an id that no access has
    hit[k] = w < words ? hit_words[w] : 0ull;
    if (k < WALK_CHUNKS) ins[k] = w < words ? ins_words[w] : 0ull;
  }
  const uint64_t left_of = base > 0 ? sorted[base - 1] : ~0ull;
  // the insertions' places in their list, all read at once
  uint32_t slot[WALK_CHUNKS];
  {
    uint64_t word[WALK_CHUNKS];
#pragma unroll
    for (int k = 0; k < WALK_CHUNKS; ++k)
      if (ins[k] >> lane & 1) word[k] = at_ins.word((uint32_t)cur[k]);
#pragma unroll
    for (int k = 0; k < WALK_CHUNKS; ++k) slot[k] = InsIndex::index(word[k], (uint32_t)cur[k]);
  }
  uint64_t stops[WALK_CHUNKS];                     // the stays that do not reach a hit
  uint32_t leave_of[WALK_CHUNKS];
#pragma unroll
  for (int k = 0; k < WALK_CHUNKS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    uint64_t right = ((uint64_t)from_right(v) << 32) | from_right(p);
    const uint64_t other = of_lane(cur[k + 1], 0);
    if (lane == WAVE - 1) right = other;
    const uint64_t right_hits = (hit[k] >> 1) | (hit[k + 1] << (WAVE - 1));
    const bool more = (uint32_t)(right >> 32) == v;
    const bool end = !(more && (right_hits >> lane & 1));
    stops[k] = __ballot(end);
    leave_of[k] = STAYS;
    if (end && ((hit[k] | ins[k]) >> lane & 1))
      leave_of[k] = walk_leaves(q, iteration, never, v, iteration(p), more, (uint32_t)right);
  }
  uint32_t carry = STAYS;
#pragma unroll
  for (int k = WALK_CHUNKS - 1; k >= 0; --k) {
    if (k == WALK_CHUNKS - 1 && !(stops[k] >> (WAVE - 1))) {
      // the stretch's last access is linked to the next stretch: on to the row's next stay that ends
      // (at the latest with its last access)
      for (int64_t ahead = base + WALK_CHUNKS * WAVE; ; ahead += WAVE) {
        const int64_t y = ahead + lane, w = ahead / WAVE;
        const uint64_t a = y < n ? sorted[y] : ~0ull, r = y + 1 < n ? sorted[y + 1] : ~0ull;
        const bool more = y + 1 < n && (uint32_t)(r >> 32) == (uint32_t)(a >> 32);
        const uint64_t h = w < words ? hit_words[w] : 0ull, h1 = w + 1 < words ? hit_words[w + 1] : 0ull;
        const uint64_t m = __ballot(!(more && (((h >> 1) | (h1 << (WAVE - 1))) >> lane & 1)));
        if (!m) continue;                          // (an access at or behind n ends)
        const int at = __ffsll((unsigned long long)m) - 1;
        uint32_t leaves = STAYS;
        if (lane == at && y < n)
          leaves = walk_leaves(q, iteration, never, (uint32_t)(a >> 32), iteration((uint32_t)a),
                               more, (uint32_t)r);
        carry = __shfl(leaves, at, WAVE);
        break;
      }
    }
    const uint64_t mine = stops[k] >> lane;        // stays that end, from this lane's on
    const uint32_t found = __shfl(leave_of[k], mine ? lane + __ffsll((unsigned long long)mine) - 1 : lane, WAVE);
    const uint32_t leaves = mine ? found : carry;
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    uint32_t rp = from_right(p);         // the next access, if it is one of the row
    const uint32_t op = of_lane((uint32_t)cur[k + 1], 0);
    if (lane == WAVE - 1) rp = op;
    if (ins[k] >> lane & 1) {
      const int32_t i = iteration(p);
      uint32_t next = NO_POSITION;
      // (no end here: a hit of the row)
      if (hand_over && !(stops[k] >> lane & 1) && (int32_t)rp < lds_off[i + 2]) hand_over[next = rp] = HANDED_OVER;
      leave_ins[slot[k]] = ins_record(leaves == (uint32_t)(i + 1) ? LEAVES_NEXT : leaves, next);
    }
    // a first access that hits is one of a start-state row
    uint32_t lv = (uint32_t)from_left(v);
    const uint64_t before = k > 0 ? of_lane(cur[k > 0 ? k - 1 : 0], WAVE - 1) : left_of;
    if (lane == 0) lv = (uint32_t)(before >> 32);
    if ((hit[k] >> lane & 1) && lv != v) leave_start[addr[v]] = leaves;
    carry = of_lane(leaves, 0);
  }
}

// The same for LRU, where hits follow from the limits (copied to LDS) and the neighbour in node order, so that one
// pass does what k_stays_links and the kernel above do.
__global__ __launch_bounds__(TB) void k_lru_walk(Stays q, const uint64_t* __restrict__ sorted, int64_t n,
                                                 const uint64_t* __restrict__ last_head,
                                                 const int32_t* __restrict__ addr,
                                                 InsIndex at_ins, uint64_t* __restrict__ leave_ins,
                                                 uint32_t* __restrict__ leave_start,
                                                 int32_t* __restrict__ hand_over) {
  extern __shared__ uint64_t lds_limits[];         // [S], then the offsets [S + 1]
  int32_t* const lds_off = reinterpret_cast<int32_t*>(lds_limits + q.S);
  for (int x = threadIdx.x; x < q.S; x += TB) lds_limits[x] = q.limits[x];
  __shared__ uint16_t s_coarse[IterFinder::COARSE + 1];
  const IterFinder find = iter_finder(lds_off, s_coarse, q.off, q.S);
  const int lane = lane_id();
  const int64_t base = ((int64_t)blockIdx.x * (TB / WAVE) + threadIdx.x / WAVE) * (WAVE * WALK_CHUNKS);
  if (base >= n) return;                           // uniform over the wave
  auto iteration = [&](uint64_t pair) {
    return (pair >> 32) != 0xFFFFFFFFull ? find((uint32_t)pair) : q.S;
  };
  // the stay of an access of row v in iteration i reaches the row's next access, in iteration j
  auto reaches = [&](uint32_t v, int32_t i, int32_t j) { return lru_key((uint32_t)i, v) >= lds_limits[j > 0 ? j - 1 : 0]; };
  auto leaves_at = [&](uint32_t v, int32_t i) {
    const int32_t e = lru_end(lds_limits, q.S, i, lru_key((uint32_t)i, v));
    return e < q.S ? (uint32_t)e : STAYS;
  };
  uint64_t cur[WALK_CHUNKS + 1];                   // behind n: an id that no access has
  int32_t it[WALK_CHUNKS + 1];
#pragma unroll
  for (int k = 0; k <= WALK_CHUNKS; ++k) {
    const int64_t x = base + k * WAVE + (k < WALK_CHUNKS ? lane : 0);
    cur[k] = x < n ? sorted[x] : ~0ull;
  }
  const uint64_t left_of = base > 0 ? sorted[base - 1] : ~0ull;
#pragma unroll
  for (int k = 0; k <= WALK_CHUNKS; ++k) it[k] = iteration(cur[k]);
  uint64_t stops[WALK_CHUNKS];                     // the stays that do not reach a hit
  uint32_t leave_of[WALK_CHUNKS];
#pragma unroll
  for (int k = 0; k < WALK_CHUNKS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32);
    uint32_t rv = from_right(v);
    int32_t rj = from_right(it[k]);
    const uint32_t ov = of_lane((uint32_t)(cur[k + 1] >> 32), 0);
    const int32_t oj = of_lane(it[k + 1], 0);
    if (lane == WAVE - 1) {
      rv = ov;
      rj = oj;
    }
    const bool valid = v != 0xFFFFFFFFu;
    const bool end = !(valid && rv == v && reaches(v, it[k], rj));
    stops[k] = __ballot(end);
    leave_of[k] = valid && end ? leaves_at(v, it[k]) : STAYS;
  }
  bool left_reaches = false;                       // (uniform: chunk 0's first pair is in range)
  {
    const uint32_t v = of_lane((uint32_t)(cur[0] >> 32), 0);
    if ((uint32_t)(left_of >> 32) == v) left_reaches = reaches(v, iteration(left_of), of_lane(it[0], 0));
  }
  uint32_t carry = STAYS;
#pragma unroll
  for (int k = WALK_CHUNKS - 1; k >= 0; --k) {
    if (k == WALK_CHUNKS - 1 && !(stops[k] >> (WAVE - 1))) {
      // the stretch's last access is linked to the next stretch: on to the row's next stay that ends
      for (int64_t ahead = base + WALK_CHUNKS * WAVE; ; ahead += WAVE) {
        const int64_t y = ahead + lane;
        const uint64_t a = y < n ? sorted[y] : ~0ull, r = y + 1 < n ? sorted[y + 1] : ~0ull;
        const int32_t i = iteration(a);
        const bool end = !(y + 1 < n && (r >> 32) == (a >> 32) && reaches((uint32_t)(a >> 32), i, iteration(r)));
        const uint64_t m = __ballot(end);
        if (!m) continue;                          // (an access at or behind n ends)
        const int at = __ffsll((unsigned long long)m) - 1;
        uint32_t leaves = STAYS;
        if (lane == at && y < n) leaves = leaves_at((uint32_t)(a >> 32), i);
        carry = __shfl(leaves, at, WAVE);
        break;
      }
    }
    const uint64_t mine = stops[k] >> lane;        // stays that end, from this lane's on
    const uint32_t found = __shfl(leave_of[k], mine ? lane + __ffsll((unsigned long long)mine) - 1 : lane, WAVE);
    const uint32_t leaves = mine ? found : carry;
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    uint32_t lv = (uint32_t)from_left(v);
    const uint64_t before = k > 0 ? of_lane(cur[k > 0 ? k - 1 : 0], WAVE - 1) : left_of;
    bool linked = lane > 0 ? !(stops[k] >> (lane - 1) & 1) : k > 0 ? !(stops[k > 0 ? k - 1 : 0] >> (WAVE - 1)) : left_reaches;
    if (lane == 0) lv = (uint32_t)(before >> 32);
    uint32_t rp = from_right(p);         // the next access, if it is one of the row
    const uint32_t op = of_lane((uint32_t)cur[k + 1], 0);
    if (lane == WAVE - 1) rp = op;
    if (v != 0xFFFFFFFFu) {
      if (lv == v ? !linked : !in_start_state(v, it[k], last_head, nullptr)) {   // a miss: inserted
        uint32_t next = NO_POSITION;
        if (hand_over && !(stops[k] >> lane & 1) && (int32_t)rp < lds_off[it[k] + 2])
          hand_over[next = rp] = HANDED_OVER;
        leave_ins[InsIndex::index(at_ins.word(p), p)] =
            ins_record(leaves == (uint32_t)(it[k] + 1) ? LEAVES_NEXT : leaves, next);
      } else if (lv != v)                            // a first access that hits is one of a start-state row
        leave_start[addr[v]] = leaves;
    }
    carry = of_lane(leaves, 0);
  }
}

// Start-state rows that the superbatch never accesses (carried caches; accessed: bitmap over ids).
__global__ __launch_bounds__(TB) void k_stays_idle(Stays q, const int32_t* __restrict__ res_id,
                                                   const uint32_t* __restrict__ accessed, int64_t cap,
                                                   uint32_t* __restrict__ leave_start) {
  const int64_t l = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (l >= cap) return;
  const uint32_t v = (uint32_t)res_id[l];
  if (accessed[v >> 5] >> (v & 31) & 1u) return;
  const int32_t e = never_end(q.never, q.S, never_levels(q.S), 0, v);
  leave_start[l] = e < q.S ? (uint32_t)e : STAYS;
}

// Turns the evicting iterations into places of the per-iteration lists of evicted lines (list of
// iteration e: from cs_offsets[e] on, filled[e] entries): a start-state row's line goes there now,
// an insertion's record keeps the place for the step that learns its line.  A block counts per
// iteration in LDS first, so that a counter sees one atomic per block.
__global__ __launch_bounds__(TB) void k_leave_places(int64_t n_ins, int64_t cap, int32_t S,
                                                     uint64_t* __restrict__ leave_ins,
                                                     const uint32_t* __restrict__ leave_start,
                                                     const int64_t* __restrict__ cs_offsets,
                                                     uint32_t* __restrict__ filled,
                                                     int32_t* __restrict__ leaving) {
  extern __shared__ uint32_t s_cnt[];     // [S]
  for (int e = threadIdx.x; e < S; e += TB) s_cnt[e] = 0;
  __syncthreads();
  const int64_t n = n_ins + cap;
  const int64_t per = ((n + gridDim.x - 1) / gridDim.x + TB - 1) / TB * TB;
  const int64_t first = (int64_t)blockIdx.x * per, last = first + per < n ? first + per : n;
  for (int64_t x = first + threadIdx.x; x < last; x += TB) {
    const uint32_t e = x < n_ins ? (uint32_t)leave_ins[x] : leave_start[x - n_ins];
    if (e < (uint32_t)S) atomicAdd(&s_cnt[e], 1u);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < S; e += TB) {
    const uint32_t c = s_cnt[e];
    s_cnt[e] = c ? (uint32_t)cs_offsets[e] + atomicAdd(&filled[e], c) : 0u;
  }
  __syncthreads();
  for (int64_t x = first + threadIdx.x; x < last; x += TB) {
    const uint32_t e = x < n_ins ? (uint32_t)leave_ins[x] : leave_start[x - n_ins];
    if (e >= (uint32_t)S) continue;
    const uint32_t at = atomicAdd(&s_cnt[e], 1u);
    const bool room = (int64_t)at < cs_offsets[e + 1];   // (always, for distinct ids)
    if (x < n_ins) leave_ins[x] = room ? at : STAYS;
    else if (room) leaving[at] = (int32_t)(x - n_ins);
  }
}

// ---- the lines: one launch per iteration -----------------------------------------------------------
//
// For more lines than the blocks of k_move_lines hold in LDS, and where these did not all run (see lines.hpp).

constexpr int64_t LARGE_CACHE = int64_t(1) << 21;   // lines from which tiles and blocks of the steps are larger

struct Step {
  uint64_t *now, *next;        // flag words: lines evicted by this iteration / the next one
  uint32_t *cnt_now, *cnt_next, *cnt_clear;   // set flags per tile of 2^tile_shift lines; cnt_clear: to be zeroed
  int64_t words, tiles;
  int32_t tile_shift, cnt_shift;   // a counter every 2^cnt_shift words
  int64_t emit_blocks, flag_blocks;
  int64_t dst, n_change;       // this iteration's records
  int64_t next_dst, next_n;    // the next iteration's
  const uint32_t* next_filled; // entries of the next iteration's list that stem from earlier iterations
  int32_t* leaving;            // lists of evicted lines
  const uint64_t* leave_ins;   // per insertion: place in `leaving`, LEAVES_NEXT or STAYS (the lower half)
  const int32_t* in_ids;
  int32_t* out_ids;
  const int32_t* ids;          // this iteration's accesses
  int32_t* src_line;           // null: not asked for
  int64_t n;
};

__device__ __forceinline__ void flag_line(const Step& s, int32_t line) {
  atomicOr((unsigned long long*)&s.next[line >> 6], 1ull << (line & 63));
  atomicAdd(&s.cnt_next[line >> s.tile_shift << s.cnt_shift], 1u);
}

// Where an iteration changes more than a sixteenth of the lines (DENSE), additions to the counters of
// a few hundred tiles queue up, and blocks of 4 096 lines have many rounds of evictions to go.  A block
// takes the lines of one tile and counts in LDS first then, as far as the tiles have room there (36 k
// lines, about 20 k changes: 51 -> 9.5 us per iteration; 1.2 M lines, 0.4 M changes: 112 -> 45).
// LRU gives lines up in the order in which they were taken, so that an iteration's lie side by side and meet in
// a few counters however few they are: DENSE as long as the tiles' counters are in LDS (100 x 150 000 accesses, 1.4 M
// lines, 22 k changes: 4 588 -> 2 863 us a call; 60 x 600 000, 4.9 M lines: 8 989 -> 4 491; 567 changes in 2.7 M lines:
// 1 716 -> 1 611).  Belady's are spread, and the small tiles of DENSE cost more than they save (1.4 M lines, 4 k changes:
// 2 192 against 2 545).
constexpr int DENSE_SHARE = 16;
constexpr int DENSE_TILES = 4096;
constexpr int64_t DENSE_ENTRIES = 2048;   // of the list of leaving lines, to a block at a time

// The lines the next iteration evicts, as far as they were taken before this one; vb: block of `blocks`.
template <bool DENSE>
__device__ __forceinline__ void flag_leaving(const Step& s, int64_t vb, int64_t blocks, uint32_t* s_tiles) {
  const int64_t have = *s.next_filled < s.next_n ? *s.next_filled : s.next_n;
  const bool in_lds = DENSE && s.tiles <= DENSE_TILES;
  if (in_lds) {
    for (int q = threadIdx.x; q < s.tiles; q += TB) s_tiles[q] = 0;
    __syncthreads();
  }
  constexpr int ITEMS = DENSE ? (int)(DENSE_ENTRIES / TB) : 1;
  for (int64_t x0 = vb * (TB * ITEMS) + threadIdx.x; x0 < have; x0 += blocks * (TB * ITEMS)) {
    int32_t line[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) line[k] = s.leaving[s.next_dst + (x0 + k * TB < have ? x0 + k * TB : x0)];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      if (x0 + k * TB >= have) continue;
      if (in_lds) {
        atomicOr((unsigned long long*)&s.next[line[k] >> 6], 1ull << (line[k] & 63));
        atomicAdd(&s_tiles[line[k] >> s.tile_shift], 1u);
      } else {
        flag_line(s, line[k]);
      }
    }
  }
  if (in_lds) {
    __syncthreads();
    for (int q = threadIdx.x; q < s.tiles; q += TB)
      if (s_tiles[q]) atomicAdd(&s.cnt_next[q << s.cnt_shift], s_tiles[q]);
  }
}

// The flagged lines in line order take the iteration's insertions (a list known up front).  Roles
// by block: [0, emit_blocks) lists and lines, LINE_WORDS flag words each; the next flag_blocks flag
// the lines the next iteration evicts, as far as they were taken before this iteration (the others
// are flagged by the emit blocks themselves); the rest looks up the lines of the iteration's hits.
// Nothing one role reads is written by another: a row that hits is not inserted by the same
// iteration, an evicted row keeps its address-table entry (its next access, a miss, does not
// read it), and flags and counts alternate between two and three copies.  DENSE: a block takes the lines of
// one tile, so that its evictions are few rounds of its threads.
template <int LINE_WORDS, bool DENSE>   // flag words (64 lines each) a block of the emit role takes
__global__ __launch_bounds__(TB) void k_step_lines(State st, Step s) {
  constexpr int STEPS = LINE_WORDS == 8 ? 3 : LINE_WORDS == 64 ? 6 : 8;
  static_assert(1 << STEPS == LINE_WORDS && LINE_WORDS <= TB, "a word per thread, found by bisection");
  __shared__ uint32_t red[TB / WAVE], smem[TB / WAVE + 1];
  __shared__ uint64_t s_word[LINE_WORDS];
  __shared__ uint32_t s_incl[LINE_WORDS];
  __shared__ uint32_t s_tiles[DENSE ? DENSE_TILES : 1];   // (the emit role: flags for the next iteration)
  const int64_t b = blockIdx.x;
  if (b >= s.emit_blocks + s.flag_blocks) {
    constexpr int ITEMS = 4;
    const int64_t base = (b - s.emit_blocks - s.flag_blocks) * (TB * ITEMS) + threadIdx.x;
    int32_t v[ITEMS], mark[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int64_t p = base + k * TB;
      v[k] = s.ids[p < s.n ? p : 0];
      mark[k] = p < s.n ? s.src_line[p] : -1;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
      if (mark[k] >= 0) mark[k] = st.addr[v[k]];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
      if (mark[k] >= 0) s.src_line[base + k * TB] = mark[k];
    return;
  }
  if (b >= s.emit_blocks) {
    flag_leaving<DENSE>(s, b - s.emit_blocks, s.flag_blocks, s_tiles);
    return;
  }
  const int64_t first_word = b * LINE_WORDS;
  const int64_t first_tile = (first_word * 64) >> s.tile_shift;
  const int64_t own_tiles = (LINE_WORDS * 64) >> s.tile_shift;
  if (threadIdx.x < own_tiles && first_tile + threadIdx.x < s.tiles)
    s.cnt_clear[(first_tile + threadIdx.x) << s.cnt_shift] = 0;
  if (s.n_change == 0) return;
  uint64_t word = 0;
  if (threadIdx.x < LINE_WORDS) {                  // whole waves
    const int64_t at = first_word + threadIdx.x;
    word = at < s.words ? s.now[at] : 0;
    if (word) s.now[at] = 0;                       // consumed
    s_word[threadIdx.x] = word;
  }
  const uint32_t flags = (uint32_t)__popcll(word);
  uint32_t total;
  const uint32_t ahead = block_exclusive_scan<uint32_t, TB>(flags, smem, total);
  if (threadIdx.x < LINE_WORDS) s_incl[threadIdx.x] = ahead + flags;
  if (DENSE && threadIdx.x < 2 * LINE_WORDS) s_tiles[threadIdx.x] = 0;   // two halves of every word
  if (total == 0) return;                          // uniform
  uint32_t counted = 0;
  for (int64_t q = threadIdx.x; q < first_tile; q += TB) counted += s.cnt_now[q << s.cnt_shift];
  const int64_t before = block_sum_u32(counted, red);
  for (uint32_t k = threadIdx.x; k < total; k += TB) {
    int lo = 0, hi = LINE_WORDS - 1;               // the word of the k-th flag
#pragma unroll
    for (int step = 0; step < STEPS; ++step) {
      const int mid = (lo + hi) >> 1;
      if (s_incl[mid] > k) hi = mid; else lo = mid + 1;
    }
    uint64_t bits = s_word[lo];
    for (uint32_t skip = k - (s_incl[lo] - (uint32_t)__popcll(bits)); skip > 0; --skip) bits &= bits - 1;
    const int32_t line = (int32_t)((first_word + lo) * 64 + (__ffsll((unsigned long long)bits) - 1));
    const int64_t at = before + k;
    if (at >= s.n_change) continue;                // (as many lines as insertions, for distinct ids)
    const int32_t gone = st.res_id[line];
    const int32_t comes = s.in_ids[s.dst + at];
    const uint32_t leaves = (uint32_t)s.leave_ins[s.dst + at];
    s.out_ids[s.dst + at] = gone;
    st.res_id[line] = comes;
    st.addr[comes] = line;
    if (leaves == LEAVES_NEXT) {
      if (DENSE) atomicOr(&s_tiles[(line >> 5) - first_word * 2], 1u << (line & 31));   // a line of the block's own
      else flag_line(s, line);
    } else if (leaves != STAYS) {
      s.leaving[leaves] = line;
    }
  }
  if (DENSE) {
    __syncthreads();
    if (threadIdx.x < LINE_WORDS) {
      const uint64_t flagged = ((uint64_t)s_tiles[2 * threadIdx.x + 1] << 32) | s_tiles[2 * threadIdx.x];
      const int64_t tile = ((first_word + threadIdx.x) * 64) >> s.tile_shift;
      uint32_t count = (uint32_t)__popcll(flagged);
      if (count) atomicOr((unsigned long long*)&s.next[first_word + threadIdx.x], flagged);
      // (a block's words are those of one tile, and fewer than a wave has lanes or as many)
      for (int d = 1; d < LINE_WORDS; d <<= 1) count += __shfl_xor(count, d, WAVE);
      if (threadIdx.x == 0 && count) atomicAdd(&s.cnt_next[tile << s.cnt_shift], count);
    }
  }
}

// the lines the first iteration evicts
template <bool DENSE>
__global__ __launch_bounds__(TB) void k_step_flags(Step s) {
  __shared__ uint32_t s_tiles[DENSE ? DENSE_TILES : 1];
  flag_leaving<DENSE>(s, blockIdx.x, gridDim.x, s_tiles);
}
