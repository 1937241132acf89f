// Belady changesets of the smallest calls: the loop over the iterations in one workgroup.  Included by
// changeset.hip only.
//
// A call on some ten thousand accesses is a chain of launches that do next to nothing, some 40 of them from the trace,
// six to an iteration in the loop over the state, with waits for the host in between.
// Here the rows are numbered by rank (in id order, so that ids compare as ranks), which makes the whole state of the
// cache fit LDS as 16-bit words, and one workgroup goes through the iterations: the same steps as the loop
// (see there), with barriers between them instead of launches.
//   k_small_ranks   rank and next accessed iteration of every access, id and first iteration of every row
//   k_small_belady  C_0, then the iterations
// 8 iterations of 3 500 accesses to 10 900 rows, 1 858 lines: from the trace 405 us a call, the loop 480; this way 219.
// On 16 384 nodes, 2 048 lines: 230, k_small_ranks 9 and k_small_belady 82 (some 20 barriers and two reads of the
// accesses an iteration, 10 us), the rest the sort and two waits for the host.
#pragma once

constexpr int SMALL_ROWS = 12288;          // five arrays of 24 KB
constexpr int SMALL_S = 256;               // iterations at most (LDS counters of a wave per iteration)
// One workgroup takes 5 us for an iteration of 600 accesses, 18 for one of 10 000; all iterations' lines in one launch
// 3 to 6, more where many iterations have cuts, behind some 250 us of other launches.  Up to 12 200 rows, by lines held
// (share of the rows), from the trace and this way: 2 x 40 (half) 253 and 134 us, 256 x 600 (0.3) 1 674 and 1 301, (0.9)
// 1 674 and 1 460, 128 x 1 200 (0.3) 1 040 and 892, 32 x 3 500 (0.3) 599 and 430, 16 x 10 000 (0.3) 643 and 405, (0.7)
// 465 and 410; beyond: 128 x 3 500 (0.3) 1 578 and 1 281, but 256 x 3 500 (0.8) 1 962 and 2 714, 100 x 10 000 (0.9)
// 1 081 and 1 801.
constexpr int64_t SMALL_IDS = 163'840;     // (16 x 10 000, some more)
constexpr uint32_t NOT_RESIDENT = 0xFFFFu;

struct Small {
  uint32_t* access;        // [total] rank | next << 16
  int32_t* id;             // [rows]
  uint32_t* first;         // [rows] first iteration
  const int64_t* off;
  int32_t rows, cap, S;
  int32_t* init_ids;
  int32_t *in_ids, *out_ids, *in_positions;
  int64_t cs_capacity;
  int64_t *cs_offsets, *miss_count;
  int32_t* src_line;       // null: not asked for
  int64_t *ready, *cs_copy;          // [S] rows of C_0 first accessed up to an iteration, [S + 1] cs_offsets, for the host
};

__global__ __launch_bounds__(TB) void k_small_ranks(const uint64_t* __restrict__ sorted, int64_t n,
                                                    const uint32_t* __restrict__ head_bases, Small s) {
  __shared__ int32_t lds_off[SMALL_S + 1];
  __shared__ uint32_t s_heads[TB / WAVE];
  load_offsets(lds_off, s.off, s.S);
  const int lane = lane_id(), wave = threadIdx.x / WAVE;
  const int64_t base = (int64_t)blockIdx.x * LOOK_TILE + wave * (WAVE * LOOK_ITEMS);
  uint64_t cur[LOOK_ITEMS + 1];            // behind n: an id that no access has
#pragma unroll
  for (int k = 0; k <= LOOK_ITEMS; ++k) {
    const int64_t x = base + k * WAVE + (k < LOOK_ITEMS ? lane : 0);
    cur[k] = x < n ? sorted[x] : ~0ull;
  }
  uint32_t before = base > 0 && base - 1 < n ? (uint32_t)(sorted[base - 1] >> 32) : 0xFFFFFFFFu;
  uint64_t heads[LOOK_ITEMS];
  uint32_t count = 0;
#pragma unroll
  for (int k = 0; k < LOOK_ITEMS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32);
    uint32_t left = from_left(v);
    if (lane == 0) left = before;
    before = of_lane(v, WAVE - 1);
    heads[k] = __ballot(v != left && v != 0xFFFFFFFFu);
    count += __popcll(heads[k]);
  }
  if (lane == 0) s_heads[wave] = count;
  __syncthreads();
  uint32_t run = head_bases[blockIdx.x];
  for (int w = 0; w < wave; ++w) run += s_heads[w];
  const uint64_t upto = lane == WAVE - 1 ? ~0ull : (2ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < LOOK_ITEMS; ++k) {
    const uint32_t v = (uint32_t)(cur[k] >> 32), p = (uint32_t)cur[k];
    uint32_t rv = from_right(v), rp = from_right(p);
    const uint64_t other = of_lane(cur[k + 1], 0);
    if (lane == WAVE - 1) {
      rv = (uint32_t)(other >> 32);
      rp = (uint32_t)other;
    }
    const uint32_t rank = run + __popcll(heads[k] & upto) - 1;
    run += __popcll(heads[k]);
    if (base + k * WAVE + lane >= n) continue;
    const uint32_t next = rv == v ? (uint32_t)iter_of(lds_off, s.S, (int32_t)rp) : (uint32_t)s.S;
    s.access[p] = rank | next << 16;
    if (heads[k] >> lane & 1) {
      s.id[rank] = (int32_t)v;
      s.first[rank] = (uint32_t)iter_of(lds_off, s.S, (int32_t)p);
    }
  }
}

__global__ __launch_bounds__(BIG) void k_small_belady(Small s) {
  constexpr int WAVES = BIG / WAVE, WORDS = SMALL_ROWS / 32;
  static_assert(SMALL_ROWS % BIG == 0 && WORDS <= BIG, "");
  __shared__ uint16_t s_line[SMALL_ROWS];  // of a row
  __shared__ uint16_t s_key[SMALL_ROWS];   // its next accessed iteration
  __shared__ uint16_t s_row[SMALL_ROWS];   // of a line
  __shared__ uint16_t s_in[SMALL_ROWS];    // rows inserted in the iteration, in the order of their positions
  __shared__ uint16_t s_out[SMALL_ROWS];   // lines evicted, in order
  __shared__ uint32_t s_bits[WORDS];       // members of the class that is selected from
  __shared__ uint32_t s_res[SMALL_S + 1], s_inc[SMALL_S + 1];   // residents, incoming rows by key
  __shared__ uint16_t s_count[WAVES][SMALL_S];
  __shared__ uint32_t smem[WAVES + 1];
  __shared__ uint32_t s_misses;
  __shared__ int32_t s_jstar, s_mode_in, s_mode_res, s_T;
  __shared__ uint32_t s_keep, s_kept;
  const int me = threadIdx.x, lane = lane_id(), wave = me / WAVE;
  const int32_t S = s.S, rows = s.rows, cap = s.cap;

  // C_0: the rows by (first access, rank).  A wave takes a stretch of rows, twice: for the iterations' numbers
  // in it and, with those in front, for the lines.
  for (int x = me; x < WAVES * SMALL_S; x += BIG) (&s_count[0][0])[x] = 0;
  for (int j = me; j <= S; j += BIG) s_res[j] = s_inc[j] = 0;
  for (int x = me; x < WORDS; x += BIG) s_bits[x] = 0;
  __syncthreads();
  const int32_t stretch = ((rows + WAVES - 1) / WAVES + WAVE - 1) / WAVE * WAVE;
  const int bits = 32 - __clz(S);
  for (int pass = 0; pass < 2; ++pass) {
    for (int32_t r0 = wave * stretch; r0 < (wave + 1) * stretch && r0 < rows; r0 += WAVE) {
      const int32_t r = r0 + lane;
      const uint32_t i = r < rows ? s.first[r] : 0u;
      uint64_t peers = __ballot(r < rows);
      for (int b = 0; b < bits; ++b) {
        const uint64_t m = __ballot((i >> b) & 1);
        peers &= (i >> b) & 1 ? m : ~m;
      }
      if (r < rows) {
        const uint32_t ahead = __popcll(peers & ((1ull << lane) - 1));
        const uint32_t at = s_count[wave][i] + ahead;    // (read by all lanes before the last of them writes)
        if (ahead + 1 == (uint32_t)__popcll(peers)) s_count[wave][i] = (uint16_t)(at + 1);
        if (pass) {
          const bool in = at < (uint32_t)cap;
          s_line[r] = (uint16_t)(in ? at : NOT_RESIDENT);
          if (in) {
            s_row[at] = (uint16_t)r;
            s_key[r] = (uint16_t)i;
            atomicAdd(&s_res[i], 1u);
            s.init_ids[at] = s.id[r];
          }
        }
      }
    }
    __syncthreads();
    if (pass) continue;
    uint32_t mine = 0;                     // (iterations: at most one to a thread)
    if (me < S)
      for (int w = 0; w < WAVES; ++w) mine += s_count[w][me];
    uint32_t total;
    uint32_t at = block_exclusive_scan<uint32_t, BIG>(mine, smem, total);
    if (me < S) {
      s.ready[me] = at + mine < (uint32_t)cap ? at + mine : (uint32_t)cap;
      for (int w = 0; w < WAVES; ++w) {
        const uint32_t c = s_count[w][me];
        s_count[w][me] = (uint16_t)at;
        at += c;
      }
    }
    __syncthreads();
  }

  uint32_t dst = 0;                        // records so far
  if (me == 0) s.cs_offsets[0] = s.cs_copy[0] = 0;
  for (int32_t i = 0; i < S; ++i) {
    const int64_t off = s.off[i];
    const int32_t n = (int32_t)(s.off[i + 1] - off);
    const uint32_t* const access = s.access + off;
    // hits get their new key, hits and misses are counted by key
    for (int j = me; j <= S; j += BIG) s_inc[j] = 0;
    if (me == 0) {
      s_misses = 0;
      s_jstar = S + 1;                     // nothing is dropped
      s_mode_in = s_mode_res = MODE_ALL;
      s_T = -1;
    }
    __syncthreads();
    uint32_t misses = 0;
    for (int32_t p = me; p < n; p += BIG) {
      const uint32_t a = access[p], r = a & 0xFFFFu, next = a >> 16, line = s_line[r];
      if (s.src_line) s.src_line[off + p] = line == NOT_RESIDENT ? -1 : (int32_t)line;
      if (line != NOT_RESIDENT) {
        s_key[r] = (uint16_t)next;         // (bucket i is not looked at any more)
        atomicAdd(&s_res[next], 1u);
      } else {
        atomicAdd(&s_inc[next], 1u);
        ++misses;
      }
    }
    misses = wave_reduce_sum(misses);
    if (lane == 0 && misses) atomicAdd(&s_misses, misses);
    __syncthreads();
    const uint32_t n_drop = s_misses;
    if (me == 0) s.miss_count[i] = n_drop;
    uint32_t n_change = 0;
    if (n_drop > 0) {                      // uniform
      // the threshold bucket, from "never" downwards
      const int32_t j = S - me;            // (buckets: at most one to a thread)
      const uint32_t R = j > i ? s_res[j] : 0u, I = j > i ? s_inc[j] : 0u;
      uint32_t total;
      const uint32_t before = block_exclusive_scan<uint32_t, BIG>(R + I, smem, total);
      if (j > i && before <= n_drop && before + R + I > n_drop) {
        const uint32_t rem = n_drop - before;
        s_jstar = j;
        s_kept = R + I - rem;
        if (rem == 0) {
          s_mode_in = s_mode_res = MODE_ALL;
        } else if (rem < I) {
          s_mode_in = MODE_SELECT;
          s_keep = I - rem;
        } else if (rem == I) {
          s_mode_in = MODE_NONE;
        } else {
          s_mode_in = MODE_NONE;
          s_mode_res = MODE_SELECT;
          s_keep = R - (rem - I);
        }
      }
      __syncthreads();
      const int32_t jstar = s_jstar, mode_in = s_mode_in, mode_res = s_mode_res;
      // the keys of the state after the iteration
      if (j > i) {
        if (j > jstar) s_res[j] = 0;
        else if (j == jstar) s_res[j] = s_kept;
        else s_res[j] += I;
      }
      if (mode_in == MODE_SELECT || mode_res == MODE_SELECT) {   // uniform
        if (mode_in == MODE_SELECT) {
          for (int32_t p = me; p < n; p += BIG) {
            const uint32_t a = access[p], r = a & 0xFFFFu;
            if ((int32_t)(a >> 16) == jstar && s_line[r] == NOT_RESIDENT) atomicOr(&s_bits[r >> 5], 1u << (r & 31));
          }
        } else {
          for (int32_t l = me; l < cap; l += BIG) {
            const uint32_t r = s_row[l];
            if (s_key[r] == jstar) atomicOr(&s_bits[r >> 5], 1u << (r & 31));
          }
        }
        __syncthreads();
        const uint32_t keep = s_keep, word = me < WORDS ? s_bits[me] : 0u, members = __popc(word);
        const uint32_t ahead = block_exclusive_scan<uint32_t, BIG>(members, smem, total);
        if (ahead < keep && ahead + members >= keep) {
          uint32_t left = word;
          for (uint32_t skip = keep - ahead; skip > 1; --skip) left &= left - 1;
          s_T = me * 32 + __ffs(left) - 1;
        }
        if (me < WORDS) s_bits[me] = 0;
        __syncthreads();
      }
      const int32_t T = s_T;
      // evicted lines, neighbouring ones to a thread
      const int32_t per = (cap + BIG - 1) / BIG, l0 = me * per;
      uint32_t gone = 0;                   // bit k: line l0 + k
      for (int32_t k = 0; k < per && l0 + k < cap; ++k) {
        const int32_t r = s_row[l0 + k], key = s_key[r];
        if (key > jstar || (key == jstar && mode_res == MODE_SELECT && r > T)) gone |= 1u << k;
      }
      uint32_t at = block_exclusive_scan<uint32_t, BIG>(__popc(gone), smem, n_change);
      for (; gone; gone &= gone - 1) s_out[at++] = (uint16_t)(l0 + __ffs(gone) - 1);
      // inserted rows, a position to a thread
      uint32_t inserted = 0;
      for (int32_t p0 = 0; p0 < n; p0 += BIG) {
        const int32_t p = p0 + me;
        const uint32_t a = p < n ? access[p] : 0u, r = a & 0xFFFFu;
        const int32_t next = a >> 16;
        const bool in = p < n && s_line[r] == NOT_RESIDENT &&
                        (next < jstar || (next == jstar && (mode_in == MODE_ALL ||
                                                            (mode_in == MODE_SELECT && (int32_t)r <= T))));
        uint32_t all;
        const uint32_t k = inserted + block_exclusive_scan<uint32_t, BIG>(in ? 1u : 0u, smem, all);
        if (in && k < SMALL_ROWS) {
          s_in[k] = (uint16_t)r;
          s_key[r] = (uint16_t)next;
          const uint32_t x = dst + k;
          if (x < s.cs_capacity) {
            s.in_ids[x] = s.id[r];
            s.in_positions[x] = p;
          }
        }
        inserted += all;
      }
      __syncthreads();
      // the k-th insertion takes the line of the k-th eviction (as many of one as of the other)
      for (uint32_t k = me; k < n_change && k < inserted; k += BIG) {
        const uint32_t line = s_out[k], out = s_row[line], in = s_in[k], x = dst + k;
        if (x < s.cs_capacity) s.out_ids[x] = s.id[out];
        s_line[out] = NOT_RESIDENT;
        s_line[in] = (uint16_t)line;
        s_row[line] = (uint16_t)in;
      }
    }
    dst += n_change;
    if (me == 0) s.cs_offsets[i + 1] = s.cs_copy[i + 1] = dst;
    __syncthreads();
  }
}
