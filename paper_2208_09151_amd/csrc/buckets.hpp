// One hop of the sampler without hash tables in HBM.  Included by sampler.hip only.
//
// A batch's candidates of a later hop are too many for one table in LDS, and in tables in HBM every
// insert is an atomic on the memory side of the fabric (27 G/s on this GPU, 57.6 M of them for a
// superbatch of 200 batches).  So the ids are dealt to buckets by hash, each small enough for a table in
// the LDS of one workgroup:
//   k_pick_tiles    a block per tile of TILE_NODES frontier nodes, a thread per node: draws the picks,
//                   reads the neighbours, sorts the tile's candidates by bucket in LDS and writes them
//                   out in that order with their rank inside the tile; further blocks do the same
//                   for the list the batch has so far, LIST_TILE ids at a time
//   k_bucket_dedup  a workgroup per bucket: inserts the bucket's share of every tile (list ids with their
//                   position, candidates with their rank, the smallest wins), then looks every
//                   candidate up: list position, or the rank of its id's first occurrence
//   k_tile_firsts   a block per tile: first-occurrence masks, the picks and first occurrences in front of
//                   every node inside its tile, tile and batch sums
//   k_bucket_emit   a block per tile: where the batch's and the tile's output starts (sums over the batches
//                   and tiles before it, no launch of their own), then list, rowptr and adj_col, put
//                   into order in LDS (the permutation never leaves the tile, so nothing is scattered in
//                   memory); in the last hop straight into the caller's ids
// Every access to memory but the neighbour reads and the places of repeated ids is a run of consecutive
// entries.  200 batches of 1 000 seeds, fanout 10/10/10, 111 M nodes, 42.7 M picks, both later hops together:
// k_pick_tiles 0.95 ms (41 M line fetches: bound by the neighbour reads), k_bucket_dedup 0.47 (LDS latency),
// k_tile_firsts 0.09, k_bucket_emit 0.27; with the tables in HBM k_pick 2.44, k_reinsert 0.25, k_table_clear 0.15,
// k_count 0.03, k_emit 0.19, k_col 0.30, k_copy_ids 0.07.  (Answers put back into candidate order by
// k_tile_firsts, then k_scan_batch, k_stage_offsets, k_emit and k_col as for the tables, and the lists copied
// at the end: 0.27 more; a superbatch of 33 batches of 777 seeds, fanout 25/10, 300 -> 233 us, of 8 of 256,
// 10/10/10, 185 -> 155, mostly launches that are gone.)
#pragma once

constexpr int TILE_NODES = TB;           // frontier nodes per tile (the tiles of k_emit and the scans)
constexpr int LIST_TILE = 2048;          // list ids per tile
constexpr int MAX_BUCKETS = 2 * TB;      // two to a thread in the scan of a tile's counts
constexpr int BUCKET_THREADS = 512;
constexpr int BUCKET_SLOTS = 4096;       // 32 KB: four workgroups of 512 threads per CU (two of twice the size: 260 instead of
                                         // 235 us per hop of 200 batches)
constexpr int BUCKET_IDS = 2000;         // ids a bucket is meant to hold: load factor 0.49
constexpr int BUCKET_IDS_MIN = 512;      // ... and at least, where there are few batches, or, on a small graph whose
constexpr int BUCKET_ENTRIES_MIN = 1024; // ids come many times over, this many entries (one batch of 26 k entries of
                                         // 5 000 ids: 17.0 us with 10 buckets, 8.1 with 26)
constexpr int BUCKET_PROBES = 512;       // a longer search ends the attempt, see k_bucket_dedup
constexpr uint32_t NO_ID = 0xFFFFFFFFu;  // an unused slot of a tile (ids are below 2^31)
constexpr int PICK_READS = 8;            // neighbour reads a thread keeps in flight
constexpr int BUCKET_K_MAX = 32;         // fanouts up to here: a thread keeps a node's picks in registers

// Buckets serve up to this many ids in a batch, a load factor of 0.72 in MAX_BUCKETS tables.  Beyond that the
// buckets are done in slices, each of which reads all of the bucket: work that grows with the square of
// the batch, where that of the tables in HBM is linear (one batch of 4 000 seeds, fanout 10/10/10, 4.4 M ids:
// 19.5 ms in slices, 2.1 in the tables; 2 000 seeds, 2.3 M ids: 4.5 and 1.1; 16 000 seeds: 211 and 7.9).
constexpr int64_t BUCKET_IDS_LIMIT = 1'500'000;

struct Buckets {
  uint32_t* id;          // [S][entries] a tile's ids by bucket (tile t of the nodes: from t * TILE_NODES * k on;
                         // list tiles: behind cand_slots)
  uint16_t* rank;        // [S][entries] their rank inside the tile
  uint16_t* start;       // [S][tiles][row] start of every bucket inside the tile
  int64_t entries, tiles;
  int64_t list_tiles_at; // first list tile (tiles of the nodes come first)
  int64_t list_at;       // first list entry
  int32_t row;           // most buckets a batch can have, plus one
  int64_t num_nodes;
};

// Buckets of a batch for a hop that starts with `n` ids in the list (all of them are the frontier):
// BUCKET_IDS of the ids that the batch can have after the hop (hop_ids) make a bucket; with few batches more
// and smaller ones, until the GPU's 256 CUs have two workgroups each (8 batches of 34 k candidates: 16 us
// with 5 buckets a batch, 7 us with 64).
__host__ __device__ __forceinline__ int64_t hop_ids(int64_t n, int k, int64_t num_nodes) {
  const int64_t ids = n + n * k;
  return ids < num_nodes ? ids : num_nodes;
}

__host__ __device__ __forceinline__ int32_t bucket_count(int64_t n, int k, int64_t num_nodes, int32_t S) {
  const int64_t ids = hop_ids(n, k, num_nodes);
  int64_t p = (ids + BUCKET_IDS - 1) / BUCKET_IDS;
  const int64_t spread = (512 + S - 1) / S;
  int64_t fill = (ids + BUCKET_IDS_MIN - 1) / BUCKET_IDS_MIN;
  const int64_t by_entries = (n + n * k + BUCKET_ENTRIES_MIN - 1) / BUCKET_ENTRIES_MIN;
  if (fill < by_entries) fill = by_entries;
  const int64_t more = spread < fill ? spread : fill;
  if (p < more) p = more;
  return (int32_t)(p < 1 ? 1 : p > MAX_BUCKETS ? MAX_BUCKETS : p);
}

// The picks of one node by one thread: a[i] = row position of draw i, i < min(deg, k) (deg <= k: the
// whole row); all other entries compare larger.  Floyd's subset rule in draw order: a position that an
// earlier draw took is replaced by the rule's own j.  The array stays in registers (every index is
// known at compile time; k is uniform).  One thread per node instead of a group of lanes per node
// draws only the words a node needs and compares registers instead of shuffling.
template <int K_MAX, typename Pos>
__device__ __forceinline__ void choose_picks(uint32_t v, int64_t deg, int k, int hop, uint64_t seed,
                                             uint32_t batch, Pos (&a)[K_MAX]) {
#pragma unroll
  for (int i = 0; i < K_MAX; ++i) a[i] = i < k ? (Pos)i : ~(Pos)0;
  if (deg <= k) return;
#pragma unroll
  for (int i = 0; i < K_MAX; ++i) {
    if (i < k) {             // (no break: the loop has to unroll)
      const uint64_t r = philox_draw(seed, v, batch, (uint32_t)hop, (uint32_t)i);
      const Pos j = (Pos)(deg - k + i);
      Pos t;
      if (sizeof(Pos) == 4) {   // (j + 1 < 2^32: the high word of a 96-bit product)
        const uint64_t x = (uint64_t)j + 1;
        t = (Pos)(((r >> 32) * x + (((r & 0xFFFFFFFFull) * x) >> 32)) >> 32);
      } else {
        t = (Pos)__umul64hi(r, (uint64_t)j + 1);
      }
      bool taken = false;
#pragma unroll
      for (int m = 0; m < i; ++m) taken |= a[m] == t;
      a[i] = taken ? j : t;
    }
  }
}

// The place of pick i among the node's picks in ascending row position.
template <int K_MAX, typename Pos>
__device__ __forceinline__ int pick_slot(const Pos (&a)[K_MAX], int i) {
  int below = 0;
#pragma unroll
  for (int m = 0; m < K_MAX; ++m) below += a[m] < a[i] ? 1 : 0;
  return below;
}

// Exclusive prefix of the tile's counts per bucket into s_start[0 .. P], start row of the tile out.
__device__ __forceinline__ uint32_t tile_starts(const uint32_t* s_count, uint32_t* s_start, int32_t P,
                                                uint32_t* smem, uint16_t* __restrict__ row) {
  const int32_t q = 2 * (int32_t)threadIdx.x;
  const uint32_t c0 = q < P ? s_count[q] : 0u, c1 = q + 1 < P ? s_count[q + 1] : 0u;
  uint32_t total;
  const uint32_t at = block_exclusive_scan<uint32_t, TB>(c0 + c1, smem, total);
  if (q < P) {
    s_start[q] = at;
    row[q] = (uint16_t)at;
  }
  if (q + 1 < P) {
    s_start[q + 1] = at + c0;
    row[q + 1] = (uint16_t)(at + c0);
  }
  if (threadIdx.x == 0) row[P] = (uint16_t)total;
  __syncthreads();
  return total;
}

// The tile's entries, sorted by bucket in LDS, to memory.
__device__ __forceinline__ void tile_store(const uint32_t* s_id, const uint16_t* s_rank, uint32_t n,
                                           uint32_t* __restrict__ id, uint16_t* __restrict__ rank) {
  __syncthreads();
  for (uint32_t x = threadIdx.x; x < n; x += TB) {
    id[x] = s_id[x];
    rank[x] = s_rank[x];
  }
}

template <int K_MAX, typename OffT, typename Pos, bool NC>
__global__ __launch_bounds__(TB) void k_pick_tiles(Tables T, Buckets B, const OffT* __restrict__ offsets,
                                                   const int32_t* __restrict__ indices,
                                                   const int64_t* __restrict__ nc_address_table,
                                                   const int32_t* __restrict__ nc_cache_array,
                                                   const int32_t* __restrict__ nfront, int k, int hop,
                                                   uint64_t seed, uint32_t first_batch, int S,
                                                   uint64_t* __restrict__ batch_total, int64_t tpb,
                                                   int slots) {
  extern __shared__ uint32_t s_id[];                              // [slots] ids, then [slots] ranks
  uint16_t* s_rank = reinterpret_cast<uint16_t*>(s_id + slots);
  __shared__ uint32_t s_count[MAX_BUCKETS], s_start[MAX_BUCKETS];
  __shared__ uint32_t smem[TB / WAVE + 1];
  const Where here = where_am_i(S, tpb);
  if (here.b < 0) return;
  const int b = here.b;
  if (here.tile == 0 && threadIdx.x == 0) batch_total[b] = 0;   // k_tile_firsts adds to it
  const int64_t nf = nfront[b];
  const int32_t P = bucket_count(nf, k, B.num_nodes, S);
  const int64_t node_tiles = (nf + TILE_NODES - 1) / TILE_NODES, list_tiles = (nf + LIST_TILE - 1) / LIST_TILE;
  const int32_t* list = T.wlist + b * T.stride_ids;
  for (int64_t tile = here.tile; tile < node_tiles + list_tiles; tile += tpb) {
    __syncthreads();                     // the tile before is stored
    for (int x = threadIdx.x; x < MAX_BUCKETS; x += TB) s_count[x] = 0;
    __syncthreads();
    if (tile < node_tiles) {
      const int64_t idx = tile * TILE_NODES + threadIdx.x;
      const int64_t nodes = nf - tile * TILE_NODES < TILE_NODES ? nf - tile * TILE_NODES : TILE_NODES;
      const int n_slots = (int)nodes * k;
      for (int x = threadIdx.x; x < n_slots; x += TB) s_id[x] = NO_ID;
      __syncthreads();
      if (idx < nf) {
        const uint32_t v = (uint32_t)list[idx];
        int64_t lo, deg;
        bool cached;
        row_of<OffT, NC>(v, offsets, nc_address_table, nc_cache_array, lo, deg, cached);
        const int c = deg < k ? (int)deg : k;
        Pos a[K_MAX];
        choose_picks<K_MAX, Pos>(v, deg, k, hop, seed, first_batch + (uint32_t)b, a);
        const int32_t* row = (cached ? nc_cache_array : indices) + lo;
#pragma unroll
        for (int h = 0; h < K_MAX; h += PICK_READS) {
          uint32_t u[PICK_READS];
#pragma unroll
          for (int i = 0; i < PICK_READS; ++i)
            if (h + i < c) u[i] = (uint32_t)row[a[h + i]];
#pragma unroll
          for (int i = 0; i < PICK_READS; ++i)
            if (h + i < c) s_id[threadIdx.x * k + pick_slot<K_MAX, Pos>(a, h + i)] = u[i];
        }
        T.cnt[b * T.fr_slots + idx] = (uint8_t)c;
      }
      __syncthreads();
      // from here on by candidate: a thread's entries are TB apart, k of them at most
      const int64_t first = tile * TILE_NODES * k;
      uint32_t u[K_MAX], at[K_MAX];      // at: bucket << 16 | place among the tile's entries of the bucket
#pragma unroll
      for (int i = 0; i < K_MAX; ++i) {
        const int x = i * TB + threadIdx.x;
        u[i] = x < n_slots ? s_id[x] : NO_ID;
        if (u[i] != NO_ID) {
          const uint32_t q = __umulhi(hash_mix(u[i]), (uint32_t)P);
          at[i] = (q << 16) | atomicAdd(&s_count[q], 1u);
        }
      }
      __syncthreads();
      const uint32_t n = tile_starts(s_count, s_start, P, smem, B.start + (b * B.tiles + tile) * B.row);
#pragma unroll
      for (int i = 0; i < K_MAX; ++i)
        if (u[i] != NO_ID) {
          const uint32_t x = s_start[at[i] >> 16] + (at[i] & 0xFFFFu);
          s_id[x] = u[i];
          s_rank[x] = (uint16_t)(i * TB + threadIdx.x);
        }
      tile_store(s_id, s_rank, n, B.id + b * B.entries + first, B.rank + b * B.entries + first);
    } else {
      constexpr int ITEMS = LIST_TILE / TB;
      const int64_t first = (tile - node_tiles) * LIST_TILE;
      uint32_t u[ITEMS], at[ITEMS];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int64_t x = first + i * TB + threadIdx.x;
        u[i] = x < nf ? (uint32_t)list[x] : NO_ID;
      }
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (u[i] != NO_ID) {
          const uint32_t q = __umulhi(hash_mix(u[i]), (uint32_t)P);
          at[i] = (q << 16) | atomicAdd(&s_count[q], 1u);
        }
      __syncthreads();
      const int64_t list_tile = B.list_tiles_at + (tile - node_tiles);
      const uint32_t n = tile_starts(s_count, s_start, P, smem, B.start + (b * B.tiles + list_tile) * B.row);
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (u[i] != NO_ID) {
          const uint32_t x = s_start[at[i] >> 16] + (at[i] & 0xFFFFu);
          s_id[x] = u[i];
          s_rank[x] = (uint16_t)(i * TB + threadIdx.x);
        }
      tile_store(s_id, s_rank, n, B.id + b * B.entries + B.list_at + first,
                 B.rank + b * B.entries + B.list_at + first);
    }
  }
}

// The bucket's entries in the tiles of a batch, dealt evenly to the threads: the shares of up to
// BUCKET_THREADS tiles (those of the list first) are laid end to end, a wave finds the share of its
// first entry and its lanes step on from there.
constexpr int BUCKET_ITEMS = 5;          // entries a thread requests at once

struct Shares {
  uint32_t end[BUCKET_THREADS];          // entries up to and with the tile's share
  int32_t shift[BUCKET_THREADS];         // + entry number = place in the batch's entries
};

struct Entries {                         // what a thread holds of them
  uint32_t u[BUCKET_ITEMS];              // id, NO_ID: none
  int32_t at[BUCKET_ITEMS];              // place in the batch's entries, ~place for one of the list
};

struct BucketOf {                        // the bucket at work
  const uint32_t* id;                    // of the batch, as below
  const uint16_t *rank, *start;
  int32_t q, row, span;                  // span: entries of a node tile
  int32_t list_tiles, tiles;             // tiles: of both kinds
  int64_t list_tiles_at, list_at;
};

// Lays out the shares of the tiles [t0, t0 + BUCKET_THREADS); returns their entries.
__device__ __forceinline__ uint32_t bucket_shares(const BucketOf& k, int32_t t0, Shares& sh, uint32_t* smem) {
  const int32_t t = t0 + threadIdx.x;
  uint32_t lo = 0, hi = 0;
  if (t < k.tiles) {
    const int64_t tile = t < k.list_tiles ? k.list_tiles_at + t : t - k.list_tiles;
    lo = k.start[tile * k.row + k.q];
    hi = k.start[tile * k.row + k.q + 1];
  }
  uint32_t total;
  const uint32_t before = block_exclusive_scan<uint32_t, BUCKET_THREADS>(hi - lo, smem, total);
  const int32_t first = t < k.list_tiles ? (int32_t)k.list_at + t * LIST_TILE : (t - k.list_tiles) * k.span;
  sh.end[threadIdx.x] = before + hi - lo;
  sh.shift[threadIdx.x] = first + (int32_t)lo - (int32_t)before;
  __syncthreads();
  return total;
}

// The entries x0 + i * BUCKET_THREADS + threadIdx.x of the shares laid out.
__device__ __forceinline__ void bucket_load(const BucketOf& k, int32_t t0, const Shares& sh, uint32_t total,
                                            uint32_t x0, Entries& e, uint32_t (&value)[BUCKET_ITEMS]) {
  const int n_tiles = k.tiles - t0 < BUCKET_THREADS ? k.tiles - t0 : BUCKET_THREADS;
#pragma unroll
  for (int i = 0; i < BUCKET_ITEMS; ++i) {
    const uint32_t x = x0 + i * BUCKET_THREADS + threadIdx.x;
    e.u[i] = NO_ID;
    if (x >= total) continue;
    int a = 0, z = n_tiles - 1;
    const uint32_t first = x & ~(uint32_t)(WAVE - 1);
    while (a < z) {
      const int mid = (a + z) >> 1;
      if (sh.end[mid] > first) z = mid; else a = mid + 1;
    }
    while (sh.end[a] <= x) ++a;
    const int32_t at = sh.shift[a] + (int32_t)x, t = t0 + a;
    const bool of_list = t < k.list_tiles;
    e.u[i] = k.id[at];
    e.at[i] = of_list ? ~at : at;
    // list position, or PEND + candidate rank
    value[i] = k.rank[at] + (of_list ? (uint32_t)(t * LIST_TILE) : PEND + (uint32_t)((t - k.list_tiles) * k.span));
  }
}

// One workgroup per (batch, bucket): insert, then look up; a bucket of the size it is meant to have
// stays in the threads' registers in between.  Where more ids fall into a bucket than its table takes
// (ids made to collide), a search that takes
// too long ends the attempt and the bucket is done in slices of the 32-bit space that an odd
// multiplier spreads the ids over, half as long after every failed attempt (a slice of length one
// holds a single id).
__global__ __launch_bounds__(BUCKET_THREADS) __attribute__((amdgpu_waves_per_eu(8))) void k_bucket_dedup(
    Tables T, Buckets B, const int32_t* __restrict__ nfront, int fanout, int S, int64_t tpb) {
  __shared__ unsigned long long tab[BUCKET_SLOTS];
  __shared__ Shares sh;
  __shared__ uint32_t smem[BUCKET_THREADS / WAVE + 1];
  __shared__ uint32_t s_full;
  const Where here = where_am_i(S, tpb);
  if (here.b < 0) return;
  const int b = here.b;
  const int32_t nf = nfront[b];
  if (nf == 0) return;   // an empty batch has no tiles, and the barriers below are in the loop over them
  const int32_t P = bucket_count(nf, fanout, B.num_nodes, S);
  BucketOf k;
  k.id = B.id + b * B.entries;
  k.rank = B.rank + b * B.entries;
  k.start = B.start + b * B.tiles * B.row;
  k.row = B.row;
  k.span = TILE_NODES * fanout;          // (places in a batch's entries stay below 2^31)
  k.list_tiles = (nf + LIST_TILE - 1) / LIST_TILE;
  k.tiles = k.list_tiles + (nf + TILE_NODES - 1) / TILE_NODES;
  k.list_tiles_at = B.list_tiles_at;
  k.list_at = B.list_at;
  uint32_t* answer = T.ref + b * T.cand_slots;
  for (k.q = (int32_t)here.tile; k.q < P; k.q += (int32_t)tpb) {
    uint64_t lo = 0, len = 1ull << 32;
    while (lo < (1ull << 32)) {          // uniform
      for (int i = threadIdx.x; i < BUCKET_SLOTS; i += BUCKET_THREADS) tab[i] = FREE_SLOT;
      if (threadIdx.x == 0) s_full = 0;
      auto mine = [&](uint32_t u) {      // (wraps below lo)
        return u != NO_ID && (uint64_t)(u * 2654435761u) - lo < len;
      };
      auto place = [&](uint32_t u, uint32_t value) {
        const unsigned long long word = ((unsigned long long)u << 32) | value;
        uint32_t h = hash_mix(u) & (BUCKET_SLOTS - 1);
        for (int probe = 0; probe < BUCKET_PROBES; ++probe) {
          // a plain look first: the ids of hubs come by the hundred, and equal addresses of a wave's
          // reads cost nothing while its atomics on them are carried out one after the other
          unsigned long long old = *(volatile unsigned long long*)&tab[h];
          if (old == FREE_SLOT) old = atomicCAS(&tab[h], FREE_SLOT, word);
          if (old == FREE_SLOT) return;
          if ((uint32_t)(old >> 32) == u) {
            if ((uint32_t)old > value) atomicMin(&tab[h], word);
            return;
          }
          h = (h + 1) & (BUCKET_SLOTS - 1);
        }
        s_full = 1;
      };
      auto look_up = [&](const Entries& e) {
#pragma unroll
        for (int i = 0; i < BUCKET_ITEMS; ++i) {
          if (!mine(e.u[i]) || e.at[i] < 0) continue;
          uint32_t h = hash_mix(e.u[i]) & (BUCKET_SLOTS - 1);
          unsigned long long word = tab[h];
          for (int probe = 1; probe < BUCKET_PROBES && (uint32_t)(word >> 32) != e.u[i]; ++probe) {
            h = (h + 1) & (BUCKET_SLOTS - 1);
            word = tab[h];
          }
          const uint32_t value = (uint32_t)word;
          answer[e.at[i]] = value < PEND ? OLD_ID | value : value - PEND;
        }
      };
      Entries e;
      uint32_t total = 0;
      for (int32_t t0 = 0; t0 < k.tiles; t0 += BUCKET_THREADS) {
        total = bucket_shares(k, t0, sh, smem);   // (barriers inside: the table is clear)
        for (uint32_t x0 = 0; x0 < total; x0 += BUCKET_THREADS * BUCKET_ITEMS) {
          if (*(volatile uint32_t*)&s_full) break;   // (no barrier in this loop)
          uint32_t value[BUCKET_ITEMS];
          bucket_load(k, t0, sh, total, x0, e, value);
#pragma unroll
          for (int i = 0; i < BUCKET_ITEMS; ++i)
            if (mine(e.u[i])) place(e.u[i], value[i]);
        }
        __syncthreads();                 // the shares may be rewritten, the table is complete
      }
      const bool held = k.tiles <= BUCKET_THREADS && total <= BUCKET_THREADS * BUCKET_ITEMS;
      if (s_full) {                      // uniform
        len /= 2;
        __syncthreads();                 // every thread has seen it
        continue;
      }
      if (held) {
        if (total) look_up(e);
      } else {
        for (int32_t t0 = 0; t0 < k.tiles; t0 += BUCKET_THREADS) {
          total = bucket_shares(k, t0, sh, smem);
          for (uint32_t x0 = 0; x0 < total; x0 += BUCKET_THREADS * BUCKET_ITEMS) {
            uint32_t value[BUCKET_ITEMS];
            bucket_load(k, t0, sh, total, x0, e, value);
            look_up(e);
          }
          __syncthreads();
        }
      }
      __syncthreads();                   // the table is cleared for the next slice or bucket
      lo += len;
    }
  }
}

// A frontier slot's word: mask of its picks that are first occurrences, first occurrences and picks of the
// tile's slots in front of it (below 2^16: a tile has at most 256 * 32 picks).
__device__ __forceinline__ uint64_t slot_word(uint32_t mask, uint32_t firsts, uint32_t picks) {
  return (uint64_t)mask | (uint64_t)firsts << 32 | (uint64_t)picks << 48;
}
// First occurrences of the tile in front of the slot's pick.
__device__ __forceinline__ uint32_t firsts_before(uint64_t word, uint32_t pick) {
  return ((uint32_t)(word >> 32) & 0xFFFFu) + __popc((uint32_t)word & ((1u << pick) - 1u));
}

// rank / k for ranks of a batch's candidates: at most BUCKET_IDS_LIMIT frontier nodes and fanouts up to 32, so
// below 2^27, where the high word of rank * ceil(2^32 / k) is exact.
__device__ __forceinline__ uint32_t slot_of(uint32_t rank, int k, uint32_t inverse) {
  return k == 1 ? rank : __umulhi(rank, inverse);
}
__device__ __forceinline__ uint32_t slot_inverse(int k) { return 0xFFFFFFFFu / (uint32_t)k + 1u; }

constexpr uint32_t NEW_HERE = 0x80000000u;   // (ids and positions are below 2^31)
constexpr int EMIT_ITEMS = 5;            // entries of a tile a thread has in flight

// One block per tile of frontier nodes, see above.  Bound by reading the answers and ranks (6 bytes per pick).
__global__ __launch_bounds__(TB) void k_tile_firsts(Tables T, Buckets B, const int32_t* __restrict__ nfront,
                                                    int k, uint64_t* __restrict__ tile_sums, int64_t tiles,
                                                    uint64_t* __restrict__ batch_total, int S,
                                                    int64_t tpb) {
  __shared__ uint32_t s_mask[TILE_NODES];
  __shared__ uint32_t smem[TB / WAVE + 1];
  const Where here = where_am_i(S, tpb);
  if (here.b < 0) return;
  const int b = here.b;
  const int64_t nf = nfront[b];
  const int32_t P = bucket_count(nf, k, B.num_nodes, S);
  const uint32_t inverse = slot_inverse(k);
  uint64_t sum = 0;                      // of the tiles of this block
  for (int64_t tile = here.tile; tile * TILE_NODES < nf; tile += tpb) {
    const uint32_t first = (uint32_t)(tile * TILE_NODES * k);
    const uint32_t* answer = T.ref + b * T.cand_slots + first;
    const uint16_t* rank = B.rank + b * B.entries + first;
    const uint32_t n = B.start[(b * B.tiles + tile) * B.row + P];
    const int64_t idx = tile * TILE_NODES + threadIdx.x;
    const uint32_t c = idx < nf ? T.cnt[b * T.fr_slots + idx] : 0u;
    s_mask[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t x0 = threadIdx.x; x0 < n; x0 += TB * EMIT_ITEMS) {
      uint32_t a[EMIT_ITEMS], r[EMIT_ITEMS];
#pragma unroll
      for (int i = 0; i < EMIT_ITEMS; ++i) {
        const uint32_t x = x0 + i * TB < n ? x0 + i * TB : x0;   // (beyond the end the first one again)
        a[i] = answer[x];
        r[i] = rank[x];
      }
#pragma unroll
      for (int i = 0; i < EMIT_ITEMS; ++i)
        if (a[i] == first + r[i]) {      // the rank of its id's first occurrence is its own
          const uint32_t slot = slot_of(r[i], k, inverse);
          atomicOr(&s_mask[slot], 1u << (r[i] - slot * k));
        }
    }
    __syncthreads();
    const uint32_t mask = s_mask[threadIdx.x];
    uint32_t total;
    const uint32_t ex = block_exclusive_scan<uint32_t, TB>(c << 16 | __popc(mask), smem, total);
    if (idx < nf) T.first[b * T.fr_slots + idx] = slot_word(mask, ex & 0xFFFFu, ex >> 16);
    const uint64_t here_sum = (uint64_t)(total >> 16) << 32 | (total & 0xFFFFu);
    if (threadIdx.x == 0) tile_sums[b * tiles + tile] = here_sum;
    sum += here_sum;
  }
  if (threadIdx.x == 0 && sum) atomicAdd((unsigned long long*)&batch_total[b], (unsigned long long)sum);
}

// What k_front_lds left of the adj of hop 0 (positions of the picks in `cand`, edges in front of every row
// in `displaced`), still to be put at its place; nlist null: nothing.
struct FrontAdj {
  const int32_t* nlist;          // [S] frontier of hop 0: the seeds kept
  const uint64_t* batch_total;   // [S] its picks and first occurrences
  int k;
};

struct EmitTo {
  int64_t* rowptr;
  int64_t rowptr_capacity;
  int32_t* col;
  int64_t col_capacity;
  int32_t* ids;                  // the last hop: the caller's list, else null
  int64_t ids_capacity;
  // where the batches' outputs start, where k_stage_offsets has laid that out, else null
  const int64_t *row_base, *col_base;
};

// The segment of hop 0 of batch b, from block `vb` of `blocks`.
__device__ __forceinline__ void front_adj_copy(const Tables& T, int b, int n0, int k, int64_t rb, int64_t cb,
                                               const EmitTo& to, int64_t vb, int64_t blocks) {
  const int32_t* pos = T.cand + (int64_t)b * T.cand_slots;
  const uint32_t* edges = reinterpret_cast<const uint32_t*>(T.displaced + (int64_t)b * T.fr_slots);   // [n0 + 1]
  for (int64_t r = vb * TB + threadIdx.x; r <= n0; r += blocks * TB)
    if (rb + r < to.rowptr_capacity) to.rowptr[rb + r] = (int64_t)edges[r];
  const int64_t ncand = (int64_t)n0 * k;
  for (int64_t r = vb * TB + threadIdx.x; r < ncand; r += blocks * TB) {
    const uint32_t node = (uint32_t)r / (uint32_t)k, pick = (uint32_t)r - node * (uint32_t)k;
    const uint32_t e = edges[node];
    if (pick < edges[node + 1] - e && cb + e + pick < to.col_capacity) to.col[cb + e + pick] = pos[r];
  }
}

// Up to here a block adds up the totals of the batches in front of its own by itself (a launch of one block
// for the prefix sums costs 5 us and another wait for the launch before it); beyond, k_stage_offsets.  Superbatches of 1
// to 1 000 seeds a batch, two and three hops on 20 000 to 50 M nodes, with the launch against without: 64 batches
// 1.03 to 1.43 times, 256 0.99 to 1.48, 512 0.99 to 1.43, 1 024 0.96 to 1.37 (1.11 on the mean; 1 000 batches of
// 100 seeds, 10/10/10, 2 906 us and 2 840, of 16 seeds, 10/10, 187 and 234).
constexpr int EMIT_BATCHES = 1024;

// ... and scans the sums of a batch's tiles; beyond, k_scan_batch (sums as long as the entries of a tile in LDS).  The
// launch against none, the same calls and 1 to 8 batches of up to 300 000 seeds: 1.00 to 1.18 times, 1.03 on the mean.
constexpr int64_t EMIT_TILES = 1024;

// One block per tile of frontier nodes, see above.  Bound by the reads and writes of a few tiles a block (18
// bytes per pick, 214 us for 37 M picks: 3.1 TB/s) where there are many, by the chain of reads where there are few:
// batch length, sums and slot words, entries, words of repeated ids.  Dynamic LDS: sums of the tiles in front of each
// (tiles_in_lds of them), [TILE_NODES * k] positions or new ids, [TILE_NODES * k] places of the new ids.
__global__ __launch_bounds__(TB) void k_bucket_emit(Tables T, Buckets B, Meta M, const int32_t* __restrict__ nfront,
                                                    int32_t* __restrict__ nlist_next, int k, int hop, int H,
                                                    const uint64_t* __restrict__ tile_sums, int64_t tiles,
                                                    const uint64_t* __restrict__ batch_total, FrontAdj front,
                                                    EmitTo to, int S, int64_t tpb, int tiles_in_lds) {
  extern __shared__ uint64_t s_tile[];
  __shared__ uint64_t smem[TB / WAVE + 1];
  __shared__ uint64_t s_word[TILE_NODES];
  const Where here = where_am_i(S, tpb);
  if (here.b < 0) return;
  const int b = here.b;
  const uint32_t nf = (uint32_t)nfront[b];
  const int64_t tiles_here = ((int64_t)nf + TILE_NODES - 1) / TILE_NODES;
  const bool last = hop == H - 1;
  uint32_t* const s_col = reinterpret_cast<uint32_t*>(s_tile + tiles_in_lds);
  uint16_t* const s_place = reinterpret_cast<uint16_t*>(s_col + TILE_NODES * k);

  // The first reads wait for nothing but the batch's length; those of the sums over batches not even for that.
  // Sums over the batches in front (of all batches for the block that writes the totals): rows, picks,
  // list lengths; of hop 0 if it is still to be placed (rows << 32 | picks: at most 1 024 seeds to a batch), of all
  // and of those in front.
  uint64_t sums[5] = {};
  if (!to.row_base) {
    const int limit = b ? b : S;
    for (int q = threadIdx.x; q < S; q += TB) {
      const uint64_t t = batch_total[q], n = (uint64_t)nfront[q];
      uint64_t f = 0;
      if (front.nlist) f = (uint64_t)(front.nlist[q] + 1) << 32 | front.batch_total[q] >> 32;
      if (q < limit) {
        sums[0] += n + 1;
        sums[1] += t >> 32;
        sums[2] += n + (t & 0xFFFFFFFFu);
      }
      sums[3] += f;
      if (q < b) sums[4] += f;
    }
  }
  const int32_t P = bucket_count(nf, k, B.num_nodes, S);
  uint32_t n = 0;
  uint64_t word = 0;
  auto request = [&](int64_t tile) {      // of the tile: its picks, the words of its slots
    const int64_t idx = tile * TILE_NODES + threadIdx.x;
    n = tile < tiles_here ? B.start[(b * B.tiles + tile) * B.row + P] : 0u;
    word = idx < nf ? T.first[b * T.fr_slots + idx] : 0ull;
  };
  request(here.tile);
  // picks and first occurrences of the tiles in front of each tile, and of all
  const uint64_t* const ahead_of = tiles_in_lds ? s_tile : tile_sums + b * tiles;
  uint64_t run = 0;
  if (tiles_in_lds)
    for (int64_t t0 = 0; t0 < tiles_here; t0 += TB) {
      const int64_t t = t0 + threadIdx.x;
      uint64_t total;
      const uint64_t ex = block_exclusive_scan<uint64_t, TB>(t < tiles_here ? tile_sums[b * tiles + t] : 0ull, smem, total);
      if (t < tiles_here) s_tile[t] = run + ex;
      run += total;
    }
  else
    run = batch_total[b];
  // where the batch's outputs start
  int64_t rb, cb, ib = 0;
  if (to.row_base) {
    rb = to.row_base[b];
    cb = to.col_base[b];
    if (last) ib = M.ids_offsets[b];
  } else {
    __shared__ uint64_t red[TB / WAVE][5];
#pragma unroll
    for (int x = 0; x < 5; ++x) {
      sums[x] = wave_reduce_sum(sums[x]);
      if (lane_id() == 0) red[threadIdx.x / WAVE][x] = sums[x];
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 5; ++x) {
      sums[x] = 0;
#pragma unroll
      for (int w = 0; w < TB / WAVE; ++w) sums[x] += red[w][x];
    }
    // what the hops before took: hop 0 follows from its sums, later ones left it in the next segment's entry
    const int64_t row_run = front.nlist ? (int64_t)(sums[3] >> 32) : hop == 0 ? 0 : M.row_off[(int64_t)hop * S];
    const int64_t col_run = front.nlist ? (int64_t)(sums[3] & 0xFFFFFFFFu) : hop == 0 ? 0 : M.col_off[(int64_t)hop * S];
    rb = row_run + (b ? (int64_t)sums[0] : 0);
    cb = col_run + (b ? (int64_t)sums[1] : 0);
    ib = b ? (int64_t)sums[2] : 0;
    const int64_t rb0 = (int64_t)(sums[4] >> 32), cb0 = (int64_t)(sums[4] & 0xFFFFFFFFu);
    if (here.tile == 0 && threadIdx.x == 0) {
      const int32_t grown = (int32_t)(nf + (uint32_t)run);
      nlist_next[b] = grown;
      M.hop_sizes[(int64_t)b * (H + 1) + hop + 1] = grown;
      if (b > 0 || hop == 0 || front.nlist) {       // (else: the entry read above)
        M.row_off[(int64_t)hop * S + b] = rb;
        M.col_off[(int64_t)hop * S + b] = cb;
      }
      if (front.nlist) {
        M.row_off[b] = rb0;
        M.col_off[b] = cb0;
      }
      if (last) M.ids_offsets[b] = ib;
      if (b == 0) {
        M.row_off[(int64_t)(hop + 1) * S] = M.totals[1] = row_run + (int64_t)sums[0];
        M.col_off[(int64_t)(hop + 1) * S] = M.totals[2] = col_run + (int64_t)sums[1];
        if (last) M.ids_offsets[S] = M.totals[0] = (int64_t)sums[2];
      }
    }
    if (front.nlist && to.rowptr)
      front_adj_copy(T, b, front.nlist[b], front.k, rb0, cb0, to, here.tile, tpb);
  }
  int32_t* const list = T.wlist + b * T.stride_ids;
  // (the last hop: the list moves to its place as a whole, the others append to it)
  int32_t* const grow = last ? to.ids + ib : list;
  const int64_t room = last ? to.ids_capacity - ib : T.stride_ids;
  if (last)
    for (int64_t j = here.tile * TB + threadIdx.x; j < nf && j < room; j += tpb * TB) grow[j] = list[j];
  if (nf == 0 && here.tile == 0 && threadIdx.x == 0 && to.rowptr && rb < to.rowptr_capacity)
    to.rowptr[rb] = 0;                              // an empty frontier still has a rowptr entry
  const uint32_t inverse = slot_inverse(k);
  for (int64_t tile = here.tile; tile < tiles_here; tile += tpb) {
    const int64_t idx = tile * TILE_NODES + threadIdx.x;
    const uint32_t first = (uint32_t)(tile * TILE_NODES * k);
    const uint32_t* answer = T.ref + b * T.cand_slots + first;
    const uint16_t* rank = B.rank + b * B.entries + first;
    const uint32_t* id = B.id + b * B.entries + first;
    __syncthreads();                                // the sums are complete; the tile before is stored
    s_word[threadIdx.x] = word;
    const uint64_t ahead = ahead_of[tile];
    const int64_t edges_ahead = (int64_t)(ahead >> 32);
    const uint32_t new_at = nf + (uint32_t)ahead;   // list position of the tile's first new id
    if (to.rowptr) {
      if (idx < nf && rb + idx < to.rowptr_capacity) to.rowptr[rb + idx] = edges_ahead + (int64_t)(word >> 48);
      if (idx == (int64_t)nf - 1 && rb + nf < to.rowptr_capacity) to.rowptr[rb + nf] = (int64_t)(run >> 32);
    }
    __syncthreads();
    for (uint32_t x0 = threadIdx.x; x0 < n; x0 += TB * EMIT_ITEMS) {
      uint32_t a[EMIT_ITEMS], r[EMIT_ITEMS], u[EMIT_ITEMS];
      uint64_t w2[EMIT_ITEMS];
#pragma unroll
      for (int i = 0; i < EMIT_ITEMS; ++i) {
        const uint32_t x = x0 + i * TB < n ? x0 + i * TB : x0;
        a[i] = answer[x];
        r[i] = rank[x];
        u[i] = id[x];
      }
#pragma unroll
      for (int i = 0; i < EMIT_ITEMS; ++i)          // the slot of the first occurrence, where that is another pick
        w2[i] = !(a[i] & OLD_ID) && a[i] != first + r[i] ? T.first[b * T.fr_slots + slot_of(a[i], k, inverse)] : 0ull;
#pragma unroll
      for (int i = 0; i < EMIT_ITEMS; ++i) {
        if (x0 + i * TB >= n) continue;
        const uint32_t slot = slot_of(r[i], k, inverse), pick = r[i] - slot * k;
        const uint64_t w = s_word[slot];
        uint32_t pos;
        if (a[i] & OLD_ID) {
          pos = a[i] & ~OLD_ID;
        } else if (a[i] == first + r[i]) {
          pos = u[i] | NEW_HERE;
          s_place[(uint32_t)(w >> 48) + pick] = (uint16_t)firsts_before(w, pick);
        } else {
          const uint32_t slot2 = slot_of(a[i], k, inverse);
          pos = nf + (uint32_t)ahead_of[slot2 / TILE_NODES] + firsts_before(w2[i], a[i] - slot2 * k);
        }
        s_col[(uint32_t)(w >> 48) + pick] = pos;
      }
    }
    const uint32_t entries = n;
    if (tile + tpb < tiles_here) request(tile + tpb);
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < entries; e += TB) {
      uint32_t pos = s_col[e];
      if (pos & NEW_HERE) {
        const uint32_t u = pos & ~NEW_HERE;
        pos = new_at + s_place[e];
        if ((int64_t)pos < room) grow[pos] = (int32_t)u;
      }
      if (to.col && cb + edges_ahead + e < to.col_capacity) to.col[cb + edges_ahead + e] = (int32_t)pos;
    }
  }
}
