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
//   k_tile_firsts   a block per tile: puts the answers back into candidate order (the permutation
//                   never leaves the tile, so nothing is scattered in memory), first-occurrence masks
//                   and tile sums
// and the lists and adj are emitted as after the tables in HBM.  Every access to memory but the
// neighbour reads is a run of consecutive entries.  200 batches of 1 000 seeds, fanout 10/10/10, 111 M
// nodes, 42.7 M picks, both later hops together: k_pick_tiles 1.03 ms (41 M line fetches, 5.1 TB/s of
// them: bound by the neighbour reads), k_bucket_dedup 0.48 (LDS latency), k_tile_firsts 0.13; with the
// tables in HBM k_pick 2.44, k_reinsert 0.25, k_table_clear 0.15, k_count 0.03, and 0.08 more in k_col.
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

// A full mix (the finaliser of MurmurHash3): the high bits choose the bucket, the low bits the slot.
__device__ __forceinline__ uint32_t bucket_hash(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  return h ^ (h >> 16);
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
                                                   int64_t tpb, int slots) {
  extern __shared__ uint32_t s_id[];                              // [slots] ids, then [slots] ranks
  uint16_t* s_rank = reinterpret_cast<uint16_t*>(s_id + slots);
  __shared__ uint32_t s_count[MAX_BUCKETS], s_start[MAX_BUCKETS];
  __shared__ uint32_t smem[TB / WAVE + 1];
  const Where here = where_am_i(S, tpb);
  if (here.b < 0) return;
  const int b = here.b;
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
      int32_t* cand = T.cand + b * T.cand_slots + first;
      uint32_t u[K_MAX], at[K_MAX];      // at: bucket << 16 | place among the tile's entries of the bucket
#pragma unroll
      for (int i = 0; i < K_MAX; ++i) {
        const int x = i * TB + threadIdx.x;
        u[i] = x < n_slots ? s_id[x] : NO_ID;
        if (u[i] != NO_ID) {
          cand[x] = (int32_t)u[i];
          const uint32_t q = __umulhi(bucket_hash(u[i]), (uint32_t)P);
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
          const uint32_t q = __umulhi(bucket_hash(u[i]), (uint32_t)P);
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
        uint32_t h = bucket_hash(u) & (BUCKET_SLOTS - 1);
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
          uint32_t h = bucket_hash(e.u[i]) & (BUCKET_SLOTS - 1);
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

// One block per tile of frontier nodes: the answers back in candidate order (in place: a tile's
// answers and its candidates share one stretch), masks of first occurrences, tile sums.
__global__ __launch_bounds__(TB) void k_tile_firsts(Tables T, Buckets B, const int32_t* __restrict__ nfront,
                                                    int k, uint64_t* __restrict__ tile_sums, int64_t tiles,
                                                    int S, int64_t tpb) {
  extern __shared__ uint32_t s_answer[];                          // [TILE_NODES * k]
  __shared__ uint64_t red[TB / WAVE];
  const Where here = where_am_i(S, tpb);
  if (here.b < 0) return;
  const int b = here.b;
  const int64_t nf = nfront[b];
  const int32_t P = bucket_count(nf, k, B.num_nodes, S);
  for (int64_t tile = here.tile; tile * TILE_NODES < nf; tile += tpb) {
    const int64_t first = tile * TILE_NODES * k;
    uint32_t* ref = T.ref + b * T.cand_slots + first;
    const uint16_t* rank = B.rank + b * B.entries + first;
    const uint32_t n = B.start[(b * B.tiles + tile) * B.row + P];
    for (uint32_t x = threadIdx.x; x < n; x += TB) s_answer[rank[x]] = ref[x];
    __syncthreads();
    const int64_t idx = tile * TILE_NODES + threadIdx.x;
    uint64_t mask = 0;
    int c = 0;
    if (idx < nf) {
      c = T.cnt[b * T.fr_slots + idx];
      for (int s = 0; s < c; ++s)
        if (s_answer[threadIdx.x * k + s] == (uint32_t)(first + threadIdx.x * k + s)) mask |= 1ull << s;
      T.first[b * T.fr_slots + idx] = mask;
    }
    const int64_t nodes = nf - tile * TILE_NODES < TILE_NODES ? nf - tile * TILE_NODES : TILE_NODES;
    for (int x = threadIdx.x; x < nodes * k; x += TB) ref[x] = s_answer[x];   // (unused slots: anything)
    uint64_t packed = wave_reduce_sum(((uint64_t)c << 32) | (uint64_t)__popcll(mask));
    if (lane_id() == 0) red[threadIdx.x / WAVE] = packed;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint64_t sum = 0;
      for (int w = 0; w < TB / WAVE; ++w) sum += red[w];
      tile_sums[b * tiles + tile] = sum;
    }
    __syncthreads();                     // `red` and the answers are rewritten for the next tile
  }
}
