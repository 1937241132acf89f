// The lines of inserted rows, all iterations in one launch.  Included by changeset.hip only, behind stays.hpp.
//
// An iteration's evicted lines, in line order, take its insertions, in the order of their list.  When every line
// is given up is known with the row that takes it (stays.hpp), so all that passes from one iteration to
// the next is how many lines of which stretch go.  A block per CU keeps, in LDS, the iteration that gives up each
// line of its stretch, and an iteration is:
//   * the block publishes how many of its lines go (one word, tagged with the iteration), finds them while the other
//     blocks' words arrive, and adds up the words of the blocks in front: the place of its lines' insertions
//   * hands the insertions their lines, and notes when these are given up again
//   * looks up the lines of a share of the iteration's accesses that hit
// What a block reads of another's is the words and the address table, both by atomics of the agent's scope, which
// neither L1 nor the L2 of an XCD answers, with all that the block wrote to the table complete (vmcnt 0) before it
// publishes; no fence, which would write back and invalidate an L2.  The lookups of iteration t begin when the block has
// published t and end before it publishes t + 1:
//   * all blocks had published t - 1, so the table holds what t - 2 wrote.  A row inserted in t - 1 that hits in t
//     is not looked up: with its insertion comes the position of that access (HANDED_OVER)
//   * nothing of t + 1 is written yet, and t itself does not write the entry of a row that hits
// The words sit in two sets in turn: a block publishes t + 2 after all have published t + 1, so after all have read t.
//
// The blocks wait for each other, so all of them have to run.  One call of the process at a time has them on a GPU, and only
// where MOVE_CALLS changesets at most are worked on: two calls' blocks with part of the CUs each would wait in vain, and blocks
// that wait keep many calls' kernels from the CUs.  The others take a launch per iteration (k_step_lines).  Still nothing
// guarantees it (other kernels may hold the CUs, other processes' blocks), so the wait is bounded: after MOVE_POLLS reads a block
// gives up and says so in its words, which ends the others' waits too, and the host starts over with the launches.  In the first
// iteration, where blocks that do not all run fail to meet, the bound is about what the iterations save.
// A read takes 0.2 us; the first wait 2 us, beside kernels of other streams (gathers, copies, products of 8 192^3) 100 us in 99
// of 100 calls, and 751 once.  10 M nodes, 100 iterations of 100 000, 300 000 lines, two, three, four and six threads
// that call all the time: 2 680, 3 650, 4 490 and 6 660 us a call (four, if one of them went this way, 4 680; with no
// turns 6 040, a third of the calls given up; all by launches 2 860, 3 615, 4 415 and 6 660); three processes 3 750 (with
// one bound for all waits 3 900, all by launches 3 510).
//
// An iteration takes 2.6 us without lookups (the words' way to memory and back 1.3, records and LDS), 4.4 with 96 000 of
// them from a table of 444 MB, 17.6 with 670 000 (two thirds of it random words at 59 G/s, the chip's rate); a launch
// per iteration, with flags and lists of leaving lines in HBM, took 7.4 and 27.6, and 13.0 where 31 000 of 105 000 lines
// change (4.1 this way).  The calls: 5 152 -> 4 375 us (33 M accesses, 573 000 lines, 200 iterations), 18 686 -> 16 546
// (154 M, 13.1 M lines), LRU of 20 iterations 715 -> 501.
#pragma once

constexpr int MOVE_THREADS = 1024;
constexpr int MOVE_CHAIN = 256;               // threads that exchange words and hand lines over
constexpr int MOVE_LOOKUPS = MOVE_THREADS - MOVE_CHAIN;
constexpr int MOVE_BLOCKS = MOVE_CHAIN;       // at most: a word to a thread
constexpr int MOVE_LIST = 2048;               // lines handed over at a time
constexpr int MOVE_ITEMS = 5;                 // lookups in flight to a thread
constexpr int64_t MOVE_LINES = 512;           // of a block, where there are few
constexpr int MOVE_POLLS = 1 << 13;           // reads of a wait; of the first one
constexpr int MOVE_MEET_MIN = 1 << 10, MOVE_MEET_SAVED = 16;   // at least, and for each iteration
constexpr int MOVE_DEVICES = 64;              // GPUs that calls take turns on; not this way on others
constexpr int MOVE_CALLS = 3;                 // calls at once on a GPU up to which one of them goes this way
constexpr int MOVE_WORDS_MAX = 35;            // words of two lines a thread has in LDS, at most (140 KB)
// ... and for LRU, which gives lines up in the order in which they were taken, so that an iteration's lie in the stretches of
// a few blocks, and the larger these are the more one block hands over.  Moved and by a launch per iteration, 300 iterations
// of 100 000 accesses, 25 000 lines each: of 3 M lines 4 477 and 5 435 us a call, 4 M 5 201 and 5 621, 4.7 M 5 996 and
// 5 674, 6 M 7 209 and 6 032, 8 M 9 382 and 6 496; of 300 000 accesses, 70 000 lines: 4.7 M 3 809 and 4 008, 6 M 4 313
// and 4 093.  (Belady's are spread: 10 M rows in a window that moves, 200 iterations of 200 000, 4 897 and 5 824.)
constexpr int MOVE_LRU_WORDS = 9;
constexpr uint32_t MOVE_GAVE_UP = 0xFFFFFFFFu;
constexpr int FINAL_ITEMS = 8;
constexpr int MOVE_TAG = 18;                  // bits for the lines of a block; above: iteration + 1, at most 2 048
static_assert(MOVE_THREADS * 2 * MOVE_WORDS_MAX < 1 << MOVE_TAG && STATIC_S_MAX < 1 << (31 - MOVE_TAG), "one word");

struct Moves {
  int32_t blocks;              // 0: not this way
  uint32_t* words;             // [2 * MOVE_BLOCKS], zero
  uint32_t* gave_up;           // zero
  int64_t per;                 // lines of a block's stretch
  uint64_t per_block;          // 2^32 / blocks, rounded up: n accesses are at most n * per_block / 2^32 to a block
  int32_t meet, polls;         // reads of the first iteration's wait, of the others'
  int32_t stop;                // iteration in which a block gives up whatever it reads; -1: none
  const uint32_t* leave_start;               // iteration that gives a line of the start state up, STAYS
  const uint64_t* leave_ins;                 // records of the insertions
  const int32_t *ids, *in_ids;
  int32_t *out_ids, *src_line;               // src_line: null, or marked
};

template <typename T>
__device__ __forceinline__ T agent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// W: words of two lines a thread has; odd, so that the threads of a wave read different banks.  The first waves
// (MOVE_CHAIN threads) exchange the words and hand the lines over, the others look the accesses up; the lines that go
// are found by all of them.
template <int W>
__global__ __launch_bounds__(MOVE_THREADS) void k_move_lines(State st, Moves m, const int64_t* __restrict__ off,
                                                             const int64_t* __restrict__ cs_offsets) {
  typedef uint16_t Pair __attribute__((ext_vector_type(2)));
  __shared__ uint32_t s_leave[W * MOVE_THREADS];    // per line the iteration that gives it up, 0xFFFF: none
  __shared__ uint32_t s_count[STATIC_S_MAX];        // lines that go, per iteration
  __shared__ uint32_t s_list[MOVE_LIST];
  __shared__ uint32_t s_waves[MOVE_THREADS / WAVE], s_before[MOVE_CHAIN / WAVE];
  __shared__ int s_stop;
  uint16_t* const leave = reinterpret_cast<uint16_t*>(s_leave);
  const int32_t S = st.S, me = blockIdx.x, blocks = gridDim.x;
  const int64_t first = me * m.per;
  const int32_t lines = (int32_t)(first >= st.cap ? 0 : st.cap - first < m.per ? st.cap - first : m.per);
  for (int t = threadIdx.x; t < S; t += MOVE_THREADS) s_count[t] = 0;
  for (int x = threadIdx.x; x < W * MOVE_THREADS; x += MOVE_THREADS) s_leave[x] = 0xFFFFFFFFu;
  if (threadIdx.x == 0) s_stop = 0;
  __syncthreads();
  for (int32_t l = threadIdx.x; l < lines; l += MOVE_THREADS) {
    const uint32_t e = m.leave_start[first + l];
    if (e >= (uint32_t)S) continue;
    leave[l] = (uint16_t)e;
    atomicAdd(&s_count[e], 1u);
  }
  const bool chain = threadIdx.x < MOVE_CHAIN;
  // the block's share of the accesses from `at` to `end`
  auto share_of = [&](int64_t at, int64_t end, int64_t& p, int64_t& to) {
    const int64_t share = (int64_t)((uint64_t)(uint32_t)(end - at + blocks - 1) * m.per_block >> 32);
    p = at + me * share + threadIdx.x - MOVE_CHAIN;
    to = at + (me + 1) * share < end ? at + (me + 1) * share : end;
  };
  // MOVE_ITEMS of them to a thread: ids and marks asked for, whether they are to be looked up (else -1), the table's
  // words, the results; nothing is waited for inside a step
  int32_t ids[MOVE_ITEMS], mark[MOVE_ITEMS], v[MOVE_ITEMS], line[MOVE_ITEMS];
  auto ask = [&](int64_t p, int64_t to) {
#pragma unroll
    for (int k = 0; k < MOVE_ITEMS; ++k) {
      ids[k] = m.ids[p + k * MOVE_LOOKUPS < to ? p + k * MOVE_LOOKUPS : 0];
      mark[k] = m.src_line[p + k * MOVE_LOOKUPS < to ? p + k * MOVE_LOOKUPS : 0];
    }
  };
  auto choose = [&](int64_t p, int64_t to) {
#pragma unroll
    for (int k = 0; k < MOVE_ITEMS; ++k) v[k] = mark[k] == LOOK_UP && p + k * MOVE_LOOKUPS < to ? ids[k] : -1;
  };
  // (the others read one word: a branch would be a wait for every load)
  auto look = [&]() {
#pragma unroll
    for (int k = 0; k < MOVE_ITEMS; ++k) line[k] = agent_load(&st.addr[v[k] >= 0 ? v[k] : 0]);
  };
  auto put = [&](int64_t p) {
#pragma unroll
    for (int k = 0; k < MOVE_ITEMS; ++k)
      if (v[k] >= 0) m.src_line[p + k * MOVE_LOOKUPS] = line[k];
  };
  int64_t dst = cs_offsets[0], dst_next = cs_offsets[1], at = off[0], at_next = off[1];
  const bool looks = !chain && m.src_line;
  int64_t p0 = 0, to = 0;
  if (looks) {
    share_of(at, at_next, p0, to);
    ask(p0, to);
    choose(p0, to);
  }
  for (int32_t t = 0; t < S; ++t) {
    const int64_t n_change = dst_next - dst;
    // what the iteration before wrote to the table is complete (its lookups are, their results were stored)
    if (chain) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    uint32_t* const words = m.words + (t & 1) * MOVE_BLOCKS;
    const uint32_t total = s_count[t];
    if (threadIdx.x == 0) agent_store(&words[me], (uint32_t)(t + 1) << MOVE_TAG | total);
    const int32_t ahead = t + 2 <= S ? t + 2 : S;
    const int64_t dst_ahead = cs_offsets[ahead], at_ahead = off[ahead];
    // the table's words for this iteration, ids and marks for the next one
    int64_t p1 = 0, to1 = 0;
    if (looks) {
      look();
      share_of(at_next, at_ahead, p1, to1);
      ask(p1, to1);
    }
    // the lines that go: bit k of a half for word k, lower line in the lower half
    constexpr int MASKS = (W + 15) / 16;
    uint32_t stays[MASKS];
    uint32_t mine = 0, rank = 0;
    auto list_from = [&](uint32_t round) {
      uint32_t r = rank;
#pragma unroll
      for (int q = 0; q < MASKS; ++q) {
        uint32_t go = ~stays[q];
        while (go) {
          const int k = __ffs((go | go >> 16) & 0xFFFFu) - 1;
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (go >> (k + 16 * h) & 1u) {
              if (r - round < (uint32_t)MOVE_LIST) s_list[r - round] = (threadIdx.x * W + q * 16 + k) * 2 + h;
              ++r;
              go &= ~(1u << (k + 16 * h));
            }
        }
      }
    };
    if (total) {                                    // uniform
      const Pair now = {(uint16_t)t, (uint16_t)t}, one = {1, 1};
#pragma unroll
      for (int q = 0; q < MASKS; ++q) {
        stays[q] = W - q * 16 < 16 ? 0xFFFFu << (W - q * 16) & 0xFFFFu : 0u;
        stays[q] |= stays[q] << 16;
#pragma unroll
        for (int k = 0; k < 16 && q * 16 + k < W; ++k) {
          const Pair x = __builtin_bit_cast(Pair, s_leave[threadIdx.x * W + q * 16 + k]) ^ now;
          stays[q] |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(x, one)) << k;
        }
        mine += 32 - __popc(stays[q]);
      }
      const uint32_t incl = wave_inclusive_scan(mine);
      if (lane_id() == WAVE - 1) s_waves[threadIdx.x / WAVE] = incl;
      __syncthreads();
      rank = incl - mine;
      for (int w = 0; w < (int)threadIdx.x / WAVE; ++w) rank += s_waves[w];
      if (mine) list_from(0);
    }
    // the words of all blocks
    if (chain) {
      uint32_t w = 0;
      bool here = (int32_t)threadIdx.x >= blocks;
      int polls = t == m.stop && me == blocks / 2 ? -1 : t == 0 ? m.meet : m.polls;
      if (polls < 0) s_stop = 1;
      while (polls >= 0) {
        if (!here) {
          w = agent_load(&words[threadIdx.x]);
          here = w >> MOVE_TAG == (uint32_t)(t + 1);
        }
        if (__all(here)) break;
        if (__any(w == MOVE_GAVE_UP) || --polls < 0) {
          s_stop = 1;
          break;
        }
      }
      const uint32_t sum = wave_reduce_sum((int32_t)threadIdx.x < me ? w & ((1u << MOVE_TAG) - 1u) : 0u);
      if (lane_id() == 0) s_before[threadIdx.x / WAVE] = sum;
    }
    __syncthreads();
    if (s_stop) {                                   // uniform
      if (threadIdx.x == 0) {
        agent_store(m.gave_up, 1u);
        agent_store(&m.words[me], MOVE_GAVE_UP);
        agent_store(&m.words[MOVE_BLOCKS + me], MOVE_GAVE_UP);
      }
      return;
    }
    if (looks) {
      put(p0);
      const bool more = p0 + MOVE_ITEMS * MOVE_LOOKUPS < to;   // a large share
      while ((p0 += MOVE_ITEMS * MOVE_LOOKUPS) < to) {
        ask(p0, to);
        choose(p0, to);
        look();
        put(p0);
      }
      if (more) ask(p1, to1);
      p0 = p1;
      to = to1;
      choose(p0, to);
    }
    if (total) {
      int64_t before = 0;
#pragma unroll
      for (int q = 0; q < MOVE_CHAIN / WAVE; ++q) before += s_before[q];
      for (uint32_t round = 0; round < total; round += MOVE_LIST) {    // uniform
        if (round) {
          __syncthreads();
          if (mine) list_from(round);
          __syncthreads();
        }
        if (!chain) continue;
        const uint32_t here = total - round < (uint32_t)MOVE_LIST ? total - round : (uint32_t)MOVE_LIST;
        for (uint32_t x = threadIdx.x; x < here; x += MOVE_CHAIN) {
          const int64_t k = before + round + x;
          const uint32_t l = s_list[x];
          if (k >= n_change) {                      // (as many lines as insertions, for distinct ids)
            leave[l] = 0xFFFFu;
            continue;
          }
          const uint64_t record = m.leave_ins[dst + k];
          const int32_t comes = m.in_ids[dst + k], gone = st.res_id[first + l];
          const uint32_t leaves = (uint32_t)record, next = (uint32_t)(record >> 32);
          const uint32_t e = leaves == LEAVES_NEXT ? (uint32_t)(t + 1) : leaves;
          const bool goes = e < (uint32_t)S && e > (uint32_t)t;
          leave[l] = goes ? (uint16_t)e : (uint16_t)0xFFFFu;
          if (goes) atomicAdd(&s_count[e], 1u);
          m.out_ids[dst + k] = gone;                // (before the table: a store in front would be waited for with `gone`)
          st.res_id[first + l] = comes;
          if (m.src_line) agent_store(&st.addr[comes], (int32_t)(first + l));
          if (next != NO_POSITION) m.src_line[next] = (int32_t)(first + l);
        }
      }
    }
    dst = dst_next;
    dst_next = dst_ahead;
    at = at_next;
    at_next = at_ahead;
  }
}

// The rows of the final state to the caller, but not where the call starts over: he may have given the array of the start
// state for them.
__global__ __launch_bounds__(TB) void k_final_lines(const int32_t* __restrict__ res_id, int64_t cap,
                                                    int32_t* __restrict__ final_ids,
                                                    const uint32_t* __restrict__ gave_up) {
  if (*gave_up) return;
  const int64_t base = (int64_t)blockIdx.x * (TB * FINAL_ITEMS) + threadIdx.x;
  int32_t v[FINAL_ITEMS];
#pragma unroll
  for (int k = 0; k < FINAL_ITEMS; ++k) v[k] = res_id[base + k * TB < cap ? base + k * TB : cap - 1];
#pragma unroll
  for (int k = 0; k < FINAL_ITEMS; ++k)
    if (base + k * TB < cap) final_ids[base + k * TB] = v[k];
}
void final_lines_async(const State& state, int32_t* final_ids, const void* gave_up, hipStream_t st) {
  hipLaunchKernelGGL(k_final_lines, dim3((unsigned)ceil_div(state.cap, TB * FINAL_ITEMS)), dim3(TB), 0, st, state.res_id,
                     state.cap, final_ids, static_cast<const uint32_t*>(gave_up));
}

// the rows and lines of the start state again, and what is to be looked up, for the launches per iteration
__global__ __launch_bounds__(TB) void k_start_lines(State st, const int32_t* __restrict__ start, int64_t total,
                                                    int32_t* __restrict__ src_line) {
  const int64_t l = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (l < st.cap) {
    const int32_t v = start[l];
    st.res_id[l] = v;
    st.addr[v] = (int32_t)l;
  }
  if (src_line && l < total && src_line[l] == HANDED_OVER) src_line[l] = LOOK_UP;
}

// A call on its GPU, and its turn to have such blocks there, from their launch until it has waited for them.
class MoveTurn {
 public:
  explicit MoveTurn(int device) : on_(device >= 0 && device < MOVE_DEVICES ? &gpus()[device] : nullptr) {
    if (on_) ++on_->calls;
  }
  ~MoveTurn() {
    give();
    if (on_) --on_->calls;
  }
  MoveTurn(const MoveTurn&) = delete;
  MoveTurn& operator=(const MoveTurn&) = delete;
  bool take() {
    mine_ = on_ && on_->calls <= MOVE_CALLS && !on_->taken.exchange(true);
    return mine_;
  }
  void give() {
    if (mine_) on_->taken = false;
    mine_ = false;
  }

 private:
  struct Gpu {
    std::atomic<int> calls{0};
    std::atomic<bool> taken{false};
  };
  static Gpu* gpus() {
    static Gpu all[MOVE_DEVICES];
    return all;
  }
  Gpu* const on_;
  bool mine_ = false;
};

// The blocks and their stretches; none for more lines than the blocks' LDS has room for, or pays for, nor in another
// call's turn.  GINEX_MOVE_POLLS: another bound of the waits, 0 for none of this; GINEX_MOVE_STOP: the iteration in which
// they give up.
int32_t moves_shape(const State& state, int64_t longest, int device, MoveTurn* turn, Moves* m) {
  const char* polls = getenv("GINEX_MOVE_POLLS");
  m->polls = polls ? atoi(polls) : MOVE_POLLS;
  m->meet = polls ? m->polls : std::min(MOVE_POLLS, std::max(MOVE_MEET_MIN, MOVE_MEET_SAVED * state.S));
  const char* stop = getenv("GINEX_MOVE_STOP");
  m->stop = stop ? atoi(stop) : -1;
  int cus = 0;
  GINEX_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device));
  int64_t blocks = std::max(ceil_div(state.cap, MOVE_LINES), ceil_div(longest, MOVE_ITEMS * MOVE_LOOKUPS));
  blocks = std::max<int64_t>(1, std::min<int64_t>(blocks, std::min(cus, MOVE_BLOCKS)));
  m->per = (ceil_div(state.cap, blocks) + 1) / 2 * 2;
  m->per_block = (uint64_t)ceil_div(int64_t(1) << 32, blocks);
  const int64_t words = state.lru ? MOVE_LRU_WORDS : MOVE_WORDS_MAX;
  m->blocks = m->polls > 0 && m->per <= MOVE_THREADS * 2 * words && turn->take() ? (int32_t)blocks : 0;
  return GINEX_OK;
}

void move_lines_async(const State& state, const Moves& m, const int64_t* off, const int64_t* cs_offsets,
                      hipStream_t st) {
  const int64_t words = ceil_div(m.per, 2 * MOVE_THREADS);
  const dim3 grid((unsigned)m.blocks), threads(MOVE_THREADS);
  if (words <= 1) hipLaunchKernelGGL(k_move_lines<1>, grid, threads, 0, st, state, m, off, cs_offsets);
  else if (words <= 3) hipLaunchKernelGGL(k_move_lines<3>, grid, threads, 0, st, state, m, off, cs_offsets);
  else if (words <= 9) hipLaunchKernelGGL(k_move_lines<9>, grid, threads, 0, st, state, m, off, cs_offsets);
  else if (words <= 17) hipLaunchKernelGGL(k_move_lines<17>, grid, threads, 0, st, state, m, off, cs_offsets);
  else hipLaunchKernelGGL(k_move_lines<MOVE_WORDS_MAX>, grid, threads, 0, st, state, m, off, cs_offsets);
}
