// mc_chains.hip -- the chain engine: exhaustive exploration on units of unequal speed with
// every workgroup's part of the visited set in its own LDS.
//
// On units of unequal speed a configuration's states up to its last dispatches are one per
// operation end of any unit and the closures of the dispatches at multiples of d; after them
// each choice of the last p units runs on by itself (mc_chains.h).  States at different clocks
// differ, so the visited set can be cut by clocks: a workgroup takes a piece (a window of a
// configuration's clocks), generates the window's states from their numbers, tests each in a
// hash set in LDS, exact on (clock, busy units), and writes the new ones to slots of their own
// in the visited set in HBM, a unit's ends one after another.  The duplicates are ends of
// several units at one clock; their slots are written empty.
//
// What bounds it.  k_superstep, which explored these models before, lists a chain state by
// state between two dispatches, in turns of the whole workgroup, and claims each state with a
// device-scope compare-and-swap in a table that has to be cleared first.  Here nothing in a
// piece waits for a state before it: a piece costs its fixed part (its tables, its window's
// counts and barriers, a chain of dependent reads: 4 us when it is alone, twice that among
// 1,024) and some 430 vector instructions per 64 states.  min_time launch by kernel trace,
// k_superstep -> here: reduction_g256_cu4_s1123 (86k states) 267 -> 15 us, matmul32_cu4_s1123
// (1.44M) 710 -> 45; check one below the optimum 180 -> 13 and 219 -> 27.  The times below, and
// mc_stats, are from the first workgroup's start to the last one's end on the device clock: 11
// and 36 us, checks 8 and 25.
//
// A workgroup has 256 threads and 18 KiB of LDS.  Its registers (124 vector registers with
// two-word keys and up to four units) let four share a CU, as many as a launch has.  Steps to
// that on matmul32_cu4_s1123, pieces of 1,024 items unless said: loops for any number of units
// and any kind of operation list 63 us, builds of their own for four units and for uniform
// phases 49; pieces of 1,536 47; no array indexed by lane in private memory (it was written to
// HBM, 51 KB for every piece) 45; a window's fields read from LDS where they are used rather
// than held in scalar registers, which spilled, the next piece's number taken while a piece is
// explored, and the closures' counts in LDS 38.
//
// Each piece stores a word to pinned memory: the steps it adds to a path, which give a
// counterexample's places and the longest path, and whether a terminal was found, whose clock
// follows from the piece.  So no counter on the device is added to, and nothing is copied.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mc_chains.h"
#include "mc_launch.h"

namespace mc {

namespace {

constexpr uint32_t kSetEmpty = 0xFFFFFFFFu;
constexpr uint32_t kChainBlock = 256;

typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) u64x2 global_u64x2;  // (a slot of W >= 2 words is
                                                               // 16-byte aligned)

// Operation ends.  UNIFORM: every configuration of the model has uniform phases and one wave.
template <bool UNIFORM>
struct DeviceEnds;
template <>
struct DeviceEnds<false> {
  GeneralEnds g;
  const CfgRec& r;
  __device__ __forceinline__ explicit DeviceEnds(const CfgRec& c) : g(general_ends(c)), r(c) {}
  __device__ __forceinline__ uint32_t at(uint32_t j) const { return r.d - rem_after(g, j); }
  __device__ __forceinline__ uint32_t upto(uint32_t x) const { return ends_upto(r, x); }
};
template <>
struct DeviceEnds<true> {
  UniformEnds g;
  const CfgRec& r;
  __device__ __forceinline__ explicit DeviceEnds(const CfgRec& c) : g(uniform_ends(c)), r(c) {}
  __device__ __forceinline__ uint32_t at(uint32_t j) const { return r.d - rem_after(g, j); }
  __device__ __forceinline__ uint32_t upto(uint32_t x) const { return ends_upto_uniform(r, x); }
};

template <int W, int M>
__device__ __forceinline__ Key<W> key_of(const ChainItem& it, uint32_t c, uint32_t clock,
                                         const Layout& L) {
  St y;
  y.cfg = c;
  y.pending = it.pending;
  y.clock = clock;
#pragma unroll
  for (int u = 0; u < kMaxCU; ++u) y.rem[u] = u < M ? it.rem[u] : 0u;
  return encode<W>(y, L);
}

// The sets of busy units of F_K in a tail window, ascending, listed by the first wavefront;
// returns their number.
__device__ __forceinline__ uint32_t list_sets(uint32_t p, uint32_t alive, uint32_t dead_n,
                                              uint8_t* list) {
  uint32_t n = 0;
  for (uint32_t b = 0; b < 1u << bits_set(alive); b += 64u) {
    const uint32_t x = b + lane_id(), set = spread_bits(x, alive);
    const bool ok = x < 1u << bits_set(alive) && tail_set(p, dead_n, set);
    const unsigned long long in = __ballot(ok);
    if (ok) list[n + (uint32_t)__popcll(in & ((1ull << lane_id()) - 1ull))] = (uint8_t)set;
    n += (uint32_t)__popcll(in);
  }
  return n;
}

__device__ __forceinline__ uint32_t unit_speed(const Layout& L, uint32_t u) {
  return u < L.m ? L.speed[u] : 1u;
}

constexpr uint32_t kChainSets = 64;  // closure counts held in LDS

struct ChainShared {
  ChainWindow w;
  uint32_t sets[kChainSets];
  uint32_t speed[kMaxCU];
  uint32_t whole[kMaxCU];
  uint32_t sets_n;
  uint8_t list[256];
  uint32_t per_set[256];  // new ends of each set
};

// The closures' counts: in LDS where they fit (read by lanes one after another), else the
// table.
__device__ __forceinline__ const uint32_t* load_sets(ChainShared& s, const ChainArgs& a) {
  const uint32_t* table = a.blob + a.sets_at;
  if (a.lcm >= kChainSets) return table;
  if (threadIdx.x <= a.lcm) s.sets[threadIdx.x] = table[threadIdx.x];
  return s.sets;
}

// Fills s.w for [s.w.t0, s.w.t1); every thread calls it.  x: *xp in scalar registers.
template <class E>
__device__ __forceinline__ void fill_window(ChainShared& s, const ChainCfg& x,
                                            const ChainCfg* xp, const ChainEnv& g, const E& ends, const ChainTail& tl,
                                            bool tail, uint32_t interval) {
  const uint32_t tid = threadIdx.x;
  const uint32_t listed = tail_listed(x, g);
  if (tid < (uint32_t)kMaxCU) {
    uint32_t whole = 0;
    const uint32_t sp = s.speed[tid];
    if (tail) whole = tail_window_unit(s.w, x, g, ends, interval, tid, sp, (listed >> tid) & 1u);
    else chain_window_unit(s.w, x, g, ends, tid, sp, xp->unit_off[tid]);
    s.whole[tid] = whole;
  }
  __syncthreads();
  if (tid == 0) {
    if (tail) tail_window_rest(s.w, x, g, tl, interval, s.whole);
    else chain_window_rest(s.w, x, g);
  }
  __syncthreads();
  if (tail && tid < 64u) {
    const uint32_t n = list_sets(x.p, s.w.alive, s.w.dead_n, s.list);
    if (tid == 0) {
      s.w.sets_n = n;
      s.w.items = n * s.w.before[kMaxCU];
    }
  }
  if (tail) __syncthreads();
}

}  // namespace

// The root (slot 0) and the SELECT states (slot 1 + c), by threads i, i + step, ..
template <int W>
__device__ __forceinline__ void write_roots(const QueryArgs& q, uint32_t i, uint32_t step) {
  for (; i <= q.n_cfg; i += step) {
    St y = {};
    y.cfg = i ? i - 1u : q.n_cfg;
    y.pending = i ? q.cfgs[i - 1u].n : 0u;
    const Key<W> k = encode<W>(y, q.L);
    unsigned long long* to =
        reinterpret_cast<unsigned long long*>(q.table) + (unsigned long long)i * W;
#pragma unroll
    for (int w = 0; w < W; ++w) to[w] = k.w[w];
  }
}

// The incumbent of branch and bound.
__global__ void k_chains_bound(Ctrl* ctrl, uint32_t T) { ctrl->bound = T; }

template <int W, int M, bool UNIFORM>
__global__ __launch_bounds__(kChainBlock) void k_chains(ChainArgs a) {
  __shared__ uint32_t set[1u << kChainSetLog2];
  __shared__ ChainShared s;
  __shared__ union {
    RoundRecord rec;
    uint32_t words[sizeof(RoundRecord) / 4];
  } s_sums;
  RoundRecord& sums = s_sums.rec;
  __shared__ uint32_t s_piece, s_T, s_skip, s_steps, s_term;
  const uint32_t tid = threadIdx.x;
  const ChainCfg* cfgs = reinterpret_cast<const ChainCfg*>(a.blob);
  const ChainTail* tails = reinterpret_cast<const ChainTail*>(a.blob + a.tails_at);
  uint32_t next = blockIdx.x;
  if (tid < (uint32_t)kMaxCU) s.speed[tid] = unit_speed(a.q.L, tid);
  if (tid == 0) {
    sums = RoundRecord{};
    sums.t_first = (uint32_t)__builtin_amdgcn_s_memrealtime();
  }
  const uint32_t* sets = load_sets(s, a);
  write_roots<W>(a.q, blockIdx.x * kChainBlock + tid, gridDim.x * kChainBlock);
  // sums of a wavefront (uniform in it)
  uint32_t states = 0, edges = 0, probes = 0, max_probe = 0, terms = 0;
  for (;;) {
    if (tid == 0) s_piece = next;
    __syncthreads();  // the piece before is done
    const uint32_t piece = uniform(s_piece);
    if (piece >= a.n_pieces) break;
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    const uint32_t c = find_piece(cfgs, a.q.n_cfg, piece);
    const ChainCfg x = load_const(cfgs + c);
    const CfgRec r = load_const(a.q.cfgs + c);
    const ChainEnv g = chain_env(r, a.q.L.speed, a.q.L.m, a.lcm, sets);
    const DeviceEnds<UNIFORM> ends(r);
    if (tid == 0) {
      uint32_t T = a.q.prune ? a.q.T : kNoClock;
      if (a.bb) {
        const uint32_t b = __hip_atomic_load(&a.q.ctrl->bound, __ATOMIC_RELAXED, kScopeAgent);
        T = b < T ? b : T;
      }
      const uint32_t stop = stop_asked(a.abort, a.watch, a.launch, piece, t0);
      if (stop) sums.error = kDevErrAbort;
      s_T = T;
      s_skip = stop;
      s_steps = s_term = 0u;
      next = a.n_pieces;
    }
    __syncthreads();
    const ChainSpan span = chain_span(x, g, piece - x.piece0, uniform(s_T));
    const bool tail = span.tail;
    const ChainTail tl = load_const(tails + (tail ? x.tail0 + span.interval : 0u));
    uint32_t steps = 0;  // of the longest path through the piece (thread 0)
    bool took = a.n_pieces <= gridDim.x;
    const auto take = [&] {  // the next piece, while this one is explored
      if (!took && tid == 0) next = gridDim.x + (atomicAdd(a.head, 1u) - a.head0);
      took = true;
    };
    uint32_t from = uniform(s_skip) ? span.t1 : span.t0;
    while (from < span.t1) {
      uint32_t to = span.t1;
      for (;;) {
        if (tid == 0) {
          s.w.t0 = from;
          s.w.t1 = to;
        }
        __syncthreads();
        fill_window(s, x, cfgs + c, g, ends, tl, tail, span.interval);
        const uint32_t items = uniform(s.w.items);
        __syncthreads();
        if (items <= kChainCap || to - from == 1u) break;
        to = from + (to - from) / 2u;
      }
      {
        uint4* s4 = reinterpret_cast<uint4*>(set);
        for (uint32_t i = tid; i < 1u << (kChainSetLog2 - 2u); i += kChainBlock)
          s4[i] = make_uint4(kSetEmpty, kSetEmpty, kSetEmpty, kSetEmpty);
        s.per_set[tid] = 0u;
      }
      __syncthreads();
      take();
      // (two loops: the fields of either kind of window fill the scalar registers)
      const auto explore = [&](auto is_tail) {
        constexpr bool kTail = decltype(is_tail)::value;
        const ChainWindow& w = s.w;  // (its lanes' fields are read as they are needed: in
                                     // scalar registers they spilled)
        const uint32_t w_t0 = uniform(w.t0);
        const uint32_t w_items = uniform(w.items);
        const uint32_t items = w_items < kChainCap ? w_items : kChainCap;
        const float per_inv = inverse(w.before[kMaxCU]);
        uint32_t ends_new = 0;
        for (uint32_t base = 0; base < items; base += kChainBlock) {
          const uint32_t i = base + tid < items ? base + tid : items - 1u;
          ChainItem it;
          uint32_t rank = 0;
          if constexpr (kTail) {
            rank = quotient(i, per_inv);
            tail_item<M>(w, x, g, ends, i - rank * w.before[kMaxCU], rank, s.list[rank], &it);
          } else {
            chain_item<M>(w, x, g, ends, r.n, i, &it);
          }
          const bool in = base + tid < items, act = in && it.active;
          const uint32_t code = it.t << g.m | it.busy;
          uint32_t at = probe_start<0x9E3779B1u>(code, 32u - kChainSetLog2, a.q.hkeep), old = code;
          if (act) old = atomicCAS(&set[at], kSetEmpty, code);
          const unsigned long long acts = __builtin_amdgcn_ballot_w64(act);
          unsigned long long met =
              __builtin_amdgcn_ballot_w64(act && old != kSetEmpty && old != code);
          uint32_t trips = 1;
          probes += (uint32_t)__popcll(acts) + (uint32_t)__popcll(met);
          while (met) {
            if (__builtin_amdgcn_inverse_ballot_w64(met)) {
              at = (at + trips) & ((1u << kChainSetLog2) - 1u);
              old = atomicCAS(&set[at], kSetEmpty, code);
            }
            met &= __builtin_amdgcn_ballot_w64(old != kSetEmpty && old != code);
            probes += (uint32_t)__popcll(met);
            if (++trips >> kChainSetLog2) break;  // (never: there are more slots than states)
          }
          max_probe = trips > max_probe ? trips : max_probe;
          const bool fresh = act && old == kSetEmpty;
          if (in) {
            const Key<W> key = key_of<W, M>(it, c, w_t0 + it.t, a.q.L);
            global_u64* kp = (global_u64*)a.q.table + (unsigned long long)it.slot * W;
            if constexpr (W == 1) {
              *kp = fresh ? key.w[0] : kEmptyWord;
            } else {
#pragma unroll
              for (int j = 0; j < W; j += 2) {
                u64x2 v;
                v.x = fresh ? key.w[j] : kEmptyWord;
                v.y = fresh ? key.w[j + 1] : kEmptyWord;
                *(global_u64x2*)(kp + j) = v;
              }
            }
          }
          if (kTail && fresh) atomicAdd(&s.per_set[rank], 1u);
          const unsigned long long news = __builtin_amdgcn_ballot_w64(fresh);
          edges += (uint32_t)__popcll(acts);
          states += (uint32_t)__popcll(news);
          if constexpr (!kTail)
            ends_new += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(fresh && it.is_end));
          const unsigned long long over =
              __builtin_amdgcn_ballot_w64(fresh && (it.pending | it.busy) == 0u);
          if (over) {
            terms += (uint32_t)__popcll(over);
            if (__builtin_amdgcn_inverse_ballot_w64(over)) {
              s_term = 1u;
              if (a.bb) atomicMin(&a.q.ctrl->bound, w_t0 + it.t);
            }
          }
        }
        // the steps this window adds to a path: every end and dispatch of the chain, and of a
        // tail the ends of the set with most
        if (!kTail && ends_new && lane_id() == 0) atomicAdd(&s_steps, ends_new);
        __syncthreads();
        if (kTail) {
          if (tid < 64u) {
            uint32_t most = 0;
            for (uint32_t q = tid; q < 256u; q += 64u) most = max(most, s.per_set[q]);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o));
            steps += most;
          }
        } else {
          steps += starts_between(g, w.k0, w.k1) + (w.part_n ? x.p : 0u);
        }
        if (tid == 0) sums.chunks += (items + kChainBlock - 1u) / kChainBlock;
      };
      if (tail) explore(std::true_type{});
      else explore(std::false_type{});
      from = to;
      __syncthreads();
    }
    take();
    // (crowded sets make more probes over a launch than 32 bits count, a window 2^23 at most)
    if (lane_id() == 0) atomicAdd(&sums.probes, (unsigned long long)probes);
    probes = 0;
    if (tid == 0) {
      __hip_atomic_store(a.words + piece, (s_steps + steps) | (s_term << 31), __ATOMIC_RELAXED,
                         kScopeSystem);
      sums.rounds += 1u;
      sums.pieces += 1u;
      const uint32_t dt = (uint32_t)(__builtin_amdgcn_s_memrealtime() - t0);
      if (dt > sums.crit) {
        sums.crit = dt;
        sums.crit_cfg = c;
      }
    }
  }
  if (lane_id() == 0) {
    atomicAdd(&sums.states, states);
    atomicAdd(&sums.edges, edges);
    if (terms) atomicAdd(&sums.terms, terms);
    atomicMax(&sums.max_probe, max_probe);
  }
  __syncthreads();
  if (tid == 0) sums.t_last = (uint32_t)__builtin_amdgcn_s_memrealtime();
  __syncthreads();
  if (tid < sizeof(RoundRecord) / 4u)
    __hip_atomic_store(reinterpret_cast<uint32_t*>(a.records + blockIdx.x) + tid,
                       s_sums.words[tid], __ATOMIC_RELAXED, kScopeSystem);
}

// ---- counterexample ---------------------------------------------------------------------
//
// The path to a terminal of configuration a.target at clock q.T, root first.  Up to the last
// dispatches every end of the chain is on it, and of each dispatch the units in index order;
// then the least set of p units whose tail ends at q.T.  The exploration counted each chain
// piece's states on the path, so a workgroup knows where its pieces' states go (base[b] for
// workgroup b); the last one lists the tail.  Within a window of clocks an end belongs to the
// lowest unit that ends there, its place is the ends before it (of each unit, by a prefix sum
// over those that belong to it) and the dispatches before it.  Every state has to be in a slot
// of its own or, an end of several units, in one of theirs, or the path is bad.
//
// It waits for its reads and barriers, window by window.  One workgroup for the whole path took
// 64 and 71 us on the two models above, a workgroup for each piece 29 and 30, most of it the
// tail's intervals, one after another.
constexpr uint32_t kPathEnds = kChainCap, kChainPathBlock = 512;

template <int W, int M, bool UNIFORM>
__global__ __launch_bounds__(kChainPathBlock) void k_chain_path(ChainArgs a, TraceOut t,
                                                               const uint32_t* base,
                                                               uint32_t per) {
  __shared__ ChainShared s;
  __shared__ uint32_t own[kPathEnds + 1], covered[kPathEnds / 32], wave_sums[kChainPathBlock / 64];
  __shared__ uint32_t s_bad, s_set, s_rank;
  const uint32_t tid = threadIdx.x, c = a.target, T = a.q.T;
  const ChainCfg* xp = reinterpret_cast<const ChainCfg*>(a.blob) + c;
  const ChainCfg x = load_const(xp);
  const ChainTail* tails = reinterpret_cast<const ChainTail*>(a.blob + a.tails_at);
  const CfgRec r = load_const(a.q.cfgs + c);
  const ChainEnv g = chain_env(r, a.q.L.speed, a.q.L.m, a.lcm, load_sets(s, a));
  const DeviceEnds<UNIFORM> ends(r);
  const unsigned long long* keys = reinterpret_cast<const unsigned long long*>(a.q.table);
  const auto there = [&](uint32_t slot, const Key<W>& k) {
    bool same = slot <= a.q.mask;
#pragma unroll
    for (int w = 0; w < W; ++w) same = same && keys[(unsigned long long)slot * W + w] == k.w[w];
    return same;
  };
  const auto put = [&](uint32_t i, const Key<W>& k) {
    if (i >= t.cap) return;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const unsigned long long at = (unsigned long long)i * W + w;
      if (at < t.host_words) t.host[at] = k.w[w];
      else t.out[at] = k.w[w];
    }
  };
  if (tid < (uint32_t)kMaxCU) s.speed[tid] = unit_speed(a.q.L, tid);
  if (tid == 0) {
    s_bad = 0u;
    s_set = 0x100u;
  }
  __syncthreads();
  const bool last = blockIdx.x + 1u == gridDim.x;
  uint32_t n = base[blockIdx.x];
  if (blockIdx.x == 0u && tid < 2u) {  // the root and the SELECT state
    St y = {};
    y.cfg = tid ? c : a.q.n_cfg;
    y.pending = tid ? r.n : 0u;
    const Key<W> k = encode<W>(y, a.q.L);
    if (!there(tid ? 1u + c : 0u, k)) s_bad = 1u;
    put(tid, k);
  }
  // the least set of p units of F_K whose tail ends at T (none where the chain ends there)
  if (tid < 256u && (tid & ~x.idle) == 0u && bits_set(tid) == x.p) {
    uint32_t end = x.K * g.d;
    for (uint32_t u = 0; u < g.m; ++u)
      if (((tid | ~x.idle) >> u) & 1u)
        end = max(end, tail_start(x, g, s.speed[u]) + s.speed[u] * g.d);
    if (end == T) atomicMin(&s_set, tid);
  }
  __syncthreads();
  const uint32_t chosen = uniform(s_set);
  bool bad = chosen > 0xFFu;
  const uint32_t on = (g.all & ~x.idle) | chosen;  // units busy in the tail
  // the workgroup's chain pieces, one at a time, or the tail's intervals
  const bool tail = last;
  uint32_t phase = last ? 0u : blockIdx.x * per;
  const uint32_t phases = last ? x.tail_n : min(phase + per, x.windows);
  for (; !bad && phase < phases; ++phase) {
    const uint32_t interval = tail ? phase : 0u;
    const ChainSpan span = chain_span(x, g, phase, kNoClock);
    uint32_t from = tail ? tail_from(x, g, interval) : span.t0;
    uint32_t end = tail ? (x.K + interval + 1u) * g.d : span.t1;
    if (tail && end > T + 1u) end = T + 1u;
    const ChainTail tl = load_const(tails + (tail ? x.tail0 + interval : 0u));
    while (from < end) {
      uint32_t to = end;
      for (;;) {
        if (tid == 0) {
          s.w.t0 = from;
          s.w.t1 = to;
        }
        __syncthreads();
        fill_window(s, x, xp, g, ends, tl, tail, interval);
        const uint32_t k = uniform(s.w.before[kMaxCU]);
        __syncthreads();
        if (k <= kPathEnds || to - from == 1u) break;
        to = from + (to - from) / 2u;
      }
      const ChainWindow& w = s.w;
      const uint32_t N = w.before[kMaxCU], set = chosen & w.alive;
      if (tid == 0) s_rank = 0u;
      for (uint32_t i = tid; i < (N + 31u) / 32u; i += kChainPathBlock) covered[i] = 0u;
      __syncthreads();
      if (tail && tid < w.sets_n && s.list[tid] == set) s_rank = tid;
      __syncthreads();
      const uint32_t rank = uniform(s_rank);
      // unit v's ends before clock `at`, from the window's first on
      const auto ends_to = [&](uint32_t v, uint32_t at) {
        uint32_t k;
        const uint32_t sp = s.speed[v];
        if (!tail) return ends_before(ends, g, sp, at) - s.w.first[v];
        return ends_of_one(ends, sp, tail_start(x, g, sp), w.t0, at, &k);
      };
      uint32_t counted = g.reps;
      if (tail) {  // the listed units of whose speed one runs
        counted = 0u;
        const uint32_t listed = tail_listed(x, g);
#pragma unroll
        for (uint32_t v = 0; v < (uint32_t)M; ++v)
          if (((listed >> v) & 1u) && (units_of_speed<M>(g, g.speed[v]) & on)) counted |= 1u << v;
      }
      const auto counts = [&](uint32_t v) { return ((counted >> v) & 1u) != 0u; };
      const auto item = [&](uint32_t i, ChainItem* it) {
        if (tail) tail_item<M>(w, x, g, ends, i, rank, set, it);
        else chain_item<M>(w, x, g, ends, r.n, i, it);
      };
      for (uint32_t i = tid; i < N; i += kChainPathBlock) {
        ChainItem it;
        item(i, &it);
        const uint32_t at = w.t0 + it.t;
        uint32_t owner = kParentNone;
        for (uint32_t v = 0; v < g.m && owner == kParentNone; ++v) {
          if (!counts(v) || !s.w.count[v]) continue;
          const uint32_t k = ends_to(v, at);
          if (ends_to(v, at + 1u) > k) owner = s.w.before[v] + k;
        }
        own[i] = owner == i ? 1u : 0u;
        if (owner < N && it.active && there(it.slot, key_of<W, M>(it, c, at, a.q.L)))
          atomicOr(&covered[owner >> 5], 1u << (owner & 31u));
      }
      __syncthreads();
      {  // exclusive prefix sum of `own`, own[N] = their number
        constexpr uint32_t kPer = kPathEnds / kChainPathBlock;
        uint32_t v[kPer], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
          const uint32_t i = tid * kPer + q;
          v[q] = i < N ? own[i] : 0u;
          sum += v[q];
        }
        uint32_t incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = __shfl_up(incl, o);
          if ((int)lane_id() >= o) incl += y;
        }
        if (lane_id() == 63u) wave_sums[tid >> 6] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
        for (uint32_t q = 0; q < tid >> 6; ++q) run += wave_sums[q];
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
          const uint32_t i = tid * kPer + q;
          if (i <= N) own[i] = run;
          run += v[q];
        }
        if (tid == kChainPathBlock - 1u && N == kPathEnds) own[N] = run;
      }
      __syncthreads();
      const uint32_t total_ends = own[N];
      const auto before = [&](uint32_t at) {  // ends of the path before clock `at`
        uint32_t k = 0;
        for (uint32_t v = 0; v < g.m; ++v)
          if (counts(v) && s.w.count[v])
            k += own[s.w.before[v] + ends_to(v, at)] - own[s.w.before[v]];
        return k;
      };
      for (uint32_t i = tid; i < N; i += kChainPathBlock) {
        if (own[i + 1u] == own[i]) continue;
        ChainItem it;
        item(i, &it);
        const uint32_t at = w.t0 + it.t;
        if (!((covered[i >> 5] >> (i & 31u)) & 1u)) s_bad = 1u;
        uint32_t k = div_up(at, g.d);
        k = k < w.k1 ? k : w.k1;
        put(n + before(at) + (tail ? 0u : starts_between(g, w.k0, k)),
            key_of<W, M>(it, c, at, a.q.L));
      }
      n += total_ends;
      if (!tail) {
        const uint32_t starts = starts_between(g, w.k0, w.k1);
        for (uint32_t y = tid; y < starts + (w.part_n ? x.p : 0u); y += kChainPathBlock) {
          uint32_t k, j, place;
          const bool part = y >= starts;
          if (part) {  // the units of the chosen set, in index order
            k = x.K;
            j = y - starts + 1u;
            place = n + y;
          } else {
            uint32_t u = 0, loc = y;
            for (; u + 1u < g.m; ++u) {
              const uint32_t cnt = div_up(w.k1, s.speed[u]) - div_up(w.k0, s.speed[u]);
              if (loc < cnt) break;
              loc -= cnt;
            }
            k = (div_up(w.k0, s.speed[u]) + loc) * s.speed[u];
            j = bits_set(idle_at(g, k) & ((2u << u) - 1u));
            place = n - total_ends + before(k * g.d + 1u) + starts_between(g, w.k0, k) + j - 1u;
          }
          uint32_t sub = (1u << j) - 1u, slot;
          if (part) {
            uint32_t left = j, at = 0;
            sub = 0;
            for (uint32_t u = 0; u < g.m; ++u)
              if ((x.idle >> u) & 1u) {
                if (left && ((chosen >> u) & 1u)) {
                  sub |= 1u << at;
                  --left;
                }
                ++at;
              }
            slot = x.slot0 + x.part_off + sub - 1u;
          } else {
            slot = x.slot0 + x.close_off + closures_before(g, k) + sub - 1u;
          }
          ChainItem it;
          chain_state<M>(w, g, r.n, k - w.kw, 0u, sub, true, &it);
          const Key<W> key = key_of<W, M>(it, c, k * g.d, a.q.L);
          if (!there(slot, key)) s_bad = 1u;
          put(place, key);
        }
        n += starts + (w.part_n ? x.p : 0u);
      }
      from = to;
      __syncthreads();
      bad = s_bad != 0u;
      if (bad) break;
    }
  }
  __syncthreads();
  if (tid == 0) {
    // (the host cleared the flag)
    if (bad || s_bad || n > t.cap || (!last && n != base[blockIdx.x + 1u]))
      __hip_atomic_store(t.host_res + 2, 1u, __ATOMIC_RELAXED, kScopeSystem);
    if (last) __hip_atomic_store(t.host_res + 1, n, __ATOMIC_RELAXED, kScopeSystem);
  }
}

// ---- launch helpers (host) ------------------------------------------------------------

// f(W, M, UNIFORM) as compile-time constants
template <class F>
hipError_t for_model(const ChainArgs& a, uint32_t W, const F& f) {
  const auto units = [&](auto w, auto uniform) {
    if (a.q.L.m <= 4u) f(w, std::integral_constant<int, 4>{}, uniform);
    else f(w, std::integral_constant<int, kMaxCU>{}, uniform);
  };
  const auto words = [&](auto uniform) {
    if (W == 1) units(std::integral_constant<int, 1>{}, uniform);
    else if (W == 2) units(std::integral_constant<int, 2>{}, uniform);
    else units(std::integral_constant<int, 4>{}, uniform);
  };
  if (a.uniform) words(std::true_type{});
  else words(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_chains(hipStream_t st, uint32_t W, uint32_t grid, const ChainArgs& a) {
  if (a.bb) hipLaunchKernelGGL(k_chains_bound, dim3(1), dim3(1), 0, st, a.q.ctrl, a.q.T);
  return for_model(a, W, [&](auto w, auto m, auto uniform) {
    hipLaunchKernelGGL((k_chains<decltype(w)::value, decltype(m)::value, decltype(uniform)::value>),
                       dim3(grid), dim3(kChainBlock), 0, st, a);
  });
}

hipError_t launch_chain_path(hipStream_t st, uint32_t W, const ChainArgs& a, const TraceOut& t,
                             uint32_t grid, const uint32_t* base, uint32_t per) {
  return for_model(a, W, [&](auto w, auto m, auto uniform) {
    hipLaunchKernelGGL(
        (k_chain_path<decltype(w)::value, decltype(m)::value, decltype(uniform)::value>),
        dim3(grid), dim3(kChainPathBlock), 0, st, a, t, base, per);
  });
}

}  // namespace mc
