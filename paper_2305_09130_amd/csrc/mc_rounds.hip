// mc_rounds.hip -- the round engine: exhaustive exploration on units alike with every
// workgroup's part of the visited set in its own LDS.
//
// On units alike a configuration's subgraph is a chain of rounds: from the state with every
// unit idle (clock r d, n - r m pending) k = min(m, n - r m) workgroups start, in any order
// (the closure: the sets of started units), and each of the C(m, k) full sets runs in lock
// step through the b operation ends to the next all-idle state.  A partition holds whole
// rounds, the head of a long round or a slice of its runs, and no two partitions generate
// the same state: rounds differ in the pending count, slices in the time left, and a state
// between two rounds belongs to the partition of the round it ends.
//
// So a duplicate can only meet its first copy within a partition, and the set that tells new
// states from found ones need not be shared: a workgroup takes a piece of a partition (at
// most kMaxPiece generated states, and the last of a partial round's runs), tests each in an
// open-addressing hash set in LDS and writes the new ones to the partition's own slots of the
// visited set in HBM, consecutive states to consecutive slots.  The set is exact: it holds the
// state's (pending, mask, time left), which is all of a state that varies within a piece, in 32
// bits.
//
// What bounds it.  k_superstep, which explored these models before, makes one device-scope
// compare-and-swap per state on a random line of a table in HBM, at the chip's limit for
// those (17 G/s); here a state costs a compare-and-swap in LDS, 8 bytes of a coalesced store
// and some 125 vector instructions per 64 states, which bound it (the vector units issue in
// about 85 of 100 cycles that they could).  min_time launch by kernel trace, k_superstep (which
// needs its table cleared besides: 330 us of the first) -> here: matmul128_vw_cu8 (58.0M states)
// 3,876 -> 226 us, matmul64_cu4 (5.15M) 457 -> 37, abstract_s1024_np4_cu4 280 -> 28,
// minimum_s1024_np4_cu4 133 -> 23; 512 uneven instances (228M) by HIP events 15.4 -> 1.11 ms.
// The other times here, and mc_stats, are from the first workgroup's start to the last one's end
// on the device clock, 7 to 9 us less than the trace has for the same launch: 218 us on
// matmul128_vw_cu8 within a tuning step (266 G states/s, 2.1 TB/s of keys written) and 209 in a
// row of queries, 29 on matmul64_cu4.
//
// The loop over a piece's items was 0.29 ms on matmul128_vw_cu8 with the operation ends and the
// places in a round computed from the configuration record for every item, the statistics
// reduced over the wavefront for every piece, and branches where selects now are.
//
// A workgroup has 256 or 512 threads (rounds_block) and up to 33 KiB of LDS, so that four share
// a CU: one's lookups and barriers between pieces overlap another's items.  Pieces of half the
// size ran slower (matmul128_vw_cu8 0.40 -> 0.47 ms when measured): a piece costs about 3 us
// beyond its items.
//
// A query of one model is one launch: it writes the root and SELECT states itself and takes its
// descriptor as an argument, no counter has to be cleared for it, and its pieces' descriptors
// are two dependent reads nearer.  With a launch before it that began the model:
// reduction_g256_cu2, load to check 85 -> 81 us, abstract_s1024_np4_cu1 121 -> 116 us.
//
// Sums go to the host as one 64-byte record per workgroup, stored to pinned memory: added to
// the model's counters instead, ten atomics of 1,024 workgroups on one line took 60 us.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mc_launch.h"
#include "mc_rounds.h"

namespace mc {

namespace {

constexpr uint32_t kSetEmpty = 0xFFFFFFFFu;

// A workgroup's sums, added to its model's counters: for launches over several models, when
// a piece of another model comes or the launch ends.
// One lane per counter: the atomics of a flush go out together, and none returns a value.
__device__ __forceinline__ void flush_sums(Ctrl* ctrl, RoundRecord& s) {
  const uint32_t tid = threadIdx.x;
  if (tid >= 64u) return;
  unsigned long long v = 0, *to = nullptr;
  switch (tid) {
    case 0: v = s.states; to = &ctrl->states; break;
    case 1: v = s.terms; to = &ctrl->terminals; break;
    case 2: v = s.edges; to = &ctrl->edges; break;
    case 3: v = s.edges - s.states; to = &ctrl->dups; break;
    case 4: v = s.probes; to = &ctrl->probes; break;
    case 5: v = s.chunks; to = &ctrl->chunks; break;
    case 6: v = s.rounds; to = &ctrl->supersteps; break;
    case 7: v = s.depth; to = &ctrl->max_depth; break;
    case 8: v = (unsigned long long)s.crit << 32 | s.crit_cfg; to = &ctrl->crit_longest; break;
    default: break;
  }
  if (v && tid < 7u) atomicAdd(to, v);
  else if (v) atomicMax(to, v);
  if (tid == 9u && s.max_probe) atomicMax(&ctrl->max_probe, s.max_probe);
  if (tid == 10u && s.pieces) atomicAdd(&ctrl->parts_done, s.pieces);
  if (tid == 0u) s = RoundRecord{};  // (the wavefront's reads above are done: one instruction
                                     // stream)
}

// What the items of a piece need of its model, configuration and query.
struct ItemEnv {
  uint32_t c, d, T, refloor, rem_bits, sp, sm, set_shift, set_mask, hkeep;
  unsigned long long keys, links;  // addresses of the set's two regions
};

// Sums of one wavefront, kept in scalar registers (but for `terms`) from piece to piece.
struct ItemSums {
  uint32_t states = 0, edges = 0, chunks = 0;
  uint32_t depth = 0;
  uint32_t last = 0;                            // the piece's last item found new (+ 1)
  uint32_t probes = 0, max_probe = 0;           // of all lanes, in this piece; of the lane with
                                                // most
  uint32_t terms = 0;                           // per lane
};

__device__ __forceinline__ uint32_t sum64(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Adds a wavefront's sums to the workgroup's.
__device__ __forceinline__ void add_sums(RoundRecord& s, ItemSums& w) {
  const uint32_t terms = sum64(w.terms);
  if (lane_id() == 0) {
    atomicAdd(&s.states, w.states);
    atomicAdd(&s.edges, w.edges);
    if (terms) atomicAdd(&s.terms, terms);
    atomicMax(&s.max_probe, w.max_probe);
    atomicMax(&s.depth, w.depth);
    if (threadIdx.x == 0) s.chunks += w.chunks;
  }
  w = ItemSums{};
}

// A select takes one scalar operand: values the items select among are kept in vector
// registers, or each select would copy one there first.
__device__ __forceinline__ void to_vector(uint32_t& x) { asm("" : "+v"(x)); }
__device__ __forceinline__ UniformEnds in_vector_registers(UniformEnds u) {
#pragma unroll
  for (int j = 0; j < kMaxPhases; ++j) {
    to_vector(u.lat[j]);
    to_vector(u.left[j]);
  }
  return u;
}
__device__ __forceinline__ GeneralEnds in_vector_registers(GeneralEnds u) {
#pragma unroll
  for (int j = 0; j < kMaxPhases; ++j) {
    to_vector(u.i0[j]);
    to_vector(u.t0[j]);
    to_vector(u.lat[j]);
    to_vector(u.la[j]);
  }
  return u;
}

// Items [from, to) of a piece: of its full rounds, or (PART) of its partial round.  Two loops,
// as the fields of one round kind fill the scalar registers.  CLOCKS: a query with a
// threshold or a floor tells states apart by their clocks.
template <int BLOCK, bool PART, bool CLOCKS, class Ends, class Model>
__device__ __forceinline__ void explore_items(const Piece& v, const Ends& ends_in, const ItemEnv& g,
                                              uint32_t from, uint32_t to, uint32_t* set,
                                              const uint8_t* masks, const Model& model,
                                              uint32_t* host_tc, ItemSums& sum) {
  const ItemBase b = item_base(v, g.c, g.d, g.rem_bits, g.sp, g.sm);
  const uint32_t wave = uniform(threadIdx.x & ~63u);
  const Ends ends = in_vector_registers(ends_in);
  for (uint32_t base = from; base < to; base += BLOCK) {
    const uint32_t i = base + threadIdx.x;
    ++sum.chunks;
    const RoundItem it = PART ? part_item(v, i, masks) : full_item(v, i);
    const ItemState x = item_state(v, b, it, rem_after(ends, it.j));
    const uint32_t code = x.code;
    bool act = i < to;
    if constexpr (CLOCKS) act = act && x.clock <= g.T;
    // the set: exact on (pending, busy, time left).  It has more slots than the piece has
    // items, so the probe sequence ends (probe_start: why this one)
    uint32_t at = probe_start(code, g.set_shift, g.hkeep), old = code;
    if (act) old = atomicCAS(&set[at], kSetEmpty, code);
    const unsigned long long acts = __builtin_amdgcn_ballot_w64(act);
    // the lanes that met another state try the next slot
    unsigned long long met = __builtin_amdgcn_ballot_w64(old != kSetEmpty && old != code);
    uint32_t trips = 1;
    sum.probes += (uint32_t)__popcll(acts) + (uint32_t)__popcll(met);
    while (met) {
      if (__builtin_amdgcn_inverse_ballot_w64(met)) {
        at = (at + trips) & g.set_mask;
        old = atomicCAS(&set[at], kSetEmpty, code);
      }
      met &= __builtin_amdgcn_ballot_w64(old != kSetEmpty && old != code);
      sum.probes += (uint32_t)__popcll(met);
      if (++trips > g.set_mask) break;  // (never: set_log2)
    }
    sum.max_probe = trips > sum.max_probe ? trips : sum.max_probe;
    bool fresh = act && old == kSetEmpty;
    const unsigned long long key = x.key;
    global_u64* kp = (global_u64*)g.keys + it.slot;
    // a continued exploration finds the states below its floor in their slots
    if constexpr (CLOCKS)
      if (x.clock < g.refloor && fresh) fresh = *kp != key;
    if (fresh) {
      *kp = key;
      // links, as the counterexample reads them: a round's end to the state its round starts
      // from (parent; none in a run slice) and the leaf its run starts from (jump), a dispatch
      // leaf to its round's start
      if (x.rem == 0u || it.is_leaf) {
        const ItemLinks l = links_of(v, i, it.q);
        const unsigned long long hi = x.rem ? kParentNone : l.leaf;
        ((global_u64*)g.links)[it.slot] = l.root | hi << 32;
        if (x.rem == 0u && x.prel + v.pmin == 0u) {
          const ModelDev md = model();
          const uint32_t end = b.clock0 + it.q * b.d + b.d;  // x.clock, needed here only
          ++sum.terms;
          md.tslot[g.c] = it.slot;
          // (a configuration has one terminal)
          if (host_tc) __hip_atomic_store(host_tc + g.c, end, __ATOMIC_RELAXED, kScopeSystem);
          else atomicMin(&md.tc[g.c], end);
          if (md.prune) md.ctrl->violated = 1u;
          if (md.bb) atomicMin(&md.ctrl->bound, end);
        }
      }
    }
    const unsigned long long news = __builtin_amdgcn_ballot_w64(fresh);
    sum.edges += (uint32_t)__popcll(acts);
    sum.states += (uint32_t)__popcll(news);
    if (news) sum.last = base + wave + 64u - (uint32_t)__builtin_clzll(news);
  }
}

// A model's root (slot 0) and SELECT states (slot 1 + c), by threads i, i + step, ..
__device__ __forceinline__ void write_roots(const ModelDev& md, uint32_t i, uint32_t step) {
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(md.table);
  for (; i <= md.n_cfg; i += step) {
    if (i == 0u) {
      keys[0] = (unsigned long long)md.n_cfg;  // configuration n_cfg, all else 0
      set_links<1>(md.table, md.mask, 0, kParentRoot, kParentNone);
    } else {
      const uint32_t c = i - 1u;
      keys[i] = (unsigned long long)c |
                (unsigned long long)md.cfgs[c].n << md.L.shift[kFPending];
      set_links<1>(md.table, md.mask, i, 0u, kParentNone);
    }
  }
}

}  // namespace

// ONE: RoundQueue::one (a.self), else the models of the queue.
// 512 threads ask for eight waves per SIMD, so that four workgroups share a CU as with 256 (left
// alone the compiler takes the scalar registers of seven: three workgroups, 219 instead of 210 us
// on matmul128_vw_cu8).
template <int BLOCK, bool GEN, bool ONE>
__global__ __launch_bounds__(BLOCK, BLOCK == 512 ? 8 : 1) void k_rounds(RoundQueue a) {
  extern __shared__ uint32_t set[];  // 1 << log2_set slots
  __shared__ uint8_t masks[256];     // a partial round's closure sets, by size and value
  __shared__ union {
    RoundRecord rec;
    uint32_t words[sizeof(RoundRecord) / 4];
  } s_sums;
  RoundRecord& sums = s_sums.rec;
  __shared__ uint32_t s_piece, s_T, s_skip;
  const uint32_t tid = threadIdx.x;
  // Thread 0: the piece taken.  The first is the workgroup's own number, and no counter is
  // touched where every piece has a workgroup.
  uint32_t next = blockIdx.x;
  if (tid == 0) {
    sums = RoundRecord{};
    sums.t_first = (uint32_t)__builtin_amdgcn_s_memrealtime();
  }
  uint32_t model = kParentNone;  // whose sums are held
  Ctrl* ctrl = nullptr;
  ItemSums sum;
  if (ONE && !a.one.refloor) write_roots(a.one, blockIdx.x * BLOCK + tid, gridDim.x * BLOCK);
  for (;;) {
    if (tid == 0) s_piece = next;
    __syncthreads();  // the piece before is done: its set, its sums
    const uint32_t taken = uniform(s_piece);
    if (taken >= a.n_pieces) break;
    const uint32_t piece = a.reverse ? a.n_pieces - 1u - taken : taken;
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    const RoundPart pt = load_const(a.parts + find_piece(a.parts, a.n_parts, piece));
    const auto get_model = [&] {
      if constexpr (ONE) return a.one;
      else return load_const(a.models + pt.model);
    };
    const ModelDev md = get_model();
    const uint32_t c = pt.cfg_flags & kRpCfg;
    const CfgRec r = load_const(md.cfgs + c);
    if (!ONE && model != pt.model) {
      if (model != kParentNone) {  // (added to again only past the barrier after the clear)
        add_sums(sums, sum);
        __syncthreads();
        flush_sums(ctrl, sums);
      }
      model = pt.model;
      ctrl = md.ctrl;
    }
    const Piece v = piece_of(pt, r, md.L.m, a.piece, piece - pt.piece0);
    if (tid == 0) {
      uint32_t T = md.prune ? md.T : kNoClock;
      if (!ONE && md.bb) {
        const uint32_t b = __hip_atomic_load(&md.ctrl->bound, __ATOMIC_RELAXED, kScopeAgent);
        T = b < T ? b : T;
      }
      // one read of the flag for the whole workgroup: others set it concurrently
      const uint32_t stop = stop_asked(a.abort, a.watch, a.launch, taken, t0);
      if (stop) sums.error = kDevErrAbort;
      s_T = T;
      s_skip = stop;
    }
    {
      uint4* s4 = reinterpret_cast<uint4*>(set);
      for (uint32_t i = tid; i < 1u << (a.log2_set - 2u); i += BLOCK)
        s4[i] = make_uint4(kSetEmpty, kSetEmpty, kSetEmpty, kSetEmpty);
    }
    if (v.partial && v.i1 > v.F)
      for (uint32_t x = tid + 1u; x <= v.all; x += BLOCK)
        masks[mask_rank(x, v.all)] = (uint8_t)x;
    __syncthreads();
    if (tid == 0) {  // taken while this piece is explored
      next = a.n_pieces;
      if (a.n_pieces > gridDim.x)
        next = gridDim.x + (atomicAdd(a.head, 1u) - (ONE ? a.head0 : 0u));
    }
    const uint32_t T = uniform(s_T);
    const bool none =  // every state past T, or below the floor of a continued exploration
        (unsigned long long)(v.r0 + v.q0) * r.d > T ||
        (unsigned long long)(v.r0 + v.q1 + 1u) * r.d < md.refloor;
    sum.last = 0;
    if (!uniform(s_skip) && !none) {
      ItemEnv g;
      g.c = c;
      g.d = r.d;
      g.T = T;
      g.refloor = md.refloor;
      g.rem_bits = 32u - (uint32_t)__clz((int)(r.d + 1u));  // code_rem_bits
      g.sp = md.L.shift[kFPending];
      g.sm = md.L.shift[kFRem];
      g.set_shift = 32u - a.log2_set;
      g.set_mask = (1u << a.log2_set) - 1u;
      g.hkeep = md.hkeep;
      g.keys = (unsigned long long)md.table;
      g.links = g.keys + (md.mask + 1ull) * 8ull;
      const auto items = [&](const auto& ends, auto clocks) {
        if (v.i0 < v.F)
          explore_items<BLOCK, false, decltype(clocks)::value>(
              v, ends, g, v.i0, v.i1 < v.F ? v.i1 : v.F, set, masks, get_model, a.host_tc, sum);
        if (v.i1 > v.F)
          explore_items<BLOCK, true, decltype(clocks)::value>(
              v, ends, g, v.i0 > v.F ? v.i0 : v.F, v.i1, set, masks, get_model, a.host_tc, sum);
      };
      const auto explore = [&](const auto& ends) {
        if (T != kNoClock || md.refloor != 0u) items(ends, std::true_type{});
        else items(ends, std::false_type{});
      };
      if constexpr (GEN) explore(general_ends(r));
      else explore(uniform_ends(r));
    }
    // (without a threshold a partition's deepest state is in its last piece)
    if (sum.last && (v.last || T != kNoClock))
      sum.depth = max(sum.depth, uniform(depth_of(v, sum.last - 1u, masks)));
    // (crowded sets make more probes over a launch than 32 bits count, a piece 2^26 at most)
    if (lane_id() == 0) atomicAdd(&sums.probes, (unsigned long long)sum.probes);
    sum.probes = 0;
    if (tid == 0) {
      sums.rounds += v.q1 - v.q0 + 1u;
      sums.pieces += 1u;
      const uint32_t dt = (uint32_t)(__builtin_amdgcn_s_memrealtime() - t0);
      if (dt > sums.crit) {
        sums.crit = dt;
        sums.crit_cfg = c;
      }
    }
  }
  add_sums(sums, sum);
  __syncthreads();
  if (a.records) {
    if (tid == 0) sums.t_last = (uint32_t)__builtin_amdgcn_s_memrealtime();
    __syncthreads();
    if (tid < sizeof(RoundRecord) / 4u)
      __hip_atomic_store(reinterpret_cast<uint32_t*>(a.records + blockIdx.x) + tid,
                         s_sums.words[tid], __ATOMIC_RELAXED, kScopeSystem);
  } else if (model != kParentNone) {
    flush_sums(ctrl, sums);
  }
}

// Counters, clocks and terminal slots of a model, its root and SELECT states.
__device__ void begin_model(const ModelDev& md) {
  const uint32_t tid = threadIdx.x;
  Ctrl* ctrl = md.ctrl;
  unsigned int* cw = reinterpret_cast<unsigned int*>(ctrl);
  for (uint32_t i = tid; i < sizeof(Ctrl) / 4; i += blockDim.x) cw[i] = 0u;
  __syncthreads();
  if (tid == 0) {
    ctrl->states = ctrl->probes = 1ull + md.n_cfg;
    ctrl->edges = md.n_cfg;
    ctrl->max_depth = 1ull;
    ctrl->levels = 2u;
    ctrl->max_probe = 1u;
    ctrl->bound = md.T;
    ctrl->target_slot = kParentNone;
  }
  for (uint32_t c = tid; c < md.n_cfg; c += blockDim.x) {
    md.tc[c] = kNoClock;
    md.tslot[c] = kParentNone;
  }
  write_roots(md, tid, blockDim.x);
}

__global__ __launch_bounds__(256) void k_rounds_begin(ModelDev md, ModelDev* dst,
                                                      unsigned int* head) {
  if (threadIdx.x == 0) {
    *dst = md;
    *head = 0u;
    if (md.refloor) {  // counters and clocks run on
      md.ctrl->parts_done = 0u;
      md.ctrl->bound = md.T;
      md.ctrl->violated = 0u;
    }
  }
  if (!md.refloor) begin_model(md);
}

__global__ __launch_bounds__(256) void k_rounds_begin_models(const ModelDev* models,
                                                             unsigned int* head) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *head = 0u;
  const ModelDev md = load_const(models + blockIdx.x);
  if (md.tslot) begin_model(md);
}

// ---- counterexample ---------------------------------------------------------------------
//
// The path to a configuration's terminal, terminal first.  A round's end links to the state
// its round starts from, which is the end of the round before: one dependent read of about a
// microsecond per round, made by the first wavefront for up to kPathRounds rounds at a time.
// The rounds' leaves are then read side by side (they name the units each round started), and
// all threads write the states: a round's run from its last state back, then its dispatches,
// the last of the units in index order first.  Every end and leaf read has to be the state the
// round structure gives, or the path is bad.  The keys go straight to pinned memory, so that
// the host waits once.  mc_trace, by way of the general chase -> here: 55 -> 17 us on
// reduction_g256_cu2, 73 -> 29 us on matmul64_cu4, 75 -> 45 us on matmul128_vw_cu8 (2,834
// states, of which decoding them on the host takes about 15).
constexpr uint32_t kPathRounds = 256, kPathBlock = 512;

template <bool GEN>
__global__ __launch_bounds__(kPathBlock) void k_round_path(QueryArgs a, const uint32_t* tslot,
                                                           uint32_t c, TraceOut t) {
  __shared__ uint32_t end[kPathRounds], leaf[kPathRounds];
  __shared__ uint8_t units[kPathRounds];
  __shared__ uint32_t s_count, s_at, s_bad;
  const uint32_t tid = threadIdx.x, m = a.L.m, all = (1u << m) - 1u;
  const CfgRec r = load_const(a.cfgs + c);
  const unsigned long long* keys = reinterpret_cast<const unsigned long long*>(a.table);
  const uint32_t sp = a.L.shift[kFPending], sm = a.L.shift[kFRem], sr = a.L.shift[kFRem + 1];
  const uint32_t target = tslot[c];
  const uint32_t rounds = (r.n + m - 1u) / m, last = r.n - (rounds - 1u) * m;  // units of the last
  const uint32_t per = r.b + m;
  uint32_t n = 0;            // states written
  uint32_t left = rounds;    // rounds before the ones written
  if (tid == 0) {
    s_at = target;
    s_bad = target == kParentNone || target > a.mask ? 1u : 0u;
  }
  __syncthreads();
  const auto put = [&](uint32_t i, unsigned long long key) {
    if (i >= t.cap) return;
    if (i < t.host_words) t.host[i] = key;
    else t.out[i] = key;
  };
  const auto run = [&](const auto& ends) {
    while (left && !s_bad) {
      const uint32_t take = left < kPathRounds ? left : kPathRounds;
      if (tid < 64u) {
        uint32_t at = s_at, k = 0;
        while (k < take && at <= a.mask) {
          const uint2 l = *reinterpret_cast<const uint2*>(slot_parent<1>(a.table, a.mask, at));
          if (tid == 0) {
            end[k] = at;
            leaf[k] = l.y;
          }
          at = l.x;
          // the end of a run slice knows its leaf only, which links to the round's start
          if (at == kParentNone && l.y <= a.mask) at = *slot_parent<1>(a.table, a.mask, l.y);
          ++k;
        }
        if (tid == 0) {
          s_at = at;
          s_count = k;
        }
      }
      __syncthreads();
      if (s_count < take && tid == 0) s_bad = 1u;
      for (uint32_t k = tid; k < s_count; k += kPathBlock) {
        const uint32_t round = left - 1u - k, started = round + 1u == rounds ? last : m;
        const uint32_t pend = r.n - round * m - started;
        const unsigned long long want = (unsigned long long)c | (unsigned long long)pend << sp;
        uint32_t mask = 0;
        bool ok = keys[end[k]] == want && leaf[k] <= a.mask;
        if (ok) {
          const unsigned long long lk = keys[leaf[k]];
          mask = (uint32_t)(lk >> sm) & all;
          ok = lk == (want | (unsigned long long)mask << sm | (unsigned long long)r.d << sr) &&
               bits_set(mask) == started;
        }
        units[k] = (uint8_t)mask;
        if (!ok) s_bad = 1u;
      }
      __syncthreads();
      if (s_bad) break;
      const uint32_t first = left == rounds ? r.b + last : per;  // states of the chunk's last round
      const uint32_t rows = first + (take - 1u) * per;
      for (uint32_t i = tid; i < rows; i += kPathBlock) {
        const uint32_t k = i < first ? 0u : 1u + (i - first) / per;
        const uint32_t off = i < first ? i : (i - first) - (k - 1u) * per;
        const uint32_t round = left - 1u - k, started = round + 1u == rounds ? last : m;
        uint32_t mask = units[k], rem = r.d;
        if (off < r.b) {
          rem = rem_after(ends, r.b - 1u - off);
        } else {  // the first of the leaf's units, fewer and fewer of them
          for (uint32_t drop = off - r.b; drop; --drop) mask &= ~(1u << (31 - __clz((int)mask)));
        }
        const uint32_t pend = r.n - round * m - (off < r.b ? started : bits_set(mask));
        put(n + i, (unsigned long long)c | (unsigned long long)pend << sp |
                       (unsigned long long)(rem ? mask : 0u) << sm | (unsigned long long)rem << sr);
      }
      n += rows;
      left -= take;
      __syncthreads();
    }
  };
  if constexpr (GEN) run(general_ends(r));
  else run(uniform_ends(r));
  if (tid == 0) {
    // the SELECT state and the root
    const bool bad = s_bad || s_at != 1u + c || n + 2u > t.cap;
    put(n, (unsigned long long)c | (unsigned long long)r.n << sp);
    put(n + 1u, (unsigned long long)a.n_cfg);
    n += 2u;
    a.ctrl->trace_len = n;
    a.ctrl->target_slot = target;
    if (bad && target != kParentNone) set_error(a.ctrl, kDevErrTrace);
    if (t.host_res) {
      t.host_res[0] = target;
      t.host_res[1] = n;
      t.host_res[2] = bad ? 1u : 0u;
    }
  }
}

// Staged descriptors: block (0, y) begins model y, every block clears a share of its slots
// but for the root's and the SELECT states', which block (0, y) writes.
__global__ __launch_bounds__(256) void k_rounds_begin_staged(const ModelDev* staged,
                                                             ModelDev* models) {
  __shared__ union {
    ModelDev md;
    uint32_t words[sizeof(ModelDev) / 4];
  } s;
  const uint32_t* from = reinterpret_cast<const uint32_t*>(staged + blockIdx.y);
  if (threadIdx.x < sizeof(ModelDev) / 4)
    s.words[threadIdx.x] =
        __hip_atomic_load(from + threadIdx.x, __ATOMIC_RELAXED, kScopeSystem);
  __syncthreads();
  const ModelDev& md = s.md;
  if (blockIdx.x == 0) {
    if (threadIdx.x < sizeof(ModelDev) / 4)
      reinterpret_cast<uint32_t*>(models + md.index)[threadIdx.x] = s.words[threadIdx.x];
    if (md.refloor) {
      if (threadIdx.x == 0) {  // counters and clocks run on
        md.ctrl->parts_done = 0u;
        md.ctrl->bound = md.T;
        md.ctrl->violated = 0u;
      }
    } else {
      begin_model(md);
    }
  }
  if (md.refloor) return;
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(md.table);
  for (uint32_t i = 1u + md.n_cfg + blockIdx.x * 256u + threadIdx.x; i < md.used;
       i += gridDim.x * 256u)
    keys[i] = kEmptyWord;
}

// ---- launch helpers (host) ------------------------------------------------------------

hipError_t launch_rounds_begin(hipStream_t st, const ModelDev& md, ModelDev* dst,
                               unsigned int* head) {
  hipLaunchKernelGGL(k_rounds_begin, dim3(1), dim3(256), 0, st, md, dst, head);
  return hipGetLastError();
}

hipError_t launch_rounds_begin_models(hipStream_t st, const ModelDev* models, uint32_t n,
                                      unsigned int* head) {
  hipLaunchKernelGGL(k_rounds_begin_models, dim3(n), dim3(256), 0, st, models, head);
  return hipGetLastError();
}

hipError_t launch_rounds_begin_staged(hipStream_t st, const ModelDev* staged, uint32_t n,
                                      ModelDev* models) {
  static_assert(sizeof(ModelDev) / 4 <= 256, "one thread per word");
  hipLaunchKernelGGL(k_rounds_begin_staged, dim3(64, n), dim3(256), 0, st, staged, models);
  return hipGetLastError();
}

hipError_t launch_round_path(hipStream_t st, const QueryArgs& q, const uint32_t* tslot,
                             uint32_t target, const TraceOut& t, bool general) {
  const dim3 one(1), block(kPathBlock);
  if (general) hipLaunchKernelGGL(k_round_path<true>, one, block, 0, st, q, tslot, target, t);
  else hipLaunchKernelGGL(k_round_path<false>, one, block, 0, st, q, tslot, target, t);
  return hipGetLastError();
}

hipError_t launch_rounds(hipStream_t st, uint32_t grid, uint32_t block, const RoundQueue& q,
                         bool general) {
  const uint32_t lds = 4u << q.log2_set;
#define MC_LAUNCH_ROUNDS_(B, G)                                                                \
  do {                                                                                         \
    if (q.self) hipLaunchKernelGGL((k_rounds<B, G, true>), dim3(grid), dim3(B), lds, st, q); \
    else hipLaunchKernelGGL((k_rounds<B, G, false>), dim3(grid), dim3(B), lds, st, q);         \
  } while (0)
#define MC_LAUNCH_ROUNDS(B)                 \
  do {                                      \
    if (general) MC_LAUNCH_ROUNDS_(B, true); \
    else MC_LAUNCH_ROUNDS_(B, false);       \
  } while (0)
  if (block == 1024) MC_LAUNCH_ROUNDS(1024);
  else if (block == 512) MC_LAUNCH_ROUNDS(512);
  else MC_LAUNCH_ROUNDS(256);
#undef MC_LAUNCH_ROUNDS
#undef MC_LAUNCH_ROUNDS_
  return hipGetLastError();
}

}  // namespace mc
