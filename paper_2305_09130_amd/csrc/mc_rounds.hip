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
// most kMaxPiece generated states), tests each in an open-addressing hash set in LDS and
// writes the new ones to the partition's own slots of the visited set in HBM, consecutive
// states to consecutive slots.  The set is exact: it holds the state's (pending, mask, time
// left), which is all of a state that varies within a piece, in 32 bits.
//
// What bounds it.  k_superstep, which explored these models before, makes one device-scope
// compare-and-swap per state on a random line of a table in HBM, at the chip's limit for
// those (17 G/s); here a state costs a compare-and-swap in LDS, 8 bytes of a coalesced store
// and about 100 vector instructions, which bound it.  min_time launch, k_superstep and its
// table's clear -> here: matmul128_vw_cu8 (58.0M states) 3.89 + 0.38 -> 0.29 ms (200 G
// states/s, 1.6 TB/s of keys written), matmul64_cu4 (5.15M) 0.44 -> 0.056 ms,
// abstract_s1024_np4_cu1 0.23 -> 0.026 ms, reduction_g256_cu2 (81k) 45 -> 6 us.
//
// A workgroup has 256 threads and up to 33 KiB of LDS, so that four share a CU: one's lookups
// and barriers between pieces overlap another's items.  Pieces of half the size ran slower
// (matmul128_vw_cu8 0.40 -> 0.47 ms when measured): a piece costs about 3 us beyond its items.
//
// Sums go to the host as one 96-byte record per workgroup, stored to pinned memory: added to
// the model's counters instead, ten atomics of 1,024 workgroups on one line took 60 us.
#include <hip/hip_runtime.h>

#include "mc_launch.h"
#include "mc_rounds.h"

namespace mc {

namespace {

constexpr uint32_t kSetEmpty = 0xFFFFFFFFu;

// Pointers read from a descriptor carry no address space, and a store through such a pointer
// counts as an LDS access too: the next wait for the set would wait for HBM.
typedef __attribute__((address_space(1))) unsigned long long global_u64;

// Uniform loads of a launch's constant tables, as scalar loads.
template <class T>
__device__ __forceinline__ T load_const(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  typedef const __attribute__((address_space(4))) uint32_t* cptr;
  cptr c = (cptr)(uintptr_t)p;
  union {
    T v;
    uint32_t w[sizeof(T) / 4];
  } u;
#pragma unroll
  for (uint32_t i = 0; i < sizeof(T) / 4; ++i) u.w[i] = c[i];
  return u.v;
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// The partition that holds piece p: the last whose first piece is at most p.  The wavefront
// looks at 64 partitions at a time (3,828 partitions: two steps).
__device__ __forceinline__ uint32_t find_part(const RoundPart* parts, uint32_t n, uint32_t p) {
  uint32_t lo = 0, len = n;
  while (len > 1u) {
    const uint32_t step = (len + 63u) / 64u, at = lane_id() * step;
    const bool le = at < len && parts[lo + at].piece0 <= p;
    const uint32_t c = (uint32_t)__popcll(__ballot(le));  // at least one: parts[lo]
    const uint32_t skip = (c - 1u) * step;
    lo += skip;
    len = step < len - skip ? step : len - skip;
  }
  return uniform(lo);
}

// A workgroup's sums, added to its model's counters: for launches over several models, when
// a piece of another model comes or the launch ends.
__device__ __forceinline__ void flush_sums(Ctrl* ctrl, RoundRecord& s) {
  if (threadIdx.x != 0) return;
  if (s.states) atomicAdd(&ctrl->states, s.states);
  if (s.terms) atomicAdd(&ctrl->terminals, s.terms);
  if (s.edges) atomicAdd(&ctrl->edges, s.edges);
  if (s.dups) atomicAdd(&ctrl->dups, s.dups);
  if (s.probes) atomicAdd(&ctrl->probes, s.probes);
  if (s.chunks) atomicAdd(&ctrl->chunks, s.chunks);
  if (s.rounds) atomicAdd(&ctrl->supersteps, s.rounds);
  if (s.pieces) atomicAdd(&ctrl->parts_done, s.pieces);
  if (s.depth) atomicMax(&ctrl->max_depth, (unsigned long long)s.depth);
  if (s.max_probe) atomicMax(&ctrl->max_probe, s.max_probe);
  if (s.crit > atomicMax(&ctrl->crit_ticks, (unsigned long long)s.crit))
    ctrl->crit_part = s.crit_cfg;
  s = RoundRecord{};
}

// What the items of a piece need of its model, configuration and query.
struct ItemEnv {
  uint32_t c, T, refloor, rb, sp, sm, sr, log2_set, hkeep;
  unsigned long long keys, links;  // addresses of the set's two regions
};

// Sums of one wavefront over a piece (states .. terms: the same in every lane).
struct ItemSums {
  uint32_t states = 0, edges = 0, terms = 0, chunks = 0;
  uint32_t probes = 0, max_probe = 0, depth = 0;  // per lane
};

// Items [from, to) of a piece: of its full rounds, or (PART) of its partial round.  Two loops,
// as the fields of one round kind fill the scalar registers.
template <int BLOCK, bool GEN, bool PART>
__device__ __forceinline__ void explore_items(const Piece& v, const CfgRec& r, const ItemEnv& g,
                                              uint32_t from, uint32_t to, uint32_t* set,
                                              const uint8_t* masks, const ModelDev* mdp,
                                              uint32_t* host_tc, ItemSums& sum) {
  const uint32_t set_mask = (1u << g.log2_set) - 1u;
  for (uint32_t base = from; base < to; base += BLOCK) {
    const uint32_t i = base + threadIdx.x;
    ++sum.chunks;
    const RoundItem it = PART ? part_item(v, i, masks) : full_item(v, i);
    const uint32_t e = it.is_cl ? 0u : (GEN ? end_at(r, it.j) : end_at_uniform(r, it.j));
    const uint32_t rem = r.d - e, clock = it.round * r.d + e, ns = bits_set(it.mask);
    const uint32_t pending = r.n - it.round * v.m - ns, busy = rem ? it.mask : 0u;
    const bool act = i < to && clock <= g.T;
    // the set: exact on (pending, busy, rem).  It has twice the slots of the piece's states,
    // so the probe sequence (linear: codes of a run spread evenly under this multiplier) ends
    const uint32_t code = state_code(v, pending, busy, rem, g.rb);
    uint32_t h = code * 0x9E3779B1u;
    if (g.hkeep) h = ((h >> 8) & ((1u << g.hkeep) - 1u)) * 0x9E3779B1u;
    uint32_t at = h >> (32u - g.log2_set), old = 0u, tries = 0;
    if (act) {
      do {
        old = atomicCAS(&set[at], kSetEmpty, code);
        at = (at + 1u) & set_mask;
        ++tries;
      } while (old != kSetEmpty && old != code && tries <= set_mask);
    }
    bool fresh = act && old == kSetEmpty;
    sum.probes += tries;
    sum.max_probe = tries > sum.max_probe ? tries : sum.max_probe;
    const unsigned long long key = (unsigned long long)g.c | (unsigned long long)pending << g.sp |
                                   (unsigned long long)busy << g.sm |
                                   (unsigned long long)rem << g.sr;
    global_u64* kp = (global_u64*)g.keys + it.slot;
    // a continued exploration finds the states below its floor in their slots
    if (clock < g.refloor && fresh) fresh = *kp != key;
    if (fresh) {
      *kp = key;
      const uint32_t dep = 1u + it.round * (v.m + r.b) + ns + (it.is_cl ? 0u : it.j + 1u);
      sum.depth = dep > sum.depth ? dep : sum.depth;
      // links, as the counterexample reads them: a dispatch leaf to its round's start, a
      // round's end to the leaf its run starts from (parent and jump)
      if (rem == 0u || it.is_leaf) {
        const unsigned long long lo = rem ? it.root : it.leaf, hi = rem ? kParentNone : it.leaf;
        ((global_u64*)g.links)[it.slot] = lo | hi << 32;
      }
    }
    const bool term = fresh && rem == 0u && pending == 0u;
    if (term) {
      const ModelDev md = load_const(mdp);
      md.tslot[g.c] = it.slot;
      // (a configuration has one terminal)
      if (host_tc) __hip_atomic_store(host_tc + g.c, clock, __ATOMIC_RELAXED, kScopeSystem);
      else atomicMin(&md.tc[g.c], clock);
      if (md.prune) md.ctrl->violated = 1u;
      if (md.bb) atomicMin(&md.ctrl->bound, clock);
    }
    sum.edges += (uint32_t)__popcll(__ballot(act));
    sum.states += (uint32_t)__popcll(__ballot(fresh));
    sum.terms += (uint32_t)__popcll(__ballot(term));
  }
}

}  // namespace

template <int BLOCK, bool GEN>
__global__ __launch_bounds__(BLOCK) void k_rounds(RoundQueue a) {
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
    sums.t_first = __builtin_amdgcn_s_memrealtime();
  }
  uint32_t model = kParentNone;  // whose sums are held
  Ctrl* ctrl = nullptr;
  for (;;) {
    if (tid == 0) s_piece = next;
    __syncthreads();  // the piece before is done: its set, its sums
    const uint32_t taken = uniform(s_piece);
    if (taken >= a.n_pieces) break;
    const uint32_t piece = a.reverse ? a.n_pieces - 1u - taken : taken;
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    const RoundPart pt = load_const(a.parts + find_part(a.parts, a.n_parts, piece));
    const ModelDev md = load_const(a.models + pt.model);
    const uint32_t c = pt.cfg_flags & kRpCfg;
    const CfgRec r = load_const(md.cfgs + c);
    if (model != pt.model) {  // the sums are added to again only past the next barrier
      if (model != kParentNone) flush_sums(ctrl, sums);
      model = pt.model;
      ctrl = md.ctrl;
    }
    const Piece v = piece_of(pt, r, md.L.m, a.piece, piece - pt.piece0);
    if (tid == 0) {
      uint32_t T = md.prune ? md.T : kNoClock;
      if (md.bb) {
        const uint32_t b = __hip_atomic_load(&md.ctrl->bound, __ATOMIC_RELAXED, kScopeAgent);
        T = b < T ? b : T;
      }
      const uint32_t stop = abort_asked(a.abort, taken);
      if (stop) {
        set_error(md.ctrl, kDevErrAbort);
        sums.error = kDevErrAbort;
      }
      s_T = T;
      // one read of the error flag for the whole workgroup: others set it concurrently
      s_skip = stop | __hip_atomic_load(&md.ctrl->error, __ATOMIC_RELAXED, kScopeAgent);
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
      next = a.n_pieces > gridDim.x ? gridDim.x + atomicAdd(a.head, 1u) : a.n_pieces;
    }
    const uint32_t T = uniform(s_T);
    const bool none =  // every state past T, or below the floor of a continued exploration
        (unsigned long long)(v.r0 + v.q0) * r.d > T ||
        (unsigned long long)(v.r0 + v.q1 + 1u) * r.d < md.refloor;
    ItemSums sum;
    if (!uniform(s_skip) && !none) {
      ItemEnv g;
      g.c = c;
      g.T = T;
      g.refloor = md.refloor;
      g.rb = 32u - (uint32_t)__clz((int)(r.d + 1u));  // code_rem_bits
      g.sp = md.L.shift[kFPending];
      g.sm = md.L.shift[kFRem];
      g.sr = md.L.shift[kFRem + 1];
      g.log2_set = a.log2_set;
      g.hkeep = md.hkeep;
      g.keys = (unsigned long long)md.table;
      g.links = g.keys + (md.mask + 1ull) * 8ull;
      const ModelDev* mdp = a.models + pt.model;
      if (v.i0 < v.F)
        explore_items<BLOCK, GEN, false>(v, r, g, v.i0, v.i1 < v.F ? v.i1 : v.F, set, masks, mdp,
                                         a.host_tc, sum);
      if (v.i1 > v.F)
        explore_items<BLOCK, GEN, true>(v, r, g, v.i0 > v.F ? v.i0 : v.F, v.i1, set, masks, mdp,
                                        a.host_tc, sum);
    }
    const unsigned long long w_probes = wave_sum(sum.probes);
    const uint32_t w_max = (uint32_t)wave_max(sum.max_probe), w_depth = (uint32_t)wave_max(sum.depth);
    if (lane_id() == 0) {
      atomicAdd(&sums.states, (unsigned long long)sum.states);
      atomicAdd(&sums.edges, (unsigned long long)sum.edges);
      if (sum.edges != sum.states)
        atomicAdd(&sums.dups, (unsigned long long)(sum.edges - sum.states));
      if (sum.terms) atomicAdd(&sums.terms, (unsigned long long)sum.terms);
      atomicAdd(&sums.probes, w_probes);
      atomicMax(&sums.max_probe, w_max);
      atomicMax(&sums.depth, w_depth);
    }
    if (tid == 0) {
      sums.chunks += sum.chunks;
      sums.rounds += v.q1 - v.q0 + 1u;
      sums.pieces += 1u;
      const uint32_t dt = (uint32_t)(__builtin_amdgcn_s_memrealtime() - t0);
      if (dt > sums.crit) {
        sums.crit = dt;
        sums.crit_cfg = c;
      }
    }
  }
  if (a.records) {
    if (tid == 0) sums.t_last = __builtin_amdgcn_s_memrealtime();
    __syncthreads();
    if (tid < sizeof(RoundRecord) / 4u)
      __hip_atomic_store(reinterpret_cast<uint32_t*>(a.records + blockIdx.x) + tid,
                         s_sums.words[tid], __ATOMIC_RELAXED, kScopeSystem);
  } else if (model != kParentNone) {
    flush_sums(ctrl, sums);
  }
}

// Counters, clocks and terminal slots of a model, its root (slot 0) and SELECT states (slot
// 1 + c).
__device__ void begin_model(const ModelDev& md) {
  const uint32_t tid = threadIdx.x;
  Ctrl* ctrl = md.ctrl;
  unsigned int* cw = reinterpret_cast<unsigned int*>(ctrl);
  for (uint32_t i = tid; i < sizeof(Ctrl) / 4; i += blockDim.x) cw[i] = 0u;
  __syncthreads();
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(md.table);
  if (tid == 0) {
    ctrl->states = ctrl->probes = 1ull + md.n_cfg;
    ctrl->edges = md.n_cfg;
    ctrl->max_depth = 1ull;
    ctrl->levels = 2u;
    ctrl->max_probe = 1u;
    ctrl->bound = md.T;
    ctrl->target_slot = kParentNone;
    keys[0] = (unsigned long long)md.n_cfg;  // the root: configuration n_cfg, all else 0
    set_links<1>(md.table, md.mask, 0, kParentRoot, kParentNone);
  }
  for (uint32_t c = tid; c < md.n_cfg; c += blockDim.x) {
    md.tc[c] = kNoClock;
    md.tslot[c] = kParentNone;
    keys[1u + c] = (unsigned long long)c | (unsigned long long)md.cfgs[c].n << md.L.shift[kFPending];
    set_links<1>(md.table, md.mask, 1u + c, 0u, kParentNone);
  }
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

hipError_t launch_rounds(hipStream_t st, uint32_t grid, uint32_t block, const RoundQueue& q,
                         bool general) {
  const uint32_t lds = 4u << q.log2_set;
#define MC_LAUNCH_ROUNDS(B)                                                                  \
  do {                                                                                       \
    if (general) hipLaunchKernelGGL((k_rounds<B, true>), dim3(grid), dim3(B), lds, st, q);   \
    else hipLaunchKernelGGL((k_rounds<B, false>), dim3(grid), dim3(B), lds, st, q);          \
  } while (0)
  if (block == 1024) MC_LAUNCH_ROUNDS(1024);
  else if (block == 512) MC_LAUNCH_ROUNDS(512);
  else MC_LAUNCH_ROUNDS(256);
#undef MC_LAUNCH_ROUNDS
  return hipGetLastError();
}

}  // namespace mc
