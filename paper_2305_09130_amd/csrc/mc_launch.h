// mc_launch.h -- host-side launch helpers of the exploration kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "mc_device.h"

namespace mc {

constexpr uint32_t kLevelBlock = 128;

struct QueryArgs {
  Ctrl* ctrl;
  uint32_t* tc;             // per-configuration least terminal clock
  const CfgRec* cfgs;
  unsigned char* table;
  unsigned long long mask;  // slots - 1
  Layout L;
  uint32_t n_cfg;
  uint32_t prune;           // check(T): drop states with clock > T
  uint32_t T;
  uint32_t max_clock;       // bound of the packed clock field
  uint32_t hkeep;           // bits of the key hash kept (0 = all; testing only)
};

// Whether work on the stream would be recorded into a graph instead of run (or, of a stream in
// an unknown state, might be).  Calls that prepare or wait for work are refused on such a stream.
inline bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

// Where a counterexample's keys go, terminal first: at most cap of them to `out` (device),
// the first host_words words of them to `host` instead (pinned memory, or null with 0 words);
// the target's slot, the path's length and whether it is bad go to host_res[0..2] if given.
struct TraceOut {
  unsigned long long* out;
  uint32_t cap;
  uint32_t host_words = 0;
  unsigned long long* host = nullptr;
  uint32_t* host_res = nullptr;
};

// Keys each thread of the persistent kernel inserts per round trip: 1 or 2 as asked,
// else (0) 2 for keys of one or two words and 1 for four-word keys, whose two-key
// kernel needs more registers than three wavefronts per SIMD allow.
inline uint32_t lane_items_for(uint32_t asked, uint32_t W) {
  return asked == 1u || asked == 2u ? asked : (W == 4u ? 1u : 2u);
}

// Library error code (MC_E_*) of a device error flag (kDevErr*).
inline int dev_error_code(unsigned int e) {
  switch (e) {
    case 0: return MC_OK;
    case kDevErrTableFull: return MC_E_TABLE_FULL;
    case kDevErrOverflow: return MC_E_OVERFLOW;
    case kDevErrSplit: return MC_E_INTERNAL;
    case kDevErrAbort: return MC_E_ABORTED;
    default: return MC_E_DEVICE;
  }
}

struct LevelArgs {
  QueryArgs q;
  uint32_t in_idx, out_idx, clr_idx;  // rotating frontier counters
  uint32_t fcap;
  const unsigned int* abort;  // host-set stop request (pinned host word), or null
};

// Saved frontier of a partition explored across several launches.
struct PartState {
  unsigned long long k[4];
  uint32_t slot, depth;
  uint32_t status;  // 0 not started, 1 in progress (one saved frontier state), 2 done
  uint32_t pad;
};
static_assert(sizeof(PartState) == 48, "PartState layout");

// One model of a persistent launch (device memory, written by the host).
struct ModelDev {
  Ctrl* ctrl;
  uint32_t* tc;
  const CfgRec* cfgs;
  Seed* seeds;
  unsigned char* table;
  unsigned long long mask;  // slots - 1
  Layout L;
  uint32_t n_cfg;
  uint32_t prune;
  uint32_t T;
  uint32_t max_clock;
  uint32_t n_parts;   // partitions of the model (entries of pstate)
  uint32_t bb;        // branch and bound: prune at min(T, ctrl->bound), every new
                      // terminal lowers ctrl->bound
  PartState* pstate;  // one per partition when partitions may yield, else null
  uint32_t hkeep;     // bits of the key hash kept (0 = all; testing only)
  uint32_t refloor;   // a continued exploration: every state with clock < refloor was
                      // inserted before, and one found again is still expanded, so the
                      // walk reaches the new states past it (0 = a fresh exploration)
  uint32_t* tslot;    // round engine: slot of each configuration's terminal (else null:
                      // the model is not explored by the round engine)
  uint32_t index;     // round engine, staged descriptors: its place in the models' array
  uint32_t used;      // ... and the slots of its plan, cleared before a fresh exploration
};

// One partition of a persistent launch: rounds [r0, r1) of one configuration's subgraph
// (r1 = kRoundsToEnd: through its terminal).  After r full rounds the subgraph of a
// configuration passes through the single state (c, r*d, n - r*m, every unit idle), so a
// block of whole rounds can be explored from that state on its own.
struct Part {
  uint32_t model, cfg, r0, r1;  // r0 = r1 = kRunSlice: a run slice [j0, j1)
  uint32_t pidx;  // index of the partition within its model (its PartState)
  uint32_t j0, j1;  // a run slice's states; else j1 > 0 caps the runs from SELECT
  uint32_t pad;
};
static_assert(sizeof(Part) == 32, "Part layout");

// Partitions of a persistent launch, largest first.
struct PartQueue {
  const ModelDev* models;
  const Part* parts;
  uint32_t n_parts;
  uint32_t batch_items;  // states generated per super-step batch before waiting (target)
  unsigned int* head;
  uint32_t slice;        // super-step levels per partition before it yields (0 = no limit)
  uint32_t reverse;      // take the partitions smallest first
  Part* yielded;         // partitions that yielded, for the next launch
  unsigned int* n_yielded;
  // host-set stop request (a pinned host word read at system scope), or null: a
  // partition taken after it is set is not explored, so the launch drains quickly and
  // every workgroup still exits normally (with it: where the launch notes its looks at the
  // word, and the number, not 0, that tells its notes from those of other launches there)
  const unsigned int* abort;
  unsigned long long* watch;
  uint32_t launch;
};

// Place of the watch word (stop_asked): the last of the 256 bytes that a handle's device
// descriptor has in its workspace.  Every workgroup reads it for every piece, so not on the line
// of the queue's head, for whose atomics the reads waited (matmul128_vw_cu8, 14,300 pieces, 0.22
// -> 0.95 ms).
constexpr size_t kWatchOff = 256 - 8;
static_assert(sizeof(ModelDev) <= kWatchOff, "the descriptor and the watch word");

// A launch of the round engine.
struct RoundQueue {
  const ModelDev* models;
  const RoundPart* parts;
  uint32_t n_parts, n_pieces;
  uint32_t piece;       // items per piece
  uint32_t log2_set;    // slots of a piece's hash set: set_log2(piece)
  uint32_t reverse;     // take the pieces last first
  unsigned int* head;
  const unsigned int* abort;  // as PartQueue
  // One model, a handle with pinned memory: every workgroup stores its sums here (grid
  // records in host memory) and every terminal its clock in host_tc; else null, and the
  // sums are added to the models' counters and the clocks to ModelDev::tc.
  struct RoundRecord* records;
  uint32_t* host_tc;
  // With records, and no incumbent to share: the launch begins the model itself (self), by its
  // descriptor; head0 is the count that head stands at.
  uint32_t self;
  uint32_t head0;
  ModelDev one;
  // with abort: as PartQueue
  unsigned long long* watch;
  uint32_t launch;
};
// One workgroup's sums over a launch (its pieces of one model, where counters are device's):
// a line of the host's cache.  A set has at most 2^31 slots, so that the counts of items and
// states fit in 32 bits.
struct RoundRecord {
  uint32_t states, terms, edges;
  uint32_t chunks, rounds, pieces;
  unsigned long long probes;
  uint32_t depth, max_probe;
  uint32_t crit, crit_cfg;  // its longest piece, in ticks
  uint32_t t_first, t_last; // device clock (100 MHz, its low bits): its first piece, its end
  uint32_t error;
  uint32_t pad;
};
static_assert(sizeof(RoundRecord) == 64, "RoundRecord layout");
// Least log2 of the slots of a hash set for pieces of `piece` items: twice as many slots, 512 at
// least.  A partition's last piece can hold kMaxEndGroup more, the last states of a partial
// round's runs; it leaves slots free even so, and on a free one every probe sequence ends.
constexpr uint32_t kMaxEndGroup = 70;  // choices of 4 units of 8
static_assert(256 + kMaxEndGroup < 512 && kMaxPiece >= 256, "auto_piece gives 256 at least");
inline uint32_t set_log2(uint32_t piece) {
  uint32_t l = 9;
  while ((1u << l) < 2u * piece) ++l;
  return l;
}
// Threads per workgroup for pieces of `piece` items, where the caller leaves them open: 512 take
// a large piece in half the turns, with the same set for twice the wavefronts (min_time launch,
// 256 -> 512: matmul64_cu4 38 -> 29 us, abstract_s1024_np4_cu4 25.3 -> 21.8,
// matmul128_vw_cu8 219 -> 210); a small one is over in a few turns, and its barriers cost more
// (checks of 256 items: 6.3 -> 8.2 us on matmul64_cu4; reduction_g256_cu2 5.3 -> 6.4).
inline uint32_t rounds_block(uint32_t piece) { return piece >= 1024u ? 512u : 256u; }
// Counters, clocks, root and SELECT states of one model (its descriptor is written to
// dst), or of every model of a queue that the round engine explores.
hipError_t launch_rounds_begin(hipStream_t st, const ModelDev& md, ModelDev* dst,
                               unsigned int* head);
hipError_t launch_rounds_begin_models(hipStream_t st, const ModelDev* models, uint32_t n,
                                      unsigned int* head);
// The same for models whose descriptors the host staged (pinned memory) for a round engine
// that continues or starts them: each is written to models[index]; the slots of those that
// start (refloor 0) are cleared, so that a scan of the set finds only states.
hipError_t launch_rounds_begin_staged(hipStream_t st, const ModelDev* staged, uint32_t n,
                                      ModelDev* models);
// The counterexample of configuration `target` after a query on the round engine; tslot: the
// slot of each configuration's terminal.
hipError_t launch_round_path(hipStream_t st, const QueryArgs& q, const uint32_t* tslot,
                             uint32_t target, const TraceOut& t, bool general);
// general: some configuration has waves or two-operation periods.
hipError_t launch_rounds(hipStream_t st, uint32_t grid, uint32_t block, const RoundQueue& q,
                         bool general);

// A launch of the chain engine (one model, a handle with pinned memory).
struct ChainArgs {
  QueryArgs q;
  const uint32_t* blob;       // ChainPlan::blob
  uint32_t lcm, tails_at, sets_at;
  uint32_t n_pieces;
  uint32_t bb;                // as ModelDev::bb
  uint32_t uniform;           // ChainPlan::uniform
  unsigned int* head;
  uint32_t head0;             // as RoundQueue
  const unsigned int* abort;  // as PartQueue
  unsigned long long* watch;
  uint32_t launch;
  RoundRecord* records;       // a record per workgroup, in pinned memory
  uint32_t target;            // launch_chain_path: the configuration
  uint32_t* words;            // per piece, in pinned memory: the steps it adds to the longest
                              // path, in bit 31 whether it holds a terminal
};
hipError_t launch_chains(hipStream_t st, uint32_t W, uint32_t grid, const ChainArgs& a);
// The counterexample of configuration a.target that ends at clock q.T, root first, by `grid`
// workgroups: `per` chain pieces each, the tail the last.  base: the place of the first state of
// each (device-readable); the caller clears t.host_res[2].
hipError_t launch_chain_path(hipStream_t st, uint32_t W, const ChainArgs& a, const TraceOut& t,
                             uint32_t grid, const uint32_t* base, uint32_t per);

template <int W>
hipError_t launch_seed(hipStream_t st, const QueryArgs& q, Seed* seeds, void* front0);
template <int W>
hipError_t launch_level(hipStream_t st, uint32_t grid, const LevelArgs& la, const void* fin,
                        void* fout);
// All models of the queue have key width W (1, 2, 4).  items: keys per lane per insert
// round trip, as for lane_items_for.  general: some configuration of some model of the
// queue has waves or two-operation periods (ModelHost::general); false selects the
// engine built for uniform phases only.  hetero: some model runs on units of unequal
// speed (ModelHost::hetero), which selects the build with determined ADVANCE chains.
hipError_t launch_super(hipStream_t st, uint32_t W, uint32_t grid, uint32_t block,
                        uint32_t items, const PartQueue& pq, bool general, bool hetero);

// Runs up to three launches (one per key width) concurrently on sub-streams forked from
// and joined back into a main stream with events; usable inside stream capture.
struct Fork {
  hipStream_t sub[3] = {nullptr, nullptr, nullptr};
  hipEvent_t fork = nullptr;
  hipEvent_t join[3] = {nullptr, nullptr, nullptr};
  hipError_t create() {
    hipError_t e = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
    for (int i = 0; i < 3 && e == hipSuccess; ++i) {
      e = hipStreamCreateWithFlags(&sub[i], hipStreamNonBlocking);
      if (e == hipSuccess) e = hipEventCreateWithFlags(&join[i], hipEventDisableTiming);
    }
    return e;
  }
  void destroy() {
    for (int i = 0; i < 3; ++i) {
      if (sub[i]) (void)hipStreamDestroy(sub[i]);
      if (join[i]) (void)hipEventDestroy(join[i]);
      sub[i] = nullptr;
      join[i] = nullptr;
    }
    if (fork) (void)hipEventDestroy(fork);
    fork = nullptr;
  }
};

// queue[w] (w = 0, 1, 2 for key widths 1, 2, 4) with n_parts == 0 are skipped
hipError_t launch_super_fork(hipStream_t main, Fork& f, const PartQueue (&queue)[3],
                             const uint32_t (&grid)[3], uint32_t block, uint32_t items,
                             bool general, bool hetero);
hipError_t launch_seed_models(hipStream_t st, const ModelDev* models, uint32_t n);
hipError_t launch_reset_models(hipStream_t st, const ModelDev* models, uint32_t n,
                               unsigned int* head, uint32_t n_heads);
// Counters and clocks kept, partition bookkeeping reset: before a launch that continues
// an exploration on the same visited set.
hipError_t launch_resume_models(hipStream_t st, const ModelDev* models, uint32_t n,
                                unsigned int* head, uint32_t n_heads);
// *out += states of the visited set (slots slots) with clock <= T; *out is not cleared.
template <int W>
hipError_t launch_count_le(hipStream_t st, const unsigned char* table, unsigned long long slots,
                           const Layout& L, const CfgRec* cfgs, uint32_t T,
                           unsigned long long* out);
template <int W>
hipError_t launch_find(hipStream_t st, const QueryArgs& q, const unsigned long long* key);
template <int W>
hipError_t launch_chase(hipStream_t st, const QueryArgs& q, const TraceOut& t);
hipError_t launch_clear(hipStream_t st, void* p, unsigned long long bytes);
hipError_t launch_reset(hipStream_t st, Ctrl* ctrl, uint32_t* tc, uint32_t n_cfg);
hipError_t launch_simulate(hipStream_t st, const QueryArgs& q, unsigned long long seed);

// ---- swarm search (Sec. 5) ----------------------------------------------------------
// One member of a swarm (device record, 80 bytes; mirrored by mc_swarm_member).
struct SwarmMember {
  unsigned long long walks, trails, steps;
  unsigned long long best_walk_start;  // member step at which the best trail's walk began
  unsigned long long first_step;       // member step at which its first trail ended (~0: none)
  unsigned long long start_ticks, first_ticks;  // device clock (100 MHz) at start / first trail
  uint32_t best_clock, best_cfg;       // kNoClock / kParentNone without trails
  uint32_t first_clock, first_cfg;     // the member's first trail
  uint32_t pad[2];
};
static_assert(sizeof(SwarmMember) == 80, "SwarmMember layout");

struct SwarmArgs {
  const CfgRec* cfgs;
  uint32_t n_cfg, m;
  unsigned long long seed;    // base seed; member i uses splitmix64(seed + i)
  unsigned long long budget;  // member steps before no new walk starts
  uint32_t members, bits_log2;
  uint32_t prune, T;          // over-time property with threshold T, else non-termination
  uint32_t* bits;             // members x 2^bits_log2 bits, zero
  SwarmMember* out;           // members records
  uint8_t speed[kMaxCU];      // speed of each unit (1 = full speed)
  // operation ends counted per interval of a workgroup's duration (k_swarm_segments), or null
  uint32_t* seg;
  uint32_t seg_lcm, seg_masks;
  uint32_t lanes;  // members per wavefront (set by launch_swarm)
};
// Members per wavefront of a swarm.  A member's walks are one serial chain, and a wavefront takes
// every branch that one of its members takes: 4,096 wavefronts (four per SIMD, as many as their
// registers let share one) hold as few members each as that allows.  Fewer wavefronts leave SIMDs
// waiting for one chain, more take turns (walks not counted by interval: 16,384 members on eight
// units of eight speeds in 1,024 wavefronts 41 ms, in 4,096 27; 8,192 members on three units of a
// long period 73 and 56, in 8,192 wavefronts 43, but 65,536 on them 96, 101 and 125).
inline uint32_t swarm_lanes(uint32_t members) {
  const uint32_t n = members / 4096u + (members % 4096u ? 1u : 0u);
  return n < 64u ? n : 64u;
}
// Whether the members' bit arrays of 2^bits_log2 bits are held in LDS: where a wavefront's fit in
// a quarter of a CU's 160 KiB, and those of the whole swarm in the chip's 256 CUs at once (else
// SwarmArgs::bits is used, and cleared before the launch).  A lookup in memory is a 1-2 us link
// of a walk's chain, but wavefronts that wait for LDS cost more: 16,384 members of 8 KiB on
// matmul32_cu4_s1123 5.7 ms in LDS, 3.5 in memory, with a long period 121 and 67 ms; 4,096 of
// them 2.3 and 2.5, on units alike 1.8 and 2.0 (2,048 members).
inline bool swarm_in_lds(uint32_t members, uint32_t bits_log2) {
  const uint32_t log2_bytes = bits_log2 - 3u;
  return (unsigned long long)swarm_lanes(members) << log2_bytes <= 40u << 10 &&
         (unsigned long long)members << log2_bytes <= 256ull * (160u << 10);
}
hipError_t launch_swarm(hipStream_t st, const SwarmArgs& a);
// Replays the walk of member seed `mseed` that began at member step `start`, writing the
// rows (cfg, clock, pending, rem[0..m-1]) of its states root first into `rows` (at most
// `cap` rows; ctrl->trace_len gets the number written, ctrl->error kDevErrTrace if more).
hipError_t launch_swarm_replay(hipStream_t st, const SwarmArgs& a, Ctrl* ctrl,
                               unsigned long long mseed, unsigned long long start,
                               uint32_t* rows, uint32_t cap);

}  // namespace mc
