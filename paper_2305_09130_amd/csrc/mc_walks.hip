// mc_walks.hip -- seeded walks of the MI355X explicit-state checker.
//
//   k_simulate      one seeded random run from the root (simulation mode, the T_ini of
//                   the tuning loop)
//   k_swarm         swarm search: many independent bitstate walkers, one per lane
//   k_swarm_replay  one member's walk again, state by state (its counterexample)
#include <hip/hip_runtime.h>

#include "mc_launch.h"

namespace mc {

// ---- simulation mode ------------------------------------------------------------------
//
// One run from the root, choosing uniformly among the successors at every step with
// the choice of step t drawn from splitmix64(seed ^ splitmix64(t)); successors are
// ordered by configuration (SELECT) and by unit index (DISPATCH).  A lock-step ADVANCE
// run has one successor per step; it is taken in one jump that counts its steps.  On units
// of one speed whole rounds are crossed at once as well: with at least m workgroups pending
// every order of the m dispatches leads through one run to the same all-idle state, and each
// round takes m + b steps (a draw depends on its step alone, so the later ones are the same).

// Units of unequal speed with no DISPATCH enabled until clock H (the first workgroup end
// while work is pending, else the last): the ADVANCE steps up to H are one per distinct
// operation end of the busy units in (clock, H].  The wavefront counts them a window at a
// time: lane l takes the (l mod p)-th next end of unit l / p (p = 64 / m); the window
// closes at the least last-slot end of any unit (no end of any unit below it is missing),
// an end counts unless a unit of lower index ends at the same time, and the state moves
// to the window's close.  Returns the steps; x is left at clock H.
__device__ uint32_t jump_unequal(St& x, const CfgRec& r, int m, const uint8_t* speed,
                                 uint32_t H) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t per = 64u / (uint32_t)m;
  const uint32_t u = lane / per, k = lane - u * per;
  uint32_t steps = 0;
  while (x.clock < H) {
    uint32_t v = 0xFFFFFFFFu;
    if (u < (uint32_t)m && x.rem[u]) {
      const uint32_t sp = speed[u];
      const uint32_t e = sp * r.d - x.rem[u];
      const uint32_t kk = ends_upto(r, e / sp) + k;
      if (kk < r.b) {
        const uint32_t tau = x.clock + sp * end_at(r, kk) - e;
        if (tau <= H) v = tau;
      }
    }
    uint32_t lim = (k + 1u == per) ? v : 0xFFFFFFFFu;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const uint32_t y = __shfl_xor(lim, o);
      lim = y < lim ? y : lim;
    }
    lim = lim < H ? lim : H;
    bool first = v <= lim;
    for (uint32_t j = 0; j < u && first; ++j) {
      // does unit j (busy until clock + rem_j) end an operation at time v?
      if (x.rem[j] == 0u || v > x.clock + x.rem[j]) continue;
      const uint32_t sj = speed[j];
      const uint32_t diff = v - x.clock + (sj * r.d - x.rem[j]);
      if (diff % sj) continue;
      const uint32_t q = diff / sj;
      if (q && ends_upto(r, q) != ends_upto(r, q - 1u)) first = false;
    }
    steps += (uint32_t)__popcll(__ballot(first));
    const uint32_t dt = lim - x.clock;
#pragma unroll
    for (int i = 0; i < kMaxCU; ++i) x.rem[i] = x.rem[i] > dt ? x.rem[i] - dt : 0u;
    x.clock = lim;
  }
  return steps;
}

__global__ void k_simulate(QueryArgs a, unsigned long long seed) {
  // every lane of the wavefront follows the same run; jump_unequal splits its windows
  if (blockIdx.x != 0 || threadIdx.x >= 64) return;
  const int m = a.L.m;
  const uint8_t* speed = a.L.speed;
  unsigned long long step = 0;
  const uint32_t c = (uint32_t)(splitmix64(seed ^ splitmix64(step)) % a.n_cfg);
  ++step;
  const CfgRec r = a.cfgs[c];
  St x{};
  x.cfg = c;
  x.pending = r.n;
  bool alike = true;
  for (int u = 1; u < m; ++u) alike = alike && speed[u] == speed[0];
  if (alike) {  // 2,048 rounds one dispatch at a time took 2.2 ms
    const uint32_t rounds = r.n / (uint32_t)m;
    x.pending -= rounds * (uint32_t)m;
    x.clock = rounds * speed[0] * r.d;
    step += (unsigned long long)rounds * ((uint32_t)m + r.b);
  }
  for (;;) {
    uint32_t freem = 0, busy = 0, brem = 0, bsp = 0;
    bool same = true;
    for (int u = 0; u < m; ++u) {
      if (x.rem[u] == 0u) {
        freem |= 1u << u;
      } else {
        if (busy && (x.rem[u] != brem || speed[u] != bsp)) same = false;
        brem = x.rem[u];
        bsp = speed[u];
        busy |= 1u << u;
      }
    }
    if (x.pending && freem) {
      const uint32_t nfree = (uint32_t)__popc(freem);
      uint32_t pick = (uint32_t)(splitmix64(seed ^ splitmix64(step)) % nfree);
      ++step;
      for (int u = 0; u < m; ++u) {
        if ((freem >> u) & 1u) {
          if (pick == 0u) {
            x.rem[u] = unit_dur<true>(r, speed, u);
            x.pending -= 1u;
            break;
          }
          --pick;
        }
      }
      continue;
    }
    if (!busy) break;
    if (same) {
      // busy units in lock step (equal speed and time left): one step per end to go
      const uint32_t e0 = bsp * r.d - brem;
      step += r.b - ends_upto(r, e0 / bsp);
      x.clock += brem;
      for (int u = 0; u < m; ++u) x.rem[u] = 0u;
    } else {
      // no DISPATCH before the first workgroup end (work pending) or the last
      uint32_t H = x.pending ? 0xFFFFFFFFu : 0u;
      for (int u = 0; u < m; ++u) {
        if (!x.rem[u]) continue;
        const uint32_t t = x.clock + x.rem[u];
        H = x.pending ? (t < H ? t : H) : (t > H ? t : H);
      }
      step += jump_unequal(x, r, m, speed, H);
    }
  }
  if (threadIdx.x == 0) {
    a.ctrl->sim_t = x.clock;
    a.ctrl->sim_cfg = c;
  }
}

// ---- swarm search (Sec. 5) -----------------------------------------------------------
//
// Swarm model checking runs many independent, incomplete searches: each member keeps a
// bit array of its own (bitstate hashing) instead of storing states, and reports the
// counterexamples it meets within a bounded number of model steps.  Against G(!FIN)
// every run reaching a terminal is a counterexample whose clock is a model time;
// against the over-time property with threshold T only terminals with clock <= T are.
// Member i (one lane) uses seed splitmix64(seed + i) and makes walks from the root: at
// its step t (counted over all its walks) it takes successor number
// splitmix64(seed_i ^ splitmix64(t)) mod k of the k successors (configurations in order
// at the root, free units in index order for DISPATCH).  With a threshold a walk ends
// at the first state with clock > T.  At every state it reaches (not the root) with
// other than exactly one successor it hashes (cfg, clock, pending, rem_0..rem_{m-1})
// with a splitmix64 chain to bit positions h mod B and (h >> 32) mod B: both set, the
// walk ends (the state was visited); else both are set.  A new terminal ends the walk
// as a counterexample (a trail).  A new walk starts only while t < budget.  The
// interior states of a lock-step run (one successor each, no bitstate lookup) are
// crossed in one jump that counts their steps, and, with a threshold, stops exactly at
// the first of them past T.

// x mod k for k in 1..8, by way of x mod 840 = lcm(1..8) in 32-bit arithmetic (a 64-bit
// remainder was most of a dispatch's instructions).
__device__ __forceinline__ uint32_t small_mod(unsigned long long x, uint32_t k) {
  constexpr uint32_t kAll = 840u, kFold = (uint32_t)((1ull << 32) % kAll);
  const uint32_t y = ((uint32_t)(x >> 32) % kAll * kFold + (uint32_t)x % kAll) % kAll;
  // y + 1/2 is at least half off a multiple of k: far more than the product's error
  const uint32_t q = (uint32_t)(((float)y + 0.5f) * __builtin_amdgcn_rcpf((float)k));
  return y - q * k;
}

// The per-unit loops of a walk run to MU (4 or 8, the least that holds the units), unrolled,
// so that the times left stay in registers.
template <int MU>  // h: splitmix64 of the configuration, the same along a walk
__device__ __forceinline__ unsigned long long swarm_hash(unsigned long long h, const St& x, int m) {
  h = splitmix64(h ^ x.clock);
  h = splitmix64(h ^ x.pending);
#pragma unroll
  for (int u = 0; u < MU; ++u)
    if (u < m) h = splitmix64(h ^ x.rem[u]);
  return h;
}

// successor count of a non-root state, its free and busy units, and whether the busy
// units are in lock step (equal speed and remaining time)
struct SwarmView {
  uint32_t k, freem, busy, brem, bsp;
  bool same;
};
template <int MU>
__device__ __forceinline__ SwarmView swarm_view(const St& x, int m, const uint8_t* speed) {
  SwarmView v{0u, 0u, 0u, 0u, 1u, true};
#pragma unroll
  for (int u = 0; u < MU; ++u) {
    if (u >= m) continue;
    if (x.rem[u] == 0u) {
      v.freem |= 1u << u;
    } else {
      if (v.busy && (x.rem[u] != v.brem || speed[u] != v.bsp)) v.same = false;
      v.brem = x.rem[u];
      v.bsp = speed[u];
      v.busy |= 1u << u;
    }
  }
  v.k = (x.pending && v.freem) ? (uint32_t)__popc(v.freem) : (v.busy ? 1u : 0u);
  return v;
}

template <int MU>
__device__ __forceinline__ void swarm_dispatch(St& x, const CfgRec& r, uint32_t freem,
                                               uint32_t pick, int m, const uint8_t* speed) {
#pragma unroll
  for (int u = 0; u < MU; ++u)
    if (((freem >> u) & 1u) && (uint32_t)__popc(freem & ((1u << u) - 1u)) == pick)
      x.rem[u] = unit_dur<true>(r, speed, u);
  x.pending -= 1u;
}

// Operation ends on units of unequal speed, counted once per swarm.  A unit starts its
// workgroups back to back from clock 0 (dispatch is eager) until none is left, so at clock
// k d unit u has run (k mod s_u) d of its workgroup, and how many distinct operation ends the
// units of a mask have in (k d, (k+1) d] depends on k mod lcm(s) alone.  Workgroups end at
// multiples of d, so a walk crosses an ADVANCE chain by adding these counts, one interval at
// a time, instead of merging the units' ends step by step: the 4,096-member swarm on
// matmul32_cu4_s1123 took 177 ms that way, on walks of up to 10^5 steps.
// a.seg[(c lcm + k) masks + M]: M the busy units (masks = 2^m), or the one count for all
// units busy (masks = 1).
__global__ __launch_bounds__(64) void k_swarm_segments(SwarmArgs a) {
  const uint32_t lane = threadIdx.x, c = blockIdx.x / a.seg_lcm, k = blockIdx.x - c * a.seg_lcm;
  const CfgRec r = a.cfgs[c];
  const int m = (int)a.m;
  uint32_t e0[kMaxCU], lo[kMaxCU], first[kMaxCU + 1];
  uint32_t total = 0;
#pragma unroll
  for (int u = 0; u < kMaxCU; ++u) {
    first[u] = total;
    e0[u] = lo[u] = 0u;
    if (u >= m) continue;
    const uint32_t sp = a.speed[u];
    e0[u] = (k % sp) * r.d;
    lo[u] = ends_upto(r, e0[u] / sp);
    total += ends_upto(r, (e0[u] + r.d) / sp) - lo[u];
  }
  first[kMaxCU] = total;
  uint32_t count = 0;  // lane M: of mask M (lane 0: of all units where masks = 1)
  for (uint32_t base = 0; base < total; base += 64u) {
    const uint32_t i = base + lane;
    uint32_t tau = 0, unit = 0, lower = 0;  // lower: units of lower index that end at tau
    if (i < total) {
      uint32_t eu = e0[0], lu = lo[0], fu = 0, su = a.speed[0];
#pragma unroll
      for (int u = 1; u < kMaxCU; ++u)
        if (u < m && i >= first[u]) {
          unit = (uint32_t)u;
          eu = e0[u];
          lu = lo[u];
          fu = first[u];
          su = a.speed[u];
        }
      tau = su * end_at(r, lu + (i - fu)) - eu;
#pragma unroll
      for (int j = 0; j < kMaxCU; ++j) {
        if (j >= m || (uint32_t)j >= unit) continue;
        const uint32_t x = e0[j] + tau, q = x / a.speed[j];
        if (q * a.speed[j] == x && ends_upto(r, q) != ends_upto(r, q - 1u)) lower |= 1u << j;
      }
    }
    if (a.seg_masks == 1u) {
      count += (uint32_t)__popcll(__ballot(i < total && lower == 0u));
    } else {
      for (uint32_t M = 1; M < a.seg_masks; ++M) {
        const bool mine = i < total && ((M >> unit) & 1u) && (lower & M) == 0u;
        const uint32_t n = (uint32_t)__popcll(__ballot(mine));
        if (lane == M) count += n;
      }
    }
  }
  if (lane < a.seg_masks) a.seg[(unsigned long long)blockIdx.x * a.seg_masks + lane] = count;
}

// A walk's ADVANCE chain on units that are not in lock step: from x on every state has
// one successor (no work pending, or no unit free) until a unit falls idle while work is
// pending, or no unit is busy.  Each busy unit keeps the index and time of its next
// operation end and its workgroup's end, so a step is the least next end and one
// operation-end lookup per unit that ends there.  t counts one model step per state, as
// one ADVANCE at a time would.  With a threshold it stops on the first state past T and
// returns true (the walk ends there).  x is left on the chain's last state.
template <int MU>
__device__ bool swarm_advance_run(St& x, const CfgRec& r, int m, const uint8_t* speed,
                                  bool prune, uint32_t T, unsigned long long& t) {
  uint32_t nx[MU], kk[MU], wend[MU], sp[MU];
  uint32_t busy = 0;
#pragma unroll
  for (int u = 0; u < MU; ++u) {
    nx[u] = 0xFFFFFFFFu;
    kk[u] = 0u;
    wend[u] = 0u;
    sp[u] = 1u;
    if (u < m && x.rem[u]) {
      sp[u] = speed[u];
      // elapsed e < sp*d; the next end sp*E[k] > e has E[k] > floor(e / sp)
      const uint32_t e = sp[u] * r.d - x.rem[u];
      kk[u] = ends_upto(r, e / sp[u]);
      wend[u] = x.clock + x.rem[u];
      nx[u] = x.clock + sp[u] * end_at(r, kk[u]) - e;
      busy |= 1u << u;
    }
  }
  bool past = false;
  for (;;) {
    uint32_t tmin = 0xFFFFFFFFu;
#pragma unroll
    for (int u = 0; u < MU; ++u) tmin = nx[u] < tmin ? nx[u] : tmin;
    x.clock = tmin;
    ++t;
    bool freed = false;
#pragma unroll
    for (int u = 0; u < MU; ++u) {
      if (nx[u] != tmin) continue;
      if (++kk[u] == r.b) {
        busy &= ~(1u << u);
        nx[u] = 0xFFFFFFFFu;
        freed = true;
      } else {
        nx[u] = wend[u] - sp[u] * r.d + sp[u] * end_at(r, kk[u]);
      }
    }
    if (prune && x.clock > T) {
      past = true;
      break;
    }
    if (!busy || (freed && x.pending)) break;
  }
#pragma unroll
  for (int u = 0; u < MU; ++u) x.rem[u] = ((busy >> u) & 1u) ? wend[u] - x.clock : 0u;
  return past;
}

// The same chain by the counts of k_swarm_segments, while those hold the busy units: x.clock
// is a multiple of d.  Returns whether the chain is at its end (else the units still busy, or
// the interval in which the clock passes T, are left to swarm_advance_run).
template <int MU>
__device__ __forceinline__ bool swarm_jump(St& x, const CfgRec& r, const SwarmArgs& a,
                                           unsigned long long& t) {
  const uint32_t all = (1u << a.m) - 1u;
  uint32_t k = x.clock / r.d;
  const uint32_t* seg = a.seg + (unsigned long long)x.cfg * a.seg_lcm * a.seg_masks;
  uint32_t at = k % a.seg_lcm;
  for (;;) {
    uint32_t busy = 0, least = 0xFFFFFFFFu;
#pragma unroll
    for (int u = 0; u < MU; ++u)
      if (u < (int)a.m && x.rem[u]) {
        busy |= 1u << u;
        least = x.rem[u] < least ? x.rem[u] : least;
      }
    if (!busy) return true;
    if ((a.seg_masks == 1u && busy != all) || (a.prune && x.clock + least > a.T)) return false;
    for (uint32_t left = least; left; left -= r.d) {  // least is a multiple of d
      t += seg[at * a.seg_masks + (a.seg_masks == 1u ? 0u : busy)];
      at = at + 1u == a.seg_lcm ? 0u : at + 1u;
    }
    x.clock += least;
#pragma unroll
    for (int u = 0; u < MU; ++u)
      if (u < (int)a.m && x.rem[u]) x.rem[u] -= least;
    if (x.pending) return true;  // a unit fell idle
  }
}

// LDS: the members' bit arrays are in LDS (swarm_in_lds), cleared here, else in a.bits.  Four
// waves per SIMD are asked for: left alone, the build for eight units takes 137 registers, which
// three share (262,144 members on eight units of eight speeds, walks not counted by interval:
// 82 -> 60 ms).
template <int MU, bool LDS>
__global__ __launch_bounds__(64, 4) void k_swarm(SwarmArgs a) {
  extern __shared__ uint32_t lds_bits[];
  if constexpr (LDS) {
    const uint32_t n4 = a.lanes << (a.bits_log2 - 7u);  // 16-byte units
    for (uint32_t j = threadIdx.x; j < n4; j += 64u)
      reinterpret_cast<uint4*>(lds_bits)[j] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }
  if (threadIdx.x >= a.lanes) return;
  const uint32_t i = blockIdx.x * a.lanes + threadIdx.x;
  if (i >= a.members) return;
  const int m = (int)a.m;
  const unsigned long long seed = splitmix64(a.seed + i);
  const unsigned long long B = 1ull << a.bits_log2;
  uint32_t* bits;
  if constexpr (LDS) bits = lds_bits + threadIdx.x * (uint32_t)(B >> 5);
  else bits = a.bits + (unsigned long long)i * (B >> 5);
  SwarmMember rec;
  rec.walks = rec.trails = rec.best_walk_start = 0ull;
  rec.first_step = ~0ull;
  rec.first_ticks = 0ull;
  rec.best_clock = rec.first_clock = kNoClock;
  rec.best_cfg = rec.first_cfg = kParentNone;
  rec.pad[0] = rec.pad[1] = 0u;
  rec.start_ticks = __builtin_amdgcn_s_memrealtime();
  unsigned long long t = 0;
  while (t < a.budget) {
    ++rec.walks;
    const unsigned long long start = t;
    const uint32_t c = (uint32_t)(splitmix64(seed ^ splitmix64(t)) % a.n_cfg);
    ++t;
    const CfgRec r = a.cfgs[c];
    St x{};
    x.cfg = c;
    x.pending = r.n;
    // One instant a time, so that the walks of a wavefront stay together: the states at x's
    // clock, each just reached by a transition (a state with one successor has no place in
    // the bitstate), through the dispatches there, then the steps to the next instant.
    const unsigned long long h0 = splitmix64((unsigned long long)c);
    bool over = false;
    while (!over) {
      SwarmView v;
      for (;;) {
        v = swarm_view<MU>(x, m, a.speed);
        if (a.prune && x.clock > a.T) {
          over = true;
          break;
        }
        if (v.k != 1u) {
          const unsigned long long h = swarm_hash<MU>(h0, x, m);
          const unsigned long long p0 = h & (B - 1ull), p1 = (h >> 32) & (B - 1ull);
          const uint32_t w0 = bits[p0 >> 5], w1 = bits[p1 >> 5];
          const uint32_t m0 = 1u << (p0 & 31ull), m1 = 1u << (p1 & 31ull);
          if ((w0 & m0) && (w1 & m1)) {  // visited
            over = true;
            break;
          }
          bits[p0 >> 5] = w0 | m0;
          bits[p1 >> 5] = (p1 >> 5) == (p0 >> 5) ? w0 | m0 | m1 : w1 | m1;
        }
        if (!(x.pending && v.freem)) break;
        const uint32_t pick = small_mod(splitmix64(seed ^ splitmix64(t)), v.k);
        ++t;
        swarm_dispatch<MU>(x, r, v.freem, pick, m, a.speed);
      }
      if (over) break;
      if (v.k == 0u) {  // a new terminal: a trail
        ++rec.trails;
        if (rec.first_step == ~0ull) {
          rec.first_step = t;
          rec.first_ticks = __builtin_amdgcn_s_memrealtime();
          rec.first_clock = x.clock;
          rec.first_cfg = x.cfg;
        }
        if (rec.best_clock == kNoClock || x.clock < rec.best_clock) {
          rec.best_clock = x.clock;
          rec.best_cfg = x.cfg;
          rec.best_walk_start = start;
        }
        break;
      }
      if (v.same) {  // a lock-step run to its end, one transition per operation end
        // ends of the busy units' grid bsp*E after the elapsed time e0
        const uint32_t e0 = v.bsp * r.d - v.brem;
        const uint32_t idx0 = ends_upto(r, e0 / v.bsp);
        if (a.prune && x.clock + v.brem > a.T) {
          // stop at the first state of the run past T
          const uint32_t idx = ends_upto(r, (a.T - x.clock + e0) / v.bsp);
          t += (unsigned long long)(idx - idx0 + 1u);
          break;
        }
        t += (unsigned long long)(r.b - idx0);
        x.clock += v.brem;
#pragma unroll
        for (int u = 0; u < MU; ++u) x.rem[u] = 0u;
        continue;
      }
      if (a.seg && swarm_jump<MU>(x, r, a, t)) continue;
      if (swarm_advance_run<MU>(x, r, m, a.speed, a.prune != 0u, a.T, t)) break;
    }
  }
  rec.steps = t;
  a.out[i] = rec;
}

// One thread: the walk of one member from member step `start`, to its terminal.
__global__ void k_swarm_replay(SwarmArgs a, Ctrl* ctrl, unsigned long long seed,
                               unsigned long long start, uint32_t* rows, uint32_t cap) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int m = (int)a.m;
  const uint32_t S = 3u + (uint32_t)m;
  uint32_t n = 0;
  bool bad = false;
  auto put = [&](const St& x, bool root) {
    if (n >= cap) {
      bad = true;
      return;
    }
    uint32_t* row = rows + (unsigned long long)n * S;
    row[0] = root ? kParentNone : x.cfg;
    row[1] = root ? 0u : x.clock;
    row[2] = root ? 0u : x.pending;
    for (int u = 0; u < m; ++u) row[3 + u] = root ? 0u : x.rem[u];
    ++n;
  };
  St x{};
  put(x, true);
  unsigned long long t = start;
  const uint32_t c = (uint32_t)(splitmix64(seed ^ splitmix64(t)) % a.n_cfg);
  ++t;
  const CfgRec r = a.cfgs[c];
  x.cfg = c;
  x.pending = r.n;
  put(x, false);
  for (;;) {
    const SwarmView v = swarm_view<kMaxCU>(x, m, a.speed);
    if (v.k == 0u || bad) break;
    if (x.pending && v.freem) {
      const uint32_t pick = (uint32_t)(splitmix64(seed ^ splitmix64(t)) % v.k);
      ++t;
      swarm_dispatch<kMaxCU>(x, r, v.freem, pick, m, a.speed);
    } else {
      advance_once(x, r, m, a.speed);
      ++t;
    }
    put(x, false);
  }
  if (bad) set_error(ctrl, kDevErrTrace);
  ctrl->trace_len = n;
}

// ---- launch helpers (host) ------------------------------------------------------------

hipError_t launch_swarm(hipStream_t st, const SwarmArgs& a) {
  if (a.seg)
    hipLaunchKernelGGL(k_swarm_segments, dim3(a.n_cfg * a.seg_lcm), dim3(64), 0, st, a);
  SwarmArgs q = a;
  q.lanes = swarm_lanes(a.members);
  const bool held = swarm_in_lds(a.members, a.bits_log2);
  const uint32_t lds = held ? q.lanes << (a.bits_log2 - 3u) : 0u;
  const dim3 grid((a.members + q.lanes - 1u) / q.lanes);
  if (a.m <= 4u) {
    if (held) hipLaunchKernelGGL((k_swarm<4, true>), grid, dim3(64), lds, st, q);
    else hipLaunchKernelGGL((k_swarm<4, false>), grid, dim3(64), 0, st, q);
  } else {
    if (held) hipLaunchKernelGGL((k_swarm<8, true>), grid, dim3(64), lds, st, q);
    else hipLaunchKernelGGL((k_swarm<8, false>), grid, dim3(64), 0, st, q);
  }
  return hipGetLastError();
}

hipError_t launch_swarm_replay(hipStream_t st, const SwarmArgs& a, Ctrl* ctrl,
                               unsigned long long mseed, unsigned long long start,
                               uint32_t* rows, uint32_t cap) {
  hipLaunchKernelGGL(k_swarm_replay, dim3(1), dim3(64), 0, st, a, ctrl, mseed, start, rows, cap);
  return hipGetLastError();
}

hipError_t launch_simulate(hipStream_t st, const QueryArgs& q, unsigned long long seed) {
  hipLaunchKernelGGL(k_simulate, dim3(1), dim3(64), 0, st, q, seed);
  return hipGetLastError();
}

}  // namespace mc
