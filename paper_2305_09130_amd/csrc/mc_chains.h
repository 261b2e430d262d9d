// mc_chains.h -- which states a piece of the chain engine (units of unequal speed) generates:
// the arithmetic from an item's number to its state and slot, for the kernels and for checks
// on the host.
//
// Dispatch is eager, so while work is pending unit u runs workgroups back to back from clock
// 0, its j-th one from j s_u d on.  The units that fall idle at clock k d are F_k = {u : s_u
// divides k}.  Up to clock K d every workgroup's start is determined but for the order of the
// dispatches at one clock: the states are one per operation end (the chain), and at every
// clock k d the sets of F_k started (the closure).  At K d fewer workgroups p are pending than
// units are idle; each set of p of F_K starts a tail, in which nothing more is dispatched and
// whose states differ by the clock and the units still busy.
#pragma once

#include <stdint.h>

#include <vector>

#include "mc_rounds.h"

namespace mc {

// One configuration of the chain engine (device table).  Its slots, from slot0: the ends of
// each unit that stands for its speed (unit_off), the closures of the intervals before K
// (close_off), the partial closure at K d (part_off), the tails (ChainTail::off).
struct ChainCfg {
  uint32_t piece0;    // pieces before this configuration's
  uint32_t windows;   // pieces of the chain: windows of `delta` cycles of [0, K d]
  uint32_t delta;
  uint32_t tail_n;    // intervals of d cycles the tails reach into, from K d on
  uint32_t tsub;      // pieces of each
  uint32_t tail0;     // the first's ChainTail
  uint32_t slot0;
  uint32_t K, p;
  uint32_t idle;      // F_K
  uint32_t close_off, part_off;
  uint32_t unit_off[kMaxCU];
};
static_assert(sizeof(ChainCfg) == 80, "ChainCfg layout");

struct ChainTail {
  uint32_t off;    // slot of its first item
  uint32_t count;  // ends of the tails' units in the interval: items per set of busy units
};

constexpr uint32_t kChainCap = 2048;       // most items of a window explored at once
constexpr uint32_t kChainSetLog2 = 12;     // slots of its hash set: twice its items
constexpr uint32_t kMaxChainPieces = 1u << 15;  // a word for each goes where a counterexample's
                                                // keys are staged
constexpr uint32_t kMaxChainIntervals = 1u << 12;  // most intervals of a window (see quotient)

// Host plan of the chain engine: the device tables as they are uploaded (configurations,
// tails, and the closure states before interval k of a period, k = 0 .. lcm).
struct ChainPlan {
  std::vector<uint32_t> blob;
  uint32_t lcm = 0, tails_at = 0, sets_at = 0;  // places in the blob, in words
  uint64_t used = 0, n_pieces = 0;
  bool uniform = false;  // every configuration has uniform phases back to back in one wave
  bool ok() const { return n_pieces != 0; }
  const ChainCfg* cfgs() const { return reinterpret_cast<const ChainCfg*>(blob.data()); }
};

// The plan; n_pieces 0 where the chain engine cannot explore the model: units alike, a period
// of more than kMaxPeriodLcm intervals, clocks of 2^31 or more, workgroups of 2^24 operation ends
// or more, more slots needed than `slots`, a state's place within a window (time, busy units)
// that does not fit in 32 bits, or more than kMaxChainPieces pieces.  The last leaves the largest
// models to k_superstep: of 1,536 items each, 32,768 pieces hold some 50 million items
// (matmul128 on units of speeds 1, 1, 2, 3, 68M states, has 67,492 and takes 19 ms there), and
// models of many thousand configurations, which need two pieces or more each.
// target: items per piece (0: chosen).
void chain_plan(const ModelHost& h, uint64_t slots, uint64_t target, ChainPlan* out);

// What the pieces of one configuration have in common.
struct ChainEnv {
  uint32_t m, all, lcm, b, d;
  const uint32_t* sets;       // closure states before interval k of a period
  uint32_t reps;              // the lowest unit of every speed
  uint32_t speed[kMaxCU];
  float inv_speed[kMaxCU];
  float inv_b, inv_d;
};

MC_HD ChainEnv chain_env(const CfgRec& r, const uint8_t* speed, uint32_t m, uint32_t lcm,
                         const uint32_t* sets) {
  ChainEnv g;
  g.m = m;
  g.all = (1u << m) - 1u;
  g.lcm = lcm;
  g.b = r.b;
  g.d = r.d;
  g.sets = sets;
  g.reps = 0;
  g.inv_b = inverse(r.b);
  g.inv_d = inverse(r.d);
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u) {
    g.speed[u] = u < m ? speed[u] : 1u;
    g.inv_speed[u] = inverse(g.speed[u]);
    bool first = u < m;
#pragma unroll
    for (uint32_t v = 0; v < u; ++v) first = first && g.speed[v] != g.speed[u];
    g.reps |= first ? 1u << u : 0u;
  }
  return g;
}

// F_k
MC_HD uint32_t idle_at(const ChainEnv& g, uint32_t k) {
  uint32_t f = 0;
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u)
    if (u < g.m && k % g.speed[u] == 0u) f |= 1u << u;
  return f;
}
// closure states at the clocks k' d, k' < k
MC_HD uint32_t closures_before(const ChainEnv& g, uint32_t k) {
  return (k / g.lcm) * g.sets[g.lcm] + g.sets[k % g.lcm];
}
// ends before clock t of workgroups run back to back from clock 0 by a unit of speed s.
// E: the operation ends of one workgroup (upto(x): how many are at most x; at(j): the j-th)
template <class E>
MC_HD uint32_t ends_before(const E& ends, const ChainEnv& g, uint32_t s, uint32_t t) {
  if (t < 2u) return 0u;
  const uint32_t x = t - 1u, j = x / (s * g.d);
  return j * g.b + ends.upto((x - j * s * g.d) / s);
}
// ends in [t0, t1) of the one workgroup that a unit of speed s starts at clock w < t0; *n0:
// those before t0
template <class E>
MC_HD uint32_t ends_of_one(const E& ends, uint32_t s, uint32_t w, uint32_t t0, uint32_t t1,
                           uint32_t* n0) {
  *n0 = ends.upto((t0 - 1u - w) / s);
  return ends.upto((t1 - 1u - w) / s) - *n0;
}

// A window [t0, t1) of a configuration's chain or (tail) of one interval of its tails.  Items:
// unit by unit the ends in it (count[u] from the first[u]-th on), then (chain) the closures'
// sets, then the partial closure's; in a tail all of a set of busy units' ends, set by set.
struct ChainWindow {
  uint32_t t0, t1, kw;           // kw = t0 / d
  uint32_t before[kMaxCU + 1];   // ends of the units before u; [kMaxCU]: all ends
  uint32_t count[kMaxCU], first[kMaxCU];
  uint32_t slot[kMaxCU];         // chain: slot of the unit's end 0; tail: of its end 0 were it
                                 // in the interval, for the first set
  uint32_t speed[kMaxCU];
  uint32_t j0[kMaxCU], idx0[kMaxCU];    // chain: workgroup and end of the first
  uint32_t km[kMaxCU], kq[kMaxCU];      // chain: kw mod s, kw / s
  uint32_t close0, close_n;      // closure states before the window, in it
  uint32_t part_n;               // sets of the partial closure
  uint32_t k0, k1;               // intervals whose closures are in the window (k1 <= K)
  uint32_t items;
  // tail
  uint32_t interval, alive, dead_n, sets_n, per;  // alive: units of F_K busy past its start
};

// Unit u's part of a chain window (u < kMaxCU); s its speed, off its ChainCfg::unit_off (given,
// as an index known at run time only would put those arrays into memory).
template <class E>
MC_HD void chain_window_unit(ChainWindow& w, const ChainCfg& x, const ChainEnv& g, const E& ends,
                             uint32_t u, uint32_t s, uint32_t off) {
  const uint32_t kw = w.t0 / g.d;
  w.speed[u] = s;
  w.km[u] = kw % s;
  w.kq[u] = kw / s;
  w.count[u] = w.first[u] = w.j0[u] = w.idx0[u] = w.slot[u] = 0u;
  if (!((g.reps >> u) & 1u)) return;
  const uint32_t a = ends_before(ends, g, s, w.t0);
  w.first[u] = a;
  w.count[u] = ends_before(ends, g, s, w.t1) - a;
  w.j0[u] = a / g.b;
  w.idx0[u] = a % g.b;
  w.slot[u] = x.slot0 + off;
}
MC_HD void window_prefix(ChainWindow& w) {
  uint32_t n = 0;
#pragma unroll
  for (int u = 0; u < kMaxCU; ++u) {
    w.before[u] = n;
    n += w.count[u];
  }
  w.before[kMaxCU] = n;
}
MC_HD uint32_t div_up(uint32_t a, uint32_t b) { return a / b + (a % b ? 1u : 0u); }
MC_HD void chain_window_rest(ChainWindow& w, const ChainCfg& x, const ChainEnv& g) {
  window_prefix(w);
  w.kw = w.t0 / g.d;
  w.k0 = div_up(w.t0, g.d);
  w.k1 = div_up(w.t1, g.d);
  const bool end = w.k1 > x.K;  // the window holds clock K d
  w.k1 = end ? x.K : w.k1;
  w.k0 = w.k0 < w.k1 ? w.k0 : w.k1;
  w.close0 = closures_before(g, w.k0);
  w.close_n = closures_before(g, w.k1) - w.close0;
  w.part_n = end && x.p ? (1u << bits_set(x.idle)) - 1u : 0u;
  w.items = w.before[kMaxCU] + w.close_n + w.part_n;
}
// dispatches at the clocks k d, k in [a, b)
MC_HD uint32_t starts_between(const ChainEnv& g, uint32_t a, uint32_t b) {
  uint32_t n = 0;
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u)
    if (u < g.m && b > a) n += div_up(b, g.speed[u]) - div_up(a, g.speed[u]);
  return n;
}

// The functions of one item are for up to M units: four or kMaxCU.
//
// A state: its clock past the window's start, the units' time left, the workgroups pending.
struct ChainItem {
  uint32_t t, busy, pending;
  uint32_t rem[kMaxCU];
  uint32_t slot;
  bool active, is_end;
};

// Bits of `set` (an index of subsets) moved to the bits of `of`.
MC_HD uint32_t spread_bits(uint32_t set, uint32_t of) {
  uint32_t out = 0, at = 0;
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u)
    if ((of >> u) & 1u) out |= ((set >> at++) & 1u) << u;
  return out;
}

// The state k - w.kw = dk intervals and `past` cycles into the window's time, `set` of F_k
// started when past is 0.
template <int M>
MC_HD void chain_state(const ChainWindow& w, const ChainEnv& g, uint32_t n, uint32_t dk,
                       uint32_t past, uint32_t set, bool closure, ChainItem* it) {
  uint32_t started = 0, busy = 0, at = 0;
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)M; ++u) {
    it->rem[u] = 0u;
    if (u >= g.m) continue;
    const uint32_t s = g.speed[u], a = w.km[u] + dk, q = quotient(a, g.inv_speed[u]);
    const uint32_t mod = a - q * s;
    bool on = true;  // past the interval's start every unit runs
    if (past == 0u && mod == 0u) {
      on = closure && ((set >> at) & 1u);
      ++at;
    }
    started += w.kq[u] + q + ((mod != 0u || on) ? 1u : 0u);
    it->rem[u] = on ? (s - mod) * g.d - past : 0u;
    busy |= on ? 1u << u : 0u;
  }
  // a unit that ends its workgroup at the window's clock has no time left
  it->busy = busy;
  it->pending = n - started;
}

// Item i of a chain window (i < items).  n: the configuration's workgroups.
template <int M, class E>
MC_HD void chain_item(const ChainWindow& w, const ChainCfg& x, const ChainEnv& g, const E& ends,
                      uint32_t n, uint32_t i, ChainItem* it) {
  uint32_t dk, past = 0, set = 0;
  bool closure = false;
  it->active = true;
  it->is_end = i < w.before[kMaxCU];
  if (it->is_end) {
    uint32_t u = 0;
#pragma unroll
    for (int v = 1; v < M; ++v) u = i >= w.before[v] ? (uint32_t)v : u;
    const uint32_t s = w.speed[u], at = i - w.before[u];
    it->slot = w.slot[u] + w.first[u] + at;
    // (a workgroup of more than kSmallRound ends holds the window's but for one wrap)
    const uint32_t y = w.idx0[u] + at;
    const uint32_t q = g.b <= kSmallRound ? quotient(y, g.inv_b) : (y >= g.b ? 1u : 0u);
    const uint32_t e = s * ends.at(y - q * g.b);
    uint32_t k = (uint32_t)((float)e * g.inv_d);
    past = e - k * g.d;
    if ((int32_t)past < 0) {
      --k;
      past += g.d;
    } else if (past >= g.d) {
      ++k;
      past -= g.d;
    }
    k += (w.j0[u] + q) * s;
    dk = k - w.kw;
  } else if (i - w.before[kMaxCU] < w.close_n) {
    closure = true;
    const uint32_t X = w.close0 + (i - w.before[kMaxCU]), per = g.sets[g.lcm];
    const uint32_t period = X / per, rest = X - period * per;
    uint32_t lo = 0, len = g.lcm;  // the last interval with sets[lo] <= rest
    while (len > 1u) {
      const uint32_t half = len >> 1;
      if (g.sets[lo + half] <= rest) {
        lo += half;
        len -= half;
      } else {
        len = half;
      }
    }
    set = rest - g.sets[lo] + 1u;
    dk = period * g.lcm + lo - w.kw;
    it->slot = x.slot0 + x.close_off + X;
  } else {
    closure = true;
    const uint32_t y = i - w.before[kMaxCU] - w.close_n;
    set = y + 1u;
    dk = x.K - w.kw;
    it->active = bits_set(set) <= x.p;
    it->slot = x.slot0 + x.part_off + y;
  }
  it->t = (w.kw + dk) * g.d + past - w.t0;
  chain_state<M>(w, g, n, dk, past, set, closure, it);
}

// ---- tails ------------------------------------------------------------------------------

// The units a tail's workgroups run on: those busy at clock K d, and (p > 0) those of F_K.
MC_HD uint32_t tail_units(const ChainCfg& x, const ChainEnv& g) {
  return x.p ? g.all : g.all & ~x.idle;
}
// Start of the workgroup that a unit of speed s runs in the tails.
MC_HD uint32_t tail_start(const ChainCfg& x, const ChainEnv& g, uint32_t s) {
  return (x.K - x.K % s) * g.d;
}
// The units whose ends are listed in the tails: the lowest of every speed.  Those of one speed
// are all idle at K d or all busy, and end alike.
MC_HD uint32_t tail_listed(const ChainCfg& x, const ChainEnv& g) {
  return g.reps & tail_units(x, g);
}
// The units of speed s.
template <int M>
MC_HD uint32_t units_of_speed(const ChainEnv& g, uint32_t s) {
  uint32_t out = 0;
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)M; ++u) out |= u < g.m && g.speed[u] == s ? 1u << u : 0u;
  return out;
}
MC_HD uint32_t tail_from(const ChainCfg& x, const ChainEnv& g, uint32_t interval) {
  return (x.K + interval) * g.d + (interval ? 0u : 1u);
}

// Unit u's part of a tail window of `interval` (s its speed; listed: it is one of
// tail_listed); returns its ends in the whole interval.
template <class E>
MC_HD uint32_t tail_window_unit(ChainWindow& w, const ChainCfg& x, const ChainEnv& g,
                                const E& ends, uint32_t interval, uint32_t u, uint32_t s,
                                bool listed) {
  w.count[u] = w.first[u] = w.slot[u] = w.j0[u] = w.idx0[u] = w.km[u] = w.kq[u] = 0u;
  w.speed[u] = s;
  if (!listed) return 0u;
  const uint32_t ws = tail_start(x, g, s);
  uint32_t n0, a;
  const uint32_t whole =
      ends_of_one(ends, s, ws, tail_from(x, g, interval), (x.K + interval + 1u) * g.d, &n0);
  w.count[u] = ends_of_one(ends, s, ws, w.t0, w.t1, &a);
  w.first[u] = a;
  w.slot[u] = 0u - n0;  // the interval's ends of the units before u are added
  return whole;
}
// whole[u]: as tail_window_unit gave them
MC_HD void tail_window_rest(ChainWindow& w, const ChainCfg& x, const ChainEnv& g,
                            const ChainTail& tl, uint32_t interval, const uint32_t* whole) {
  window_prefix(w);
  uint32_t n = x.slot0 + tl.off;
#pragma unroll
  for (int u = 0; u < kMaxCU; ++u) {
    w.slot[u] += n;
    n += whole[u];
  }
  w.kw = w.t0 / g.d;
  w.interval = interval;
  w.alive = 0;
  const uint32_t run = x.p ? x.idle : 0u;
#pragma unroll
  for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u)
    if (((run >> u) & 1u) && g.speed[u] > interval) w.alive |= 1u << u;
  w.dead_n = bits_set(run) - bits_set(w.alive);
  w.per = tl.count;
  w.close0 = w.close_n = w.part_n = w.k0 = w.k1 = 0u;
}
// Whether some choice of p units of F_K has exactly the units `set` of w.alive.
MC_HD bool tail_set(uint32_t p, uint32_t dead_n, uint32_t set) {
  const uint32_t n = bits_set(set);
  return n <= p && p - n <= dead_n;
}

// End i of a tail window for the rank-th set of busy units of F_K.
template <int M, class E>
MC_HD void tail_item(const ChainWindow& w, const ChainCfg& x, const ChainEnv& g, const E& ends,
                     uint32_t i, uint32_t rank, uint32_t set, ChainItem* it) {
  uint32_t u = 0;
#pragma unroll
  for (int v = 1; v < M; ++v) u = i >= w.before[v] ? (uint32_t)v : u;
  const uint32_t s = w.speed[u], n = w.first[u] + (i - w.before[u]);
  it->slot = w.slot[u] + n + rank * w.per;
  it->is_end = true;
  const uint32_t t = (x.K - x.K % s) * g.d + s * ends.at(n);
  it->t = t - w.t0;
  // an end of units of F_K: of one of the set, or the last of one that was started beside it
  const bool chosen = (x.idle >> u) & 1u;
  it->active = !chosen || (set & units_of_speed<M>(g, s)) != 0u ||
               (!((w.alive >> u) & 1u) && bits_set(set) < x.p);
  it->pending = 0u;
  it->busy = 0u;
  const uint32_t on = (g.all & ~x.idle) | set;
#pragma unroll
  for (uint32_t v = 0; v < (uint32_t)M; ++v) {
    it->rem[v] = 0u;
    if (v >= g.m || !((on >> v) & 1u)) continue;
    const uint32_t end = (x.K - x.K % g.speed[v] + g.speed[v]) * g.d;
    it->rem[v] = end > t ? end - t : 0u;
    it->busy |= it->rem[v] ? 1u << v : 0u;
  }
}

// The window of piece `local` of a configuration, up to clock T (t0 >= t1: nothing).
struct ChainSpan {
  uint32_t t0, t1, interval;
  bool tail;
};
MC_HD ChainSpan chain_span(const ChainCfg& x, const ChainEnv& g, uint32_t local, uint32_t T) {
  ChainSpan s;
  const uint32_t end = x.K * g.d + 1u;
  s.tail = local >= x.windows;
  s.interval = 0;
  if (!s.tail) {
    s.t0 = local * x.delta;
    s.t1 = local + 1u == x.windows ? end : s.t0 + x.delta;
  } else {
    const uint32_t l = local - x.windows;
    s.interval = l / x.tsub;
    const uint32_t part = l - s.interval * x.tsub, step = div_up(g.d, x.tsub);
    const uint32_t base = (x.K + s.interval) * g.d;
    s.t0 = part * step < g.d ? base + part * step : base + g.d;
    s.t1 = part * step + step < g.d ? s.t0 + step : base + g.d;
    s.t0 = s.t0 < end ? end : s.t0;
  }
  if (T < 0x7FFFFFFFu && s.t1 > T + 1u) s.t1 = T + 1u;
  return s;
}

}  // namespace mc
