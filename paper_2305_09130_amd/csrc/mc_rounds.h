// mc_rounds.h -- which states a piece of the round engine generates: the arithmetic from an
// item's number to its state and slots, for the kernel and for checks on the host.
#pragma once

#include <stdint.h>

#include "mc_model.h"

#ifdef __HIP__
#define MC_HD \
  __attribute__((host)) __attribute__((device)) inline __attribute__((always_inline))
#else
#define MC_HD inline
#endif

namespace mc {

MC_HD uint32_t mul24(uint32_t a, uint32_t b) { return (a & 0xFFFFFFu) * (b & 0xFFFFFFu); }
// 1 / n to within a unit in the last place
MC_HD float inverse(uint32_t n) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf((float)n);
#else
  return 1.0f / (float)n;
#endif
}
MC_HD uint32_t bits_set(uint32_t v) { return (uint32_t)__builtin_popcount(v); }

// Items [i0, i1) of a partition (RoundPart gives the item order), and what is common to them.
struct Piece {
  uint32_t m, all;           // units, the mask of all
  uint32_t n, b;             // the configuration's workgroups and operation ends
  uint32_t r0, nfull;        // the partition's first round and full rounds
  uint32_t ja, jb, cl, per;  // run states, closure items and items of a full round
  uint32_t F;                // items of the full rounds
  uint32_t sets, choices, p; // of the partial round: closure sets, choices of p units
  uint32_t slot0, link;
  uint32_t i0, i1;
  uint32_t q0, q1, loc0;     // first and last round of the piece, from r0; i0's place in it
  float per_inv;             // 1 / per
  float choices_inv;         // 1 / choices
  uint32_t jj0, l0;          // run state and choice of the first item past the full rounds'
                             // and the closure's that the piece holds
  uint32_t y0;               // that item's number
  bool last;                 // the partition's last piece
  uint32_t pmin;             // least pending count of the piece's states
  uint32_t xloc;             // place in a round of its end, where the runs stop before it
  bool closure, extra, partial;
};

// x / n given 1 / n, for n up to kSmallRound and x below 2^15: x + 1/2 is at least half off
// every multiple of n, 2^-16 of it, and the product is off by 2^-22 of it at most.
constexpr uint32_t kSmallRound = 8192;
MC_HD uint32_t quotient(uint32_t x, float inv) {
  return (uint32_t)(((float)x + 0.5f) * inv);
}

MC_HD Piece piece_of(const RoundPart& pt, const CfgRec& r, uint32_t m, uint32_t piece,
                     uint32_t nth) {
  Piece v;
  v.m = m;
  v.all = (1u << m) - 1u;
  v.n = r.n;
  v.b = r.b;
  v.closure = (pt.cfg_flags & kRpClosure) != 0u;
  v.extra = (pt.cfg_flags & kRpEndExtra) != 0u;
  v.partial = (pt.cfg_flags & kRpPartial) != 0u;
  v.r0 = pt.r0;
  v.nfull = v.closure ? pt.a : (v.partial ? 0u : 1u);
  v.ja = v.closure ? 0u : pt.a;
  v.jb = pt.jb;
  v.cl = v.closure ? v.all : 0u;
  v.per = v.cl + (v.jb - v.ja) + (v.extra ? 1u : 0u);
  v.F = v.nfull * v.per;
  v.xloc = v.extra ? v.per - 1u : 0xFFFFFFFFu;
  v.slot0 = pt.slot0;
  v.link = pt.link;
  v.sets = 0;
  v.choices = 1;
  v.p = 0;
  if (v.partial) {
    v.p = r.n % m;
    for (uint32_t j = 1; j <= v.p; ++j) {
      v.choices = v.choices * (m - j + 1u) / j;
      v.sets += v.choices;
    }
  }
  const uint32_t items =
      v.F + (v.partial ? (v.closure ? v.sets : 0u) + v.choices * (v.jb - v.ja) : 0u);
  // the last states of a partial round's runs are one state: they share a piece
  const uint32_t group = v.partial && v.jb == r.b ? v.choices : 1u;
  v.i0 = nth * piece;
  v.last = items - v.i0 <= piece + group;  // nth + 1 >= (items - group) / piece
  v.i1 = v.last ? items : v.i0 + piece;
  v.per_inv = inverse(v.per);
  v.q0 = v.i0 < v.F ? v.i0 / v.per : v.nfull;
  v.loc0 = v.i0 - v.q0 * v.per;
  // (a piece reaches into one more round at most where rounds are longer than it)
  const uint32_t x1 = v.i1 - 1u - v.i0 + v.loc0;
  v.q1 = v.i1 > v.F               ? v.nfull
         : v.per <= kSmallRound ? v.q0 + quotient(x1, v.per_inv)
                                : v.q0 + (x1 >= v.per ? 1u : 0u);
  v.choices_inv = inverse(v.choices);
  const uint32_t runs = v.F + (v.closure ? v.sets : 0u);
  v.y0 = v.i0 > runs ? v.i0 : runs;
  v.jj0 = v.l0 = 0u;
  if (v.partial && v.i0 > runs) {
    v.jj0 = (v.i0 - runs) / v.choices;
    v.l0 = v.i0 - runs - v.jj0 * v.choices;
  }
  const uint32_t after = (v.r0 + v.q1 + 1u) * m;
  v.pmin = r.n > after ? r.n - after : 0u;
  return v;
}

struct RoundItem {
  uint32_t q;        // its round, from the piece's first
  uint32_t mask, j;  // the started units; the run state (closure: none)
  uint32_t slot;
  bool is_cl, is_leaf;
};

// Item i of the full rounds (i < F).
MC_HD RoundItem full_item(const Piece& v, uint32_t i) {
  RoundItem t;
  t.slot = v.slot0 + i;
  const uint32_t x = i - v.i0 + v.loc0;
  uint32_t loc;
  if (v.per <= kSmallRound) {
    t.q = quotient(x, v.per_inv);
    loc = x - mul24(t.q, v.per);
  } else {
    t.q = x >= v.per ? 1u : 0u;
    loc = x - (t.q ? v.per : 0u);
  }
  t.is_cl = loc < v.cl;
  t.mask = t.is_cl ? loc + 1u : v.all;
  t.is_leaf = loc + 1u == v.cl;
  t.j = v.ja + loc - v.cl;
  t.j = loc == v.xloc ? v.b - 1u : t.j;
  return t;
}

// Item i of the partial round (i >= F).  masks: its closure sets by size and value.
MC_HD RoundItem part_item(const Piece& v, uint32_t i, const uint8_t* masks) {
  RoundItem t;
  t.slot = v.slot0 + i;
  const uint32_t y = i - v.F, s = v.closure ? v.sets : 0u;
  t.q = v.nfull - v.q0;
  t.is_cl = y < s;
  // run states and choices from those of the piece's first run item
  const uint32_t z = t.is_cl ? 0u : i - v.y0 + v.l0, jj = quotient(z, v.choices_inv);
  const uint32_t l = z - jj * v.choices;
  t.j = v.ja + v.jj0 + jj;
  t.mask = i < v.i1 ? (uint32_t)masks[t.is_cl ? y : v.sets - v.choices + l] : 0u;
  t.is_leaf = t.is_cl && y + v.choices >= v.sets;
  if (!t.is_cl && t.j + 1u == v.b) t.slot -= l;  // the runs' one last state
  return t;
}

// The slots that an item's links name: of the all-idle state its round starts from (not known
// in a slice, whose partition holds the round's leaf instead), and of the dispatch leaf its
// run starts from.
struct ItemLinks {
  uint32_t root, leaf;
};

MC_HD ItemLinks links_of(const Piece& v, uint32_t i, uint32_t q) {
  ItemLinks k;
  if (i < v.F) {
    const uint32_t first = (v.q0 + q) * v.per;
    k.root = !v.closure ? kParentNone : first ? v.slot0 + first - 1u : v.link;
    k.leaf = v.closure ? v.slot0 + first + v.cl - 1u : v.link;
  } else {
    const uint32_t y = i - v.F, s = v.closure ? v.sets : 0u;
    const uint32_t l = y < s ? 0u : (y - s) % v.choices;
    k.root = !v.closure ? kParentNone : v.F ? v.slot0 + v.F - 1u : v.link;
    k.leaf = v.closure ? v.slot0 + v.F + v.sets - v.choices + l : v.link + l;
  }
  return k;
}

// Path length from the root to the state of item i.  Along a partition's items it falls only
// among the closure sets of one round, which are all at one clock, so all new or none, and
// end on the deepest: over a query, the last new items of its pieces hold the deepest state.
MC_HD uint32_t depth_of(const Piece& v, uint32_t i, const uint8_t* masks) {
  const RoundItem t = i < v.F ? full_item(v, i) : part_item(v, i, masks);
  return 1u + (v.r0 + v.q0 + t.q) * (v.m + v.b) + bits_set(t.mask) + (t.is_cl ? 0u : t.j + 1u);
}

// The place of set x in a partial round's closure list: sets of fewer units first, then by
// value.
MC_HD uint32_t mask_rank(uint32_t x, uint32_t all) {
  const uint32_t nx = bits_set(x);
  uint32_t at = 0;
  for (uint32_t y = 1; y <= all; ++y) {
    const uint32_t ny = bits_set(y);
    at += (ny < nx || (ny == nx && y < x)) ? 1u : 0u;
  }
  return at;
}

// A state's code in a piece's set: exact on (pending, busy mask, time left), which is all of
// a state that differs within a piece (rounds_model checks that it fits).  item_state forms it
// for an item; this is for checks on the host.
MC_HD uint32_t state_code(const Piece& v, uint32_t pending, uint32_t busy, uint32_t rem,
                          uint32_t rem_bits) {
  return (pending - v.pmin) << (v.m + rem_bits) | rem << v.m | busy;
}

// What the states of a piece's items have in common: of configuration c, d cycles long, with keys
// that hold the pending count at bit sp and the units at bit sm.
struct ItemBase {
  uint32_t d, code_shift, sp, sm;
  uint32_t prel0;   // pending past Piece::pmin before the piece's first round
  uint32_t clock0;  // that round's clock
  uint64_t key0;
};

MC_HD ItemBase item_base(const Piece& v, uint32_t c, uint32_t d, uint32_t rem_bits, uint32_t sp,
                         uint32_t sm) {
  ItemBase b;
  b.d = d;
  b.code_shift = v.m + rem_bits;
  b.sp = sp;
  b.sm = sm;
  b.prel0 = v.n - (v.r0 + v.q0) * v.m - v.pmin;
  b.clock0 = (v.r0 + v.q0) * d;
  b.key0 = (uint64_t)c + ((uint64_t)v.pmin << sp);
  return b;
}

struct ItemState {
  uint32_t rem;    // time left
  uint32_t prel;   // pending past Piece::pmin
  uint32_t clock;  // (32 bits, as terminal clocks fit)
  uint32_t code;
  uint64_t key;
};

// An item's state; run: the time left after its run state.
MC_HD ItemState item_state(const Piece& v, const ItemBase& b, const RoundItem& it, uint32_t run) {
  ItemState s;
  s.rem = it.is_cl ? b.d : run;
  s.prel = b.prel0 - mul24(it.q, v.m) - bits_set(it.mask);
  s.clock = b.clock0 + it.q * b.d + (b.d - s.rem);
  const uint32_t low = s.rem << v.m | (s.rem ? it.mask : 0u);
  s.code = s.prel << b.code_shift | low;
  s.key = (b.key0 + (uint64_t)s.prel * (1u << b.sp)) + ((uint64_t)low << b.sm);
  return s;
}

// Where a code's probe sequence starts in a set of 2^(32 - shift) slots; it goes on 1, 2, 3, ..
// slots further at every probe, which reaches all of them.  keep: bits kept (0: all; testing
// only).  The codes of a piece are a lattice (time left by round), which a multiplication alone
// maps to another: for some operation times many lie together, and steps of one slot walk
// through all of them.  With such steps and the multiplier 0x9E3779B1, the probes of a
// wavefront's slowest lane, averaged over a piece, came to 311 at worst over 720 models of all
// kinds with operation times 1 to 42 (counted on the host), and to 2.1 - 3.4 by kind of model;
// so, to 8, and to 1.4 - 2.5.  A second multiplication takes the lattice away, and with it what
// keeps the codes of one run apart: 3 - 5.4.  min_time launch, mean (most) over 21 settings of
// the operation times, then -> now: abstract_s1024_np4_cu1 35 (184) -> 25 (27) us,
// minimum_s1024_np4_cu4 21 (40) -> 19.5 (20), matmul64_cu4 37.5 (42) -> 37.8 (40),
// matmul128_vw_cu8 246 (320) -> 227 (241).
// Windows of clocks are lattices that the first multiplier suits better (it is the chain
// engine's): 1.1 - 2.6 probes against 1.2 - 3.0.
template <uint32_t MUL = 0xEB91CE37u>
MC_HD uint32_t probe_start(uint32_t code, uint32_t shift, uint32_t keep) {
  uint32_t h = code * MUL;
  if (keep) h = ((h >> 8) & ((1u << keep) - 1u)) * MUL;
  return h >> shift;
}

// Time left after run state j of a workgroup of a configuration: d - end_at(j), with the
// phases' terms that do not depend on j taken out of the loop over a piece's items.
// Uniform phases (one operation per period, back to back, one wave): the end of operation j
// of a phase is off + j lat.  Products are of 24-bit factors (rounds_model and chain_plan check
// b; models with operations of kLongOperation cycles take GeneralEnds).
struct UniformEnds {
  uint32_t i1, i2, i3;     // first operations of the later phases (none: all-ones)
  uint32_t lat[4], left[4];  // time left = left - j lat
};

MC_HD UniformEnds uniform_ends(const CfgRec& r) {
  UniformEnds u;
  for (int j = 0; j < kMaxPhases; ++j) {
    u.lat[j] = r.lat[j];
    u.left[j] = r.d - r.t0[j] + (r.i0[j] - 1u) * r.lat[j];
  }
  u.i1 = r.nph > 1u ? r.i0[1] : 0xFFFFFFFFu;
  u.i2 = r.nph > 2u ? r.i0[2] : 0xFFFFFFFFu;
  u.i3 = r.nph > 3u ? r.i0[3] : 0xFFFFFFFFu;
  return u;
}

MC_HD uint32_t rem_after(const UniformEnds& u, uint32_t j) {
  uint32_t lat = u.lat[0], left = u.left[0];
  lat = j >= u.i1 ? u.lat[1] : lat;
  left = j >= u.i1 ? u.left[1] : left;
  lat = j >= u.i2 ? u.lat[2] : lat;
  left = j >= u.i2 ? u.left[2] : left;
  lat = j >= u.i3 ? u.lat[3] : lat;
  left = j >= u.i3 ? u.left[3] : left;
  return left - mul24(j, lat);
}

// Any phases: waves of dw cycles with bw ends; phases of one or two operations per period.
struct GeneralEnds {
  uint32_t bw, recip, dw, d;  // recip = floor(2^32 / bw)
  uint32_t i1, i2, i3;
  uint32_t i0[4], t0[4], lat[4], la[4];
};

MC_HD GeneralEnds general_ends(const CfgRec& r) {
  GeneralEnds u;
  u.bw = r.bw;
  u.recip = r.bw > 1u ? (uint32_t)((1ull << 32) / r.bw) : 0xFFFFFFFFu;
  u.dw = r.dw;
  u.d = r.d;
  for (int j = 0; j < kMaxPhases; ++j) {
    u.i0[j] = r.i0[j];
    u.t0[j] = r.t0[j];
    u.lat[j] = r.lat[j];
    u.la[j] = r.la[j];
  }
  u.i1 = r.nph > 1u ? r.i0[1] : 0xFFFFFFFFu;
  u.i2 = r.nph > 2u ? r.i0[2] : 0xFFFFFFFFu;
  u.i3 = r.nph > 3u ? r.i0[3] : 0xFFFFFFFFu;
  return u;
}

MC_HD uint32_t rem_after(const GeneralEnds& u, uint32_t j) {
  uint32_t w = (uint32_t)(((uint64_t)j * u.recip) >> 32);  // j / bw, or one less
  uint32_t k = j - mul24(w, u.bw);
  if (k >= u.bw) {
    k -= u.bw;
    ++w;
  }
  uint32_t i0 = u.i0[0], t0 = u.t0[0], lat = u.lat[0], la = u.la[0];
  i0 = k >= u.i1 ? u.i0[1] : i0;
  t0 = k >= u.i1 ? u.t0[1] : t0;
  lat = k >= u.i1 ? u.lat[1] : lat;
  la = k >= u.i1 ? u.la[1] : la;
  i0 = k >= u.i2 ? u.i0[2] : i0;
  t0 = k >= u.i2 ? u.t0[2] : t0;
  lat = k >= u.i2 ? u.lat[2] : lat;
  la = k >= u.i2 ? u.la[2] : la;
  i0 = k >= u.i3 ? u.i0[3] : i0;
  t0 = k >= u.i3 ? u.t0[3] : t0;
  lat = k >= u.i3 ? u.lat[3] : lat;
  la = k >= u.i3 ? u.la[3] : la;
  const uint32_t q = k - i0, half = la ? 1u : 0u;
  // one operation per period: t0 + (q + 1) lat; two: t0 + (q / 2) lat + (la, then lat)
  const uint32_t step = half && !(q & 1u) ? la : lat;
  return u.d - w * u.dw - t0 - (q >> half) * lat - step;
}

}  // namespace mc
