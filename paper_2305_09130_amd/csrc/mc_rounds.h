// mc_rounds.h -- which states a piece of the round engine generates: the arithmetic from an
// item's number to its state and slots, for the kernel and for checks on the host.
#pragma once

#include <stdint.h>

#include "mc_model.h"

#ifdef __HIP__
#define MC_HD __host__ __device__ __forceinline__
#else
#define MC_HD inline
#endif

namespace mc {

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
  uint32_t magic;            // reciprocal of per, for items of the piece
  uint32_t pmin;             // least pending count of the piece's states
  bool closure, extra, partial;
};

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
  uint32_t pieces = (items - group + piece - 1u) / piece;
  pieces = pieces ? pieces : 1u;
  v.i0 = nth * piece;
  v.i1 = nth + 1u == pieces ? items : v.i0 + piece;
  v.q0 = v.i0 < v.F ? v.i0 / v.per : v.nfull;
  v.loc0 = v.i0 - v.q0 * v.per;
  v.q1 = v.i1 > v.F ? v.nfull : (v.i1 - 1u) / v.per;
  // an item's place past loc0 is below kMaxPiece + 70 + per: exact for per up to 2^13 (0 for
  // per = 1, a slice of one state), and beyond that a piece reaches into one more round at
  // most
  v.magic = v.per <= 8192u ? 0xFFFFFFFFu / v.per + 1u : 0u;
  const uint32_t after = (v.r0 + v.q1 + 1u) * m;
  v.pmin = r.n > after ? r.n - after : 0u;
  return v;
}

struct RoundItem {
  uint32_t round, mask, j;  // mask: the started units; j: the run state (closure: none)
  uint32_t slot, root, leaf;
  bool is_cl, is_leaf;
};

// Item i of the full rounds (i < F).
MC_HD RoundItem full_item(const Piece& v, uint32_t i) {
  RoundItem t;
  t.slot = v.slot0 + i;
  const uint32_t x = i - v.i0 + v.loc0;
  const uint32_t q = v.magic ? (uint32_t)(((uint64_t)x * v.magic) >> 32) : (x >= v.per ? 1u : 0u);
  const uint32_t loc = x - q * v.per, first = (v.q0 + q) * v.per;
  t.round = v.r0 + v.q0 + q;
  t.is_cl = loc < v.cl;
  t.mask = t.is_cl ? loc + 1u : v.all;
  t.is_leaf = t.is_cl && loc + 1u == v.cl;
  t.j = v.ja + loc - v.cl;
  if (v.extra && loc + 1u == v.per) t.j = v.b - 1u;
  t.root = first ? v.slot0 + first - 1u : v.link;
  t.leaf = v.closure ? v.slot0 + first + v.cl - 1u : v.link;
  return t;
}

// Item i of the partial round (i >= F).  masks: its closure sets by size and value.
MC_HD RoundItem part_item(const Piece& v, uint32_t i, const uint8_t* masks) {
  RoundItem t;
  t.slot = v.slot0 + i;
  const uint32_t y = i - v.F, s = v.closure ? v.sets : 0u;
  t.round = v.r0 + v.nfull;
  t.is_cl = y < s;
  const uint32_t z = t.is_cl ? 0u : y - s, jj = z / v.choices, l = z - jj * v.choices;
  t.j = v.ja + jj;
  t.mask = i < v.i1 ? (uint32_t)masks[t.is_cl ? y : v.sets - v.choices + l] : 0u;
  t.is_leaf = t.is_cl && y + v.choices >= v.sets;
  t.root = v.F ? v.slot0 + v.F - 1u : v.link;
  t.leaf = v.closure ? v.slot0 + v.F + v.sets - v.choices + l : v.link + l;
  if (!t.is_cl && t.j + 1u == v.b) t.slot -= l;  // the runs' one last state
  return t;
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
// a state that differs within a piece (rounds_model checks that it fits).
MC_HD uint32_t state_code(const Piece& v, uint32_t pending, uint32_t busy, uint32_t rem,
                          uint32_t rem_bits) {
  return (((pending - v.pmin) << v.m | busy) << rem_bits) | rem;
}

}  // namespace mc
