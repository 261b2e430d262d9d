// Walks every piece of a round-engine plan on the host, with the arithmetic the kernel uses,
// and prints what it found: one line per model read from stdin.
//
// Input, one model per line: kind m s0 s1 s2 Lg Ll Lc Lb target piece floor T n_cfg, then
// n_cfg rows of 4 parameters.  The plan is trimmed to clocks in [floor, T] unless T is
// 4294967295.  Output: "ok states slots" or what is wrong.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <set>
#include <unordered_set>
#include <vector>

#include "mc_model.h"
#include "mc_rounds.h"

using namespace mc;

int main() {
  mc_desc d;
  for (;;) {
    std::memset(&d, 0, sizeof(d));
    unsigned long long target, floor, T;
    unsigned piece;
    if (std::scanf("%u %u %u %u %u %u %u %u %u %llu %u %llu %llu %u", &d.kind, &d.n_cu, &d.size[0],
                   &d.size[1], &d.size[2], &d.lat_global, &d.lat_local, &d.lat_compute,
                   &d.lat_barrier, &target, &piece, &floor, &T, &d.n_cfg) != 14)
      return 0;
    std::vector<uint32_t> params(4ull * d.n_cfg);
    for (auto& p : params)
      if (std::scanf("%u", &p) != 1) return 1;
    d.params = params.data();
    ModelHost h;
    std::string err;
    if (build_model(&d, &h, &err)) {
      std::printf("invalid %s\n", err.c_str());
      continue;
    }
    if (!rounds_model(h)) {
      std::printf("not a round-engine model\n");
      continue;
    }
    std::vector<PartPlan> plan;
    plan_parts(h, target, &plan);
    RoundPlan base, own;
    round_plan(h, 0, plan, &base);
    const RoundPlan* rp = &base;
    if (T != 0xFFFFFFFFull) {
      trim_rounds(h, base, floor, T, &own);
      rp = &own;
    }
    const uint64_t pieces = number_pieces(const_cast<RoundPlan*>(rp), piece);
    // slot -> key, over all pieces: a slot belongs to one piece and one state
    std::vector<uint64_t> key(base.used, ~0ull);
    std::vector<uint32_t> owner(base.used, ~0u);
    uint64_t states = 0;
    const char* bad = nullptr;
    uint32_t deepest = 0, claimed = 0;  // over all states; over every piece's last new item
    std::unordered_set<uint64_t> seen;
    for (size_t i = 0; i < rp->parts.size() && !bad; ++i) {
      const RoundPart& pt = rp->parts[i];
      const uint32_t c = pt.cfg_flags & kRpCfg;
      const CfgRec& r = h.cfgs[c];
      const uint32_t rb = code_rem_bits(r);
      const uint64_t last = i + 1 < rp->parts.size() ? rp->parts[i + 1].piece0 : pieces;
      uint64_t items = 0;
      for (uint64_t q = pt.piece0; q < last && !bad; ++q) {
        const Piece v = piece_of(pt, r, h.m, piece, (uint32_t)(q - pt.piece0));
        if (v.i0 != items || v.i1 <= v.i0 || v.i1 > rp->items[i]) bad = "item ranges";
        items = v.i1;
        uint8_t masks[256];
        if (v.partial)
          for (uint32_t x = 1; x <= v.all; ++x) masks[mask_rank(x, v.all)] = (uint8_t)x;
        std::unordered_set<uint32_t> set;
        uint32_t last_new = 0;
        for (uint32_t k = v.i0; k < v.i1 && !bad; ++k) {
          const RoundItem t = k < v.F ? full_item(v, k) : part_item(v, k, masks);
          if (t.is_cl ? false : t.j >= r.b) { bad = "run state"; break; }
          const uint32_t round = v.r0 + v.q0 + t.q;
          const ItemLinks lk = links_of(v, k, t.q);
          if (!t.is_cl && (rem_after(general_ends(r), t.j) != r.d - end_at_host(r, t.j) ||
                           (!h.general &&
                            rem_after(uniform_ends(r), t.j) != r.d - end_at_host(r, t.j))))
            bad = "time left";
          const uint32_t e = t.is_cl ? 0u : (uint32_t)end_at_host(r, t.j);
          const uint32_t rem = r.d - e, ns = bits_set(t.mask), busy = rem ? t.mask : 0u;
          const uint64_t clock = (uint64_t)round * r.d + e;
          const uint64_t pend64 = (uint64_t)r.n - (uint64_t)round * h.m - ns;
          if (pend64 > r.n) { bad = "pending"; break; }
          const uint32_t pending = (uint32_t)pend64;
          if (T != 0xFFFFFFFFull && clock > T) continue;
          const uint32_t code = state_code(v, pending, busy, rem, rb);
          if (code == 0xFFFFFFFFu || pending < v.pmin ||
              ((uint64_t)(pending - v.pmin) << (h.m + rb)) >> 32)
            bad = "code range";
          if (t.slot < 1 + h.n_cfg || t.slot >= base.used || (lk.root >= base.used && (v.closure || lk.root != kParentNone)) ||
              lk.leaf >= base.used)
            bad = "slot range";
          if (bad) break;
          uint32_t f[kFields] = {0};
          f[kFCfg] = c;
          f[kFPending] = pending;
          for (uint32_t u = 0; u < h.m; ++u) f[kFRem + u] = (busy >> u) & 1u ? rem : 0u;
          uint64_t w[4];
          encode_key_host(h.layout, f, w);
          uint32_t back[kFields];
          decode_key_host(h.layout, w, back, h.cfgs.data());
          if (back[kFClock] != clock) bad = "clock";
          const bool fresh = set.insert(code).second;
          if (fresh != seen.insert(w[0]).second) bad = "a state in two pieces, or a code of two";
          if (fresh) {
            const uint32_t dep = 1 + round * (h.m + r.b) + ns + (t.is_cl ? 0 : t.j + 1);
            deepest = std::max(deepest, dep);
            last_new = k;
            if (owner[t.slot] != ~0u) bad = "slot of two states";
            owner[t.slot] = (uint32_t)q;
            key[t.slot] = w[0];
            if (floor == 0 || clock >= floor) ++states;
          } else if (owner[t.slot] != q || key[t.slot] != w[0]) {
            bad = "a state's second slot";
          }
        }
        if (set.size() > piece + 1u) bad = "set size";
        if (!bad && !set.empty()) claimed = std::max(claimed, depth_of(v, last_new, masks));
      }
      if (!bad && items != rp->items[i]) bad = "items";
    }
    if (!bad && claimed != deepest) bad = "depth";
    // links: a leaf's root is the idle state its round starts from, a round's end's leaf the
    // full set of its round
    for (size_t i = 0; i < rp->parts.size() && !bad && T == 0xFFFFFFFFull; ++i) {
      const RoundPart& pt = rp->parts[i];
      const uint32_t c = pt.cfg_flags & kRpCfg;
      const CfgRec& r = h.cfgs[c];
      const uint64_t last = i + 1 < rp->parts.size() ? rp->parts[i + 1].piece0 : pieces;
      for (uint64_t q = pt.piece0; q < last && !bad; ++q) {
        const Piece v = piece_of(pt, r, h.m, piece, (uint32_t)(q - pt.piece0));
        uint8_t masks[256];
        if (v.partial)
          for (uint32_t x = 1; x <= v.all; ++x) masks[mask_rank(x, v.all)] = (uint8_t)x;
        for (uint32_t k = v.i0; k < v.i1 && !bad; ++k) {
          const RoundItem t = k < v.F ? full_item(v, k) : part_item(v, k, masks);
          const uint32_t round = v.r0 + v.q0 + t.q;
          const ItemLinks lk = links_of(v, k, t.q);
          uint32_t f[kFields] = {0};
          uint64_t w[4];
          if (t.is_leaf) {
            f[kFCfg] = c;
            f[kFPending] = r.n - round * h.m;
            encode_key_host(h.layout, f, w);
            const bool select = lk.root == 1 + c && round == 0;
            if (!select && key[lk.root] != w[0]) bad = "root link";
          }
          if (!t.is_cl && t.j + 1 == r.b) {
            f[kFCfg] = c;
            f[kFPending] = r.n - round * h.m - bits_set(t.mask);
            for (uint32_t u = 0; u < h.m; ++u) f[kFRem + u] = (t.mask >> u) & 1u ? r.d : 0u;
            encode_key_host(h.layout, f, w);
            if (key[lk.leaf] != w[0]) bad = "leaf link";
          }
        }
      }
    }
    if (bad) std::printf("bad %s\n", bad);
    else std::printf("ok %llu %llu\n", (unsigned long long)(states + (floor ? 0 : 1 + h.n_cfg)),
                     (unsigned long long)base.used);
  }
}
