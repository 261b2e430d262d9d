// What k_rounds makes of every item of a plan: the state, its code and its packed key as the
// kernel forms them (item_state), against the state that the round structure gives, packed by
// encode_key_host; and the links of a plan, trimmed to a range of clocks or not, against the
// states that the whole plan holds in the slots they name.
//
// Input, one model per line: kind m s0 s1 s2 Lg Ll Lc Lb target piece floor T n_cfg, then n_cfg
// rows of 4 parameters.  Output: "ok items links" or what is wrong.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

#include "mc_model.h"
#include "mc_rounds.h"

using namespace mc;

namespace {

struct State {
  uint32_t round, pending, busy, rem;
  uint64_t clock;
};

State state_of(const RoundItem& t, const Piece& v, const CfgRec& r) {
  State s;
  s.round = v.r0 + v.q0 + t.q;
  const uint32_t end = t.is_cl ? 0u : (uint32_t)end_at_host(r, t.j);
  s.rem = r.d - end;
  s.busy = s.rem ? t.mask : 0u;
  s.pending = r.n - s.round * v.m - bits_set(t.mask);
  s.clock = (uint64_t)s.round * r.d + end;
  return s;
}

uint64_t key_of(const ModelHost& h, uint32_t c, uint32_t pending, uint32_t busy, uint32_t rem) {
  uint32_t f[kFields] = {0};
  f[kFCfg] = c;
  f[kFPending] = pending;
  for (uint32_t u = 0; u < h.m; ++u) f[kFRem + u] = (busy >> u) & 1u ? rem : 0u;
  uint64_t w[4];
  encode_key_host(h.layout, f, w);
  return w[0];
}

// f(part, piece, item number, item) for every item of the plan
template <class F>
void each_item(const ModelHost& h, RoundPlan* p, uint32_t piece, const F& f) {
  const uint64_t pieces = number_pieces(p, piece);
  for (size_t i = 0; i < p->parts.size(); ++i) {
    const RoundPart& pt = p->parts[i];
    const CfgRec& r = h.cfgs[pt.cfg_flags & kRpCfg];
    const uint64_t last = i + 1 < p->parts.size() ? p->parts[i + 1].piece0 : pieces;
    for (uint64_t q = pt.piece0; q < last; ++q) {
      const Piece v = piece_of(pt, r, h.m, piece, (uint32_t)(q - pt.piece0));
      uint8_t masks[256];
      if (v.partial)
        for (uint32_t x = 1; x <= v.all; ++x) masks[mask_rank(x, v.all)] = (uint8_t)x;
      for (uint32_t k = v.i0; k < v.i1; ++k)
        f(pt, v, k, k < v.F ? full_item(v, k) : part_item(v, k, masks));
    }
  }
}

}  // namespace

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
    if (build_model(&d, &h, &err) || !rounds_model(h)) {
      std::printf("not a round-engine model\n");
      continue;
    }
    std::vector<PartPlan> plan;
    plan_parts(h, target, &plan);
    RoundPlan whole, own;
    round_plan(h, 0, plan, &whole);
    const char* bad = nullptr;
    // the slots of the whole plan: the root, the SELECT states, the items
    std::vector<uint64_t> key(whole.used, ~0ull);
    for (uint32_t c = 0; c < h.n_cfg; ++c) key[1 + c] = key_of(h, c, h.cfgs[c].n, 0u, 0u);
    each_item(h, &whole, piece, [&](const RoundPart& pt, const Piece& v, uint32_t, const RoundItem& t) {
      const uint32_t c = pt.cfg_flags & kRpCfg;
      const State s = state_of(t, v, h.cfgs[c]);
      key[t.slot] = key_of(h, c, s.pending, s.busy, s.rem);
    });
    if (T == 0xFFFFFFFFull) own = whole;
    else trim_rounds(h, whole, floor, T, &own);
    const uint32_t sp = h.layout.shift[kFPending], sm = h.layout.shift[kFRem];
    uint64_t items = 0, links = 0;
    each_item(h, &own, piece, [&](const RoundPart& pt, const Piece& v, uint32_t k, const RoundItem& t) {
      const uint32_t c = pt.cfg_flags & kRpCfg;
      const CfgRec& r = h.cfgs[c];
      const State s = state_of(t, v, r);
      if (s.clock > T) return;  // (a test of its own in the kernel, on a clock that is checked)
      ++items;
      const uint32_t run = h.general ? rem_after(general_ends(r), t.j) : rem_after(uniform_ends(r), t.j);
      const ItemState x = item_state(v, item_base(v, c, r.d, code_rem_bits(r), sp, sm), t, run);
      if (x.rem != s.rem || x.prel + v.pmin != s.pending || x.clock != s.clock) bad = "state";
      if (x.code != state_code(v, s.pending, s.busy, s.rem, code_rem_bits(r))) bad = "code";
      if (x.key != key_of(h, c, s.pending, s.busy, s.rem)) bad = "key";
      if (x.key != key[t.slot]) bad = "slot";
      if (x.rem != 0u && !t.is_leaf) return;
      ++links;
      const ItemLinks l = links_of(v, k, t.q);
      const uint64_t root = key_of(h, c, r.n - s.round * h.m, 0u, 0u);
      if (l.root != kParentNone && (l.root >= whole.used || key[l.root] != root)) bad = "root link";
      if (l.root == kParentNone && v.closure) bad = "no root link";
      if (x.rem) return;
      const uint64_t leaf = key_of(h, c, s.pending, t.mask, r.d);
      if (l.leaf >= whole.used || key[l.leaf] != leaf) bad = "leaf link";
    });
    if (bad) std::printf("bad %s\n", bad);
    else std::printf("ok %llu %llu\n", (unsigned long long)items, (unsigned long long)links);
  }
}
