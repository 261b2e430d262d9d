// Walks every piece of a chain-engine plan on the host, with the arithmetic the kernel uses,
// and compares the states with a breadth-first search of the model.
//
// Input, one model per line: kind m s0 s1 s2 Lg Ll Lc Lb target T n_cfg, m speeds, then n_cfg
// rows of 4 parameters.  The pieces stop at clock T.  Output: "ok states slots items" or what
// is wrong.
#include <algorithm>
#include <array>
#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <vector>

#include "mc_chains.h"
#include "mc_model.h"

using namespace mc;

namespace {

struct Ends {
  const CfgRec& r;
  uint32_t at(uint32_t j) const { return (uint32_t)end_at_host(r, j); }
  uint32_t upto(uint32_t x) const { return (uint32_t)ends_le(r, x); }
};

typedef std::array<uint32_t, 2 + kMaxCU> State;  // clock, pending, time left per unit

// Every state of configuration r with clock <= T, its SELECT state included.
std::set<State> search(const CfgRec& r, const ModelHost& h, uint32_t T) {
  std::set<State> seen;
  State s{};
  s[1] = r.n;
  std::vector<State> todo{s};
  seen.insert(s);
  const auto push = [&](const State& y) {
    if (y[0] <= T && seen.insert(y).second) todo.push_back(y);
  };
  while (!todo.empty()) {
    const State x = todo.back();
    todo.pop_back();
    uint32_t idle = 0, busy = 0;
    for (uint32_t u = 0; u < h.m; ++u) (x[2 + u] ? busy : idle) |= 1u << u;
    if (x[1] && idle) {
      for (uint32_t u = 0; u < h.m; ++u)
        if ((idle >> u) & 1u) {
          State y = x;
          --y[1];
          y[2 + u] = h.speed[u] * r.d;
          push(y);
        }
      continue;
    }
    if (!busy) continue;
    uint32_t step = ~0u;  // to the next operation end of any busy unit
    for (uint32_t u = 0; u < h.m; ++u)
      if (x[2 + u]) {
        const uint32_t e = h.speed[u] * r.d - x[2 + u];
        const uint32_t k = (uint32_t)ends_le(r, e / h.speed[u]);
        step = std::min(step, h.speed[u] * (uint32_t)end_at_host(r, k) - e);
      }
    State y = x;
    y[0] += step;
    for (uint32_t u = 0; u < h.m; ++u) y[2 + u] -= x[2 + u] ? step : 0u;
    push(y);
  }
  return seen;
}

}  // namespace

int main() {
  mc_desc d;
  for (;;) {
    std::memset(&d, 0, sizeof(d));
    unsigned long long target, T;
    if (std::scanf("%u %u %u %u %u %u %u %u %u %llu %llu %u", &d.kind, &d.n_cu, &d.size[0],
                   &d.size[1], &d.size[2], &d.lat_global, &d.lat_local, &d.lat_compute,
                   &d.lat_barrier, &target, &T, &d.n_cfg) != 12)
      return 0;
    std::vector<uint32_t> speed(d.n_cu);
    for (auto& v : speed)
      if (std::scanf("%u", &v) != 1) return 1;
    d.unit_speed = speed.data();
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
    ChainPlan plan;
    chain_plan(h, 1ull << 31, target, &plan);
    if (!plan.ok()) {
      std::printf("not a chain-engine model\n");
      continue;
    }
    const ChainTail* tails = reinterpret_cast<const ChainTail*>(plan.blob.data() + plan.tails_at);
    const uint32_t* sets = plan.blob.data() + plan.sets_at;
    std::vector<char> taken(plan.used, 0);
    const char* bad = nullptr;
    uint64_t states = 1 + d.n_cfg, items = 0, pieces = 0;
    for (uint32_t c = 0; c < d.n_cfg && !bad; ++c) {
      const ChainCfg x = plan.cfgs()[c];
      const CfgRec& r = h.cfgs[c];
      const Ends ends{r};
      const ChainEnv g = chain_env(r, h.layout.speed, h.m, plan.lcm, sets);
      std::set<State> found;  // over the pieces: a state comes from one of them
      const uint32_t n = x.windows + x.tail_n * x.tsub;
      if (x.piece0 != pieces) bad = "pieces are not numbered one after another";
      pieces += n;
      for (uint32_t local = 0; local < n && !bad; ++local) {
        const ChainSpan s = chain_span(x, g, local, (uint32_t)T);
        std::map<uint32_t, State> piece;  // by code
        for (uint32_t from = s.t0, to; from < s.t1 && !bad; from = to) {
          ChainWindow w;
          uint32_t whole[kMaxCU] = {0};
          std::vector<uint32_t> masks;
          for (to = s.t1;; to = from + (to - from) / 2) {
            w.t0 = from;
            w.t1 = to;
            if (s.tail) {
              for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u)
                whole[u] = u < h.m ? tail_window_unit(w, x, g, ends, s.interval, u, g.speed[u],
                                                      (tail_listed(x, g) >> u) & 1u)
                                   : (w.count[u] = w.first[u] = w.slot[u] = 0u);
              tail_window_rest(w, x, g, tails[x.tail0 + s.interval], s.interval, whole);
              masks.clear();
              for (uint32_t b = 0; b < 1u << bits_set(w.alive); ++b) {
                const uint32_t set = spread_bits(b, w.alive);
                if (tail_set(x.p, w.dead_n, set)) masks.push_back(set);
              }
              w.items = (uint32_t)masks.size() * w.before[kMaxCU];
            } else {
              for (uint32_t u = 0; u < (uint32_t)kMaxCU; ++u)
                chain_window_unit(w, x, g, ends, u, g.speed[u], x.unit_off[u]);
              chain_window_rest(w, x, g);
            }
            if (w.items <= kChainCap) break;
            if (to - from == 1) {
              bad = "one clock has more items than a window holds";
              break;
            }
          }
          items += w.items;
          for (uint32_t i = 0; i < w.items && !bad; ++i) {
            ChainItem it;
            if (s.tail) {
              const uint32_t per = w.before[kMaxCU], rank = i / per;
              h.m <= 4 ? tail_item<4>(w, x, g, ends, i - rank * per, rank, masks[rank], &it)
                       : tail_item<kMaxCU>(w, x, g, ends, i - rank * per, rank, masks[rank], &it);
            } else {
              h.m <= 4 ? chain_item<4>(w, x, g, ends, r.n, i, &it)
                       : chain_item<kMaxCU>(w, x, g, ends, r.n, i, &it);
            }
            if (it.slot < 1 + d.n_cfg || it.slot >= plan.used || taken[it.slot]++) {
              bad = "a slot is out of range or has two items";
              break;
            }
            if (!it.active) continue;
            if (it.t >= to - from) bad = "a clock is outside its window";
            State y{};
            y[0] = from + it.t;
            y[1] = it.pending;
            uint32_t busy = 0;
            for (uint32_t u = 0; u < h.m; ++u) {
              y[2 + u] = it.rem[u];
              if (it.rem[u]) busy |= 1u << u;
            }
            if (busy != it.busy) bad = "busy units";
            const uint32_t code = (y[0] - s.t0) << h.m | busy;
            if (code >> h.m != y[0] - s.t0) bad = "a code does not fit";
            auto ins = piece.emplace(code, y);
            if (!ins.second && ins.first->second != y) bad = "two states have one code";
          }
        }
        for (auto& kv : piece)
          if (!found.insert(kv.second).second) bad = "a state comes from two pieces";
      }
      if (bad) break;
      State sel{};
      sel[1] = r.n;
      found.insert(sel);
      const std::set<State> want = search(r, h, (uint32_t)T);
      if (found != want) {
        std::printf("cfg %u: %zu states, search %zu; ", c, found.size(), want.size());
        for (auto& y : want)
          if (!found.count(y)) {
            std::printf("missing clock %u pending %u", y[0], y[1]);
            break;
          }
        for (auto& y : found)
          if (!want.count(y)) {
            std::printf("extra clock %u pending %u", y[0], y[1]);
            break;
          }
        bad = " states differ";
      }
      states += found.size() - 1;
    }
    if (!bad && pieces != plan.n_pieces) bad = "pieces";
    if (bad) std::printf("%s\n", bad);
    else
      std::printf("ok %llu %llu %llu\n", (unsigned long long)states,
                  (unsigned long long)plan.used, (unsigned long long)items);
  }
}
