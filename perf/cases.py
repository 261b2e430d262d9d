"""The work users have this checker do, as cases that can be timed and compared.

A tuning query is the unit of use: load a kernel's model, find the least model time and the
configurations attaining it, take the counterexample that names the parameters, and prove
the time minimal.  The listed cases cover it at every size the repository is configured
for (81 thousand to 58 million states), on every model kind, on units alike and of unequal
speed, through each of the search drivers (one exhaustive run, bisection over check(T),
branch and bound, swarm), batched and served.  `draw` spreads over the same ranges: odd
unit counts, random parameter subsets, other sizes and latencies.

Models are plain dicts as the package takes them, with the parameter table as a uint32
array (as a caller holds it).  A seed gives the latencies; a case gives everything else.
"""
from __future__ import annotations

import functools
import itertools
import math
import random

import numpy as np
import torch  # noqa: F401  (first: the package shares the HIP runtime that torch loads)

import paper_2305_09130_amd as mc

NO_CLOCK = 0xFFFFFFFF
MAX_STATES = 58_006_261       # the largest listed model
MAX_STATES_UNEQUAL = 1_500_000
PATH_ROWS = 1 << 15           # counterexamples are padded to a common length up to this
BATCH_STATES = 1 << 20        # instances of a batch or of a served pool are at most this large


def pow2(lo: int, hi: int) -> list[int]:
    return [1 << e for e in range(lo, hi + 1)]


# ---- models --------------------------------------------------------------------------------
#
# A case names a model by its shape: kind, size, m (units), the domains of its parameters,
# optionally unit speeds and a subset of the domain.  Row order is lexicographic.

def domain(shape: dict) -> list[tuple[int, int, int, int]]:
    e = shape["size"].bit_length() - 1
    kind = shape["kind"]
    if kind == "reduction":
        rows = [(wg, ts, 0, 0) for wg, ts in
                itertools.product(pow2(0, min(e, shape["wg"])), pow2(0, shape["ts"]))]
    elif kind == "matmul":
        rows = [(x, y, t, v) for x, y, t, v in
                itertools.product(pow2(0, 4), pow2(0, 4), pow2(0, 3), pow2(0, shape["vw"]))
                if t <= shape["size"] and x <= shape["size"] and y * v <= shape["size"]]
    else:  # the paper's unit models: WG and TS from 2 to S/2
        rows = [(wg, ts, 0, 0) for wg, ts in itertools.product(pow2(1, e - 1), pow2(1, e - 1))]
    if shape.get("subset"):
        rng = random.Random(shape["subset_seed"])
        rows = sorted(rng.sample(rows, min(shape["subset"], len(rows))))
    return rows


def latencies(kind: str, seed: int) -> tuple[int, int]:
    """Global and local latency: 20..40 and 2..4 cycles; 3..40 and 1..3 on the paper's unit
    platform, whose own figures are 4 and 1."""
    if kind in ("abstract", "minimum"):
        return 3 + seed % 38, 1 + seed // 38 % 3
    return 20 + seed % 21, 2 + seed // 21 % 3


def make_model(shape: dict, seed: int) -> dict:
    kind, size = shape["kind"], shape["size"]
    lg, ll = latencies(kind, seed)
    model = {"kind": kind, "m": shape["m"], "Lg": lg, "Ll": ll, "Lc": 1, "Lb": 0,
             "params": np.array(domain(shape), dtype=np.uint32)}
    if kind == "reduction":
        model["G"] = size
    elif kind == "matmul":
        model["M"] = model["N"] = model["K"] = size
    else:
        model["S"], model["NP"] = size, 4
    if shape.get("speed"):
        model["speed"] = [int(c) for c in shape["speed"].split(",")]
    return model


def shape_of(case: dict) -> dict:
    return {k: case[k] for k in ("kind", "size", "m", "wg", "ts", "vw", "speed", "subset",
                                 "subset_seed") if k in case}


@functools.lru_cache(maxsize=8)
def mix_shapes(seed: int, count: int) -> tuple:
    """Shapes of the uneven mix: kind 50/50, size 2^6..2^12, 2, 4 or 8 units, 12..200 rows of
    the kind's domain, redrawn above 2^20 states."""
    rng = random.Random(seed)
    out = []
    while len(out) < count:
        kind = rng.choice(("reduction", "matmul"))
        while True:
            shape = {"kind": kind, "size": 1 << rng.randint(6, 12), "m": rng.choice((2, 4, 8)),
                     "wg": 10, "ts": 6, "vw": 2, "subset": rng.randint(12, 200),
                     "subset_seed": rng.randrange(1 << 30)}
            # equal units: the count does not depend on the latencies
            if count_states(make_model(shape, 0)) <= BATCH_STATES:
                out.append(shape)
                break
    return tuple(out)


def mix_models(case: dict, seed: int) -> list[dict]:
    return [make_model(s, seed * 4099 + i)
            for i, s in enumerate(mix_shapes(case["mix"], case["models"]))]


# ---- what the answers are, from the models alone --------------------------------------------
#
# On units alike every run of a configuration proceeds in lock-step rounds, so its terminals
# share one clock and its states have a closed form.

def operation_ends(model: dict, row) -> tuple[int, np.ndarray]:
    """Workgroups n and the ascending distinct operation ends E of one workgroup."""
    p0, p1, p2, p3 = (int(v) for v in row)
    lg, ll, lc, lb = model["Lg"], model["Ll"], model["Lc"], model["Lb"]
    kind = model["kind"]
    if kind == "reduction":
        n = model["G"] // p0
        ops = [(-(-model["G"] // (p0 * p1)), lg), (p0.bit_length() - 1, ll), (1, lb), (p1, lc)]
        waves = 1
    elif kind == "matmul":
        v, k = p3 or 1, model["K"]
        n = (model["M"] // p0) * (model["N"] // (p1 * v))
        ops = [(2 * k, lg), (k * (1 + v), ll), (2 * (k // p2), lb), (k * v, lc)]
        waves = 1
    else:
        s, np_ = model["S"], model["NP"]
        n = max(1, s // (p0 * p1))
        waves = max(1, p0 // np_)
        if kind == "minimum":
            ops = [(waves * p1, lg), (min(p0, np_) - 1, ll), (1, lg)]
            waves = 1
        else:
            tile, wait = ll * p1 + 1, max(0, (lg - ll) * p1)
            ops = [(1, lg * p1 + 1), (1, tile)] + [(1, wait), (1, tile)] * (s // p1 - 1)
            ops += [(1, lg + 1)]
    lens = np.concatenate([np.full(c, t, dtype=np.int64) for c, t in ops if c > 0])
    ends = np.cumsum(np.tile(lens[lens > 0], waves))
    return n, ends


class Table:
    """Per configuration: n, d, b and the closed forms, on units alike."""

    def __init__(self, model: dict):
        self.m = m = model["m"]
        self.rows = []
        seen = {}
        for row in model["params"]:
            key = tuple(int(v) for v in row)
            if key not in seen:
                seen[key] = operation_ends(model, row)
            self.rows.append(seen[key])
        self.clock = np.array([-(-n // m) * int(e[-1]) for n, e in self.rows], dtype=np.int64)
        self.depth = 1 + max(n + -(-n // m) * len(e) for n, e in self.rows)

    def count(self, T: int) -> int:
        """States with clock <= T, the root included."""
        m, total = self.m, 1
        for n, e in self.rows:
            d, q, p = int(e[-1]), n // m, n % m
            full = min(q, T // d)
            c = 1 + full * ((1 << m) - 1 + len(e))
            upto = int(np.searchsorted(e, T - full * d, side="right"))
            if full < q:
                c += (1 << m) - 1 + upto
            elif p:
                c += sum(math.comb(m, j) for j in range(1, p + 1))
                c += math.comb(m, p) * min(upto, len(e) - 1) + (1 if upto == len(e) else 0)
            total += c
        return total


def count_states(model: dict) -> int:
    try:
        return mc.mc_describe(model)["states"]
    except mc.McError:
        return 1 << 62  # not representable


def argmin_of(clocks: np.ndarray) -> np.ndarray:
    return np.flatnonzero(clocks == clocks.min()).astype(np.int64)


# ---- cases ---------------------------------------------------------------------------------

def listed() -> list[dict]:
    return [
        # A small kernel tuned interactively: launches and waits are most of its time.
        {"name": "tune_reduction_g256_cu2", "do": "tune", "kind": "reduction", "size": 256,
         "m": 2, "wg": 5, "ts": 2},
        # The paper's abstract kernel on its own platform: one unit, so single long runs.
        {"name": "tune_abstract_s1024_cu1", "do": "tune", "kind": "abstract", "size": 1024, "m": 1},
        # The paper's Minimum kernel, four units of four elements.
        {"name": "tune_minimum_s1024_cu4", "do": "tune", "kind": "minimum", "size": 1024, "m": 4},
        # An ordinary kernel: a tiled matrix product on four units, 5.15 million states.
        {"name": "tune_matmul64_cu4", "do": "tune", "kind": "matmul", "size": 64, "m": 4, "vw": 0},
        # The largest query: 300 configurations on eight units, 58 million states.
        {"name": "tune_matmul128_vw_cu8", "do": "tune", "kind": "matmul", "size": 128, "m": 8,
         "vw": 2},
        # Units of unequal speed, small: dispatch choices change the time.
        {"name": "tune_reduction_g256_cu4_unequal", "do": "tune", "kind": "reduction",
         "size": 256, "m": 4, "wg": 5, "ts": 2, "speed": "1,1,2,3"},
        # Units of unequal speed, two-word states.
        {"name": "tune_matmul32_cu4_unequal", "do": "tune", "kind": "matmul", "size": 32, "m": 4,
         "vw": 0, "speed": "1,1,2,3"},
        # The paper's own loop: a simulated run bounds the time, then bisection over check(T).
        {"name": "bisect_matmul64_cu4", "do": "bisect", "kind": "matmul", "size": 64, "m": 4,
         "vw": 0},
        # Branch and bound from a simulated run's time, on the largest model.
        {"name": "bound_matmul128_vw_cu8", "do": "bound", "kind": "matmul", "size": 128, "m": 8,
         "vw": 2},
        # Many kernels tuned at once: 512 uneven instances in one replayed launch sequence.
        {"name": "batch_512", "do": "batch", "mix": 3, "models": 512},
        # A tuning service: a burst of queries on 32 models whose states do not all fit.
        {"name": "serve_32_models", "do": "serve", "mix": 4, "models": 32, "queries": 128,
         "arena_mib": 256},
        # Incomplete search: a swarm of seeded walks, each with a bit array of its own.
        {"name": "swarm_matmul32_cu4_unequal", "do": "swarm", "kind": "matmul", "size": 32,
         "m": 4, "vw": 0, "speed": "1,1,2,3", "members": 4096, "bits": 16, "budget": 2000},
    ]


def draw(rng: random.Random) -> dict:
    do = rng.choices(("tune", "unequal", "bisect", "bound", "batch", "serve", "swarm"),
                     weights=(8, 3, 2, 2, 2, 2, 1))[0]
    if do == "batch":
        return {"do": "batch", "mix": rng.randrange(1000), "models": round(2 ** rng.uniform(3, 9))}
    if do == "serve":
        return {"do": "serve", "mix": rng.randrange(1000), "models": rng.randint(4, 32),
                "queries": round(2 ** rng.uniform(4, 7)), "arena_mib": rng.choice((128, 256, 512))}
    unequal = do in ("unequal", "swarm")
    top = MAX_STATES_UNEQUAL if unequal else MAX_STATES
    target = math.exp(rng.uniform(math.log(4000), math.log(top)))
    best = None
    for _ in range(400):  # the candidate whose state count is nearest the drawn target
        kind = rng.choice(("reduction", "matmul", "abstract", "minimum"))
        size = 1 << (rng.randint(3, 7) if kind == "matmul" else rng.randint(5, 11))
        shape = {"kind": kind, "size": size, "m": rng.randint(1, 8), "wg": rng.randint(3, 10),
                 "ts": rng.randint(2, 6), "vw": rng.randint(0, 2), "subset": rng.randint(3, 200),
                 "subset_seed": rng.randrange(1 << 30)}
        if unequal:
            shape["m"] = rng.randint(2, 4)
            shape["size"] = min(size, 512 if kind != "matmul" else 32)
            shape["speed"] = ",".join(str(rng.randint(1, 3)) for _ in range(shape["m"]))
            if len(set(shape["speed"].split(","))) == 1:
                continue
        n = count_states(make_model(shape, 0))
        if n > top or (unequal and n > 3 * target):
            continue
        off = abs(math.log(n / target))
        if best is None or off < best[0]:
            best = (off, shape)
        if off < 0.3:
            break
    case = dict(best[1], do="tune" if do == "unequal" else do)
    if do == "swarm":
        case.update(members=round(2 ** rng.uniform(8, 12)), bits=12,
                    budget=round(2 ** rng.uniform(7, 11)))
    return case


# ---- running a case ------------------------------------------------------------------------

def served_queries(case: dict, models: list[dict], seed: int) -> list[tuple[int, int, int]]:
    """(model, kind, T): half minimum queries, half checks at 0.8 to 1.5 times the minimum."""
    rng = random.Random(seed * 7919 + case["mix"])
    least = [int(Table(m).clock.min()) for m in models]
    out = []
    for _ in range(case["queries"]):
        i = rng.randrange(len(models))
        if rng.random() < 0.5:
            out.append((i, mc.MC_QUERY_CHECK, int(rng.uniform(0.8, 1.5) * least[i])))
        else:
            out.append((i, mc.MC_QUERY_MIN_TIME, 0))
    return out


def prepare(case: dict, seed: int) -> dict:
    do = case["do"]
    state = {"do": do, "case": case}
    if do == "batch":
        state["batch"] = mc.Batch(mix_models(case, seed), mc.make_batch_opts(use_graph=True))
        return state
    if do == "serve":
        models = mix_models(case, seed)
        state["engine"] = mc.Engine(case["arena_mib"] << 20)
        state["queries"] = [(models[i], kind, T)
                            for i, kind, T in served_queries(case, models, seed)]
        state["width"] = max(len(m["params"]) for m in models)
        return state
    # one handle and one workspace for query after query, as a tuning loop keeps them
    state["model"] = make_model(shape_of(case), seed)
    log2_slots = 0
    if do == "swarm":  # the members' bit arrays live in the visited set's memory
        log2_slots = max(16, (case["members"] * (1 << case["bits"]) // 8 // 8).bit_length())
    state["handle"] = mc.Model(state["model"], log2_slots=log2_slots)
    state["path_rows"] = path_rows(state["model"])
    state["seed"] = seed
    return state


def path_rows(model: dict) -> int:
    """Rows that hold any counterexample of a model, where it has just one per time; 0 on
    models where several are equally good (a last round with a choice of units, or units of
    unequal speed)."""
    if "speed" in model:
        return 0
    t = Table(model)
    return t.depth + 1 if all(n % t.m == 0 for n, _ in t.rows) else 0


def counterexample(state: dict) -> dict:
    """What the counterexample is read for, its parameters and time, and its rows where it is
    the only one (padded with -1 unless the longest is beyond reason)."""
    handle, most = state["handle"], state["path_rows"]
    rows = handle.mc_trace()
    cfg = int(rows[-1][0])
    out = {"params": np.array(handle.mc_config(cfg), dtype=np.int64), "time": int(rows[-1][1])}
    if most:
        out["rows"] = np.full((most if most <= PATH_ROWS else len(rows), rows.shape[1]), -1,
                              dtype=np.int64)
        out["rows"][:len(rows)] = rows
    return out


def attaining(configurations, width: int) -> np.ndarray:
    """The set of configurations as a mask."""
    mask = np.zeros(width, dtype=np.int64)
    mask[np.asarray(configurations, dtype=np.int64)] = 1
    return mask


def clocks_array(clocks) -> np.ndarray:
    if None in clocks:
        clocks = [NO_CLOCK if c is None else c for c in clocks]
    return np.array(clocks, dtype=np.int64)


def run(state: dict):
    do = state["do"]
    if do == "batch":
        batch = state["batch"]
        t_min, states = batch.mc_batch_min_time()
        clocks = [clocks_array(batch.mc_batch_terminal_clocks(i)) for i in range(batch.n)]
        return {"t_min": np.array(t_min, dtype=np.int64),
                "states": np.array(states, dtype=np.int64), "clocks": np.concatenate(clocks)}
    if do == "serve":
        eng = state["engine"]
        tickets = [eng.mc_engine_submit(*q) for q in state["queries"]]
        eng.drain()
        rows, argmin = [], np.zeros((len(tickets), state["width"]), dtype=np.int64)
        for k, t in enumerate(tickets):
            r = eng.mc_engine_poll(t)
            rows.append((r["status"], r["violated"], r["t_min"], r["n_argmin"], r["states"]))
            argmin[k, eng.mc_engine_argmin(t)] = 1
            eng.mc_engine_release(t)
        return {"results": np.array(rows, dtype=np.int64), "argmin": argmin}
    h, model = state["handle"], state["model"]
    h.mc_model_reload(model)
    if do == "tune":
        t_min, argmin = h.mc_min_time()
        st = h.last_stats
        out = {"t_min": t_min, "argmin": attaining(argmin, h.n_cfg),
               "clocks": clocks_array(h.mc_terminal_clocks()), "states": st["states"],
               "path": counterexample(state)}
        if "speed" not in model:  # elsewhere they depend on the order of the search
            out["levels"], out["terminals"] = st["levels"], st["terminals"]
        out["violated"] = int(h.mc_check(t_min - 1))
        out["check_states"] = h.last_stats["states"]
        return out
    if do == "bisect":
        t_min, checks = h.mc_tune_bisect(state["seed"])
        return {"t_min": t_min, "checks": checks, "states": h.last_stats["states"],
                "path": counterexample(state)}
    if do == "bound":
        t_run, _ = h.mc_simulate(state["seed"])
        t_min, argmin = h.mc_min_time_bb(t_run)
        return {"t_run": t_run, "t_min": t_min, "argmin": attaining(argmin, h.n_cfg),
                "path": counterexample(state)}
    case = state["case"]
    r = h.mc_swarm(case["members"], case["bits"], case["budget"], state["seed"])
    members = h.mc_swarm_members(case["members"])
    fields = ("walks", "trails", "steps", "best_walk_start", "best_clock", "best_cfg")
    return {"best": np.array([r["best_clock"], r["best_cfg"], r["best_member"], r["trails"],
                              r["walks"], r["steps"]], dtype=np.int64),
            "members": np.array([[m[f] for f in fields] for m in members], dtype=np.int64)}


# ---- what a pass cannot do without ---------------------------------------------------------

def work(case: dict) -> dict:
    """Bytes: every state a query has to find is written once, as its packed key.  The search
    has no floating-point operations."""
    do = case["do"]
    if do == "batch":
        models = mix_models(case, 0)
        info = [mc.mc_describe(m) for m in models]
        return {"bytes": sum(8 * i["key_words"] * i["states"] for i in info), "flops": 0}
    if do == "serve":
        # every model asked for is explored at least once
        models = mix_models(case, 0)
        total = 0
        most: dict[int, int] = {}
        for i, kind, T in served_queries(case, models, 0):
            most[i] = max(most.get(i, 0), T if kind == mc.MC_QUERY_CHECK else NO_CLOCK)
        for i, T in most.items():
            total += 8 * mc.mc_describe(models[i])["key_words"] * Table(models[i]).count(T)
        return {"bytes": total, "flops": 0}
    if do == "swarm":  # the members' bit arrays are cleared, their records written
        return {"bytes": case["members"] * ((1 << case["bits"]) // 8 + 80), "flops": 0}
    model = make_model(shape_of(case), 0)
    info = mc.mc_describe(model)
    key = 8 * info["key_words"]
    if "speed" in model:
        return {"bytes": key * info["states"], "flops": 0}
    t = Table(model)
    least = int(t.clock.min())
    below = t.count(least - 1)
    if do == "tune":
        return {"bytes": key * (info["states"] + below), "flops": 0}
    return {"bytes": key * below, "flops": 0}


def exact(case: dict, seed: int):
    do = case["do"]
    if do == "swarm" or "speed" in case:
        return None
    if do == "batch":
        tables = [Table(m) for m in mix_models(case, seed)]
        return {"t_min": np.array([t.clock.min() for t in tables], dtype=np.int64),
                "states": np.array([t.count(NO_CLOCK) for t in tables], dtype=np.int64),
                "clocks": np.concatenate([t.clock for t in tables])}
    if do == "serve":
        models = mix_models(case, seed)
        tables = [Table(m) for m in models]
        queries = served_queries(case, models, seed)
        rows = []
        argmin = np.zeros((len(queries), max(len(m["params"]) for m in models)), dtype=np.int64)
        for k, (i, kind, T) in enumerate(queries):
            t = tables[i]
            check = kind == mc.MC_QUERY_CHECK
            least = int(t.clock.min())
            met = not check or least <= T
            best = argmin_of(t.clock) if met else np.zeros(0, dtype=np.int64)
            rows.append((0, int(check and met), least if met else NO_CLOCK, len(best),
                         t.count(T if check else NO_CLOCK)))
            argmin[k, best] = 1
        return {"results": np.array(rows, dtype=np.int64), "argmin": argmin}
    model = make_model(shape_of(case), seed)
    t = Table(model)
    least = int(t.clock.min())
    best = argmin_of(t.clock)
    path = {"params": np.array(model["params"][best[0]], dtype=np.int64), "time": least}
    if path_rows(model):
        path["rows"] = None  # any order of the dispatches at one instant is a valid path
    if do == "bisect":
        return {"t_min": least, "checks": None, "states": None, "path": path}
    if do == "bound":
        return {"t_run": None, "t_min": least, "argmin": attaining(best, len(t.rows)), "path": path}
    return {"t_min": least, "argmin": attaining(best, len(t.rows)), "clocks": t.clock,
            "states": t.count(NO_CLOCK), "path": path, "levels": t.depth + 1,
            "terminals": len(t.rows), "violated": 0, "check_states": t.count(least - 1)}
