"""The chain engine (units of unequal speed) at its edges, against the CPU oracle, bit-exact:
fewer workgroups than units, tails of many choices and of none, eight units of eight speeds,
windows split because one holds too many items, operation lists of waves, more pieces than
workgroups, crowded hash sets, keys of one to four words, a period left to the other engine."""
import pytest

import oracle
import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_09130_amd as mc
    return mc


def _red(G, m, wg, ts, sp, Lg=9, Ll=2):
    return w.with_speeds(w.reduction_model(G, m, wg, ts, Lg, Ll), sp)


CASES = {
    "fewer_workgroups_than_units": (_red(64, 8, [16, 32, 64], [1, 2], [1, 2, 3, 1, 2, 3, 1, 2]), {}),
    "one_workgroup": (_red(64, 3, [64], [1], [3, 1, 2]), {}),
    "eight_speeds": (_red(256, 8, [1, 2, 4], [1, 4], [8, 7, 6, 5, 4, 3, 2, 1]), {}),
    "many_choices": (_red(128, 8, [2, 4, 8], [1, 2], [1, 1, 1, 1, 1, 1, 1, 2]), {}),
    "no_unit_idle_alone": (_red(256, 2, [1, 2], [1], [2, 4]), {}),
    "slow_unit": (_red(128, 4, [1, 4], [1], [64, 1, 1, 1]), {}),
    "split_windows": (w.with_speeds(w.matmul_model(16, 16, 256, 3, [16], [1], [1], [1], 23, 3),
                                    [1, 2, 3]), {"part_states": 2048}),
    "more_pieces_than_workgroups": (_red(512, 3, [1, 2], [1, 2], [1, 2, 3]),
                                    {"part_states": 32, "grid": 3}),
    "crowded_sets": (_red(128, 4, [1, 2], [1, 2], [1, 2, 3, 4]), {"test_hash_bits": 3}),
    "four_words": (_red(64, 8, [1, 2, 4], [1, 2], [1, 2, 3, 4, 1, 2, 3, 4], 37, 3), {}),
    "long_period": (_red(32, 3, [1, 2], [1], [64, 63, 61]), {}),
    # 6,986 states in 8,192 slots, fewer than the 9,099 items: the other engine
    "few_slots": (_red(128, 3, [1], [2], [1, 2, 4]), {"log2_slots": 13}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_edges(mc, name):
    model, opts = CASES[name]
    print(f"[gpu] {name} {w.describe(model)}", flush=True)
    r = oracle.explore(model)
    g = mc.Model(model, **opts)
    for again in range(2):  # the second on the first one's slots
        assert g.mc_min_time() == (r["t_min"], r["argmin"])
        st = g.last_stats
        assert (st["states"], st["terminals"]) == (r["reachable"], r["terminals"])
        assert r["levels"] <= st["levels"] <= g.mc_model_info_get()["max_depth"] + 1
        assert st["cas_fail"] == st["probes"] - st["states"] - st["dups"]
        assert g.mc_terminal_clocks() == r["tc"]
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
        for T in sorted({0, r["t_min"] // 2, r["t_min"] - 1, r["t_min"], max(r["tc"]) - 1,
                         max(r["tc"]) + 5}):
            q = oracle.explore(model, T=T, trace=False)
            assert g.mc_check(T) == q["violated"], T
            assert g.last_stats["states"] == q["reachable"], T
            assert g.mc_terminal_clocks() == q["tc"], T
            if q["violated"]:
                oracle.check_trace(model, g.mc_trace(), max_clock=T)
        assert g.mc_min_time_bb(0) == (r["t_min"], r["argmin"])
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
        assert g.mc_tune_bisect(r["t_min"] // 2)[0] == r["t_min"]
    g.close()


def test_engines_and_models_in_turn(mc):
    """One handle: a chain query, the level engine, a swarm, a chain query, then models alike
    and of unequal speed loaded in turn."""
    a, b = CASES["eight_speeds"][0], w.reduction_model(64, 4, [1, 2], [1, 2], 9, 2)
    ra, rb = oracle.explore(a, trace=False), oracle.explore(b, trace=False)
    g = mc.Model(a)
    for k in range(3):
        assert g.mc_min_time() == (ra["t_min"], ra["argmin"])
        g.mc_set_engine(1)
        assert g.mc_min_time() == (ra["t_min"], ra["argmin"])
        assert g.last_stats["states"] == ra["reachable"]
        oracle.check_trace(a, g.mc_trace(), target_clock=ra["t_min"], cfgs=ra["argmin"])
        g.mc_set_engine(0)
        g.mc_swarm(8, 12, 2000, 1, None)
        assert g.mc_min_time() == (ra["t_min"], ra["argmin"])
        assert g.last_stats["states"] == ra["reachable"]
        oracle.check_trace(a, g.mc_trace(), target_clock=ra["t_min"], cfgs=ra["argmin"])
        g.mc_model_reload(b)
        assert g.mc_min_time() == (rb["t_min"], rb["argmin"])
        assert g.last_stats["states"] == rb["reachable"]
        g.mc_model_reload(a)
    g.close()


def test_stop_request(mc):
    """A stop set before the query ends it at its first look, and the next one runs."""
    model = CASES["many_choices"][0]
    r = oracle.explore(model, trace=False)
    g = mc.Model(model)
    g.mc_abort()
    with pytest.raises(mc.McError) as e:
        g.mc_min_time()
    assert e.value.code == mc.MC_E_ABORTED
    assert g.mc_min_time() == (r["t_min"], r["argmin"])
    g.close()


def test_workspace_without_room_for_the_tables(mc):
    """The chain engine's tables can need more room than the partitions of the table engine, for
    which a workspace was always enough: the least one that is taken holds the latter's."""
    import torch
    model = _red(64, 4, [1, 2, 4, 8], [1, 2], [1, 2, 3, 4])
    model["params"] = model["params"] * 32
    r = oracle.explore(model, trace=False)
    n_cfg = len(model["params"])
    # 80 bytes of table for a configuration, and its tails', against 32 for one partition: taken
    # uncut (part_states all-ones), so that there is one each
    cut = dict(part_states=0xFFFFFFFF)
    full = mc.mc_workspace_bytes(model, mc.make_opts(**cut))
    ws = torch.empty(full, dtype=torch.uint8, device="cuda:0")
    for less in (0, 48 * n_cfg // 256 * 256):
        g = mc.Model(model, workspace=ws[:full - less], **cut)
        assert g.mc_min_time() == (r["t_min"], r["argmin"]), less
        assert g.last_stats["states"] == r["reachable"], less
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
        g.close()


@pytest.mark.parametrize("m,speed", [(1, 5), (2, 2), (8, 3)])
def test_units_of_one_speed_above_one(mc, m, speed):
    """All fall idle together, with and without a last round of a few."""
    for G, wg in ((256, [1, 2, 8]), (16, [2, 4, 16])):
        model = _red(G, m, wg, [1, 4], [speed] * m)
        r = oracle.explore(model)
        g = mc.Model(model)
        assert g.mc_min_time() == (r["t_min"], r["argmin"])
        assert g.last_stats["states"] == r["reachable"]
        assert g.mc_terminal_clocks() == r["tc"]
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
        for T in (r["t_min"] // 2, r["t_min"] - 1, r["t_min"]):
            q = oracle.explore(model, T=T, trace=False)
            assert g.mc_check(T) == q["violated"], T
            assert g.last_stats["states"] == q["reachable"], T
        assert g.mc_min_time_bb(0) == (r["t_min"], r["argmin"])
        g.close()


@pytest.mark.parametrize("name", sorted(CASES))
def test_trace_after_bisection(mc, name):
    model, opts = CASES[name]
    r = oracle.explore(model, trace=False)
    g = mc.Model(model, **opts)
    for seed in (1, 2, 3):
        assert g.mc_tune_bisect(seed)[0] == r["t_min"]
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
    g.close()
