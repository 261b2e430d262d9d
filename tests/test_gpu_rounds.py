"""The round engine (units alike), the counted swarm walks and the jumped simulation at their
edges, against the CPU oracle, bit-exact."""
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


CASES = {
    # a last round with a choice of units, and nothing else
    "partial_round_only": (w.reduction_model(64, 8, [16, 32], [1], 9, 2), {}),
    "partial_last_rounds": (w.reduction_model(512, 7, [1, 2, 4], [1, 2], 5, 2), {}),
    "one_workgroup": (w.reduction_model(64, 3, [64], [1], 9, 2), {}),
    # rounds longer than a piece, cut into heads and run slices
    "long_rounds": (w.matmul_model(8, 8, 1024, 8, [2, 8], [8], [1], [1], 20, 2), {}),
    "run_slices": (w.matmul_model(8, 8, 1024, 8, [2, 8], [8], [1], [1], 20, 2),
                   {"part_states": 1024}),
    # lists of waves and of two operations per period
    "waves": (w.abstract_paper(64, 4), {}),
    "more_pieces_than_workgroups": (w.reduction_model(1024, 2, [1, 2], [1], 4, 2),
                                    {"part_states": 64, "grid": 2}),
    "crowded_sets": (w.reduction_model(256, 3, [1, 2], [1, 2], 4, 2), {"test_hash_bits": 3}),
    "wide_workgroups": (w.reduction_model(256, 4, [1, 2], [1, 2], 4, 2), {"block": 1024}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_round_engine_edges(mc, name):
    model, opts = CASES[name]
    print(f"[gpu] {name} {w.describe(model)}", flush=True)
    r = oracle.explore(model)
    g = mc.Model(model, **opts)
    for again in range(2):  # the second on the first one's slots
        assert g.mc_min_time() == (r["t_min"], r["argmin"])
        st = g.last_stats
        assert (st["states"], st["levels"], st["terminals"]) == (
            r["reachable"], r["levels"], r["terminals"])
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


def test_set_without_room_for_every_item(mc):
    """A set of as many slots as states but not as items is left to the other engine; a smaller
    one fills up and says so."""
    model = w.reduction_model(512, 7, [1, 2, 4], [1, 2], 5, 2)
    r = oracle.explore(model, trace=False)
    k = (r["reachable"] - 1).bit_length()
    for log2_slots in (k, k + 1):
        g = mc.Model(model, log2_slots=log2_slots)
        assert g.mc_min_time() == (r["t_min"], r["argmin"])
        assert g.last_stats["states"] == r["reachable"]
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
        g.close()
    g = mc.Model(model, log2_slots=k - 2)
    with pytest.raises(mc.McError) as e:
        g.mc_min_time()
    assert e.value.code == mc.MC_E_TABLE_FULL
    g.close()


def test_stop_request_between_queries(mc):
    model = CASES["partial_last_rounds"][0]
    r = oracle.explore(model, trace=False)
    g = mc.Model(model)
    for k in range(2):
        g.mc_abort()
        with pytest.raises(mc.McError) as e:
            g.mc_min_time()
        assert e.value.code == mc.MC_E_ABORTED
        assert g.mc_min_time() == (r["t_min"], r["argmin"])
        assert g.last_stats["states"] == r["reachable"]
    g.close()


KEYS = ("walks", "trails", "steps", "best_walk_start", "first_step", "best_clock", "best_cfg",
        "first_clock", "first_cfg")


@pytest.mark.parametrize("speeds", [[1, 2], [1, 1, 2, 3], [3, 1, 2, 1, 2], [2, 3, 4, 5, 6, 7, 8, 1],
                                    [64, 63, 61]])
@pytest.mark.parametrize("bits_log2", [10, 18, 19])
def test_swarm_walks_counted_by_interval(mc, speeds, bits_log2):
    """Counts per set of busy units up to four units, for all of them beyond, none where the
    period is long; bit arrays in LDS up to 2^18 bits, in memory past that."""
    model = w.with_speeds(w.reduction_model(128, len(speeds), [1, 2, 8], [1, 2], 9, 2), speeds)
    r = oracle.explore(model, trace=False)
    g = mc.Model(model, log2_slots=20)
    for T in (None, r["t_min"] - 1, (r["t_min"] + max(r["tc"])) // 2):
        g.mc_swarm(5, bits_log2, 20000, 3, T)
        for a, b in zip(g.mc_swarm_members(5), oracle.swarm(model, 3, 5, 20000, bits_log2, T)):
            assert {k: a[k] for k in KEYS} == {k: b[k] for k in KEYS}, T
    g.close()


@pytest.mark.parametrize("m,speed", [(1, 1), (3, 1), (5, 1), (3, 2), (8, 3)])
def test_simulated_rounds(mc, m, speed):
    """Whole rounds crossed at once on units of one speed, with and without a partial one."""
    for G, wg in ((16, [16]), (64, [4]), (512, [1, 2])):
        model = w.reduction_model(G, m, wg, [1], 9, 2)
        if speed > 1:
            model = w.with_speeds(model, [speed] * m)
        g = mc.Model(model)
        for seed in range(1, 6):
            assert g.mc_simulate(seed) == oracle.simulate(model, seed), (G, wg, seed)
        g.close()


@pytest.mark.parametrize("speeds", [None, [1], [1, 1], [1, 2], [2, 2, 1]])
def test_operations_of_2_24_cycles_and_more(mc, speeds):
    """Operation times past 24 bits: clocks, counts up to a clock and every row of a path (the
    abstract kernel with Lg <= Ll loads a tile of TS items in Lg TS + 1 cycles)."""
    model = w.unit_model("abstract", 64, 4, len(speeds) if speeds else 2, [1, 2, 4],
                         [8, 16, 32] if not speeds else [8, 16], 1 << 20, 1 << 20)
    if speeds and set(speeds) != {1}:
        model = w.with_speeds(model, speeds)
    print(f"[gpu] {w.describe(model)} {speeds}", flush=True)
    r = oracle.explore(model)
    g = mc.Model(model)
    assert g.mc_min_time() == (r["t_min"], r["argmin"])
    assert g.last_stats["states"] == r["reachable"]
    oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
    for T in (1 << 24, r["t_min"] // 3, r["t_min"] - 1, r["t_min"], max(r["tc"]) - 1):
        q = oracle.explore(model, T=T, trace=False)
        assert g.mc_check(T) == q["violated"], T
        assert g.last_stats["states"] == q["reachable"], T
        if q["violated"]:
            oracle.check_trace(model, g.mc_trace(), max_clock=T)
    assert g.mc_tune_bisect(1)[0] == r["t_min"]
    g.close()


@pytest.mark.parametrize("speeds", [[1, 2, 3], [8, 7, 6, 5, 4, 3, 2, 1], [64, 63, 61]])
@pytest.mark.parametrize("members,bits_log2", [(1280, 18), (1281, 18), (4096, 10), (4097, 10), (8193, 13),
                                               (3, 19), (2, 21), (1, 25)])
def test_swarm_sizes(mc, speeds, members, bits_log2):
    """The largest swarm whose bit arrays are in LDS and the smallest in memory; the largest of
    one member to a wavefront and the smallest of more; one member's array larger than a
    quarter of a CU's LDS, and than all of it."""
    model = w.with_speeds(w.reduction_model(64, len(speeds), [1, 4], [1, 2], 9, 2), speeds)
    need = members * (80 + (1 << bits_log2) // 8) + (1 << 20)
    g = mc.Model(model, log2_slots=(need // 8).bit_length())
    g.mc_swarm(members, bits_log2, 150, 7, None)
    want = oracle.swarm(model, 7, members, 150, bits_log2, None)
    for a, b in zip(g.mc_swarm_members(members), want):
        assert {k: a[k] for k in KEYS} == {k: b[k] for k in KEYS}
    g.close()


@pytest.mark.parametrize("name", sorted(CASES))
def test_trace_after_bisection(mc, name):
    """Its path crosses states of several continued explorations, each on a trimmed plan."""
    model, opts = CASES[name]
    r = oracle.explore(model, trace=False)
    g = mc.Model(model, **opts)
    for seed in (1, 2, 3):
        assert g.mc_tune_bisect(seed)[0] == r["t_min"]
        oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"], cfgs=r["argmin"])
    g.close()
