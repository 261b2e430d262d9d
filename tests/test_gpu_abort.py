"""A stop request from the host (mc_abort) ends a query early with MC_E_ABORTED, every
kernel of it exits normally, and the handle answers the next query exactly."""
import sys
import threading
import time

import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def mc():
    import torch
    assert torch.cuda.is_available()
    import paper_2305_09130_amd as mc
    return mc


@pytest.mark.parametrize("engine", [0, 1])
def test_abort_before_the_query(mc, engine):
    """A request made while no query runs stops the next one; the one after is exact."""
    model = workloads.reduction_g256()
    ref = oracle.explore(model, trace=False)
    _say(f"abort before min_time, engine {engine}")
    g = mc.Model(model, engine=engine)
    g.mc_abort()
    with pytest.raises(mc.McError) as e:
        g.mc_min_time()
    assert e.value.code == mc.MC_E_ABORTED
    t_min, argmin = g.mc_min_time()
    assert (t_min, argmin) == (ref["t_min"], ref["argmin"])
    assert g.last_stats["states"] == ref["reachable"]
    g.mc_abort()
    with pytest.raises(mc.McError) as e:
        g.mc_check(ref["t_min"])
    assert e.value.code == mc.MC_E_ABORTED
    assert g.mc_check(ref["t_min"]) is True
    g.close()


def test_abort_from_another_thread_stops_a_long_query(mc):
    """The plain level engine needs one launch per BFS level (331,777 levels, seconds);
    a request from another thread 50 ms in stops it within a batch of launches."""
    import torch
    model = workloads.matmul_64()
    g = mc.Model(model, engine=mc.MC_ENGINE_LEVEL)
    _say("level engine on matmul64_cu4, abort after 50 ms")
    timer = threading.Timer(0.05, g.mc_abort)
    t0 = time.perf_counter()
    timer.start()
    with pytest.raises(mc.McError) as e:
        g.mc_min_time()
    dt = time.perf_counter() - t0
    timer.join()
    assert e.value.code == mc.MC_E_ABORTED
    assert dt < 1.0, dt
    torch.cuda.synchronize()
    # the handle still answers exactly (the super-step engine, for speed)
    g.mc_set_engine(mc.MC_ENGINE_SUPERSTEP)
    t_min, argmin = g.mc_min_time()
    assert g.last_stats["states"] == 5_151_061
    assert t_min == 512 * model["Lg"] + 512 * model["Ll"] + 256
    g.close()


def _few(m, wg, ts, speeds, copies):
    return workloads.with_speeds(
        dict(workloads.reduction_model(256, m, wg, ts, 9, 2),
             params=workloads.reduction_model(256, m, wg, ts, 9, 2)["params"] * copies), speeds)


# Searches by one workgroup, which takes its items one after another: fewer than 64 of them, and
# in the round engine's case more, some milliseconds each.  Crowded sets make the pieces last.
MID_QUERY = {
    "table": (_few(3, [1], [1], [64, 63, 61], 30), {"part_states": 0xFFFFFFFF}),
    "chains": (_few(4, [1], [1], [1, 1, 2, 3], 2), {"part_states": 2048, "test_hash_bits": 1}),
    "rounds": (workloads.matmul_64(), {"test_hash_bits": 1}),
}


@pytest.mark.parametrize("name", sorted(MID_QUERY))
def test_abort_while_items_are_left(mc, name):
    """A request during the query is seen as the next item is taken, however few there are, and
    is used up by it: the next query is not stopped."""
    model, opts = MID_QUERY[name]
    g = mc.Model(model, grid=1, **opts)
    _say(f"{name}: {workloads.describe(model)}")
    if name != "rounds":
        t0 = time.perf_counter()
        whole = g.mc_min_time()
        full = time.perf_counter() - t0
        _say(f"whole query {1e3 * full:.1f} ms, {g.last_stats['parts']} items")
    else:
        full = 0.2
    started = threading.Event()

    def ask():
        started.wait()
        end = time.perf_counter() + full / 4
        while time.perf_counter() < end:
            pass
        g.mc_abort()

    thread = threading.Thread(target=ask)
    thread.start()
    t0 = time.perf_counter()
    started.set()
    with pytest.raises(mc.McError) as e:
        g.mc_min_time()
    dt = time.perf_counter() - t0
    thread.join()
    _say(f"stopped after {1e3 * dt:.1f} ms")
    assert e.value.code == mc.MC_E_ABORTED
    if name == "rounds":  # a request after 50 ms of a second or more
        assert dt < 0.1, dt
    else:
        assert dt < 0.8 * full, (dt, full)
        assert g.mc_min_time() == whole
    g.close()
