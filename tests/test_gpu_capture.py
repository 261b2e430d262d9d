"""Calls on a stream that is being captured: those that wait for the stream are refused, the
capture goes on, and the handle answers the next query exactly."""
import contextlib

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


@contextlib.contextmanager
def _capture(graph):
    graph.capture_begin()
    try:
        yield
    finally:
        graph.capture_end()


def _refused(mc, f):
    with pytest.raises(mc.McError) as e:
        f()
    assert e.value.code == mc.MC_E_DEVICE


@pytest.mark.parametrize("kind", ["round", "chain", "table"])
def test_model(mc, kind):
    """Loads, reloads and queries, for models of each engine; more pieces than workgroups, so
    that a launch takes the count of pieces up where the one before left it."""
    import torch
    model = w.reduction_model(512, 3, [1, 2], [1, 2], 9, 2)
    if kind == "chain":
        model = w.with_speeds(model, [1, 2, 3])
    elif kind == "table":
        model = w.with_speeds(w.reduction_model(32, 3, [1, 2], [1], 9, 2), [64, 63, 61])
    other = w.reduction_model(64, 2, [1, 2], [1], 9, 2)
    r = oracle.explore(model)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ws, room = (torch.empty(1 << 26, dtype=torch.uint8, device="cuda:0") for _ in range(2))
        g = mc.Model(model, grid=2, part_states=32, workspace=ws)
        x = torch.zeros(4, device="cuda:0")
        stream.synchronize()
        for before in range(2):  # before the handle's first query, and after it
            graph = torch.cuda.CUDAGraph()
            with _capture(graph):
                x.add_(1)
                _refused(mc, lambda: mc.Model(model, workspace=room))
                _refused(mc, lambda: g.mc_model_reload(other))
                _refused(mc, g.mc_min_time)
                _refused(mc, lambda: g.mc_min_time_bb(0))
                _refused(mc, lambda: g.mc_check(5))
                _refused(mc, lambda: g.mc_simulate(1))
                _refused(mc, lambda: g.mc_tune_bisect(1))
                _refused(mc, lambda: g.mc_swarm(4, 10, 100, 1))
                _refused(mc, lambda: mc.mc_min_time_static(model, stream=stream))
            for k in range(2):
                assert g.mc_min_time() == (r["t_min"], r["argmin"])
                assert g.last_stats["states"] == r["reachable"]
                oracle.check_trace(model, g.mc_trace(), target_clock=r["t_min"],
                                   cfgs=r["argmin"])
            graph.replay()
        stream.synchronize()
        assert x.tolist() == [2.0] * 4
        g.close()


def test_batch(mc):
    import torch
    models = [w.reduction_model(64, 3, [1, 2], [1, 2], 9, 2),
              w.with_speeds(w.reduction_model(64, 3, [1, 2], [1, 2], 9, 2), [1, 2, 3])]
    refs = [oracle.explore(m, trace=False) for m in models]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        b = mc.Batch(models)
        x = torch.zeros(4, device="cuda:0")
        stream.synchronize()
        for before in range(2):
            graph = torch.cuda.CUDAGraph()
            with _capture(graph):
                x.add_(1)
                _refused(mc, b.mc_batch_min_time)
            assert b.mc_batch_min_time() == ([r["t_min"] for r in refs],
                                             [r["reachable"] for r in refs])
            graph.replay()
        stream.synchronize()
        assert x.tolist() == [2.0] * 4
        b.close()


def test_engine_step(mc):
    import torch
    models = [w.reduction_model(64, 3, [1, 2], [1, 2], 9, 2),
              w.with_speeds(w.reduction_model(64, 3, [1, 2], [1, 2], 9, 2), [1, 2, 3])]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        e = mc.Engine(64 << 20)
        x = torch.zeros(4, device="cuda:0")
        stream.synchronize()
        for model in models:
            r = oracle.explore(model, trace=False)
            t = e.mc_engine_submit(model, mc.MC_QUERY_MIN_TIME)
            graph = torch.cuda.CUDAGraph()
            with _capture(graph):
                x.add_(1)
                _refused(mc, e.mc_engine_step)
            graph.replay()
            e.drain()
            out = e.mc_engine_poll(t)
            assert (out["status"], out["t_min"], out["states"]) == (0, r["t_min"], r["reachable"])
            assert e.mc_engine_argmin(t) == r["argmin"]
            e.mc_engine_release(t)
        stream.synchronize()
        assert x.tolist() == [2.0] * 4
        e.close()
