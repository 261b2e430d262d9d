"""The chain engine's arithmetic on the host: every piece of every plan walked with the
functions the kernel uses (csrc/mc_chains.h), built with gcc.  The states have to be those of
a breadth-first search of the model, each from exactly one piece, in a slot of one item, with a
code that no other state of the piece has."""
import os
import random
import shutil
import subprocess
from types import SimpleNamespace

import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_09130_amd", "csrc")
KINDS = {"reduction": 0, "matmul": 1, "abstract": 2, "minimum": 3}


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("chains") / "driver")
    subprocess.check_call([cxx, "-O2", "-g", "-std=c++17", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC,
                           os.path.join(ROOT, "tests", "chains_driver.cpp"),
                           os.path.join(CSRC, "mc_model.cpp"), "-pthread", "-o", exe])

    def run(cases):
        text = "\n".join(_line(*c) for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True)
        assert out.returncode == 0, out.stderr[-2000:]
        lines = out.stdout.splitlines()
        assert len(lines) == len(cases)
        return lines
    return run


def _line(model, target, T):
    k = model["kind"]
    size = {"reduction": lambda: (model["G"], 0, 0),
            "matmul": lambda: (model["M"], model["N"], model["K"])}.get(
                k, lambda: (model["S"], model["NP"], 0))()
    head = (KINDS[k], model["m"], *size, model["Lg"], model["Ll"], model.get("Lc", 1),
            model.get("Lb", 0), target, T, len(model["params"]), *model["speed"])
    return " ".join(map(str, head)) + "\n" + "\n".join(
        " ".join(map(str, row)) for row in model["params"])


def _models():
    w = workloads
    fast = w.reduction_model
    return (w.tiny_hetero_models(701, 40, max_cu=8) + w.tiny_hetero_models(702, 20)
            + [w.with_speeds(fast(256, m, [1, 2, 8], [1, 4], 9, 2), sp) for m, sp in (
                (2, [2, 2]), (3, [1, 2, 3]), (4, [4, 4, 2, 1]), (5, [5, 3, 1, 1, 2]),
                (8, [1, 1, 1, 1, 1, 1, 1, 2]), (8, [8, 7, 6, 5, 4, 3, 2, 1]), (6, [9, 8] * 3),
                (7, [64, 1, 1, 1, 1, 1, 1]))]
            + [w.with_speeds(w.matmul_model(16, 16, 256, 3, [16], [1], [1], [1], 23, 3),
                             [1, 2, 3])])


@pytest.mark.parametrize("target", [0, 32, 2048])
def test_pieces_hold_the_states_of_a_search(driver, target):
    rng = random.Random(target)
    cases = []
    for m in _models():
        if len(set(m["speed"])) > 1:
            cases += [(m, target, 0x7FFFFFFF), (m, target, rng.randint(0, 400)),
                      (m, target, rng.randint(0, 4000))]
    for case, line in zip(cases, driver(cases)):
        assert line.startswith("ok "), (workloads.describe(case[0]), case[1:], line)


def test_models_left_to_the_other_engine(driver):
    """Units alike, and a period of 64 * 63 * 61 intervals."""
    w = workloads
    alike = w.with_speeds(w.reduction_model(64, 2, [1], [1], 9, 2), [1, 1])
    long = w.with_speeds(w.reduction_model(64, 3, [1], [1], 9, 2), [64, 63, 61])
    assert driver([(m, 0, 0x7FFFFFFF) for m in (alike, long)]) == ["not a chain-engine model"] * 2


@pytest.mark.parametrize("rows,log2_slots", [(9392, 22), (23482, 21)])
def test_static_scratch_holds_what_it_held(rows, log2_slots):
    """mc_min_time_static does not explore windows of clocks, so their tables take no room of its
    scratch: 134,215,936 and 134,217,728 of its 134,217,728 bytes are enough for these models'
    other tables (the second's to the byte).  Without a GPU a call gets as far as the device."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("a test of the sizes, without a GPU")
    import paper_2305_09130_amd as mc
    G = 8 if log2_slots == 22 else 32
    model = workloads.with_speeds(workloads.reduction_model(G, 8, [1], [1], 9, 2),
                                  [1, 1, 2, 2] * 2)
    for n, code in ((rows, mc.MC_E_DEVICE), (rows + 8, mc.MC_E_NOMEM)):
        with pytest.raises(mc.McError) as e:
            mc.mc_min_time_static(dict(model, params=model["params"] * n),
                                  mc.make_opts(log2_slots=log2_slots, part_states=0xFFFFFFFF),
                                  stream=SimpleNamespace(cuda_stream=0))
        assert e.value.code == code, n


@pytest.mark.parametrize("target", [0, 32, 2048])
def test_units_of_one_speed_above_one(driver, target):
    """All fall idle together, and one unit is listed for all."""
    cases = []
    for m, speed in ((1, 5), (2, 2), (3, 3), (4, 2), (8, 3), (8, 64)):
        for G, wg in ((256, [1, 2, 8]), (16, [2, 4, 16])):  # the second: a last round of a few
            model = workloads.with_speeds(workloads.reduction_model(G, m, wg, [1, 4], 9, 2),
                                          [speed] * m)
            cases += [(model, target, T) for T in (0x7FFFFFFF, 40 * speed, 3000)]
    for case, line in zip(cases, driver(cases)):
        assert line.startswith("ok "), (workloads.describe(case[0]), case[1:], line)
