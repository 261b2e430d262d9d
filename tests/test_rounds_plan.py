"""The round engine's arithmetic on the host: every piece of every plan walked with the
functions the kernel uses (csrc/mc_rounds.h), built with gcc.  Each state of the model has to
come from exactly one piece, in a slot of its own inside the slots counted for it, with a code
that no other state of the piece has; links have to name the states they stand for; and a
plan trimmed to a range of clocks has to give the states of that range, as counted by the
oracle's closed forms."""
import os
import shutil
import subprocess

import pytest

import workloads
from oracle import closed_form as cf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_09130_amd", "csrc")
KINDS = {"reduction": 0, "matmul": 1, "abstract": 2, "minimum": 3}


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("rounds") / "driver")
    subprocess.check_call([cxx, "-O2", "-g", "-std=c++17", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC,
                           os.path.join(ROOT, "tests", "rounds_driver.cpp"),
                           os.path.join(CSRC, "mc_model.cpp"), "-pthread", "-o", exe])

    def run(cases):
        text = "\n".join(_line(*c) for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True)
        assert out.returncode == 0, out.stderr[-2000:]
        lines = out.stdout.splitlines()
        assert len(lines) == len(cases)
        return lines
    return run


def _line(model, target, piece, floor=0, T=0xFFFFFFFF):
    k = model["kind"]
    size = {"reduction": lambda: (model["G"], 0, 0),
            "matmul": lambda: (model["M"], model["N"], model["K"])}.get(
                k, lambda: (model["S"], model["NP"], 0))()
    head = (KINDS[k], model["m"], *size, model["Lg"], model["Ll"], model.get("Lc", 1),
            model.get("Lb", 0), target, piece, floor, T, len(model["params"]))
    return " ".join(map(str, head)) + "\n" + "\n".join(
        " ".join(map(str, row)) for row in model["params"])


def _models(seed):
    tiny = workloads.tiny_models(seed, 24, max_cu=8) + workloads.tiny_unit_models(seed, 12, 8)
    return tiny + [
        workloads.reduction_model(512, 3, [1, 2, 8, 256, 512], [1, 2], 23, 3),
        workloads.reduction_model(2048, 5, [512, 1024], [1, 64], 3, 2, Lb=1),  # partial rounds
        workloads.matmul_model(16, 16, 16, 7, [1, 2, 4], [1, 4], [1, 8], [1, 2], 29, 2),
        workloads.matmul_model(8, 8, 1024, 8, [2, 8], [8], [1], [1], 20, 2),   # long rounds
        workloads.abstract_paper(64, 4), workloads.minimum_paper(128, 6),
    ]


@pytest.mark.parametrize("target,piece", [(0, 256), (1, 7), (32, 300), (2048, 256),
                                          (16384, 4096)])
def test_every_state_in_one_place(driver, target, piece):
    models = _models(target + piece)
    lines = driver([(m, target, piece) for m in models])
    for model, line in zip(models, lines):
        words = line.split()
        assert words[0] == "ok", (line, workloads.describe(model))
        want = cf.summary(model, with_E=False)["reachable"]
        assert int(words[1]) == want, workloads.describe(model)
        # slots beyond the states: the copies of a partial round's last state only
        assert want <= int(words[2]) <= want + 69 * len(model["params"])


@pytest.mark.parametrize("target", [0, 1, 2048])
def test_trimmed_plans(driver, target):
    cases, want = [], []
    for model in _models(7 + target):
        pc = cf.per_config(model, with_E=False)
        top = max(c["tc"] for c in pc)
        d0 = pc[0]["d"]
        for lo, hi in ((0, 0), (0, top // 3), (0, d0 - 1), (0, d0), (d0, 2 * d0), (top // 3 + 1,
                       top // 2), (d0 + 1, top - 1), (1, top)):
            if lo <= hi < top:
                cases.append((model, target, 256, lo, hi))
                want.append(cf.count_le(model, hi) - (cf.count_le(model, lo - 1) if lo else 0))
    for case, line, n in zip(cases, driver(cases), want):
        words = line.split()
        assert words[0] == "ok", (line, workloads.describe(case[0]), case[1:])
        assert int(words[1]) == n, (line, n, workloads.describe(case[0]), case[1:])


@pytest.mark.parametrize("m", [1, 2])
def test_operations_of_2_24_cycles_and_more(driver, m):
    """One operation per phase may last longer than a 24-bit product holds: the abstract kernel
    with Lg <= Ll loads a tile of TS items in Lg TS + 1 cycles."""
    models = [workloads.unit_model("abstract", 64, 4, m, [1, 2, 4], [ts], 1 << 20, 1 << 20)
              for ts in (16, 32)]
    for model, line in zip(models, driver([(x, 0, 256) for x in models])):
        words = line.split()
        assert words[0] == "ok", (line, workloads.describe(model))
        assert int(words[1]) == cf.summary(model, with_E=False)["reachable"]


def test_a_plan_far_larger_than_the_set():
    """A model of 9 billion states, a set of 2^16 slots and a partition wanted for every state: a
    check of small T is a use of it, so the load must not fail for want of host memory.  Without
    a GPU it gets as far as the stream."""
    import ctypes

    import torch
    if torch.cuda.is_available():
        pytest.skip("loads into memory that is not there")
    import paper_2305_09130_amd as mc
    model = workloads.reduction_model(1 << 24, 8, [4], [1 << 11], 1, 1)
    model["params"] = model["params"] * 4
    opts = mc.make_opts(log2_slots=16, part_states=1)
    need = mc.mc_workspace_bytes(model, opts)
    desc, keep = mc.make_desc(model)
    h = ctypes.c_void_p()
    rc = mc._lib.mc_model_load(ctypes.byref(desc), ctypes.byref(opts), ctypes.c_void_p(256),
                               ctypes.c_size_t(need), None, ctypes.byref(h))
    assert rc == mc.MC_E_DEVICE


@pytest.fixture(scope="module")
def items_driver(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("round_items") / "driver")
    subprocess.check_call([cxx, "-O2", "-g", "-std=c++17", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC,
                           os.path.join(ROOT, "tests", "round_items_driver.cpp"),
                           os.path.join(CSRC, "mc_model.cpp"), "-pthread", "-o", exe])

    def run(cases):
        text = "\n".join(_line(*c) for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True)
        assert out.returncode == 0, out.stderr[-2000:]
        return out.stdout.splitlines()
    return run


@pytest.mark.parametrize("target", [0, 32, 2048])
def test_states_keys_and_links_as_the_kernel_forms_them(items_driver, target):
    """On whole plans and on trimmed ones, whose partitions start at a later round and link to
    the end of the one before, which an earlier exploration found."""
    cases = []
    for model in _models(70 + target):
        top = max(c["tc"] for c in cf.per_config(model, with_E=False))
        cases += [(model, target, 256)] + [
            (model, target, 256, lo, hi) for lo, hi in (
                (0, top // 2), (top // 3 + 1, top // 2), (top // 2 + 1, top - 1), (1, top - 1))
            if lo <= hi]
    lines = items_driver(cases)
    assert len(lines) == len(cases)
    for case, line in zip(cases, lines):
        assert line.startswith("ok "), (line, workloads.describe(case[0]), case[1:])
