"""What the library's host side asks of the HIP runtime, without a GPU (tests/fake_hip.c): handles that fit the memory only
without the pipeline kernels or with shorter order lists, memory given back, grids that every launch can have, the ring kernel's lanes per machine."""
from __future__ import annotations

import ctypes
import json
import os
import re
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ATTRIBUTES = ("-DLDS_ATTRIBUTE=74", "-DCU_ATTRIBUTE=63")     # hipDeviceAttributeMaxSharedMemoryPerBlock, ...MultiprocessorCount


def _in_child(shim):
    """Runs in a process of its own, where the library's calls resolve to the shim."""
    sys.path.insert(0, os.path.dirname(HERE))
    fake = ctypes.CDLL(shim, ctypes.RTLD_GLOBAL)
    fake.fake_used.restype = ctypes.c_size_t
    fake.fake_budget.argtypes = [ctypes.c_size_t]
    from paper_2503_09357_amd import dagsched, workloads as W
    lib = dagsched.load(import_torch_first=False)
    some = ctypes.c_void_p(1 << 20)                           # (nothing is read or written through it)

    def problem(stages, micros, scale, n_cand, split=True):
        ids, src, dst = W.pipeline_dag(stages, micros, split_w=split)
        fixed = np.zeros(len(ids), np.int32)
        for (_, s, _), v in ids.items():
            fixed[v] = s
        rp, ci = W.csr_from_edges(len(ids), src, dst)
        rng = np.random.default_rng(1)
        dur = rng.integers(1, 9, len(ids)) * scale + rng.integers(0, scale, len(ids))
        return dagsched._HostProblem(stages, rp, ci, dur, rng.integers(1, 5, (stages, stages)) * scale, rng.integers(-3, 4, len(ids)), n_cand, 0, 0,
                                     shared_placement=fixed)

    def make(hp, calls, budget=1 << 62):
        fake.fake_budget(budget)
        h, i = ctypes.c_void_p(), dagsched.Info()
        out = dict(rc=lib.dagsched_create(ctypes.byref(hp.desc), ctypes.byref(h)))
        if out["rc"] == 0:
            lib.dagsched_get_info(h, ctypes.byref(i))
            out.update(dagsched._info_dict(i), used=fake.fake_used(), calls=[])
            for n in calls:
                fake.fake_launches()
                rc = lib.dagsched_evaluate(h, n, some, some, some, some, some, some, None)
                out["calls"].append((rc, fake.fake_launches()))
            lib.dagsched_destroy(h)
        return dict(out, left=fake.fake_used())

    got = {}
    for name, args in (("optimistic", (8, 32, 37, 65536)), ("exact", (16, 128, 1, 2048)), ("fused for ring", (3, 20, 1, 20000)),
                       ("fused for general", (8, 16, 1, 32768))):
        hp = problem(*args)
        full = make(hp, (7,))
        got[name] = (full, make(hp, (7,), full["used"] - 1))
    got["after a refusal"] = make(problem(3, 20, 1, 20000), (7,))
    got["many"] = make(problem(5, 1, 20011, 2 ** 26), (1, 2 ** 20 + 1, 2 ** 24 + 1, 2 ** 26))
    # entries of a candidate's order list: what 64 candidates more add to the handle (the planner's choice does not change there)
    got["list entries"] = {}
    for name, (machines, n, fanin, window) in LISTS.items():
        rng = np.random.default_rng(n + machines)
        rp, ci = W.random_dag(rng, n, fanin, window=window)
        args = (rng.integers(1, 9, n), rng.integers(1, 5, (machines, machines)), rng.integers(-3, 4, n))
        per_wave = 64 // (1 << (machines - 1).bit_length())
        used = []
        for n_cand in (64 * 256, 64 * 257):
            hp = dagsched._HostProblem(machines, rp, ci, *args, n_cand, 0, 0, shape=dict(cand_per_block=per_wave, placement_mode=1, ring_slots=8, feeders=2, state_bits=16))
            used.append(make(hp, ())["used"])
        got["list entries"][name] = (used[1] - used[0]) // 128
    # the ring kernel that is launched: lanes per machine and kind, of every shape that tests/test_gpu_ring_lanes.py asks for
    fake.fake_kernel.restype = ctypes.c_char_p
    got["lanes"] = []
    for machines, n, fanin in RING_PROBLEMS:
        per_wave = 64 // (1 << (machines - 1).bit_length())
        for lanes in (1, 2, 4):
            if lanes > per_wave:
                continue
            g = per_wave // lanes
            w = W.random_instance(np.random.default_rng(machines * 10000 + n), n, machines, 2 * g + 3, max_fanin=fanin, frac_arbitrary=0.25, frac_bad=0.15)
            for bits in (16, 32):
                for pib, ring, feeders in RING_SHAPES:
                    if pib == 2 and machines > 16:
                        continue
                    hp = dagsched._HostProblem(machines, w.row_ptr, w.col_idx, w.dur, w.comm, w.mem_delta, w.n_cand, 0, 0, shape=dict(
                        cand_per_block=g, placement_mode=pib, ring_slots=ring, feeders=feeders, state_bits=bits, ignore_shared_placement=1))
                    made = make(hp, (w.n_cand,))
                    names = [fake.fake_kernel(i).decode() for i in range(made["calls"][0][1])]
                    of = [[int(x) for x in re.findall(r"Li(\d+)E", m)] for m in re.findall(r"relax_ring_kernelI((?:Li\d+E)+)", " ".join(names))]
                    got["lanes"].append((lanes, bits, pib, ring, feeders, made["variant"], of))
    # lists of op parts: without the memory for them, and where they would take more than 1 GiB
    rng = np.random.default_rng(9)
    rp, ci = W.random_dag(rng, 2000, 40, window=100)
    args = (rng.integers(1, 9, 2000), rng.integers(1, 5, (8, 8)), rng.integers(-3, 4, 2000))
    small, *more = (dagsched._HostProblem(8, rp, ci, *args, n, 0, 0) for n in (400, 2 ** 17, 2 ** 17 + 64))
    full = make(small, (400,))
    got["many parts"] = [full, make(small, (400,), full["used"] - 1), *(make(hp, (7,)) for hp in more)]
    print(json.dumps(got))


# (machines, operations, fan-in) and (place of the placement bytes, slots, feeders) of test_lanes_per_machine there
RING_PROBLEMS = [(1, 1, 1), (1, 130, 2), (2, 3, 1), (3, 65, 4), (4, 64, 9), (7, 333, 1), (8, 257, 14), (11, 1200, 3), (16, 515, 6), (17, 700, 2), (31, 1024, 40), (32, 2049, 9)]
RING_SHAPES = [(1, 4, 1), (1, 4, 2), (1, 8, 2), (1, 8, 3), (2, 8, 1), (0, 8, 2), (0, 16, 3)]
# (machines, operations, fan-in, window) of tests/test_gpu_ring_lanes.py
LISTS = {"one operation to a machine": (64, 70, 9, 40), "a long chain": (16, 1464, 9, 25), "the same, odd": (32, 1025, 14, 30), "wide": (16, 1403, 9, None),
         "many parts": (8, 301, 60, 100), "more parts": (16, 700, 62, 90)}


@pytest.fixture(scope="module")
def seen(tmp_path_factory):
    shim = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", *ATTRIBUTES, os.path.join(HERE, "fake_hip.c"), "-o", shim, "-ldl"], check=True)
    from paper_2503_09357_amd import _build
    _build.ensure_hip()
    run = subprocess.run([sys.executable, os.path.abspath(__file__), shim], stdout=subprocess.PIPE, check=True, timeout=600)
    return json.loads(run.stdout)


@pytest.mark.parametrize("name,form,without,launches", [
    ("optimistic", (4, 1), (4, 0), (3, 3)), ("exact", (3, 1), (3, 0), (3, 1)), ("fused for ring", (6, 0), (3, 0), (3, 1))])
def test_a_handle_that_fits_only_without_the_pipeline_kernels(seen, name, form, without, launches):
    """One byte less than it takes: the kernel planned besides takes every call."""
    full, short = seen[name]
    assert (full["rc"], full["variant"], full["two_launches"]) == (0, *form)
    assert (short["rc"], short["variant"], short["two_launches"]) == (0, *without) and short["used"] < full["used"]
    assert full["calls"] == [[0, launches[0]]] and short["calls"] == [[0, launches[1]]]
    assert full["left"] == short["left"] == 0


def test_no_handle_where_nothing_is_planned_besides(seen):
    full, short = seen["fused for general"]
    assert (full["rc"], full["variant"], full["kernel_kind"]) == (0, 6, 3) and full["calls"] == [[0, 3]]
    assert short["rc"] == -4 and full["left"] == short["left"] == 0


def test_a_refused_handle_leaves_no_error_behind(seen):
    """The launches of the next handle do not report that there was no memory for the one before."""
    assert seen["fused for general"][1]["rc"] == -4 and seen["after a refusal"]["calls"][0][0] == 0


@pytest.mark.parametrize("name", list(LISTS))
def test_order_lists_of_operations_or_of_parts(seen, name):
    """With one lane per machine the order lists hold operations where chains are long for what a machine has to do, else op parts."""
    n = LISTS[name][1]
    assert (seen["list entries"][name] == (n + 63) // 64 * 64) == (name in ("one operation to a machine", "a long chain", "the same, odd"))
    assert seen["list entries"][name] >= n


def test_the_ring_kernel_has_the_lanes_it_is_asked_for(seen):
    """As many lanes per machine as the candidates of a workgroup leave a wavefront, where that is built: placement bytes in L2 with sixteen slots and
    three feeders two at most, and one where no operation waits for more than one other (the kind of one predecessor has two feeders)."""
    counted = {1: 0, 2: 0, 4: 0}
    for lanes, bits, pib, ring, feeders, variant, kernels in seen["lanes"]:
        if variant not in (3, 4, 5):
            continue
        slots, launched_feeders, _, where, kind, _, sub = kernels[0]
        assert (slots, launched_feeders, where) == (ring, feeders, pib)
        assert sub == (lanes if feeders < 3 else 1 if kind == 3 else min(lanes, 2)), (lanes, bits, pib, ring, feeders, kernels)
        counted[sub] += 1
    assert min(counted.values()) > 50, counted


def test_lists_of_parts_that_do_not_fit(seen):
    """A byte less than lists of op parts take: a handle with lists of operations and one lane per machine.  Beyond 1 GiB of them nobody asks for the memory."""
    full, short, large, larger = seen["many parts"]
    assert (full["rc"], short["rc"], large["rc"], larger["rc"]) == (0, 0, 0, 0) and full["variant"] == short["variant"] == large["variant"]
    assert full["used"] - short["used"] > 400 * 2 * 2000 and short["cand_per_block"] == large["cand_per_block"] == 8
    assert (larger["used"] - large["used"]) // 64 < 2 * 2048 + 2048 and full["calls"] == short["calls"]
    assert [x["left"] for x in seen["many parts"]] == [0, 0, 0, 0]


def test_grids_of_large_batches(seen):
    """No dimension of a grid counts 2^32 threads or more."""
    assert seen["many"]["two_launches"] == 1 and seen["many"]["calls"] == [[0, 3]] * 4


if __name__ == "__main__":
    _in_child(sys.argv[1])
