"""Ring kernel with several lanes per machine (as many as the candidates of a workgroup leave a wavefront, up to four), operations of
several parts expanded into the order lists, the accountants' stretches of a machine: against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2503_09357_amd import workloads as W
from test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("machines,n,fanin", [
    (1, 1, 1), (1, 130, 2), (2, 3, 1), (3, 65, 4), (4, 64, 9), (7, 333, 1), (8, 257, 14), (11, 1200, 3), (16, 515, 6), (17, 700, 2), (31, 1024, 40), (32, 2049, 9)])
@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_lanes_per_machine(gpu_lib, machines, n, fanin, lanes):
    """Every cell format, ring and place of the placement bytes that is built with as many lanes (or with fewer: tests/test_host_launches.py sees which
    kernel each of these launches): machines without operations and with one, lists that end in the middle of a round, cycles, malformed
    candidates, limits, an odd last workgroup."""
    rng = np.random.default_rng(machines * 10000 + n)
    per_wave = 64 // (1 << (machines - 1).bit_length())
    if lanes > per_wave:
        pytest.skip("a wavefront has fewer lanes to a machine")
    g = per_wave // lanes
    w = W.random_instance(rng, n, machines, 2 * g + 3, max_fanin=fanin, frac_arbitrary=0.25, frac_bad=0.15)
    w.weight = rng.integers(0, 9, n).astype(np.int64)
    w.mem_limit = rng.integers(2, 12 + 9 * n // machines, machines).astype(np.int64)
    seen = set()
    for bits in (16, 32):
        for pib, ring, feeders in ((1, 4, 1), (1, 4, 2), (1, 8, 2), (1, 8, 3), (2, 8, 1), (0, 8, 2), (0, 16, 3)):
            if pib == 2 and machines > 16:
                continue
            with gpu_lib.shape_defaults(cand_per_block=g, placement_mode=pib, ring_slots=ring, feeders=feeders, state_bits=bits):
                _, info = assert_parity(gpu_lib, w, layout=(bits + pib) & 1)
            if info["variant"] in (3, 4, 5):
                assert (info["cand_per_block"], info["ring_slots"], info["state_bits"]) == (g, ring, bits)
                seen.add((bits, pib, ring))
    assert {(16, 1, 4), (16, 1, 8), (16, 0, 8), (32, 1, 8), (32, 0, 8)} <= seen, seen


@pytest.mark.parametrize("machines,lanes", [(32, 2), (16, 4), (5, 2)])
def test_range_stops_and_cycles(gpu_lib, machines, lanes):
    """16-bit end times that some candidates leave: the operation that the range stops is the head's, whatever waits behind it has its
    predecessors ended too; those candidates are evaluated again, cycles are not."""
    rng = np.random.default_rng(77 + machines)
    w = W.random_instance(rng, 900, machines, 61, max_fanin=2, max_dur=9, frac_arbitrary=0.3, frac_bad=0.1)
    per_wave = 64 // (1 << (machines - 1).bit_length())
    w.dur = (w.dur * 37 + 1).astype(np.int32)
    z = assert_parity(gpu_lib, w)[0][0]
    w.dur = (w.dur * (65535 / np.median(z[z > 0]))).astype(np.int32)     # about half of them beyond the range
    with gpu_lib.shape_defaults(cand_per_block=per_wave // lanes, state_bits=16, placement_mode=1, ring_slots=8, feeders=2):
        (z, _, _, f), info = assert_parity(gpu_lib, w)
    assert info["variant"] == 4 and (z > 65534).any() and (z[f == 0] <= 65534).any() and (f == 1).any(), info


@pytest.mark.parametrize("machines,n,fanin,window", [(64, 70, 9, 40), (16, 1464, 9, 25), (32, 1025, 14, 30), (16, 1403, 9, None), (8, 301, 60, 100), (16, 700, 62, 90), (5, 3000, 30, 200)])
def test_lists_of_operations_and_of_parts(gpu_lib, machines, n, fanin, window):
    """One lane per machine, operations of up to 16 parts: lists of operations where chains are long or machines have next to nothing to do (the
    first three), of op parts elsewhere (tests/test_host_launches.py sees which); candidates that are cyclic, have a rank twice, a rank too large,
    a machine that is not there; several wavefronts to a candidate and several candidates to one."""
    rng = np.random.default_rng(n + machines)
    rp, ci = W.random_dag(rng, n, fanin, window=window)
    per_wave = 64 // (1 << (machines - 1).bit_length())
    pl, rk = W.list_schedules(rp, ci, machines, 3 * per_wave + 2, n)
    for c in range(0, len(pl), 5):                           # a machine's order reversed, a rank twice, a rank too large, no such machine
        same = np.nonzero(pl[c] == pl[c, 0])[0]
        rk[c, same] = len(same) - 1 - rk[c, same]
    for c in range(1, len(pl), 7):
        v = int(rng.integers(0, n))
        same = np.nonzero(pl[c] == pl[c, v])[0]
        if c % 3 == 0:
            rk[c, v] = len(same)
        elif c % 3 == 1:
            pl[c, v] = machines
        else:
            rk[c, v] = rk[c, same[0]]
    w = W.Workload("lists", machines, rp, ci, rng.integers(1, 9, n).astype(np.int32), rng.integers(1, 5, (machines, machines)).astype(np.int32),
                   rng.integers(-3, 4, n).astype(np.int64), pl, rk, weight=rng.integers(0, 9, n).astype(np.int64),
                   mem_limit=np.full(machines, 12 + 9 * n // machines, np.int64))
    for bits in (16, 32):
        for pib, ring, feeders, block in ((1, 8, 2, 0), (1, 8, 1, 1024), (0, 8, 2, 512), (0, 16, 3, 0), (2, 8, 2, 0)):
            if pib == 2 and machines > 16:
                continue
            with gpu_lib.shape_defaults(cand_per_block=per_wave, placement_mode=pib, ring_slots=ring, feeders=feeders, block_threads=block, state_bits=bits):
                assert_parity(gpu_lib, w, layout=(bits + pib) & 1)


@pytest.mark.parametrize("machines,width,levels,fanin,window", [(16, 50, 300, 9, True), (8, 20, 100, 30, False)])
def test_lists_that_would_take_too_much(gpu_lib, machines, width, levels, fanin, window):
    """Handles for batches whose lists of op parts would take more than 1 GiB: lists of operations, also in window mode (both launches of it)."""
    rng = np.random.default_rng(width)
    n = width * levels
    src, dst = [], []
    for v in range(width, n):
        lo = max(0, v // width - 2) * width
        for u in rng.choice(np.arange(lo, v // width * width), size=min(fanin, v // width * width - lo), replace=False):
            src.append(u)
            dst.append(v)
    rp, ci = W.csr_from_edges(n, np.array(src), np.array(dst))
    pl, rk = W.list_schedules(rp, ci, machines, 11, n)
    same = np.nonzero(pl[3] == pl[3, 0])[0]
    rk[3, same] = len(same) - 1 - rk[3, same]                # a cycle
    rk[5, 7] = n                                             # a rank too large
    w = W.Workload("long lists", machines, rp, ci, rng.integers(1, 9, n).astype(np.int32), rng.integers(1, 5, (machines, machines)).astype(np.int32),
                   rng.integers(-3, 4, n).astype(np.int64), pl, rk)
    for big in (11, 60000):
        with gpu_lib.Evaluator.for_workload(w, max_candidates=big, shared_placement=None) as ev:
            info = ev.info()
            assert (info["window_log2"] > 0) == window and info["kernel_kind"] == 0 and info["variant"] in (3, 4), info
            import torch
            z, b, pk, f = (t.cpu().numpy() for t in ev.evaluate(torch.from_numpy(pl).cuda(), torch.from_numpy(rk).cuda()))
        zo, bo, pko, fo = oracle.Problem.of(w).evaluate(pl, rk, threads=8)
        assert (f == fo).all() and (z == zo).all() and (b == bo).all() and (pk == pko).all() and (fo != 0).sum() >= 2
