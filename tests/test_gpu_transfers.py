"""Evaluation with channel contention against the oracle where its fast path changes shape: one, two and four lanes per
machine, one to 64 candidates per workgroup, deep and shallow rings, operations with many outputs, and what it leaves to
the other kernel (orders that do not follow the producers, more than 255 inputs, more than 65000 operations and edges).
The shapes and the number of candidates left over are asserted, not assumed."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import test_gpu_channels as T
from paper_2503_09357_amd import workloads as W

pytestmark = pytest.mark.gpu


def _star(rng, n, fan, inward):
    """A chain of n operations plus `fan` edges into the last or out of the first one."""
    src, dst = list(range(n - 1)), list(range(1, n))
    for k in range(1, fan + 1):
        src.append(k if inward else 0)
        dst.append(n - 1 if inward else k + 1)
    return W.csr_from_edges(n, src, dst)


@pytest.mark.parametrize("n,p,c,kind", [
    (5, 1, 3, "random"), (300, 2, 700, "random"), (301, 4, 1500, "dense"), (257, 8, 3000, "sparse"), (900, 16, 520, "dense"),
    (1000, 17, 300, "random"), (640, 32, 1030, "dense"), (700, 33, 90, "sparse"), (800, 64, 300, "dense"), (4000, 64, 40, "random"),
    (16000, 7, 9, "random"), (25000, 5, 3, "sparse"), (150, 5, 40, "out"), (300, 5, 40, "in"), (420, 9, 20, "in255"), (20000, 6, 3, "large")])
def test_shapes_of_the_fast_path(gpu_lib, n, p, c, kind):
    rng = np.random.default_rng(n)
    if kind in ("out", "in", "in255"):
        rp, ci = _star(rng, n, {"out": 120, "in": 280, "in255": 254}[kind], kind != "out")
    else:
        rp, ci = W.random_dag(rng, n, {"dense": 6, "random": 3, "sparse": 1, "large": 6}[kind], window=400)
    pl, rk = W.list_schedules(rp, ci, p, c, n)
    for i in range(0, c, 7):                                 # some cycles and some malformed candidates
        j = np.nonzero(pl[i] == pl[i, 0])[0]
        rk[i, j] = rk[i, j][::-1].copy()
    if c > 5:
        rk[3, n // 2] = -1
        pl[5, n // 3] = p
    w = W.Workload("transfers n=%d p=%d %s" % (n, p, kind), p, rp, ci, rng.integers(0, 9, n).astype(np.int32),
                   rng.integers(0, 90, (p, p)).astype(np.int32), rng.integers(-5, 6, n).astype(np.int64), pl, rk)
    if n % 2:
        w.weight, w.mem_limit = rng.integers(0, 9, n).astype(np.int64), np.full(p, 5 * n // p + 20, np.int64)
    er = W.fcfs_edge_ranks(rp, ci, p, pl, rk)
    some = np.arange(c) % 5 == 1                             # orders that do not follow the producers, and bad ones
    er[some] = T._shuffle_some_channels(rng, W.Workload("", p, rp, ci, w.dur, w.comm, w.mem_delta, pl[some], rk[some]), er[some])
    if c > 9:
        er[8] = er[8] + 1
    T._parity(gpu_lib, w, er, layout=n % 2, repeats=2)


@pytest.mark.parametrize("p,c", [(1, 70), (3, 2100), (9, 600), (16, 40), (17, 300), (32, 40), (32, 600), (40, 40)])
def test_messages_of_one_operation_share_a_channel(gpu_lib, p, c):
    """Seven messages per operation, most of them over the same channel, and channels that everything waits for: the lanes
    of a machine send them side by side, with delays laid out for lanes that stay in step."""
    rng = np.random.default_rng(100 * p + c)
    n, fan = 420, 7
    src = np.repeat(np.arange(n - fan), fan)
    dst = src + np.tile(np.arange(1, fan + 1), n - fan)
    rp, ci = W.csr_from_edges(n, src, dst)
    where = np.unique([0, p // 2, p - 1])[rng.integers(0, len({0, p // 2, p - 1}), n)].astype(np.int32)
    pl, rk = W.list_schedules(rp, ci, p, c, n, fixed_placement=where)
    w = W.Workload("shared channels p=%d" % p, p, rp, ci, rng.integers(0, 4, n).astype(np.int32),
                   rng.integers(20, 90, (p, p)).astype(np.int32), rng.integers(-5, 6, n).astype(np.int64), pl, rk)
    T._parity(gpu_lib, w, W.fcfs_edge_ranks(rp, ci, p, pl, rk), repeats=3)


@pytest.mark.parametrize("p,c,fan_in", [(2, 17000, 0), (4, 9000, 0), (8, 4200, 0), (3, 9000, 150), (16, 40, 0), (32, 40, 200)])
def test_orders_left_to_the_other_kernel_beside_others(gpu_lib, p, c, fan_in):
    """Candidates whose orders do not follow the producers share a wavefront with candidates whose orders do: theirs are
    brought to a halt (also past operations with more than 127 inputs), the others run on."""
    rng = np.random.default_rng(p + c)
    n = 40 + 2 * fan_in
    rp, ci = _star(rng, n, fan_in, True) if fan_in else W.random_dag(rng, n, 4)
    pl, rk = W.list_schedules(rp, ci, p, c, n)
    w = W.Workload("mixed orders p=%d" % p, p, rp, ci, rng.integers(0, 9, n).astype(np.int32), rng.integers(0, 30, (p, p)).astype(np.int32),
                   rng.integers(-5, 6, n).astype(np.int64), pl, rk)
    er = W.fcfs_edge_ranks(rp, ci, p, pl, rk)
    some = np.arange(c) % 11 == 3
    some[c // 2:c // 2 + 64] = True                          # a whole workgroup's
    er[some] = T._shuffle_some_channels(rng, W.Workload("", p, rp, ci, w.dur, w.comm, w.mem_delta, pl[some], rk[some]), er[some], every=1)
    T._parity(gpu_lib, w, er, repeats=2)


@pytest.mark.parametrize("p,c", [(64, 2200), (3, 8500)])
def test_several_candidates_per_workgroup_of_the_other_kernel(gpu_lib, p, c):
    """More candidates with orders of their own than the other kernel has workgroups (1024 with 64 machines, 4096 with few,
    on 256 CUs): its rows of scratch are used again, while what the candidate before read of them may still be cached."""
    rng = np.random.default_rng(p)
    n = 40
    rp, ci = W.random_dag(rng, n, 6)
    pl, rk = W.list_schedules(rp, ci, p, c, n)
    src = W.edges_from_csr(rp, ci)[0]
    w = W.Workload("rows p=%d" % p, p, rp, ci, rng.integers(0, 9, n).astype(np.int32), rng.integers(0, 30, (p, p)).astype(np.int32),
                   rng.integers(-5, 6, n).astype(np.int64), pl, rk)
    er = W.fcfs_edge_ranks(rp, ci, p, pl, rk)
    if p > 3:
        er = T._shuffle_some_channels(rng, w, er, every=1)
    else:                                                    # (those would all be cycles) two messages of one operation trade places
        for i in range(c):
            key = np.where(pl[i, src] != pl[i, ci], src * p + pl[i, ci], -1 - np.arange(len(src)))
            k = [np.nonzero(key == x)[0] for x in np.unique(key[key >= 0])]
            k = max(k, key=len)[:2]
            er[i, k] = er[i, k[::-1]]
    T._parity(gpu_lib, w, er, repeats=2)


@pytest.mark.parametrize("n,p", [(1, 1), (70, 3)])
def test_operations_without_edges(gpu_lib, n, p):
    """Tables of no entries among the others, some channels missing, limits."""
    rng = np.random.default_rng(n)
    rp, ci = W.csr_from_edges(n, [], [])
    pl, rk = W.list_schedules(rp, ci, p, 20, n)
    comm = rng.integers(0, 9, (p, p)).astype(np.int32)
    if p > 1:
        comm[0, 1] = -1
    w = W.Workload("no edges", p, rp, ci, rng.integers(0, 9, n).astype(np.int32), comm, rng.integers(-5, 6, n).astype(np.int64), pl, rk,
                   weight=rng.integers(0, 9, n).astype(np.int64), mem_limit=np.full(p, 5 * n // p + 20, np.int64))
    T._parity(gpu_lib, w, W.fcfs_edge_ranks(rp, ci, p, pl, rk))


@pytest.mark.parametrize("n,p,reach,most,shape", [       # shape: candidates, lanes, slots, threads, teams
    (40, 1, 1, 33000, (64, 1, 32, 512, 8)), (200, 1, 1, 17000, (64, 1, 32, 1024, 16)), (41, 2, 1, 16500, (32, 1, 32, 512, 8)),
    (60, 4, 1, 8300, (16, 1, 32, 512, 8)), (61, 4, 2, 4200, (8, 2, 32, 512, 8)), (60, 8, 1, 4200, (8, 1, 32, 512, 8)),
    (700, 4, 1, 8300, (16, 1, 16, 512, 8)), (1000, 4, 1, 4200, (16, 1, 32, 1024, 16)), (1500, 8, 1, 4200, (8, 1, 16, 512, 8)),
    (2500, 8, 2, 2100, (4, 2, 16, 512, 4)), (5000, 4, 2, 1100, (4, 4, 32, 1024, 4)), (90, 16, 2, 30, (1, 4, 32, 512, 1)), (90, 33, 2, 30, (1, 1, 32, 512, 1))])
def test_small_batches_on_handles_for_large_ones(gpu_lib, n, p, reach, most, shape):
    """1, one less and one more than a workgroup's candidates, and several workgroups' on a handle made for many more."""
    import torch
    rng = np.random.default_rng(n + p)
    G = shape[0]
    c = 3 * G + 2
    step = np.arange(n)
    src, dst = np.concatenate([step[:n - r - 1] for r in range(1, reach + 1)]), np.concatenate([step[r + 1:] for r in range(1, reach + 1)])
    rp, ci = W.csr_from_edges(n, src, dst)
    pl, rk = W.list_schedules(rp, ci, p, c, n)
    if p > 1:
        pl[2, 0] = p
    w = W.Workload("G=%d" % G, p, rp, ci, rng.integers(0, 9, n).astype(np.int32), rng.integers(0, 30, (p, p)).astype(np.int32),
                   rng.integers(-5, 6, n).astype(np.int64), pl, rk, weight=rng.integers(0, 9, n).astype(np.int64),
                   mem_limit=np.full(p, 6 * n // p + 30, np.int64))
    fcfs = W.fcfs_edge_ranks(rp, ci, p, pl, rk)
    er = T._shuffle_some_channels(rng, w, fcfs.copy(), every=5)
    strange = (er != fcfs).any(axis=1) & (pl < p).all(axis=1)
    dev = torch.device("cuda", 0)
    print("[transfers] n=%d p=%d shape=%s" % (n, p, shape), flush=True)
    with gpu_lib.Evaluator.for_workload(w, max_candidates=most, contention=True, shared_placement=None) as ev:
        for size in (1, max(1, G - 1), G + 1, c):
            want = oracle.Problem.of(w).evaluate_contended(pl[:size], rk[:size], er[:size], 0, threads=8)
            got = ev.evaluate_contended(*(torch.from_numpy(a[:size]).to(dev) for a in (pl, rk, er)))
            info = ev.contended_info()
            assert all((a.cpu().numpy() == b).all() for a, b in zip(got, want)), size
            assert tuple(info[k] for k in ("cand_per_block", "lanes_per_machine", "ring_slots", "block_threads", "ingest_teams")) == shape
            assert info["left_over"] == strange[:size].sum()
