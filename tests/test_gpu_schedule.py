"""Start and end times of one schedule against the oracle where the kernel's split changes: lanes per machine (4 or
2), one relaxer or two, end times in LDS and in the L2, every ring depth (8 slots only with two relaxers), operations of many parts (more than the ring
holds), phases of 8 to 64 steps."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2503_09357_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,fanin,window", [
    (1, 1, 1, None), (2, 64, 1, None), (700, 1, 5, 30), (513, 8, 40, None), (514, 9, 33, 200), (640, 16, 17, 100), (641, 17, 9, 90),
    (1300, 32, 8, 60), (1301, 33, 5, 60), (400, 8, 90, 200), (401, 1, 70, 100), (700, 40, 14, 60), (301, 64, 90, 120), (3000, 64, 12, 300), (19400, 64, 4, 400), (24000, 64, 4, 400), (24000, 5, 3, 200), (28500, 31, 4, 500), (50001, 12, 4, 300)])
def test_schedule_at_the_edges_of_its_splits(gpu_lib, n, p, fanin, window):
    import torch
    rng = np.random.default_rng(n)
    print("[schedule] n=%d p=%d fanin=%d" % (n, p, fanin), flush=True)
    w = W.random_instance(rng, n, p, 1, max_fanin=fanin, max_dur=60000 if n < 20000 else 9000, max_comm=4000, frac_arbitrary=0.0, frac_bad=0.0) \
        if window is None else None
    if w is None:
        rp, ci = W.random_dag(rng, n, fanin, window=window)
        pl, rk = W.list_schedules(rp, ci, p, 1, n)
        w = W.Workload("window", p, rp, ci, rng.integers(0, 20000, n).astype(np.int32), rng.integers(0, 3000, (p, p)).astype(np.int32),
                       rng.integers(-3, 4, n).astype(np.int64), pl, rk)
    if n == 3000:                                            # the last of a topological order gets 1500 predecessors
        src, dst = W.edges_from_csr(w.row_ptr, w.col_idx)
        order = np.lexsort((w.rank[0],))
        last = [v for v in range(n) if w.row_ptr[v] == w.row_ptr[v + 1]][-1]
        more = np.array([v for v in order if v != last][:1500])
        rp, ci = W.csr_from_edges(n, np.concatenate([src, more]), np.concatenate([dst, np.full(len(more), last)]))
        pl, rk = W.list_schedules(rp, ci, p, 1, n)
        w = W.Workload("one wide operation", p, rp, ci, w.dur, w.comm, w.mem_delta, pl, rk)
    prob = oracle.Problem.of(w)
    dev = torch.device("cuda", 0)
    with gpu_lib.Evaluator.for_workload(w, max_candidates=1, shared_placement=None) as ev:
        rk2 = w.rank[0].copy()                               # the second order is a cycle wherever it can be one
        same = np.nonzero(w.placement[0] == w.placement[0, 0])[0]
        rk2[same] = len(same) - 1 - rk2[same]
        for rk in (w.rank[0], rk2):
            s, e, f = (t.cpu().numpy() for t in ev.schedule(torch.from_numpy(w.placement[0]).to(dev), torch.from_numpy(rk).to(dev)))
            flag, so, eo, _, _ = prob.schedule(w.placement[0], rk)
            assert int(f[0]) == flag
            assert (s == so).all() and (e == eo).all() if flag == 0 else (s == -1).all() and (e == -1).all()


@pytest.mark.parametrize("n,p", [(1, 1), (300, 1), (514, 9), (700, 64), (19400, 64), (24000, 5)])
def test_schedule_with_limits_and_missing_channels(gpu_lib, n, p):
    """Memory limits that are just met, exceeded by one on the last machine in use, exceeded together with a cycle and with
    a channel that is not there; end times in LDS and in the L2."""
    import dataclasses

    import torch
    rng = np.random.default_rng(n + p)
    print("[schedule limits] n=%d p=%d" % (n, p), flush=True)
    rp, ci = W.random_dag(rng, n, 3, window=200)
    pl, rk = W.list_schedules(rp, ci, p, 1, n)
    w = W.Workload("limits", p, rp, ci, rng.integers(0, 300, n).astype(np.int32), rng.integers(0, 90, (p, p)).astype(np.int32),
                   rng.integers(-3, 4, n).astype(np.int64), pl, rk, weight=rng.integers(0, 20, n).astype(np.int64),
                   mem_limit=np.full(p, 1 << 40, np.int64))
    peak = oracle.Problem.of(w).evaluate(pl, rk, 0, 1)[2][0]
    last = int(pl.max())
    rk2 = rk[0].copy()                                       # every machine's order reversed
    for j in range(p):
        idx = np.nonzero(pl[0] == j)[0]
        rk2[idx] = len(idx) - 1 - rk2[idx]
    src, dst = W.edges_from_csr(rp, ci)
    a, b = pl[0][src], pl[0][dst]
    comm = w.comm.copy()
    if (a != b).any():
        k = np.nonzero(a != b)[0][-1]
        comm[a[k], b[k]] = oracle.NO_CHANNEL
    short = peak.copy()
    short[last] -= 1
    seen = set()
    for limit in (peak, short):
        for cm in (w.comm, comm):
            v = dataclasses.replace(w, mem_limit=limit, comm=cm)
            prob = oracle.Problem.of(v)
            with gpu_lib.Evaluator.for_workload(v, max_candidates=1, shared_placement=None) as ev:
                for r in (rk[0], rk2):
                    flag = int(prob.evaluate(pl, r[None], 0, 1)[3][0])
                    s, e, f = (t.cpu().numpy() for t in ev.schedule(*(torch.from_numpy(x).to("cuda:0") for x in (pl[0], r))))
                    assert int(f[0]) == flag
                    seen.add(flag)
                    if flag:
                        assert (s == -1).all() and (e == -1).all()
                    else:
                        _, so, eo, _, _ = prob.schedule(pl[0], r)
                        assert (s == so).all() and (e == eo).all()
    assert {0, oracle.FLAG_OVER_MEMORY} <= seen
    assert n == 1 or oracle.FLAG_CYCLIC in seen
    assert p == 1 or oracle.FLAG_NO_CHANNEL in seen


@pytest.mark.parametrize("n,p,fanin", [(3, 2, 1), (65, 3, 9), (130, 16, 14), (131, 17, 5), (260, 32, 9), (90, 33, 3), (400, 40, 6), (611, 64, 20)])
def test_orders_of_every_kind(gpu_lib, n, p, fanin):
    """Lists that end on any lane of a machine, machines without operations, cycles through one machine and through several (of both
    relaxers beyond 32), malformed candidates."""
    import torch
    rng = np.random.default_rng(n * 100 + p)
    w = W.random_instance(rng, n, p, 24, max_fanin=fanin, frac_arbitrary=0.4, frac_bad=0.2)
    prob = oracle.Problem.of(w)
    seen = set()
    with gpu_lib.Evaluator.for_workload(w, max_candidates=1, shared_placement=None) as ev:
        for pl, rk in zip(w.placement, w.rank):
            s, e, f = (t.cpu().numpy() for t in ev.schedule(torch.from_numpy(pl).cuda(), torch.from_numpy(rk).cuda()))
            flag, so, eo, _, _ = prob.schedule(pl, rk)
            assert int(f[0]) == flag
            assert (s == so).all() and (e == eo).all() if flag == 0 else (s == -1).all() and (e == -1).all()
            seen.add(flag)
    assert 0 in seen and (n < 65 or 1 in seen), seen


@pytest.mark.parametrize("p,fillers,lengths", [(33, 0, 40), (64, 0, 40), (64, 31000, 16)])
@pytest.mark.parametrize("upper", [True, False])
def test_one_relaxer_ends_while_the_other_waits(gpu_lib, p, fillers, lengths, upper):
    """Beyond 32 machines: a chain over two machines of one relaxer and an operation of the other that waits for its end, for every
    length up to some phases; end times in LDS and (fillers in front of the chain) in the L2.  Whichever step of a phase the first relaxer's
    last one is, the second has to see it."""
    import torch
    here = np.arange(32, p) if upper else np.arange(0, 32)   # the chain's half
    one, two = (32, min(33, p - 1)) if upper else (0, 1)
    waits = 0 if upper else p - 1
    for k in range(1, lengths + 1):
        n = fillers + k + 1
        chain = fillers + np.arange(k + 1)
        rp, ci = W.csr_from_edges(n, chain[:-1], chain[1:])
        pl = np.concatenate([here[np.arange(fillers) % len(here)], np.where(np.arange(k) % 2, two, one), [waits]]).astype(np.int32)
        rk = np.zeros(n, np.int32)
        for m in np.unique(pl):
            at = np.nonzero(pl == m)[0]
            rk[at] = np.arange(len(at))
        w = W.Workload("chain", p, rp, ci, np.full(n, 2, np.int32), np.full((p, p), 3, np.int32), np.zeros(n, np.int64), pl[None], rk[None])
        flag, so, eo, _, _ = oracle.Problem.of(w).schedule(pl, rk)
        assert flag == 0
        with gpu_lib.Evaluator.for_workload(w, max_candidates=1, shared_placement=None) as ev:
            s, e, f = (t.cpu().numpy() for t in ev.schedule(torch.from_numpy(pl).cuda(), torch.from_numpy(rk).cuda()))
        assert int(f[0]) == 0 and (s == so).all() and (e == eo).all(), k
