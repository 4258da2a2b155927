"""What a user of this package has it do, as cases that can be timed: the batched evaluation of candidate schedules on
the workload families of ``workloads.py`` from 64 to 50000 operations, and the calls around it (the local search that
has the evaluation in its loop, the evaluation with channel contention, the start and end times of one schedule, the
coarsening in front of the planning).

A case names the graph (family and sizes), what is done with it, and the options in use:

  do        evaluate | contended | search | search_orders | schedule | coarsen
  graph     1f1b | zero_bubble | bidirectional | moe | layered | random    (see _graph)
  cands     candidates in the batch (search: per iteration)
  minor     candidate-minor arrays instead of candidate-major ones
  micros    durations and delays as measured times in microseconds (makespans beyond 16 bits), not small units
  limits    static memory per operation and a memory limit per machine (eq. (16))
  chain     machines in a chain: only neighbours have a channel (eq. (10)); pipelines only
"""
from __future__ import annotations

import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2503_09357_amd import dagsched as ds
from paper_2503_09357_amd import search
from paper_2503_09357_amd import workloads as W

ITERATIONS = 10          # of a search pass
MOST_ENTRIES = 6144 * 16384


def _case(name, do, graph, cands=1, a=0, b=0, p=1, minor=False, micros=False, limits=False, chain=False):
    c = dict(do=do, graph=graph, a=a, b=b, p=p, cands=cands, minor=minor, micros=micros, limits=limits, chain=chain)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest batch: a planner that tries the orders of a four-stage 1F1B pipeline.  Launches and host time count.
        _case("evaluate_1f1b", "evaluate", "1f1b", 1024, 4, 8, 4),
        # Many candidates of a middling pipeline whose stage -> machine map is given (split backward, 1 % cyclic orders).
        _case("evaluate_zero_bubble", "evaluate", "zero_bubble", 65536, 8, 32, 8),
        # A bidirectional pipeline with communication operations, map given: the largest batch in bytes.
        _case("evaluate_bidirectional", "evaluate", "bidirectional", 16384, 16, 64, 16),
        # Operator-level planning of a 61-layer MoE: every candidate places the operators anew.
        _case("evaluate_moe", "evaluate", "moe", 4096, 61, 8, 32),
        # The largest graph: a layered multi-modal model of 50000 operations on 64 machines.
        _case("evaluate_layered", "evaluate", "layered", 1024, 400, 125, 64),
        # Nothing round: odd sizes, no layers, candidate-minor arrays, times in microseconds, memory limits.
        _case("evaluate_ragged", "evaluate", "random", 2051, 3001, 0, 11, minor=True, micros=True, limits=True),
        # Ten steps of the local search over placements and orders with the batch of the README.
        _case("search_moe", "search", "moe", 256, 61, 8, 32),
        # Ten steps over the orders alone, the map given, on a cluster where only neighbours are connected.
        _case("search_zero_bubble", "search_orders", "zero_bubble", 4096, 8, 32, 8, chain=True),
        # One transfer at a time per channel, a placement per candidate.
        _case("contended_moe", "contended", "moe", 512, 61, 8, 32),
        # The same for a pipeline: few machines, many candidates.
        _case("contended_zero_bubble", "contended", "zero_bubble", 2048, 8, 32, 8),
        # The chosen schedule's start and end times, for a chart or for the runtime that carries it out.
        _case("schedule_moe", "schedule", "moe", 1, 61, 8, 32),
        # Coarsening to the size a MIP solver takes: the scale of the paper's random graph (200 operations to 40).
        _case("coarsen_random", "coarsen", "random", 1, 200, 40, 1),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    do = rng.choice(["evaluate"] * 6 + ["search", "search_orders", "contended", "contended", "schedule", "coarsen"])
    if do == "coarsen":
        n = _log(rng, 40, 400)
        return _case(None, do, "random", 1, n, max(1, n // rng.randint(2, 8)), 1)
    pipes, free = ["1f1b", "zero_bubble", "bidirectional"], ["moe", "layered", "random"]
    graph = rng.choice(pipes if do == "search_orders" else pipes + free)
    p, b = 0, 0
    if graph in ("1f1b", "zero_bubble"):
        p = rng.randint(2, 16)
        a, b = p, _log(rng, 4, 64)
        n = a * b * (2 if graph == "1f1b" else 3)
    elif graph == "bidirectional":
        p = 2 * rng.randint(2, 8)
        a, b = p, 2 * _log(rng, 4, 32)
        n = 6 * a * b
    elif graph == "moe":
        a, b, p = _log(rng, 4, 61), rng.randint(1, 8), rng.randint(4, 32)
        n = 24 * a * b
    elif graph == "layered":
        a, b, p = _log(rng, 24, 400), rng.randint(16, 125), rng.randint(8, 64)
        n = a * b
    else:
        a, p = _log(rng, 60, 6000), rng.randint(2, 40)
        n = a
    most = {"evaluate": min(65536, MOST_ENTRIES // n), "search": min(4096, MOST_ENTRIES // (8 * n)),
            "search_orders": min(4096, MOST_ENTRIES // (8 * n)), "contended": min(2048, 512 * 37072 // (3 * n)), "schedule": 1}[do]
    cands = _log(rng, min(64, most), most)
    return _case(None, do, graph, cands, a, b, p, minor=do == "evaluate" and rng.random() < 0.25, micros=rng.random() < 0.25,
                 limits=do in ("evaluate", "contended") and rng.random() < 0.25, chain=do != "schedule" and graph in ("1f1b", "zero_bubble") and rng.random() < 0.25)


# ----------------------------------------------------------------------------- inputs

def _graph(c, rng):
    """-> (n, src, dst, placement [n] every candidate uses or None, group [n] of operations that share a machine or None)."""
    kind, a, b, p = c["graph"], c["a"], c["b"], c["p"]
    if kind in ("1f1b", "zero_bubble"):          # a stages, b micro-batches, stage s on machine s
        ids, src, dst = W.pipeline_dag(a, b, split_w=kind == "zero_bubble")
        fixed = np.zeros(len(ids), np.int32)
        for (_, s, _), v in ids.items():
            fixed[v] = s
        return len(ids), src, dst, fixed, None
    if kind == "bidirectional":                  # a stages, b micro-batches, fed from both ends; F, B, W and a transfer of each
        k, s = np.meshgrid(np.arange(b), np.arange(a), indexing="ij")
        off = {"F": 2 * s, "CF": 2 * s + 1}
        off.update({x: 2 * a + 4 * (a - 1 - s) + i for i, x in enumerate(("B", "CB", "W", "CW"))})
        node = {x: k * 6 * a + o for x, o in off.items()}
        pairs = [(node["F"], node["CF"]), (node["F"], node["B"]), (node["B"], node["CB"]), (node["B"], node["W"]), (node["W"], node["CW"]),
                 (node["CF"][:, :-1], node["F"][:, 1:]), (node["CB"][:, 1:], node["B"][:, :-1])]
        fixed = np.zeros(6 * a * b, np.int32)
        for x in node:
            fixed[node[x]] = np.where(k < b // 2, s, a - 1 - s)
        return len(fixed), np.concatenate([x.ravel() for x, _ in pairs]), np.concatenate([y.ravel() for _, y in pairs]), fixed, None
    if kind == "moe":                            # a layers of attention, gate, dispatch, 8 experts, combine; b micro-batches, both directions
        roles = 12
        per_dir = a * roles
        edges = []
        for l in range(a):
            r = l * roles
            edges += [(r, r + 1), (r + 1, r + 2), (r, r + 11)] + [(r + 2, r + 3 + e) for e in range(8)] + [(r + 3 + e, r + 11) for e in range(8)]
            if l + 1 < a:
                edges.append((r + 11, r + roles))
        e = np.array(edges)
        op = np.arange(per_dir)
        back = lambda x: 2 * per_dir - 1 - x     # mirror image: last layer first, roles reversed
        src1, dst1 = np.concatenate([e[:, 0], back(e[:, 1]), op]), np.concatenate([e[:, 1], back(e[:, 0]), back(op)])
        shift = (np.arange(b) * 2 * per_dir)[:, None]
        group = np.concatenate([op, op[::-1]])
        return 2 * per_dir * b, (src1 + shift).ravel(), (dst1 + shift).ravel(), None, np.tile(group, b).astype(np.int32)
    if kind == "layered":                        # a levels of b operations, two branches that merge at 3/8 of the depth, fan-in 1..4
        levels, width = a, b
        merge, split = 3 * levels // 8, width // 2
        l, i = (x[1:] for x in np.meshgrid(np.arange(levels), np.arange(width), indexing="ij"))
        lo, hi = np.where((l < merge) & (i >= split), split, 0), np.where((l < merge) & (i < split), split, width)
        src, dst = [], []
        fan = rng.integers(1, 5, l.shape)
        for j in range(4):                       # the first from the level above, the others from up to three levels above
            up = 1 if j == 0 else 1 + rng.integers(0, np.minimum(3, l))
            u = (l - up) * width + lo + (rng.random(l.shape) * (hi - lo)).astype(np.int64)
            src.append(u[fan > j])
            dst.append((l * width + i)[fan > j])
        e = np.unique(np.stack([np.concatenate(src), np.concatenate(dst)]), axis=1)
        return levels * width, e[0], e[1], None, None
    row_ptr, col = W.random_dag(rng, a, 3)       # a operations, up to three inputs from anywhere before
    src, dst = W.edges_from_csr(row_ptr, col)
    return a, src, dst, None, None


def _problem(c, seed):
    rng = np.random.default_rng(seed)
    p = c["p"]
    n, src, dst, fixed, group = _graph(c, rng)
    row_ptr, col = W.csr_from_edges(n, src, dst)
    dur = np.maximum(1, np.rint(np.exp(1.5 + 0.5 * rng.standard_normal(n)))).astype(np.int64)
    comm = rng.integers(1, 5, (p, p))
    if c["micros"]:
        dur, comm = dur * 37 + rng.integers(0, 37, n), comm * 30
    comm = comm.astype(np.int32)
    if c["chain"]:
        j = np.arange(p)
        comm[np.abs(j[:, None] - j[None, :]) > 1] = ds.NO_CHANNEL
    np.fill_diagonal(comm, 0)
    kw = {}
    if c["limits"]:
        kw = dict(weight=rng.integers(0, 20, n), mem_limit=np.full(p, int(10 * n / p * 1.1) + 60))
    return rng, fixed, group, dict(n_devices=p, row_ptr=row_ptr, col_idx=col, dur=dur.astype(np.int32), comm=comm,
                                   mem_delta=rng.integers(-3, 4, n), **kw)


def _candidates(c, rng, prob, fixed, group, count):
    """Randomized list schedules; of every hundred candidates of a larger batch one has two operations of a machine
    trading places, as a search makes them: most of those are cyclic.  -> placement, rank: device int32 [count, n]."""
    n, p, seed = len(prob["dur"]), c["p"], int(rng.integers(1 << 62))
    dev = torch.device("cuda", 0)
    pl, rk = (torch.empty((count, n), dtype=torch.int32, device=dev) for _ in range(2))
    pick = rng.integers(1 << 62, size=count) if count >= 100 else np.ones(count, np.int64)

    def chunk(at):
        hi = min(count, at + step)
        a, b = W.list_schedules(prob["row_ptr"], prob["col_idx"], p, hi - at, seed, fixed_placement=fixed, group=group, first_cand=at)
        for i in np.nonzero(pick[at:hi] % 100 == 0)[0]:
            same = np.nonzero(a[i] == a[i, pick[at + i] // 100 % n])[0]
            u, v = same[pick[at + i] // 7 % len(same)], same[pick[at + i] // 11 % len(same)]
            b[i, u], b[i, v] = b[i, v], b[i, u]
        return at, hi, a, b

    step = max(1, min(-(-count // 32), 4_000_000 // n))
    with ThreadPoolExecutor(min(16, os.cpu_count() or 1)) as pool:
        for at, hi, a, b in pool.map(chunk, range(0, count, step)):
            pl[at:hi].copy_(torch.from_numpy(a))
            rk[at:hi].copy_(torch.from_numpy(b))
    return pl, rk


def _channel_orders(prob, p, pl, rk):
    """First come, first served orders of every channel's transfers (by the producer's rank, then by edge): device int32 [C, E]."""
    src, dst = (torch.from_numpy(x.astype(np.int64)).to(pl.device) for x in W.edges_from_csr(prob["row_ptr"], prob["col_idx"]))
    out = torch.zeros((pl.shape[0], len(src)), dtype=torch.int32, device=pl.device)
    for at in range(0, pl.shape[0], 256):
        a, b, r = pl[at:at + 256, src].long(), pl[at:at + 256, dst].long(), rk[at:at + 256, src].long()
        ch = torch.where(a != b, a * p + b, p * p)
        _, order = torch.sort(ch * pl.shape[1] + r, dim=1, stable=True)
        ch = ch.gather(1, order)
        pos = torch.arange(ch.shape[1], device=ch.device).expand_as(ch)
        head = torch.ones_like(ch, dtype=torch.bool)
        head[:, 1:] = ch[:, 1:] != ch[:, :-1]
        rank = pos - torch.cummax(torch.where(head, pos, 0), dim=1)[0]
        out[at:at + 256].scatter_(1, order, torch.where(ch < p * p, rank, 0).int())
    return out


def prepare(case, seed):
    c = case
    if c["do"] == "coarsen":                     # host arrays in and out
        rng = np.random.default_rng(seed)
        row_ptr, col = W.random_dag_bounded_degree(rng, c["a"], 3)
        n = c["a"]
        most = dict(row_ptr=n + 1, col_idx=3 * n, dur=n, mem_delta=n, mem_req=n)
        return dict(do="coarsen", most=most, args=(row_ptr, col, rng.integers(1, 20, n), rng.integers(-3, 4, n), rng.integers(0, 10, n)),
                    kw=dict(target=c["b"], edge_dur_max=200, edge_mem_max=200, nonedge_dur_max=80, nonedge_mem_max=80))
    rng, fixed, group, prob = _problem(c, seed)
    searching = c["do"].startswith("search")
    pl, rk = _candidates(c, rng, prob, fixed, group, 1 if searching else c["cands"])
    st = dict(do=c["do"], seed=seed, cands=c["cands"])
    if c["do"] == "contended":
        st["er"] = _channel_orders(prob, c["p"], pl, rk)
    if c["minor"]:
        pl, rk = pl.t().contiguous(), rk.t().contiguous()
    ev = ds.Evaluator(max_candidates=c["cands"], layout=ds.CAND_MINOR if c["minor"] else ds.CAND_MAJOR,
                      shared_placement=None if c["do"] == "search" else fixed, contention=c["do"] == "contended", **prob)
    st.update(ev=ev, out=ev.alloc_outputs(c["cands"]))
    st.update(pl=pl, rk=rk) if c["do"] in ("evaluate", "contended") else st.update(pl=pl[0].clone(), rk=rk[0].clone())
    return st


# ----------------------------------------------------------------------------- one pass

def run(st):
    do = st["do"]
    if do == "coarsen":
        got = ds.coarsen(*st["args"], **st["kw"])
        for k, most in st["most"].items():       # as long as any seed's results can be
            full = np.zeros(most, got[k].dtype)
            full[:len(got[k])] = got[k]
            got[k] = full
        return got
    ev, pl, rk = st["ev"], st["pl"], st["rk"]
    if do == "evaluate":
        return ev.evaluate(pl, rk, st["out"])
    if do == "contended":
        return ev.evaluate_contended(pl, rk, st["er"], st["out"])
    if do == "schedule":
        return ev.schedule(pl, rk)
    return search.local_search(ev, pl, rk, ITERATIONS, st["cands"], seed=st["seed"], orders_only=do == "search_orders")


def _sizes(c):
    if c["do"] == "coarsen":
        return c["a"], 2 * c["a"]
    a, b = c["a"], c["b"]
    return {"1f1b": lambda: (2 * a * b, b * (3 * a - 2)), "zero_bubble": lambda: (3 * a * b, b * (4 * a - 2)),
            "bidirectional": lambda: (6 * a * b, b * (7 * a - 2)), "moe": lambda: (24 * a * b, b * (52 * a - 2)),
            "layered": lambda: (a * b, 5 * a * b // 2), "random": lambda: (a, 3 * a // 2)}[c["graph"]]()


def work(case):
    """Bytes: the candidates and the problem read once, the results written once.  Operations: one addition and one
    maximum per DAG edge and per chain edge of every candidate (coarsening: only the graph has to be read and written)."""
    c = case
    n, e = _sizes(c)
    problem = 4 * (n + 1) + 4 * e + 12 * n + 4 * c["p"] ** 2 + (8 * n if c["limits"] else 0)
    results = 16 + 8 * c["p"]
    if c["do"] == "coarsen":
        return {"bytes": problem + 8 * n + 4 * n + 28 * c["b"] + 8 * c["b"], "flops": 0}
    if c["do"] == "schedule":
        return {"bytes": problem + 16 * n + 4, "flops": 2 * (e + n)}
    passes = ITERATIONS if c["do"].startswith("search") else 1
    reads = 16 if c["do"].startswith("search") else 8 * n + (4 * e if c["do"] == "contended" else 0)   # a search hands over random words only
    return {"bytes": problem + passes * c["cands"] * (reads + results), "flops": passes * c["cands"] * 2 * (2 * e if c["do"] == "contended" else e) + 2 * n}


def tolerance(case):
    return "exact"                               # every result is a whole number
