"""Host side of the kernels whose operations share end-time cells: an operation may take over a cell only when every
reader of the one before it is itself or precedes it in the DAG, by any path (checked against all ancestors)."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2503_09357_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("cells") / "share_cells.so")
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-std=c++17", "-I", os.path.join(HERE, "..", "paper_2503_09357_amd", "csrc"),
                    os.path.join(HERE, "share_cells_driver.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def _preds(n, src, dst):
    order = np.argsort(dst, kind="stable")
    ptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(dst, minlength=n), out=ptr[1:])
    return ptr, np.ascontiguousarray(np.asarray(src)[order], np.int32)


def _ancestors(n, ptr, idx):
    succ, left = [[] for _ in range(n)], np.diff(ptr)
    for v in range(n):
        for u in idx[ptr[v]:ptr[v + 1]]:
            succ[u].append(v)
    todo, anc = [v for v in range(n) if left[v] == 0], [0] * n
    while todo:
        u = todo.pop()
        for v in succ[u]:
            anc[v] |= anc[u] | (1 << u)
            left[v] -= 1
            if left[v] == 0:
                todo.append(v)
    return anc


def _share(lib, n, src, dst, read, max_user=1 << 20):
    rp, ri = _preds(n, src, dst)
    qp, qi = _preds(n, np.asarray(src)[read], np.asarray(dst)[read])
    cell, user = np.zeros(n, np.int32), np.zeros(n, np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    cells = lib.share_cells(n, p(rp), p(ri), p(qp), p(qi), max_user, p(cell), p(user))
    anc, readers, by_cell = _ancestors(n, rp, ri), [[] for _ in range(n)], {}
    for v in range(n):
        for u in qi[qp[v]:qp[v + 1]]:
            readers[u].append(v)
    for v in range(n):
        assert (cell[v] > 0) == bool(readers[v])
        if readers[v]:
            by_cell.setdefault(int(cell[v]), []).append((int(user[v]), v))
    assert sorted(by_cell) == list(range(1, cells + 1))
    for held in by_cell.values():
        held.sort()
        assert [k for k, _ in held] == list(range(1, len(held) + 1)) and len(held) <= max_user
        for (_, u), (_, x) in zip(held, held[1:]):
            assert all(w == x or (anc[x] >> w) & 1 for w in readers[u]), (u, x)
    return cells


@pytest.mark.parametrize("seed", range(40))
def test_a_cell_is_taken_over_only_behind_its_readers(lib, seed):
    rng = np.random.default_rng(seed)
    n = int(rng.choice([1, 2, 3, 63, 64, 65, 300, 511, 512, 513, 1100]))
    rp, ci = W.random_dag(rng, n, int(rng.integers(1, 6)), window=int(rng.integers(2, 700)), dup_prob=0.1)
    src, dst = W.edges_from_csr(rp, ci)
    if seed % 2:                                              # ids that are no topological order
        perm = rng.permutation(n)
        src, dst = perm[src], perm[dst]
    _share(lib, n, src, dst, rng.random(len(src)) < rng.choice([0.3, 1.0]), int(rng.choice([1, 2, 5, 1 << 20])))


def test_chains_and_pipelines_hand_their_cells_on(lib):
    for parts in (1, 3):                                      # chains side by side, numbered one after the other and mixed
        n = 1500 * parts
        for step in (1, parts):
            v = np.arange(n - step)
            keep = (v % 1500 != 1499) if step == 1 else np.ones(len(v), bool)
            src, dst = v[keep], v[keep] + step
            assert _share(lib, n, src, dst, np.ones(len(src), bool)) == (parts if step == 1 or parts > 1 else 1)
    w = W.gen_config(4, n_cand=1)                             # MoE graph without forward -> backward edges and shortcuts that other paths imply
    src, dst = W.edges_from_csr(w.row_ptr, w.col_idx)
    keep = (dst - src < 12) & ~np.isin((dst - src) * 100 + src % 12, [1100])
    assert _share(lib, w.n_nodes, src[keep], dst[keep], np.ones(int(keep.sum()), bool)) <= 200
