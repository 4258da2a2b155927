"""dagsched_coarsen against the oracle where its kernels change: graphs around 256 and 512 operations (rows of four and of
eight words in LDS, then the kernel that works in the L2), chains and wide graphs, requirements beyond 32 bits."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2503_09357_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 255, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("kind", ["random", "chains", "wide"])
def test_coarsen_around_the_row_sizes(gpu_lib, n, kind):
    ds = gpu_lib
    rng = np.random.default_rng(n)
    print("[coarsen] n=%d %s" % (n, kind), flush=True)
    if kind == "random":
        rp, ci = W.random_dag_bounded_degree(rng, n, 3)
    elif kind == "chains":                                   # seven chains side by side: every depth has seven operations
        rp, ci = W.csr_from_edges(n, list(range(n - 7)), list(range(7, n)))
    else:                                                    # one source, n - 2 operations, one sink
        rp, ci = W.csr_from_edges(n, [0] * (n - 2) + list(range(1, n - 1)), list(range(1, n - 1)) + [n - 1] * (n - 2))
    dur, mem, req = rng.integers(0, 20, n), rng.integers(-3, 4, n), rng.integers(0, 10, n)
    for scale, kw in ((1, dict(target=n // 5, edge_dur_max=100, edge_mem_max=60, nonedge_dur_max=40, nonedge_mem_max=30)),
                      (1 << 33, dict(target=1, edge_dur_max=ds.NO_MERGES, nonedge_dur_max=60, nonedge_mem_max=25 << 33)),
                      (1, dict(target=3))):
        if kw["target"] == 3 and n > 257:
            continue                                         # (the oracle takes long to merge a large graph down)
        got, want = ds.coarsen(rp, ci, dur, mem, req * scale, **kw), oracle.coarsen(rp, ci, dur, mem, req * scale, **kw)
        for key in want:
            assert np.array_equal(got[key], want[key]), (key, kw)
