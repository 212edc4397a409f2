"""Core numbers whose deep core's rows are built with local ids by vertex
(graphs of at most 2^21 vertices) and by rank (one vertex more), with deleted
and inserted edges in them; against the oracle."""
import numpy as np
import pytest

import bigraph_gen
import oracle
from tests.gpu_util import ensure_built, say, to_dev

pytestmark = pytest.mark.gpu

pkg = None


@pytest.fixture(scope="module", autouse=True)
def _setup():
    global pkg
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ensure_built()
    import paper_2606_07148_amd as p
    pkg = p
    yield


@pytest.mark.parametrize("n_upper,n_lower,m", [(3, 2, 4), (700, 500, 9_000),
                                               (1_200_000, 897_152, 3_000_000),
                                               (1_200_000, 897_153, 3_000_000)])
def test_by_vertex_and_by_rank(n_upper, n_lower, m):
    if m < 100:
        eu, ev = np.array([0, 0, 1, 2], np.int32), np.array([0, 1, 1, 0], np.int32)
    else:
        eu, ev = bigraph_gen.chung_lu(n_upper, n_lower, m, 2.2, 2.2, min(400, n_lower // 2), 61)
    g = pkg.abcore_build_csr(n_upper, n_lower, to_dev(eu), to_dev(ev))
    key = np.unique(eu.astype(np.int64) * n_lower + ev)
    for step in range(3):
        say("top ids", n_upper, n_lower, "step", step)
        if step == 1:  # delete, then insert (in rows of the deep core too)
            gone = key[:: max(2, len(key) // 20)]
            for k in gone.tolist():
                pkg.abcore_query(g, k // n_lower, k % n_lower, -1, 1, 1)
            key = np.setdiff1d(key, gone)
        if step == 2:
            hub = int(np.bincount(key // n_lower).argmax())
            new = [hub * n_lower + v for v in range(min(40, n_lower))]
            new = np.setdiff1d(np.array(new, np.int64), key)
            for k in new.tolist():
                pkg.abcore_query(g, k // n_lower, k % n_lower, 1, 1, 1)
            key = np.union1d(key, new)
        ref = oracle.Graph(n_upper, n_lower, (key // n_lower).astype(np.int32),
                           (key % n_lower).astype(np.int32))
        core, mx = pkg.abcore_core_numbers(g)
        want = oracle.core_numbers(ref)
        assert np.array_equal(core.cpu().numpy(), want) and mx == int(want.max())
    g.destroy()
