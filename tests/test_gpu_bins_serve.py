"""Served queries whose rounds are binned (graphs of at least 2^22 vertices) on
versioned views: equal to the same queries one at a time with every round
pushed by atomics, and to the oracle on sampled ones."""
import numpy as np
import pytest

import bigraph_gen
import oracle
from tests.gpu_util import ensure_built, say, serve_all, to_dev

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


@pytest.mark.parametrize("slots,window", [(1, 1), (4, 8)])
def test_served_on_views(slots, window):
    nU, nL, m = 1_500_007, 2_999_999, 15_000_000
    eu, ev = bigraph_gen.chung_lu(nU, nL, m, 2.2, 2.2, 20_000, 71)
    key = np.unique(eu.astype(np.int64) * nL + ev)
    rng = np.random.default_rng(72)
    # deletions and insertions around few vertices, so that views differ in
    # the rows the rounds walk
    rows = key[np.isin(key // nL, rng.integers(0, nU, 3000))]
    gone = rng.choice(rows, 20, replace=False)
    new = np.setdiff1d(gone + 1, key)[:12]
    ops = [(k, -1) for k in gone.tolist()] + [(k, 1) for k in new.tolist()]
    ops += [(k, 1) for k in gone[:8].tolist()] + [(k, -1) for k in new[:6].tolist()]
    th = [(3, 2), (8, 4), (20, 10), (2, 2), (60, 30)]
    ups = {"u": [k // nL for k, _ in ops], "v": [k % nL for k, _ in ops],
           "op": [o for _, o in ops], "alpha": [th[i % 5][0] for i in range(len(ops))],
           "beta": [th[i % 5][1] for i in range(len(ops))]}
    alone = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    pkg.abcore_set_option(alone, pkg.ABCORE_OPT_PULL, 1)
    want = []
    for i in range(len(ops)):
        say("alone", i)
        want.append(pkg.abcore_query(alone, *[ups[k][i] for k in
                                              ("u", "v", "op", "alpha", "beta")]))
    alone.destroy()
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    for pull in (0, 2):
        say("served, pull", pull)
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, pull)
        pkg.abcore_serve_start(g, 64, slots, window)
        served = serve_all(g, ups, 64)
        for i, (ans, bits) in enumerate(want):
            assert served[i]["bits"] == bits and bool(served[i]["answer"]) == ans, (pull, i)
        pkg.abcore_serve_stop(g)
        if pull == 0:  # back to the first graph
            for k, o in reversed(ops):
                pkg.abcore_query(g, k // nL, k % nL, -o, 2, 2)
    final = set(key.tolist())
    for k, o in ops:
        (final.add if o > 0 else final.discard)(k)
    fin = np.array(sorted(final), np.int64)
    ref = oracle.Graph(nU, nL, (fin // nL).astype(np.int32), (fin % nL).astype(np.int32))
    a, b = ups["alpha"][-1], ups["beta"][-1]
    member = oracle.compute(ref, a, b)
    assert want[-1][1] == int(member[ups["u"][-1]]) | int(member[nU + ups["v"][-1]]) << 1
    g.destroy()
