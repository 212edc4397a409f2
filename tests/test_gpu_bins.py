"""Binned push rounds (graphs of at least 2^22 vertices): first rounds from
the scan's bitmap and later ones from the queue, after pulled and pushed first
rounds, on sizes that leave a partial last bucket and bitmap word, with split
rows in the frontier, after updates, and in nested batches; against the
oracle."""
import numpy as np
import pytest

import bigraph_gen
import oracle
from tests.gpu_util import bits_np, ensure_built, say, to_dev

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


GRAPHS = {
    "uniform": lambda: (2_500_001, 1_800_003) + tuple(
        bigraph_gen.uniform(2_500_001, 1_800_003, 12_000_000, 21)),
    "skewed": lambda: (1_500_007, 2_999_999) + tuple(
        bigraph_gen.chung_lu(1_500_007, 2_999_999, 30_000_000, 2.1, 2.1, 50_000, 22)),
}


@pytest.fixture(scope="module")
def graphs():
    return {k: f() for k, f in GRAPHS.items()}


def _check(g, ref, a, b, tag):
    want = oracle.pack(oracle.compute(ref, a, b))
    got = bits_np(pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC))[: len(want)]
    assert np.array_equal(got, want), (tag, a, b)


@pytest.mark.parametrize("name,queries", [
    ("uniform", [(1, 1), (3, 4), (5, 7), (4, 8), (9, 2), (40, 40)]),
    ("skewed", [(1, 1), (4, 3), (10, 8), (24, 12), (70, 70), (200, 90), (5000, 5000)])])
def test_index_free_queries(graphs, name, queries):
    nU, nL, eu, ev = graphs[name]
    ref = oracle.Graph(nU, nL, eu, ev)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    pkg.abcore_set_option(g, pkg.ABCORE_OPT_RANK_ORDER, 2)
    for a, b in queries:
        for pull in (0, 2):  # the device's choice, and rounds after a pulled one
            say("bins", name, a, b, "pull", pull)
            pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, pull)
            _check(g, ref, a, b, f"{name} pull {pull}")
    g.destroy()


def test_after_updates(graphs):
    nU, nL, eu, ev = graphs["uniform"]
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    pairs = set(zip(eu[:2000].tolist(), ev[:2000].tolist()))
    gone = sorted(pairs)[::100]
    new = [(int(eu[i]), nL - 1 - i) for i in range(0, 2000, 100)]
    present = set(zip(eu.tolist(), ev.tolist()))
    new = [e for e in new if e not in present]
    for op, (u, v) in [(-1, e) for e in gone] + [(1, e) for e in new]:
        pkg.abcore_query(g, u, v, op, 2, 2)
    key = np.setdiff1d(eu.astype(np.int64) * nL + ev,
                       np.array([u * nL + v for u, v in gone], np.int64))
    key = np.union1d(key, np.array([u * nL + v for u, v in new], np.int64))
    ref = oracle.Graph(nU, nL, (key // nL).astype(np.int32), (key % nL).astype(np.int32))
    for a, b in [(3, 4), (5, 7)]:
        say("bins after updates", a, b)
        _check(g, ref, a, b, "updated")
    g.destroy()


def test_nested_batch(graphs):
    nU, nL, eu, ev = graphs["skewed"]
    ref = oracle.Graph(nU, nL, eu, ev)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    alphas, betas = [1, 3, 6, 6, 12, 30, 60], [2, 3, 4, 9, 9, 16, 40]
    want = [oracle.pack(oracle.compute(ref, a, b)) for a, b in zip(alphas, betas)]
    for order in (1, 2):
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_RANK_ORDER, order)
        for replay in range(3):
            say("bins batch", order, replay)
            out = pkg.abcore_compute_batch(g, alphas, betas)
            for i, w in enumerate(want):
                assert np.array_equal(bits_np(out[i])[: len(w)], w), (order, replay, i)
    g.destroy()
