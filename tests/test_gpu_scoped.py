"""Scoped queries whose scan resets the workspace: two components with their
bounds inside a bitmap word, frontiers pushed and pulled, other computations
of the same handle in between, and rejected updates; against the oracle."""
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


def _two(nU1, nL1, m1, nU2, nL2, m2, seed):
    a = bigraph_gen.uniform(nU1, nL1, m1, seed)
    b = bigraph_gen.uniform(nU2, nL2, m2, seed + 1)
    return (nU1 + nU2, nL1 + nL2, np.concatenate([a[0], b[0] + nU1]).astype(np.int32),
            np.concatenate([a[1], b[1] + nL1]).astype(np.int32))


@pytest.mark.parametrize("pull", [0, 1, 2])
@pytest.mark.parametrize("sizes", [(4, 4, 4, 3, 3, 3), (37, 29, 200, 70, 61, 500),
                                   (1000, 900, 9000, 15_001, 12_007, 150_000)])
def test_between_other_computations(sizes, pull):
    nU, nL, eu, ev = _two(*sizes, 51)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, pull)
    rng = np.random.default_rng(52)
    edges = {(int(u), int(v)) for u, v in zip(eu, ev)}
    ups = {k: [] for k in ("u", "v", "op", "alpha", "beta")}
    for i in range(24):
        if i % 3 == 0 and edges:
            u, v = sorted(edges)[rng.integers(len(edges))]
            op = -1
            edges.discard((u, v))
        else:
            u, v, op = int(rng.integers(nU)), int(rng.integers(nL)), 1
            if i % 3 == 1:  # rejected if present
                edges.add((u, v))
            else:
                u, v, op = (*sorted(edges)[0], 1) if edges else (u, v, -1)
        for k, x in zip(ups, (u, v, op, 1 + i % 5, 1 + i % 7)):
            ups[k].append(x)
    want = oracle.gfq_stream(nU, nL, eu, ev, ups)
    for i, (st, ans, bits) in enumerate(want):
        say("scoped", sizes, "pull", pull, "update", i, st)
        args = [ups[k][i] for k in ("u", "v", "op", "alpha", "beta")]
        if st != "OK":
            with pytest.raises(pkg.AbcoreError):
                pkg.abcore_query(g, *args)
        else:
            assert pkg.abcore_query(g, *args) == (ans, bits), i
        if i % 4 == 0:  # leaves the workspace used
            pkg.abcore_compute(g, 2, 3, pkg.ABCORE_GCC, stats=i % 8 == 0)
        if i % 6 == 0:
            pkg.abcore_compute_batch(g, [1, 2], [1, 2])
    present = {(int(u), int(v)) for u, v in zip(eu, ev)}
    for i, (st, _, _) in enumerate(want):
        e = (ups["u"][i], ups["v"][i])
        if st == "OK":
            (present.add if ups["op"][i] > 0 else present.discard)(e)
    fin = np.array(sorted(present), np.int32).reshape(-1, 2)
    ref = oracle.Graph(nU, nL, fin[:, 0].copy(), fin[:, 1].copy())
    got = bits_np(pkg.abcore_compute(g, 2, 2, pkg.ABCORE_GCC))
    assert np.array_equal(got, oracle.pack(oracle.compute(ref, 2, 2)))
    g.destroy()
