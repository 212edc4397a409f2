"""Component labels of sparse graphs without long rows, which merge more often
and then unite the lower vertices' first entries, and of graphs just outside
that rule (half an edge to 7/4 edges a vertex, rows of at most 64 entries):
labels, labels after deletions and insertions, and connected parts of cores,
against the oracle."""
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


def _path(k):
    r = np.random.RandomState(7)
    pu, pv = r.permutation(k + 1), r.permutation(k)
    return k + 1, k, np.concatenate([pu[:-1], pu[1:]]), np.concatenate([pv, pv])


def _tree(k):
    """Lower i hangs on an earlier upper vertex, upper i + 1 on an earlier
    lower one; ids shuffled."""
    r = np.random.RandomState(8)
    i = np.arange(k)
    a, b = (r.rand(k) * (i + 1)).astype(int), (r.rand(k) * (i + 1)).astype(int)
    pu, pv = r.permutation(k + 1), r.permutation(k)
    return k + 1, k, pu[np.concatenate([a, i + 1])], pv[np.concatenate([i, b])]


def _uniform(nU, nL, m):
    return (nU, nL) + tuple(bigraph_gen.uniform(nU, nL, m, 13))


def _stars(d):
    """50 upper vertices of d lower ones each, consecutive ones sharing one."""
    eu = np.repeat(np.arange(50), d)
    ev = (np.arange(50)[:, None] * (d - 1) + np.arange(d)).ravel()
    return 50, 50 * d, eu, ev


def _block(nU, nL, eu, ev):
    """The same with a complete block of 100 by 100 beside it: more edges than
    vertices, rows of 100 entries."""
    k = np.arange(100 * 100)
    return (nU + 100, nL + 100, np.concatenate([eu, nU + k // 100]),
            np.concatenate([ev, nL + k % 100]))


GRAPHS = {
    "path": lambda: _path(4000),
    "tree": lambda: _tree(4000),
    # of 3,500 vertices: half as many edges, 7/4 of them, and the next
    "half": lambda: _uniform(2000, 1500, 1750),
    "past half": lambda: _uniform(2000, 1500, 1751),
    "7/4": lambda: _uniform(2000, 1500, 6125),
    "past 7/4": lambda: _uniform(2000, 1500, 6126),
    "rows of 64": lambda: _stars(64),
    "rows of 65": lambda: _stars(65),
    "large": lambda: _uniform(150_000, 150_000, 290_000),
    "path and block": lambda: _block(*_path(4000)),
    "half and block": lambda: _block(*_uniform(2000, 1500, 1750)),
    "one lower vertex": lambda: (60, 1, np.arange(50), np.zeros(50, np.int64)),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_labels(name):
    nU, nL, eu, ev = GRAPHS[name]()
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    key = np.unique(np.asarray(eu, np.int64) * nL + ev)

    def check():
        ref = oracle.Graph(nU, nL, (key // nL).astype(np.int32), (key % nL).astype(np.int32))
        assert np.array_equal(pkg.abcore_components(g).cpu().numpy(), oracle.components(ref))
        return ref

    ref = check()
    r = np.random.default_rng(9)
    for q, (a, b) in zip([0, nU] + r.integers(0, nU + nL, 4).tolist(),
                         [(1, 1), (1, 2), (2, 1), (1, 1), (2, 2), (1, 1)]):
        say("sparse part", name, q, a, b)
        want = oracle.community(ref, q, a, b, True)
        bits, size = pkg.abcore_community(g, q, a, b, connected=True)
        w = oracle.pack(want)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32)[: len(w)], w)
        assert size == int(want.sum())
    gone = r.choice(key, 24, replace=False)
    new = np.setdiff1d(r.integers(0, nU * nL, 12), key)
    for op, ks in ((-1, gone), (1, new), (1, gone[:6])):
        for i, k in enumerate(ks.tolist()):
            say("sparse update", name, op, k)
            pkg.abcore_query(g, k // nL, k % nL, op, 1, 1)
            key = np.setdiff1d(key, [k]) if op < 0 else np.union1d(key, [k])
            if i % 3 == 0:
                check()
    g.destroy()
