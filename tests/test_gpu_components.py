"""Component labels on the device: shapes on which the hooks, the merges and
the completion of the union-find each have to do the joining, before and
after updates (labels are integers: compared exactly with the oracle)."""
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
    """The path u0 v0 u1 v1 ... with ids shuffled: chains of parents."""
    r = np.random.RandomState(7)
    pu, pv = r.permutation(k + 1).astype(np.int32), r.permutation(k).astype(np.int32)
    eu = np.concatenate([pu[:-1], pu[1:]])
    ev = np.concatenate([pv, pv])
    return k + 1, k, eu, ev


def _shape(name):
    if name == "path":
        return _path(3000)
    if name == "pairs":  # every component one edge
        k = np.arange(5000, dtype=np.int32)
        return 5000, 5000, k, k[::-1].copy()
    if name == "stars":  # hubs of both layers, joined by one edge
        a = np.arange(1, 4000, dtype=np.int32)
        eu = np.concatenate([np.zeros(3999, np.int32), a, [0]]).astype(np.int32)
        ev = np.concatenate([a, np.zeros(3999, np.int32), [0]]).astype(np.int32)
        return 4000, 4000, eu, ev
    if name == "sparse":  # about as many components as edges
        return (3001, 2003) + tuple(bigraph_gen.uniform(3001, 2003, 2500, 11))
    if name == "skewed":
        return (2000, 1000) + tuple(bigraph_gen.chung_lu(2000, 1000, 9000, 2.1, 2.1, 500, 12))
    return 1, 1, np.zeros(1, np.int32), np.zeros(1, np.int32)


@pytest.mark.parametrize("name", ["path", "pairs", "stars", "sparse", "skewed", "edge"])
def test_labels_match_oracle(name):
    nU, nL, eu, ev = _shape(name)
    say("components", name)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    want = oracle.components(oracle.Graph(nU, nL, eu, ev))
    assert np.array_equal(pkg.abcore_components(g).cpu().numpy(), want)
    g.destroy()


@pytest.mark.parametrize("name,seed", [("path", 1), ("pairs", 2), ("stars", 3), ("sparse", 4),
                                       ("skewed", 5), ("edge", 6)])
def test_labels_after_deletions_match_oracle(name, seed):
    """Deletions of bridges, leaves, label vertices and edges on cycles, more
    than 16 of them in one hub's row (its first entries become tombstones),
    then re-insertions: labels after each."""
    nU, nL, eu, ev = _shape(name)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    pkg.abcore_components(g)
    edges = sorted(set(zip(eu.tolist(), ev.tolist())))
    r = np.random.RandomState(seed)
    hub = int(np.bincount(eu).argmax())
    picks = [e for e in edges if e[0] == hub][:20]
    picks += [edges[i] for i in r.permutation(len(edges))[:15]]
    picks = list(dict.fromkeys(picks))
    left = set(edges)
    for op, (u, v) in [(-1, e) for e in picks] + [(1, e) for e in picks[::3]]:
        say("update", name, op, u, v)
        pkg.abcore_query(g, u, v, op, 1, 1)
        (left.discard if op < 0 else left.add)((u, v))
        cur = np.array(sorted(left), np.int32).reshape(-1, 2)
        want = oracle.components(oracle.Graph(nU, nL, cur[:, 0].copy(), cur[:, 1].copy()))
        assert np.array_equal(pkg.abcore_components(g).cpu().numpy(), want), (op, u, v)
    g.destroy()


@pytest.mark.parametrize("inserted", [0, 1, 64, 65, 200])
def test_export_after_updates(inserted):
    """The exported CSR of an updated graph: rows of both sides of the piece
    length (64) and a hub of 3,000 entries, tombstones in some, and `inserted`
    new edges of one row (its list held in LDS up to 64)."""
    r = np.random.RandomState(inserted)
    nU, nL = 300, 4000
    rows = {0: 3000, 1: 64, 2: 65, 3: 1, 5: 63, 6: 128, 7: 129}
    eu = np.concatenate([np.full(d, u) for u, d in rows.items()] + [r.randint(8, nU, 2000)])
    ev = np.concatenate([r.permutation(3700)[:d] for d in rows.values()] +
                        [r.randint(0, 3700, 2000)])
    left = set(zip(eu.tolist(), ev.tolist()))
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    gone = [e for u in (0, 2, 3, 6) for e in sorted(x for x in left if x[0] == u)[::40]]
    # (lower ids from 3700 on have no edges yet; the smaller ones interleave)
    new = [(0, v) for v in range(4000) if (0, v) not in left][::3][:inserted]
    for op, (u, v) in [(-1, e) for e in gone] + [(1, e) for e in new]:
        pkg.abcore_query(g, u, v, op, 2, 2)
        (left.discard if op < 0 else left.add)((u, v))
    off, cols = [t.cpu().numpy() for t in pkg.abcore_export_csr(g)]
    pairs = sorted(left)
    deg = np.bincount([u for u, _ in pairs] + [nU + v for _, v in pairs], minlength=nU + nL)
    assert np.array_equal(off, np.concatenate([[0], np.cumsum(deg)]))
    want = [nU + v for _, v in pairs] + [u for u, v in sorted(pairs, key=lambda e: (e[1], e[0]))]
    assert np.array_equal(cols, np.array(want, np.int32))
    g.destroy()


@pytest.mark.parametrize("a,b", [(1, 1), (2, 1), (1, 2), (2, 2)])
@pytest.mark.parametrize("name", ["path", "pairs", "stars", "sparse", "skewed", "edge"])
def test_connected_part_of_a_core(name, a, b):
    """The connected part of a core around members and non-members, on parts
    of every size (long chains of members among them), before and after
    deletions."""
    nU, nL, eu, ev = _shape(name)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    r = np.random.RandomState(8)
    left = sorted(set(zip(eu.tolist(), ev.tolist())))
    for step in range(2):
        cur = np.array(left, np.int32).reshape(-1, 2)
        ref = oracle.Graph(nU, nL, cur[:, 0].copy(), cur[:, 1].copy())
        for q in [0, nU] + r.randint(0, nU + nL, 4).tolist():
            say("connected part", name, a, b, q)
            want = oracle.community(ref, q, a, b, True)
            bits, size = pkg.abcore_community(g, q, a, b, connected=True)
            w = oracle.pack(want)
            assert np.array_equal(bits.cpu().numpy().view(np.uint32)[: len(w)], w), q
            assert size == int(want.sum())
        for u, v in left[1::97]:
            pkg.abcore_query(g, u, v, -1, a, b)
        left = [e for i, e in enumerate(left) if i % 97 != 1]
    g.destroy()
