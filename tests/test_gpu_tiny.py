"""Queries that run in one workgroup each (graphs that fit its LDS): rows at
the edges of a piece (32 entries) and across many, layers at the edges of a
bitmap word and of the workgroup, the largest graph of the range and the next
one, batches of more than one launch, and graphs after updates; against the
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


def _rows(lengths, n_lower):
    """Upper row i holds the first lengths[i] lower vertices."""
    eu = np.repeat(np.arange(len(lengths)), lengths).astype(np.int32)
    ev = np.concatenate([np.arange(k) for k in lengths]).astype(np.int32)
    return len(lengths), n_lower, eu, ev


def _cut(n_upper, n_lower, m, seed):
    eu, ev = bigraph_gen.uniform(n_upper, n_lower, m + m // 8, seed)
    key = np.unique(eu.astype(np.int64) * n_lower + ev)
    key = np.random.default_rng(seed).choice(key, m, replace=False)
    return n_upper, n_lower, (key // n_lower).astype(np.int32), (key % n_lower).astype(np.int32)


GRAPHS = {
    "one edge": lambda: (1, 1, np.zeros(1, np.int32), np.zeros(1, np.int32)),
    "no edge": lambda: (3, 30, np.zeros(0, np.int32), np.zeros(0, np.int32)),
    # a chain of rows that fall one after the other
    "stairs": lambda: _rows([1, 2, 3, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129], 200),
    "hub": lambda: _rows([4000] + [1] * 500 + [40] * 523, 4001),
    "word": lambda: (512, 512) + tuple(bigraph_gen.uniform(512, 512, 4_000, 31)),
    "past": lambda: (513, 512) + tuple(bigraph_gen.uniform(513, 512, 4_100, 32)),
    "skewed": lambda: (1_777, 901) + tuple(
        bigraph_gen.chung_lu(1_777, 901, 30_000, 2.1, 2.1, 800, 33)),
    # 40,960 pairs are the most of single queries, 163,840 of a batch; then one more
    "most": lambda: _cut(6_000, 5_000, 40_960, 34),
    "one more": lambda: _cut(6_000, 5_000, 40_961, 34),
    "most of a batch": lambda: _cut(4_000, 3_000, 163_840, 37),
    "past a batch": lambda: _cut(4_000, 3_000, 163_841, 37),
    "many vertices": lambda: (10_000, 9_000) + tuple(
        bigraph_gen.uniform(10_000, 9_000, 20_000, 35)),
}
THRESHOLDS = [(1, 1), (2, 2), (3, 2), (1, 9), (7, 3), (12, 14), (33, 1), (5000, 1),
              (2**32 - 1, 2**32 - 1)]


@pytest.mark.parametrize("name", list(GRAPHS))
def test_against_oracle(name):
    nU, nL, eu, ev = GRAPHS[name]()
    ref = oracle.Graph(nU, nL, eu, ev)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    want = {q: oracle.pack(oracle.compute(ref, min(q[0], 2**31 - 1), min(q[1], 2**31 - 1)))
            for q in THRESHOLDS}
    for rank_order in (2, 0):
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_RANK_ORDER, rank_order)
        for a, b in THRESHOLDS:
            say("tiny", name, a, b)
            got = bits_np(pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC))
            assert np.array_equal(got, want[(a, b)]), (name, a, b)
            plus = bits_np(pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC_PLUS))
            assert np.array_equal(plus, got), (name, a, b)
            # the general path, which keeps the statistics
            out, st = pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC, stats=True)
            assert np.array_equal(bits_np(out), got) and st["removed"] == nU + nL - int(
                oracle.unpack(got, nU + nL).sum())
    # a batch of one launch, and of one query past it
    for q in (1, 3, 4, 256, 257):
        say("tiny batch", name, q)
        pairs = [THRESHOLDS[i % len(THRESHOLDS)] for i in range(q)]
        got = bits_np(pkg.abcore_compute_batch(g, [p[0] for p in pairs], [p[1] for p in pairs]))
        for i, p in enumerate(pairs):
            assert np.array_equal(got[i], want[p]), (name, q, i)
    g.destroy()


def test_after_updates():
    nU, nL, eu, ev = GRAPHS["skewed"]()
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    key = np.unique(eu.astype(np.int64) * nL + ev)
    rng = np.random.default_rng(36)
    gone = rng.choice(key, 40, replace=False)
    new = np.setdiff1d(rng.integers(0, nU * nL, 60), key)[:20]
    for op, ks in ((-1, gone), (1, new)):  # (inserted edges: the general path)
        for k in ks.tolist():
            pkg.abcore_query(g, k // nL, k % nL, op, 2, 2)
        key = np.setdiff1d(key, ks) if op < 0 else np.union1d(key, ks)
        ref = oracle.Graph(nU, nL, (key // nL).astype(np.int32), (key % nL).astype(np.int32))
        for a, b in [(2, 2), (4, 7), (9, 20)]:
            say("tiny after updates", op, a, b)
            got = bits_np(pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC))
            assert np.array_equal(got, oracle.pack(oracle.compute(ref, a, b))), (op, a, b)
    g.destroy()
