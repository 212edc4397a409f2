"""Which rounds are binned: the launches of a query on each side of the rule,
first rounds that the device bins, and inserted edges at split rows of binned
rounds; results are the oracle's."""
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
        bigraph_gen.chung_lu(1_500_007, 2_999_999, 20_000_000, 2.1, 2.1, 50_000, 22)),
    "small": lambda: (2_000_000, 1_800_003) + tuple(
        bigraph_gen.uniform(2_000_000, 1_800_003, 12_000_000, 21)),
}
ROUNDS = 3  # of a single query: pull, split rows, and two launches a round


def _frontier(ref, a, b):
    """Entries of the rows below the thresholds, and of the others."""
    d = ref.degrees()
    thr = np.where(np.arange(ref.n) < ref.n_upper, a, b)
    return int(d[d < thr].sum()), int(d[d >= thr].sum())


def _query(g, ref, a, b):
    want = oracle.pack(oracle.compute(ref, a, b))
    pkg.abcore_kernel_timing(g, 1)  # PULL: resets
    bits, st = pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC, stats=True)
    assert np.array_equal(bits_np(bits)[: len(want)], want), (a, b)
    return pkg.abcore_kernel_timing(g, 1)[1], st


@pytest.mark.parametrize("name,queries", [
    ("uniform", [(1, 1), (2, 2), (3, 4), (4, 5), (5, 7), (9, 2), (40, 40)]),
    ("skewed", [(1, 1), (2, 2), (10, 8), (24, 12), (70, 70)]),
    ("small", [(3, 4), (5, 7), (9, 2)])])
def test_launches_follow_the_rule(name, queries):
    nU, nL, eu, ev = GRAPHS[name]()
    ref = oracle.Graph(nU, nL, eu, ev)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    pkg.abcore_set_option(g, pkg.ABCORE_OPT_RANK_ORDER, 2)
    pkg.abcore_set_option(g, pkg.ABCORE_OPT_TIMING, 1)
    sides, first = set(), 0
    for a, b in queries:
        f0, rest = _frontier(ref, a, b)
        many = ref.n >= 1 << 22 and f0 >= ref.n // 16 + (1 << 20)
        for pull in (0, 2):
            pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, pull)
            launches, st = _query(g, ref, a, b)
            say("rule", name, a, b, "pull", pull, "frontier", f0, rest, launches, st["pulled"])
            assert launches == (2 + 2 * ROUNDS if many else 1)
            if many and pull == 0 and not st["pulled"]:
                first += 1  # pushed, of n / 16 entries and more: binned
                assert f0 < rest
        sides.add(many)
    assert sides == ({False} if name == "small" else {False, True})
    assert first >= (0 if name == "small" else 1)
    g.destroy()


def test_inserted_edges_at_split_rows():
    nU, nL, eu, ev = GRAPHS["skewed"]()
    base = np.unique(eu.astype(np.int64) * nL + ev)
    ref = oracle.Graph(nU, nL, eu, ev)
    d = ref.degrees()
    # rows of 65 to 69 entries (pieces) fall in the first round at (70, 70),
    # rows of 70 to 75 mostly later
    rng = np.random.default_rng(3)
    up = rng.choice(np.flatnonzero((d[:nU] > 64) & (d[:nU] < 76)), 24, replace=False)
    lo = rng.choice(np.flatnonzero((d[nU:] > 64) & (d[nU:] < 76)), 24, replace=False)
    new = np.setdiff1d(np.concatenate([up[:12] * nL + lo[:12], up[12:] * nL + lo[:12],
                                       up[:12] * nL + lo[12:]]).astype(np.int64), base)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    for k in new.tolist():
        pkg.abcore_query(g, k // nL, k % nL, 1, 5000, 5000)
    key = np.union1d(base, new)
    ref = oracle.Graph(nU, nL, (key // nL).astype(np.int32), (key % nL).astype(np.int32))
    pkg.abcore_set_option(g, pkg.ABCORE_OPT_TIMING, 1)
    for a, b in [(70, 70), (72, 66), (76, 76), (40, 90)]:
        for pull in (0, 2):
            say("inserted at split rows", a, b, "pull", pull)
            pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, pull)
            assert _query(g, ref, a, b)[0] == 2 + 2 * ROUNDS
    g.destroy()


def test_handles_of_different_bucket_sizes():
    """A handle with large buckets stays usable while others with smaller ones
    come and go (the kernels' LDS limits are the device's, not a handle's);
    compared with the same queries pushed by atomics."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)

    def build(nU, nL, m):
        eu = torch.randint(0, nU, (m,), dtype=torch.int32, device="cuda", generator=gen)
        ev = torch.randint(0, nL, (m,), dtype=torch.int32, device="cuda", generator=gen)
        g = pkg.abcore_build_csr(nU, nL, eu, ev)
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_RANK_ORDER, 2)
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_TIMING, 1)
        return g

    def same(g, a, b):
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, 1)
        want = bits_np(pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC)).copy()
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, 0)
        pkg.abcore_kernel_timing(g, 1)
        assert np.array_equal(bits_np(pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC)), want)
        assert pkg.abcore_kernel_timing(g, 1)[1] == 2 + 2 * ROUNDS

    large = build(10_000_000, 7_000_000, 40_000_000)  # 32,768 vertices to a bucket
    say("buckets: large alone")
    same(large, 4, 5)
    small = build(2_400_000, 1_900_000, 12_000_000)   # 8,192
    say("buckets: both")
    same(small, 4, 6)
    same(large, 4, 5)
    small.destroy()
    same(large, 4, 5)
    large.destroy()
