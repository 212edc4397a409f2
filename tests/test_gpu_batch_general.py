"""The general path of batches and queries on small graphs, which by default
run in one workgroup each: nested scans, the captured launches and their
replays, also after updates; and the same around the one-workgroup path's
limit.  Against the oracle."""
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


def _build(nU, nL, eu, ev, general):
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    if general:
        # a wait limit of the caller's own (here the default's value) leaves
        # the one-workgroup path
        pkg.abcore_set_option(g, pkg.ABCORE_OPT_SPIN_LIMIT, 1 << 23)
    return g


def _batch(g, ref, alphas, betas):
    want = oracle.batch(ref, [min(a, 2**31 - 1) for a in alphas],
                        [min(b, 2**31 - 1) for b in betas])
    got = bits_np(pkg.abcore_compute_batch(g, alphas, betas))
    assert np.array_equal(got[:, : want.shape[1]], want)
    return got


def _pairs(q, hi, seed, extra=()):
    a, b = bigraph_gen.loguniform_pairs(q, 1, hi, seed)
    return ([int(x) for x in a] + [x for x, _ in extra],
            [int(x) for x in b] + [y for _, y in extra])


@pytest.mark.parametrize("general", [False, True])
def test_uniform_batch(general):
    spec = bigraph_gen.CONFIGS[1]
    eu, ev = bigraph_gen.make_graph(spec)
    ref = oracle.Graph(spec["n_upper"], spec["n_lower"], eu, ev)
    maxdeg = int(ref.degrees().max())
    alphas, betas = _pairs(40, 24, 1001, [(1, 1), (3, 2), (3, 2), (maxdeg + 1, 1),
                                          (1, maxdeg + 1), (2**31, 5), (7, 7), (7, 7)])
    g = _build(spec["n_upper"], spec["n_lower"], eu, ev, general)
    for replay in range(3):
        say("general", general, "replay", replay)
        got = _batch(g, ref, alphas, betas)
        for i in (0, 7, 14, 41, 43):
            one = bits_np(pkg.abcore_compute(g, alphas[i], betas[i], pkg.ABCORE_GCC))
            assert np.array_equal(one[: got.shape[1]], got[i])
            plus = bits_np(pkg.abcore_compute(g, alphas[i], betas[i], pkg.ABCORE_GCC_PLUS))
            assert np.array_equal(plus[: got.shape[1]], got[i])
    g.destroy()


@pytest.mark.parametrize("general", [False, True])
def test_few_edges(general):
    eu = np.array([0, 0, 1, 1, 2], np.int32)
    ev = np.array([0, 1, 0, 1, 2], np.int32)
    g = _build(4, 3, eu, ev, general)
    ref = oracle.Graph(4, 3, eu, ev)
    say("five edges, general", general)
    for alphas, betas in [([1], [1]), ([2, 1, 2, 3, 1], [2, 1, 2, 1, 3])]:
        for _ in range(3):
            _batch(g, ref, alphas, betas)
    g.destroy()
    e = np.zeros(0, np.int32)
    g = _build(3, 2, e, e, general)
    _batch(g, oracle.Graph(3, 2, e, e), [1, 2, 1], [1, 1, 2])
    g.destroy()


# pairs: far below, and past the limit of a batch of four queries and more
@pytest.mark.parametrize("m,general", [(15_000, True), (15_000, False), (200_000, False)])
def test_after_updates(m, general):
    nU, nL = (3000, 2000) if m < 100_000 else (12_000, 9_000)
    spec = dict(kind="chung_lu", n_upper=nU, n_lower=nL, m=m, gamma_upper=2.1,
                gamma_lower=2.1, cap=400, seed=402)
    eu, ev = bigraph_gen.make_graph(spec)
    g = _build(nU, nL, eu, ev, general)
    alphas, betas = _pairs(30, 12, 1402)
    for _ in range(2):  # the launches are captured, and replayed
        _batch(g, oracle.Graph(nU, nL, eu, ev), alphas, betas)
    ups = bigraph_gen.update_stream(spec, eu, ev, 120, 1403, qlo=1, qhi=4)
    keys = set(int(a) * nL + int(b) for a, b in zip(eu, ev))
    for i in range(len(ups["u"])):
        pkg.abcore_query(g, ups["u"][i], ups["v"][i], ups["op"][i], 1, 1)
        k = int(ups["u"][i]) * nL + int(ups["v"][i])
        (keys.add if ups["op"][i] > 0 else keys.discard)(k)
        if i % 60 in (0, 59):
            kk = np.array(sorted(keys), np.int64)
            ref = oracle.Graph(nU, nL, (kk // nL).astype(np.int32), (kk % nL).astype(np.int32))
            say("after update", i, "pairs", m, "general", general)
            for _ in range(2):
                _batch(g, ref, alphas, betas)
    g.destroy()
