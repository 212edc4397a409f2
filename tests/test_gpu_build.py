"""The build at the sizes where its key fields, sorts and row batches can go
wrong: layers of one vertex and of powers of two and their neighbours, rows of
the piece length (64) and around it, repeated pairs.  The CSR is compared
with the oracle's, the degree-rank copy through queries that run on it."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("nU,nL,m", [
    (1, 1, 1), (1, 1, 7), (1, 70, 400), (70, 1, 400), (2, 64, 300), (64, 65, 9000),
    (127, 128, 5000), (128, 129, 5001), (256, 255, 30000), (1023, 1025, 40000),
    (5000, 3, 6000), (3, 5000, 6000), (4096, 4097, 100_000)])
def test_build_and_rank_copy(nU, nL, m):
    say("build", nU, nL, m)
    r = np.random.RandomState(nU * 31 + nL)
    # squared uniforms: some long rows in both layers, and repeated pairs
    eu = (r.rand(m) ** 2 * nU).astype(np.int32)
    ev = (r.rand(m) ** 2 * nL).astype(np.int32)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    ref = oracle.Graph(nU, nL, eu, ev)
    pairs = np.unique(eu.astype(np.int64) * nL + ev)
    u, v = pairs // nL, pairs % nL
    assert g.m == len(pairs)
    deg = np.concatenate([np.bincount(u, minlength=nU), np.bincount(v, minlength=nL)])
    off, cols = [t.cpu().numpy() for t in pkg.abcore_export_csr(g)]
    assert np.array_equal(off, np.concatenate([[0], np.cumsum(deg)]))
    o = np.lexsort((u, v))
    assert np.array_equal(cols, np.concatenate([u * 0 + nU + v, u[o]]).astype(np.int32))
    pkg.abcore_set_option(g, pkg.ABCORE_OPT_PULL, 2)  # always on the rank copy
    for a, b in [(1, 1), (2, 3), (int(deg[:nU].mean()) + 1, 2), (2, int(deg[nU:].mean()) + 1)]:
        want = oracle.pack(oracle.compute(ref, a, b))
        bits, st = pkg.abcore_compute(g, a, b, pkg.ABCORE_GCC, stats=True)
        assert st["rank_order"] == 1
        assert np.array_equal(bits_np(bits)[: len(want)], want), (a, b)
    g.destroy()
