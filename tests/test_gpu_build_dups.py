"""Deduplication of the build at the edges of its tiles (4,096 keys) and waves
(1,024): runs of equal pairs that start, end or lie across an edge, one pair
only, and none repeated; against numpy."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("m", [1, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 12_289, 300_000])
@pytest.mark.parametrize("kind", ["one", "distinct", "runs", "hub"])
def test_duplicates(m, kind):
    r = np.random.RandomState(m)
    nU, nL = 701, 997
    if kind == "one":
        key = np.full(m, 5 * nL + 7, np.int64)
    elif kind == "distinct":
        key = r.permutation(nU * nL)[:m].astype(np.int64)
    elif kind == "runs":  # lengths 1 to 200
        key = np.repeat(np.arange(m, dtype=np.int64), r.randint(1, 200, m))[:m] % (nU * nL)
    else:  # one row holds half of the pairs, many of them repeated
        key = np.where(r.rand(m) < 0.5, 3 * nL + r.randint(0, nL, m), r.randint(0, nU * nL, m))
    key = r.permutation(key)
    say("dups", m, kind)
    g = pkg.abcore_build_csr(nU, nL, to_dev((key // nL).astype(np.int32)),
                             to_dev((key % nL).astype(np.int32)))
    want = np.unique(key)
    u, v = want // nL, want % nL
    assert g.m == len(want)
    off, cols = [t.cpu().numpy() for t in pkg.abcore_export_csr(g)]
    deg = np.concatenate([np.bincount(u, minlength=nU), np.bincount(v, minlength=nL)])
    assert np.array_equal(off, np.concatenate([[0], np.cumsum(deg)]))
    assert np.array_equal(cols, np.concatenate([nU + v, u[np.lexsort((u, v))]]).astype(np.int32))
    g.destroy()
