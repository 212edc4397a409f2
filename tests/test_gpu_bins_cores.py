"""Core numbers whose levels are binned (graphs of at least 2^22 vertices):
uniform and skewed rows, a partial last bucket, and levels after deletions and
insertions; against the oracle."""
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


@pytest.mark.parametrize("name", ["uniform", "skewed"])
def test_core_numbers(name):
    if name == "uniform":
        nU, nL = 2_500_001, 1_800_003
        eu, ev = bigraph_gen.uniform(nU, nL, 12_000_000, 21)
    else:
        nU, nL = 1_500_007, 2_999_999
        eu, ev = bigraph_gen.chung_lu(nU, nL, 20_000_000, 2.1, 2.1, 50_000, 22)
    g = pkg.abcore_build_csr(nU, nL, to_dev(eu), to_dev(ev))
    key = np.unique(eu.astype(np.int64) * nL + ev)
    for step in range(2):
        if step == 1:
            gone = key[:: len(key) // 12]
            new = np.setdiff1d(gone + 1, key)
            for op, ks in ((-1, gone), (1, new)):
                for k in ks.tolist():
                    pkg.abcore_query(g, k // nL, k % nL, op, 1, 1)
            key = np.union1d(np.setdiff1d(key, gone), new)
        say("binned cores", name, "step", step)
        ref = oracle.Graph(nU, nL, (key // nL).astype(np.int32), (key % nL).astype(np.int32))
        want = oracle.core_numbers(ref)
        for _ in range(2):
            core, mx = pkg.abcore_core_numbers(g)
            assert np.array_equal(core.cpu().numpy(), want) and mx == int(want.max())
            pkg.abcore_set_option(g, pkg.ABCORE_OPT_KCORE_SWITCH, 1000 if step else 0)
    g.destroy()
