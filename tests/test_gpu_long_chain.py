"""A peel that is one long chain of dependent removals: a single wave works
for seconds while every other wave of the asynchronous peel waits, which must
not be taken for a hang."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits_np, ensure_built, say, to_dev

pytestmark = pytest.mark.gpu

# 1.4 million removals one after the other: 3.5 s at 2.5 us each
CHAIN = 700_000


def test_long_chain():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ensure_built()
    import paper_2606_07148_amd as pkg
    # the path u0 - l0 - u1 - l1 - ... up to u_k, which is on a 4-cycle
    k = CHAIN
    i = np.arange(k)
    eu = np.concatenate([i, i + 1, [k, k, k + 1, k + 1]]).astype(np.int32)
    ev = np.concatenate([i, i, [k, k + 1, k, k + 1]]).astype(np.int32)
    n = k + 2
    ref = oracle.Graph(n, n, eu, ev)
    want = oracle.pack(oracle.compute(ref, 2, 2))
    g = pkg.abcore_build_csr(n, n, to_dev(eu), to_dev(ev))
    say("chain of", 2 * k, "removals")
    bits, st = pkg.abcore_compute(g, 2, 2, pkg.ABCORE_GCC, stats=True)
    assert np.array_equal(bits_np(bits)[: len(want)], want)
    assert st["removed"] == 2 * n - 4
    g.destroy()
