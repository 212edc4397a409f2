"""Device memory of builds: the temporaries are gone before the working set is
allocated."""
import pytest

import bigraph_gen
from tests.gpu_util import ensure_built, say, to_dev

pytestmark = pytest.mark.gpu

pkg = None
MB = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def _setup():
    global pkg
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ensure_built()
    import paper_2606_07148_amd as p
    pkg = p
    yield
    p.abcore_set_memory_budget(0)


@pytest.mark.parametrize("nU,nL,m", [(3_000, 2_000, 12_000), (6_000_000, 6_000_000, 1_000_000)])
def test_build_peak(nU, nL, m):
    """Many vertices, few edges: the temporaries (five 64-bit words a vertex)
    and the working set never stand side by side."""
    eu, ev = bigraph_gen.uniform(nU, nL, m, 5)
    deu, dev = to_dev(eu), to_dev(ev)
    base, _ = pkg.abcore_device_memory(reset_peak=True)
    g = pkg.abcore_build_csr(nU, nL, deu, dev)
    held, peak = pkg.abcore_device_memory()
    r = pkg.abcore_graph_report(g)
    g.destroy()
    n = nU + nL
    phases = r["graph_bytes"] + r["ranks_bytes"] + 40 * (n + 1)
    say("build peak", peak - base, "held", held - base, "phases", phases)
    limit = max(held - base, phases + 8 * MB if n > 1_000_000 else 0)
    assert peak - base <= limit
    # and under that budget the build succeeds
    pkg.abcore_set_memory_budget(base + limit)
    try:
        pkg.abcore_build_csr(nU, nL, deu, dev).destroy()
    finally:
        pkg.abcore_set_memory_budget(0)
