"""The degree plan of graphs whose blocks of 1,024 vertices are one group (up to
2^20 vertices, one scan kernel) and of larger ones: tier counts against the
degrees, and the labels of a call on that plan against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 1023, 1024, 1025, 65537, (1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_tiers_of_every_size(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as gsl
    rng = np.random.default_rng(n)
    far = min(n, 4 * 1024)
    # hubs of every tier among the first vertices and in the last block, short rows between, a third of them isolated
    u = [rng.integers(0, n, size=n // 2)]
    v = [np.minimum(n - 1, u[0] + rng.integers(1, 40, size=u[0].size))]
    for k, d in enumerate((33, 64, 65, 129, 513, 1025, 2049, 4097)):
        for x in (k, n - 1 - k):
            if 0 <= x < n and d < far:
                u.append(np.full(d, x))
                v.append(rng.choice(far, d, replace=False))
    u, v = np.concatenate(u), np.concatenate(v)
    key = np.unique(np.concatenate([u * n + v, v * n + u]))
    rows, cols = key // n, (key % n).astype(np.int32)
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=off[1:])
    g = graphgen.Graph(off, cols, None, name="tiers")
    deg = np.diff(off)
    say("plan n=%d nnz=%d longest=%d isolated=%d" % (n, g.nnz, deg.max(), (deg == 0).sum()))
    dev = to_device(g)
    bounds = [0, 32, 64, 128, 512, 1024, 2048, 4096, 1 << 40]
    want = [int((deg == 0).sum())] + [int(((deg > a) & (deg <= b)).sum()) for a, b in zip(bounds, bounds[1:])]
    r = oracle.lpa(g, 3, 0.0)
    for layout in ("original", "renumbered") if n > (1 << 18) else ("renumbered",):
        lab, st = gsl.gsl_lpa_ex(*dev, 3, 0.0, layout=layout)
        assert [t["vertices"] for t in st["tiers"]][:9] == want
        assert st["max_degree"] == deg.max() and st["nnz"] == g.nnz
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
