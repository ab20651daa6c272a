"""Hub rows with float weights: chunks staged by hash partition and merged, in
one batch or many, with and without hashed sub-passes.  The weights are
multiples of 1/16 below 64, so every sum is exact and the labels equal the
oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gsl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as m
    m.load()
    yield m
    m.gsl_set_hub_limits(0, 0)


def hubs(degrees, n, seed):
    rng = np.random.default_rng(seed)
    base = graphgen.planted(n, 200, 0.05, n // 2, seed)
    rows, cols = [np.repeat(np.arange(n), np.diff(base.offsets))], [base.cols.astype(np.int64)]
    for k, d in enumerate(degrees):
        v = rng.choice(np.arange(len(degrees), n), d, replace=False)
        rows += [np.full(d, k), v]
        cols += [v, np.full(d, k)]
    key = np.unique(np.concatenate(rows) * n + np.concatenate(cols))
    return graphgen.from_entries(n, key // n, key % n)


@pytest.mark.parametrize("staging,claims", [(0, 0), (2048 * 8, 0), (1 << 16, 33)])
@pytest.mark.parametrize("layout", ["original", "renumbered"])
def test_hubs(gsl, staging, claims, layout):
    g = hubs([2049, 2100, 4096, 4097, 6145, 30000, 65000], 70000, 4)
    u = np.repeat(np.arange(g.n), np.diff(g.offsets))
    h = np.minimum(u, g.cols).astype(np.int64) * 7919 + np.maximum(u, g.cols)
    w = ((h * 2654435761 >> 7) % 1024 / 16.0).astype(np.float32)
    off, cols, _ = to_device(g)
    wd = torch.from_numpy(w).cuda()
    say("f32 hubs staging=%d claims=%d %s" % (staging, claims, layout))
    for iters in (1, 20):
        r = oracle.lpa_f32(g, w, iters, 0.0)
        gsl.gsl_set_hub_limits(staging, claims)
        try:
            lab, st = gsl.gsl_lpa_f32(off, cols, wd, iters, 0.0, layout=layout)
        finally:
            gsl.gsl_set_hub_limits(0, 0)
        assert st["iterations"] == r.iterations and list(st["changed"][:r.iterations]) == list(r.dn)
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
