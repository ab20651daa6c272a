"""Modularity over rows of every way they are shared (a thread, a wavefront, the
workgroup) and communities from one for all vertices to one each, against the
oracle: the sums are whole numbers, so the value is equal to the last bit."""
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
    return m


def graph(n, hubs, weighted, seed):
    rng = np.random.default_rng(seed)
    rows, cols = [rng.integers(0, n, 3 * n)], [rng.integers(0, n, 3 * n)]
    for d in hubs:
        c = int(rng.integers(0, n))
        v = rng.choice(n, d, replace=False)
        rows += [np.full(d, c)]
        cols += [v]
    u, v = np.concatenate(rows), np.concatenate(cols)
    key = np.unique(np.concatenate([u, v]) * n + np.concatenate([v, u]))
    u, v = key // n, key % n
    return graphgen.from_entries(n, u, v, (np.minimum(u, v) * 31 + np.maximum(u, v)) % 17 if weighted else None)


@pytest.mark.parametrize("n,hubs", [(1, []), (255, [32, 33, 200]), (257, [64]), (9001, [4096, 4097, 8000]),
                                    (300007, [5000, 70000, 299999])])
@pytest.mark.parametrize("weighted", [False, True])
def test_modularity(gsl, n, hubs, weighted):
    g = graph(n, hubs, weighted, n)
    off, cols, w = to_device(g)
    rng = np.random.default_rng(n)
    say("quality n=%d longest=%d" % (n, np.diff(g.offsets).max()))
    for lab in (np.zeros(n), np.arange(n), rng.integers(0, max(1, n // 300), n), np.minimum(rng.geometric(0.5, n), n) - 1):
        lab = lab.astype(np.int32)
        q = gsl.gsl_modularity(off, cols, w, torch.from_numpy(lab).cuda())
        assert q == oracle.modularity(g, lab)
