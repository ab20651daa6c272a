"""Cluster order where hubs lend their ids to all that they name: stars and
chains of leaves around a few vertices, ids shuffled.  Labels against the
oracle, no tolerance; and the order of a star takes no longer than a few times
that of a graph without hubs (an atomic per leaf on one counter took 17 times)."""
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


def tree(n, parent_of, seed):
    """Vertex v joined to parent_of(v), every fifth to its predecessor too (less than half of the entries are the
    hubs'), ids shuffled but for the first, which are the hubs."""
    perm = np.r_[:2000, 2000 + np.random.default_rng(seed).permutation(n - 2000)].astype(np.int64)
    v = np.arange(1, n)
    u, w = np.r_[perm[v], perm[2005:n:5]], np.r_[perm[parent_of(v)], perm[2004:n - 1:5]]
    key = np.unique(np.concatenate([u * n + w, w * n + u]))
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=off[1:])
    return graphgen.Graph(off, (key % n).astype(np.int32), None, name="tree")


def star(v, hubs=1):
    return np.where(v < hubs, 0, v % hubs)


def two_deep(v):  # 40 hubs, 30 middle vertices each, the rest around those
    return np.where(v < 40, 0, np.where(v < 1240, v % 40, 40 + v % 1200))


@pytest.mark.parametrize("shape", ["star", "stars", "deep"])
def test_labels(gsl, shape):
    n = 2000003
    g = tree(n, {"star": star, "stars": lambda v: star(v, 7), "deep": two_deep}[shape], 3)
    say("cluster %s n=%d longest=%d" % (shape, n, np.diff(g.offsets).max()))
    off, cols, w = to_device(g)
    before = gsl.gsl_route_counts()["clustered"]
    lab, st = gsl.gsl_lpa_ex(off, cols, w, 20, 0.05)
    assert gsl.gsl_route_counts()["clustered"] == before + 1 and st["renumbered"]
    r = oracle.lpa(g, 20, 0.05)
    np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
    assert st["iterations"] == r.iterations and list(st["changed"][:r.iterations]) == list(r.dn)


def test_the_order_of_a_star_takes_no_longer(gsl):
    n = 4000000
    ms = []
    for parent_of in (lambda v: v - 1, star):  # a path, a star
        off, cols, w = to_device(tree(n, parent_of, 4))
        runs = [gsl.gsl_lpa_ex(off, cols, w, 8, 0.05, split=False, timing=True)[1] for _ in range(4)]
        assert all(st["renumbered"] for st in runs)
        ms.append(min(st["ms_reorder"] for st in runs[1:]))
    say("order and copy: path %.2f ms, star %.2f ms" % tuple(ms))
    assert ms[1] < 4 * ms[0]
