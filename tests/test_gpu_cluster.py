"""Graphs of short rows whose neighbours lie far apart run in cluster order:
same labels and sweeps as the oracle and as the caller's own layout, weighted
or not, with longer rows and isolated vertices beside the short ones.  All
results are whole numbers: equality, no tolerance."""
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


def shuffled_road(n, seed, extra_rows=0, isolated=0, wmax=0):
    """A road graph under a random numbering, `isolated` more vertices without
    entries, and `extra_rows` vertices that each get 50 more neighbours."""
    g = graphgen.road_knn(n, 2, seed)
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n + isolated)
    rows = np.repeat(np.arange(n), np.diff(g.offsets))
    u, v = perm[rows], perm[g.cols]
    if extra_rows:
        hub = np.repeat(perm[rng.choice(n, extra_rows, replace=False)], 50)
        far = perm[rng.integers(0, n, hub.size)]
        keep = hub != far
        u, v = np.concatenate([u, hub[keep], far[keep]]), np.concatenate([v, far[keep], hub[keep]])
    key = np.unique(u.astype(np.int64) * (n + isolated) + v)
    u, v = key // (n + isolated), key % (n + isolated)
    w = None
    if wmax:
        w = ((np.minimum(u, v) * 7919 + np.maximum(u, v)) % wmax + 1).astype(np.uint32)
    off = np.zeros(n + isolated + 1, dtype=np.int64)
    np.cumsum(np.bincount(u, minlength=n + isolated), out=off[1:])
    return graphgen.Graph(off, v.astype(np.int32), w, name="shuffled-road")


@pytest.mark.parametrize("n,extra,isolated,wmax", [(2000000, 0, 0, 0), (2100037, 301, 7001, 9)])
def test_cluster_order(gsl, n, extra, isolated, wmax):
    g = shuffled_road(n, 5, extra, isolated, wmax)
    off, cols, w = to_device(g)
    say("cluster n=%d nnz=%d" % (g.n, g.nnz))
    r = oracle.lpa(g, 20, 0.05)
    lab, st = gsl.gsl_lpa_ex(off, cols, w, 20, 0.05)
    assert st["renumbered"]
    np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
    assert st["iterations"] == r.iterations and list(st["changed"][:r.iterations]) == list(r.dn)
    plain, st0 = gsl.gsl_lpa_ex(off, cols, w, 20, 0.05, layout="original")
    assert not st0["renumbered"] and torch.equal(lab, plain)
    few, st1 = gsl.gsl_lpa_ex(off, cols, w, 7, 0.05, split=False)  # too few sweeps to pay for the order
    assert not st1["renumbered"]
    np.testing.assert_array_equal(few.cpu().numpy(), oracle.lpa(g, 7, 0.05, split=False).labels)


def test_near_ids_stay(gsl):
    g = graphgen.from_entries(2100000, np.r_[np.arange(2099999), np.arange(1, 2100000)],
                              np.r_[np.arange(1, 2100000), np.arange(2099999)], name="path")
    off, cols, w = to_device(g)
    lab, st = gsl.gsl_lpa_ex(off, cols, w, 8, 0.0)
    assert not st["renumbered"]
    np.testing.assert_array_equal(lab.cpu().numpy(), oracle.lpa(g, 8, 0.0).labels)


def test_f32_negative_zero(gsl):
    """A weight of -0 counts as 0 (it never wins a row's first sweep)."""
    g = shuffled_road(2000003, 6)
    off, cols, _ = to_device(g)
    u = np.repeat(np.arange(g.n), np.diff(g.offsets))
    w = ((np.minimum(u, g.cols).astype(np.int64) * 31 + np.maximum(u, g.cols)) % 5).astype(np.float32)
    w[w == 0] = -0.0
    r = oracle.lpa_f32(g, w, 8, 0.05)
    lab, st = gsl.gsl_lpa_f32(off, cols, torch.from_numpy(w).cuda(), 8, 0.05)
    assert st["renumbered"]
    np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
