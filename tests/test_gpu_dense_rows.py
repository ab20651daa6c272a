"""Graphs with many rows of more than 64 entries through the calls that keep the
caller's layout: one launch while those rows cost less than the launches saved,
the general path beyond, wherever in the graph they lie.  Labels against the
oracle, no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402
from tests.test_gpu_routes import Took  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gsl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as m
    m.load()
    return m


def graph(n, deg, rows, wmax=0, together=False, seed=7):
    """A ring of n vertices with 8 neighbours each; `rows` of them, spread or `together`, joined in a ring of their
    own to `deg` more."""
    rng = np.random.default_rng(seed)
    heavy = n // 3 + rng.permutation(rows) if together else rng.permutation(n)[:rows]
    i, k = np.arange(n), np.arange(1, deg // 2 + 1 if rows > deg else 1)
    u = np.concatenate([np.repeat(heavy, k.size)] + [i] * 4)
    v = np.concatenate([heavy[(np.arange(rows)[:, None] + k) % rows].ravel()] + [(i + h) % n for h in range(1, 5)])
    key = np.unique(np.concatenate([u * n + v, v * n + u]))
    r, c = key // n, (key % n).astype(np.int32)
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(r, minlength=n), out=off[1:])
    w = ((np.minimum(r, c) * 31 + np.maximum(r, c)) % wmax + 1).astype(np.uint32) if wmax else None
    return graphgen.Graph(off, c, w, name="dense")


# (vertices, row length, such rows, weights, together) -> one launch?
CASES = [
    (256, 80, 200, 0, False, True), (256, 80, 200, 9, False, False),   # one workgroup
    (4000, 100, 400, 0, False, True), (4000, 100, 3900, 0, False, True),
    (4000, 100, 400, 9, False, True), (4000, 100, 3900, 9, False, False),
    (4000, 300, 3900, 0, False, False), (4000, 900, 2000, 0, False, False), (8000, 700, 900, 9, False, False),
    (60000, 700, 800, 0, False, True), (60000, 700, 9000, 0, False, False),
    (130000, 300, 1300, 0, False, True), (130000, 300, 4000, 9, False, False),  # several windows a workgroup
    (60000, 700, 800, 0, True, False), (60000, 300, 640, 9, True, False),  # those rows in a few windows, past any sample
]


@pytest.mark.parametrize("n,deg,rows,wmax,together,one", CASES)
def test_many_long_rows(gsl, n, deg, rows, wmax, together, one):
    g = graph(n, deg, rows, wmax, together)
    d = np.diff(g.offsets)
    say("dense n=%d rows above 64: %d, above 512: %d, longest %d w=%d" % (n, (d > 64).sum(), (d > 512).sum(), d.max(), wmax))
    assert d.max() <= 2048
    dev, ref = to_device(g), oracle.lpa(g)
    for call in (lambda: gsl.gsl_lpa_noalloc(*dev), lambda: gsl.gsl_lpa_graphs([dev])[0][0],
                 lambda: gsl.gsl_lpa_ex(*dev, layout="original")[0]):
        with Took(gsl) as t:
            lab = call()
        assert t.routes == {"one_launch" if one else "declined": 1}
        np.testing.assert_array_equal(lab.cpu().numpy(), ref.labels)


@pytest.mark.parametrize("wmax", [0, 9])
def test_sessions(gsl, wmax):
    """Steps run in one launch while no resident graph is too dense for it, and again after it has left."""
    gs = [graph(3000, 100, 200, wmax), graph(100, 20, 50, wmax), graph(2500, 600, 1400, wmax, seed=3), graph(5000, 8, 1, wmax)]
    refs = [oracle.lpa(g, 20, 0.05) for g in gs]
    s = gsl.Session(20000, 2000000, max_graphs=8, weighted=bool(wmax))
    seen = []
    for part in (gs[:2], gs[2:], gs[:1]):
        dev = [to_device(g) for g in part]
        live = {}
        for g, (ticket, status, lab) in zip(part, s.add(dev)):
            assert status == gsl.GSL_OK
            live[ticket] = (g, lab)
        with Took(gsl) as t:
            while live:
                for ticket, ran in s.step(5):
                    g, lab = live.pop(ticket)
                    r = refs[[x is g for x in gs].index(True)]
                    assert ran == r.iterations
                    np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
        seen.append(t.routes.get("one_launch", 0))
        say("session part: %s" % t.routes)
    assert seen[0] > 0 and seen[2] > 0
    # the dense graph's steps run kernel by kernel; those of the one beside it may outlast it
    assert seen[1] < 4
    s.close()
