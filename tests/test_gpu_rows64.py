"""Many rows of 33 - 64 entries with unit weights, a thread each: every length
at the edges of the sorting networks, rows out of order, repeated entries and
self loops, beside graphs with fewer such rows (lanes and a table).  Equality
with the oracle, no tolerance."""
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


def ring(n, half, odd):
    """Vertex v joined to v +- 1 .. half[v] where its neighbour reaches as far."""
    v = np.arange(n, dtype=np.int64)
    rows, cols = [], []
    for h in range(1, int(half.max()) + 1):
        u = v[(half >= h) & (np.roll(half, -h) >= h)]
        rows += [u, (u + h) % n]
        cols += [(u + h) % n, u]
    if odd:
        u = v[(v % 61 == 0) & (half < 30)]
        rows += [u, u]
        cols += [u, u]
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    perm = np.random.default_rng(n).permutation(n) if odd else v
    order = np.random.default_rng(1).permutation(rows.size) if odd else np.lexsort((cols, rows))
    return graphgen.from_entries(n, perm[rows[order]], perm[cols[order]])


@pytest.mark.parametrize("n,odd", [(300011, False), (300011, True), (270000, False)])
def test_rows(gsl, n, odd):
    half = np.full(n, 20)
    for k, h in enumerate((17, 20, 21, 24, 25, 32, 16, 33)):
        half[k * n // 10:(k + 1) * n // 10] = h
    if n == 270000:
        half[40000:] = 8  # fewer than 2^16 rows of 33 - 64 entries
    g = ring(n, half, odd)
    d = np.diff(g.offsets)
    say("rows64 n=%d odd=%s 33-64: %d" % (n, odd, ((d > 32) & (d <= 64)).sum()))
    off, cols, w = to_device(g)
    for iters in (1, 4):
        r = oracle.lpa(g, iters, 0.0, split=False)
        lab, st = gsl.gsl_lpa_ex(off, cols, w, iters, 0.0, split=False, layout="original")
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
        assert list(st["changed"][:r.iterations]) == list(r.dn)
