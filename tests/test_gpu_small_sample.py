"""Small graphs whose rows decide between the one launch and the general path:
most entries in long rows (told from a sample of the rows), nearly half of them
(told after the first sweep, or not at all), and a single long row.  Every route
gives the same labels as the oracle: whole numbers, equality, no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu


# cliques of 81 vertices (6,480 entries in rows of 80) and of 5 (20 entries)
@pytest.mark.parametrize("long,short", [(1, 0), (3, 1), (10, 2000), (10, 3000), (10, 4000), (1, 400), (0, 60)])
@pytest.mark.parametrize("layout", ["auto", "original"])
def test_share_of_long_rows(long, short, layout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as gsl
    sizes = [81] * long + [5] * short
    n = sum(sizes)
    g = graphgen.cliques(sizes, perm=np.random.default_rng(n).permutation(n))
    deg = np.diff(g.offsets)
    say("long rows hold %.2f of the entries, n=%d, %s" % (deg[deg > 64].sum() / max(g.nnz, 1), n, layout))
    off, cols, w = to_device(g)
    r = oracle.lpa(g, 20, 0.05)
    lab, st = gsl.gsl_lpa_ex(off, cols, w, 20, 0.05, layout=layout)
    np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
    assert st["iterations"] == r.iterations and st["nnz"] == g.nnz and st["max_degree"] == deg.max()


def test_one_row_beyond_the_sample():
    """A star on few vertices (always sampled) and on many (found by its window)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as gsl
    for n in (2200, 60000):
        g = graphgen.from_undirected(n, [(0, v) for v in range(1, 2120)] + [(v, v + 1) for v in range(1, n - 1)])
        say("star n=%d" % n)
        off, cols, w = to_device(g)
        lab, _ = gsl.gsl_lpa_ex(off, cols, w, 20, 0.05)
        np.testing.assert_array_equal(lab.cpu().numpy(), oracle.lpa(g, 20, 0.05).labels)
