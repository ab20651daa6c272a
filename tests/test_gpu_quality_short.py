"""Modularity of graphs whose rows have 31 to 129 entries: a thread's rows, one
entry a lane of a wavefront, and more.  The integer parts are exact, so the
value agrees with the oracle's to the last rounding of its two divisions."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wmax", [0, 7])
@pytest.mark.parametrize("deg", [30, 32, 34, 62, 64, 66, 128])
def test_rows(deg, wmax):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as gsl
    n = 3001
    v = np.arange(n)
    k = np.arange(1, deg // 2 + 1)
    u, c = np.repeat(v, k.size), (v[:, None] + k).ravel() % n
    extra = np.arange(0, n, 7)  # some rows one entry longer, or with a self loop
    u, c = np.concatenate([u, extra, [5, 9]]), np.concatenate([c, (extra + n // 2) % n, [5, 9]])
    ws = None if not wmax else (u * 13 + c) % wmax + 1
    g = graphgen.from_undirected(n, list(zip(u.tolist(), c.tolist())), ws)
    labels = (v // 40 * 40).astype(np.int32)
    say("modularity rows of %d: longest %d" % (deg, np.diff(g.offsets).max()))
    off, cols, w = to_device(g)
    q = gsl.gsl_modularity(off, cols, w, torch.from_numpy(labels).cuda())
    assert abs(q - oracle.modularity(g, labels)) <= 1e-12
