"""The loop's first sweep and the thread-per-vertex kernel's sorting networks
on graphs too large for the one-launch path: rows at the edges of the networks
(8, 16, 24, 32 entries), rows in any order, with repeated entries and entries
of their own vertex, weights that tie or are zero.  All results are whole
numbers: equality with the oracle, no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu
N = 2 ** 18 + 77


@pytest.fixture(scope="module")
def gsl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as m
    m.load()
    return m


def circulant(longest, weighted, odd, seed):
    """Vertex v joined to v +- 1 .. h, fewer for some stretches of vertices, so
    that wavefronts see rows of one length or of many; `odd` graphs also have
    rows out of order, repeated entries and self loops."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(N)
    half = np.full(N, longest // 2)
    half[N // 4:N // 2] = rng.integers(1, longest // 2 + 1, N // 2 - N // 4)
    half[N // 2:N // 2 + N // 8] = max(1, longest // 4)
    rows, cols = [], []
    for h in range(1, longest // 2 + 1):
        u = np.flatnonzero((half >= h) & (np.roll(half, -h) >= h))
        v = (u + h) % N
        rows += [u, v]
        cols += [v, u]
    if odd:
        loops = np.flatnonzero((np.arange(N) % 97 == 0) & (half < longest // 2))
        twice = loops + 1
        rows += [loops, twice % N, (twice + 1) % N]
        cols += [loops, (twice + 1) % N, twice % N]
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    if not odd:
        perm = np.arange(N)
    u, v = perm[rows], perm[cols]
    w = np.where(u == v, 9, (np.minimum(u, v) * 31 + np.maximum(u, v)) % 4) if weighted else None
    order = np.argsort(rng.random(u.size), kind="stable") if odd else np.lexsort((v, u))
    return graphgen.from_entries(N, u[order], v[order], None if w is None else w[order])


@pytest.mark.parametrize("longest", [8, 16, 24, 32])
@pytest.mark.parametrize("weighted,odd", [(False, False), (True, False), (False, True), (True, True)])
def test_first_sweeps(gsl, longest, weighted, odd):
    g = circulant(longest, weighted, odd, longest)
    off, cols, w = to_device(g)
    say("first sweep longest=%d nnz=%d" % (np.diff(g.offsets).max(), g.nnz))
    for iters in (1, 4):
        r = oracle.lpa(g, iters, 0.0, split=False)
        lab, st = gsl.gsl_lpa_ex(off, cols, w, iters, 0.0, split=False, layout="original")
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels, err_msg="%d sweeps" % iters)
        assert list(st["changed"][:r.iterations]) == list(r.dn)
