"""Sweeps that read near labels from windows in LDS (8 M vertices and more whose
entries lie near their vertices): rows in and out of order, rows of 17 - 32
entries and longer ones between the short, single graphs and a batch, and a
label array that is not aligned (no windows).  All results are whole numbers:
equality with the oracle, no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu
N = (1 << 23) + 60013


@pytest.fixture(scope="module")
def gsl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as m
    m.load()
    return m


def band(n, reach, wide, backwards):
    """Vertex v joined to v +- each of `reach`; the first `wide` vertices also to
    v +- 3 .. 22 (rows of up to 46 entries)."""
    v = np.arange(n, dtype=np.int64)
    rows, cols = [], []
    for h in reach:
        rows += [v[:-h], v[h:]]
        cols += [v[h:], v[:-h]]
    for h in range(3, 23) if wide else ():
        u = v[:wide] if h % 2 else v[:wide // 2]
        rows += [u, u + h]
        cols += [u + h, u]
    key = np.unique(np.concatenate(rows) * n + np.concatenate(cols))
    u, c = (key // n), (key % n).astype(np.int32)
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(u, minlength=n), out=off[1:])
    if backwards:  # every row in descending order
        c = c[off[u] + off[u + 1] - 1 - np.arange(c.size)]
    return graphgen.Graph(off, c, None, name="band")


@pytest.mark.parametrize("backwards", [False, True])
def test_windows(gsl, backwards):
    g = band(N, (1, 5000), 200000, backwards)
    off, cols, w = to_device(g)
    d = np.diff(g.offsets)
    say("near n=%d nnz=%d longest=%d" % (g.n, g.nnz, d.max()))
    r = oracle.lpa(g, 4, 0.0, split=False)
    lab, st = gsl.gsl_lpa_ex(off, cols, w, 4, 0.0, split=False)
    assert not st["renumbered"]
    np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
    assert list(st["changed"][:r.iterations]) == list(r.dn)
    buf = torch.empty(g.n + 1, dtype=torch.int32, device="cuda")
    shifted = gsl.gsl_lpa(off, cols, w, 7, 0.0, out=buf[1:])
    assert torch.equal(shifted, gsl.gsl_lpa(off, cols, w, 7, 0.0))


def test_batch(gsl):
    gs = [graphgen.planted(n, max(1, n // 2000), 0.01 if n > 20000 else 0.4, n // 2, n) for n in (30000, 200, 90001)]
    gs.insert(1, band(N - 100000, (2, 3), 0, False))
    vb = np.cumsum([0] + [g.n for g in gs]).astype(np.int64)
    eb = np.cumsum([0] + [g.nnz for g in gs]).astype(np.int64)
    off = np.concatenate([g.offsets[:-1] + e for g, e in zip(gs, eb)] + [eb[-1:]])
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    labels, sweeps, _ = gsl.gsl_lpa_batched(t(vb), t(eb), t(off), t(np.concatenate([g.cols for g in gs])), None, 9, 0.01)
    labels, sweeps = labels.cpu().numpy(), sweeps.cpu().numpy()
    for i, g in enumerate(gs):
        r = oracle.lpa(g, 9, 0.01)
        np.testing.assert_array_equal(labels[vb[i]:vb[i + 1]], r.labels, err_msg="graph %d" % i)
        assert sweeps[i] == r.iterations
