"""Calls that run in one launch (small graphs and batches) against the oracle,
at the sizes where that kernel changes what it does: one workgroup or several,
workgroups that read each other's counts or follow the first, rows kept from
sweep to sweep or read again, and every way a row is shared among lanes.  All
results are whole numbers: equality, no tolerance."""
import os
import subprocess
import sys

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


def check(gsl, g, max_iters=20, tol=0.05, shift=0, tag=""):
    off, cols, w = to_device(g)
    if shift:
        buf = torch.zeros(cols.numel() + 4, dtype=cols.dtype, device=cols.device)
        buf[shift:shift + cols.numel()] = cols
        cols = buf[shift:shift + cols.numel()]
    for split in (False, True):
        r = oracle.lpa(g, max_iters, tol, split=split)
        lab, st = gsl.gsl_lpa_ex(off, cols, w, max_iters, tol, split=split, layout="original")
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels, err_msg="%s split=%s" % (tag, split))
        k = min(r.iterations, 64)
        assert st["iterations"] == r.iterations and list(st["changed"][:k]) == list(r.dn[:k]), tag
        deg = np.diff(g.offsets)
        assert st["nnz"] == g.nnz and st["max_degree"] == deg.max()
        for t in range(2, k):
            if r.dn[t - 2] * 8 <= g.n:
                assert st["processed"][t] == r.processed[t], (tag, t)
        assert st["processed"][0] == (deg > 0).sum() and st["edges"][0] == g.nnz
        if r.iterations <= 64:  # the per-sweep arrays hold that many
            for key in ("processed", "edges", "changed"):
                assert sum(x[key] for x in st["tiers"]) == sum(st[key]), (tag, key)


@pytest.mark.parametrize("n", [1, 2, 127, 255, 256, 257, 384, 385, 32768, 32769, 65536, 65537, 131072, 131073])
@pytest.mark.parametrize("wmax", [0, 9])
def test_sizes(gsl, n, wmax):
    g = graphgen.planted(n, max(1, n // 120), 0.12 if n > 240 else 0.5, n // 2, 3 + n % 7, wmin=0, wmax=wmax)
    say("small n=%d nnz=%d wmax=%d" % (g.n, g.nnz, wmax))
    check(gsl, g, tag="n=%d w=%d" % (n, wmax))
    if n <= 385:
        check(gsl, g, 100, 0.0, tag="n=%d w=%d to the end" % (n, wmax))


@pytest.mark.parametrize("wmax", [0, 5])
@pytest.mark.parametrize("n", [2300, 40000])
def test_row_lengths(gsl, n, wmax):
    """Rows at the bounds of every way a row is shared, the longest the kernel
    takes among them, then one longer (the general path)."""
    rng = np.random.default_rng(n + wmax)
    base = graphgen.planted(n, n // 50, 0.2, n // 4, 5)
    rows = np.repeat(np.arange(n), np.diff(base.offsets))
    keep = rows < base.cols
    for longest in (2048, 2049):
        u, v = [rows[keep]], [base.cols[keep].astype(np.int64)]
        for k, d in enumerate((15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1025, 2047, longest)):
            x = n - 1 - 3 * k
            u.append(np.full(d, x))
            v.append(rng.choice(n // 2, d, replace=d > n // 2))  # duplicates where the row is longer than the range
        u, v = np.concatenate(u), np.concatenate(v)
        u = np.append(u, [7, n - 1])  # self loops
        v = np.append(v, [7, n - 1])
        ws = None if not wmax else rng.integers(0, wmax + 1, size=u.size)
        g = graphgen.from_undirected(n, list(zip(u.tolist(), v.tolist())), ws)
        say("rows n=%d longest %d" % (n, np.diff(g.offsets).max()))
        check(gsl, g, 40, 0.0, tag="rows n=%d longest %d w=%d" % (n, longest, wmax))


@pytest.mark.parametrize("shift", [0, 1, 3])
def test_unaligned_columns(gsl, shift):
    check(gsl, graphgen.planted(5003, 50, 0.2, 4000, 3), shift=shift, tag="shift %d" % shift)
    check(gsl, graphgen.planted(201, 5, 0.4, 200, 3), shift=shift, tag="shift %d" % shift)


def test_overflow_and_bad_offsets(gsl):
    for n in (10, 3000):
        g = graphgen.from_undirected(n, [(0, 1), (0, 2), (1, 2)], [1 << 31, 1 << 31, 1])
        off, cols, w = to_device(g)
        with pytest.raises(gsl.GslError) as e:
            gsl.gsl_lpa(off, cols, w)
        assert e.value.code == gsl.GSL_EOVERFLOW
        bad = off.clone()
        bad[0] = 1
        with pytest.raises(gsl.GslError) as e:
            gsl.gsl_lpa(bad, cols, None)
        assert e.value.code == gsl.GSL_EINVAL
        check(gsl, graphgen.planted(n, 2, 0.5, n, 3) if n < 100 else graphgen.planted(n, 60, 0.2, n, 3))


def test_batches_across_windows(gsl):
    """Graphs of sizes around the window of 128 vertices, in one batch."""
    b = graphgen.batched_planted(90, 11, nmin=3, nmax=700, kmin=1, kmax=6)
    off, cols, _ = to_device(b)
    vb, eb = torch.from_numpy(b.vtx_base).cuda(), torch.from_numpy(b.edge_base).cuda()
    lab, sweeps, _ = gsl.gsl_lpa_batched(vb, eb, off, cols)
    lab, sweeps = lab.cpu().numpy(), sweeps.cpu().numpy()
    for k in range(b.num_graphs):
        r = oracle.lpa(b.subgraph(k))
        assert sweeps[k] == r.iterations, k
        np.testing.assert_array_equal(lab[b.vtx_base[k]:b.vtx_base[k + 1]], r.labels, err_msg="graph %d" % k)


def test_a_wait_that_runs_out_takes_the_general_path():
    """With no patience at all the workgroups leave at the first meeting that is
    not complete when they look, and the call still returns the oracle's
    labels (a process of its own: the limit is read once)."""
    code = ("import numpy as np, torch, graphgen, oracle, paper_2403_01261_amd as m\n"
            "g = graphgen.planted(30000, 300, 0.1, 30000, 3)\n"
            "o, c = torch.from_numpy(g.offsets).cuda(), torch.from_numpy(g.cols).cuda()\n"
            "for k in range(3):\n"
            "    assert np.array_equal(m.gsl_lpa(o, c).cpu().numpy(), oracle.lpa(g).labels)\n"
            "print('same labels')\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=110,
                       env=dict(os.environ, GSL_SMALL_WAIT_TICKS="0"))
    assert r.returncode == 0 and "same labels" in r.stdout, r.stderr[-2000:]
