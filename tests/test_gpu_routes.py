"""Which way calls run: the small ones in one launch, those it cannot take on
the general path, and the kernels chosen there -- so that a test that compares
labels also knows whose labels they are.  Labels against the oracle, no
tolerance."""
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import graphgen  # noqa: E402
import oracle  # noqa: E402
from tests import test_gpu_near, test_gpu_rows64  # noqa: E402
from tests.gpu_util import say, to_device  # noqa: E402

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def gsl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_01261_amd as m
    m.load()
    return m


class Took:
    """The routes taken inside a with block (those with a count)."""

    def __init__(self, gsl):
        self.gsl = gsl

    def __enter__(self):
        self.before = self.gsl.gsl_route_counts()
        return self

    def __exit__(self, *exc):
        after = self.gsl.gsl_route_counts()
        self.routes = {k: after[k] - self.before[k] for k in after if after[k] != self.before[k]}


def planted(n, wmax=0):
    return graphgen.planted(n, max(1, n // 120), 0.12, n // 2, 3 + n % 7, wmin=1 if wmax else 0, wmax=wmax)


# one workgroup, workgroups that read each other's words (up to 256), workgroups
# led by the first, and the largest taken
@pytest.mark.parametrize("n,wmax", [(200, 0), (200, 9), (10000, 0), (32768, 9), (32769, 0), (131072, 9), (262144, 0)])
def test_small_graphs_run_in_one_launch(gsl, n, wmax):
    g = planted(n, wmax)
    say("routes n=%d wmax=%d" % (n, wmax))
    ref = oracle.lpa(g).labels
    for call in (gsl.gsl_lpa, gsl.gsl_lpa_noalloc):
        with Took(gsl) as t:
            lab = call(*to_device(g))
        np.testing.assert_array_equal(lab.cpu().numpy(), ref)
        assert t.routes == {"one_launch": 1}, call.__name__


def test_batches_and_sessions_run_in_one_launch(gsl):
    gs = [planted(n) for n in (300, 2000, 501)]
    refs = [oracle.lpa(g) for g in gs]
    dev = [to_device(g) for g in gs]
    with Took(gsl) as t:
        labels, _, _ = gsl.gsl_lpa_graphs(dev)
    assert t.routes == {"one_launch": 1}
    vb = np.cumsum([0] + [g.n for g in gs])
    eb = np.cumsum([0] + [g.nnz for g in gs])
    off = np.concatenate([g.offsets[:-1] + e for g, e in zip(gs, eb)] + [eb[-1:]])
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    with Took(gsl) as t:
        cat, _, _ = gsl.gsl_lpa_batched(up(vb), up(eb), up(off), up(np.concatenate([g.cols for g in gs])))
    assert t.routes == {"one_launch": 1}
    cat = cat.cpu().numpy()
    for k, r in enumerate(refs):
        np.testing.assert_array_equal(labels[k].cpu().numpy(), r.labels)
        np.testing.assert_array_equal(cat[vb[k]:vb[k + 1]], r.labels)
    s = gsl.Session(int(vb[-1]), int(eb[-1]), max_graphs=4)
    out = [x[2] for x in s.add(dev)]
    steps = done = 0
    with Took(gsl) as t:
        while done < len(gs):
            done += len(s.step(4))
            steps += 1
    assert t.routes == {"one_launch": steps}
    s.close()
    for lab, r in zip(out, refs):
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)


def test_what_one_launch_cannot_take(gsl):
    star = graphgen.from_undirected(2050, [(0, k) for k in range(1, 2050)])  # a row of 2,049
    dense = graphgen.planted(2048, 4, 0.4, 1000, 3)  # all rows above 64: renumbered
    for g in (star, dense):
        off, cols, w = to_device(g)
        with Took(gsl) as t:
            lab = gsl.gsl_lpa(off, cols, w)
        assert t.routes == {"declined": 1}
        np.testing.assert_array_equal(lab.cpu().numpy(), oracle.lpa(g).labels)
    few = graphgen.cliques([80] * 20 + [5] * 400)  # most entries in rows above 64, but few such rows
    dev, ref = to_device(few), oracle.lpa(few).labels
    for layout, want in (("auto", "declined"), ("original", "one_launch")):
        with Took(gsl) as t:
            lab, _ = gsl.gsl_lpa_ex(*dev, layout=layout)
        assert t.routes == {want: 1}
        np.testing.assert_array_equal(lab.cpu().numpy(), ref)
    g = planted(262145)
    with Took(gsl) as t:
        lab = gsl.gsl_lpa(*to_device(g))
    assert t.routes.keys() <= {"rows64"}  # not tried
    np.testing.assert_array_equal(lab.cpu().numpy(), oracle.lpa(g).labels)


def test_kernels_of_the_general_path(gsl):
    with Took(gsl) as t:
        test_gpu_near.test_batch(gsl)
    assert t.routes == {"windows": 1}
    g = test_gpu_near.band(test_gpu_near.N, (1, 5000), 200000, False)
    off, cols, w = to_device(g)
    out = torch.empty(g.n + 1, dtype=torch.int32, device="cuda")
    for labels, want in ((out[:-1], {"windows": 1}), (out[1:], {})):
        with Took(gsl) as t:
            gsl.gsl_lpa(off, cols, w, 2, 0.0, out=labels)
        t.routes.pop("rows64", None)  # some of the wide rows
        assert t.routes == want
    with Took(gsl) as t:
        test_gpu_rows64.test_rows(gsl, 300011, False)
    assert t.routes == {"rows64": 2}
    with Took(gsl) as t:
        test_gpu_rows64.test_rows(gsl, 270000, False)
    assert t.routes == {}


def test_calls_in_one_launch_at_the_same_time(gsl):
    """Four threads, a stream each, all calls small: beside each other they
    share the device or take the general path; nobody waits for the limit."""
    sizes = (900, 6001, 9000, 30000)
    gs = [planted(n) for n in sizes]
    refs = [oracle.lpa(g).labels for g in gs]
    dev = [to_device(g) for g in gs]
    calls, bad = 60, []

    def work(k):
        ctx = gsl.Context()
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(calls):
                lab = ctx.lpa_graphs([dev[k]])[0][0]
                if not np.array_equal(lab.cpu().numpy(), refs[k]):
                    bad.append(k)
        ctx.close()

    with Took(gsl) as t:
        ts = [threading.Thread(target=work, args=(k,)) for k in range(len(gs))]
        [x.start() for x in ts]
        [x.join() for x in ts]
    assert not bad
    say("at the same time: %s" % t.routes)
    assert t.routes.get("one_launch", 0) + t.routes.get("busy", 0) + t.routes.get("ran_out", 0) == calls * len(gs)
    assert t.routes.get("one_launch", 0) > 0 and "declined" not in t.routes


def run_without_patience(code):
    """Runs `code` (which prints a route dict last) with waits that give up at once: in a process of its own, as the
    limit is read once."""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=110,
                       env=dict(os.environ, GSL_SMALL_WAIT_TICKS="0"))
    assert r.returncode == 0, r.stderr[-2000:]
    return eval(r.stdout.strip().split("\n")[-1])


def test_a_wait_that_runs_out_is_counted():
    routes = run_without_patience(
        "import numpy as np, torch, graphgen, oracle, paper_2403_01261_amd as m\n"
        "g = graphgen.planted(30000, 300, 0.1, 30000, 3)\n"
        "o, c = torch.from_numpy(g.offsets).cuda(), torch.from_numpy(g.cols).cuda()\n"
        "assert np.array_equal(m.gsl_lpa(o, c).cpu().numpy(), oracle.lpa(g).labels)\n"
        "print(m.gsl_route_counts())\n")
    assert routes["ran_out"] == 1 and routes["one_launch"] == 0
    routes = run_without_patience(
        "import paper_2403_01261_amd as m\n"
        "from tests import test_gpu_session_small as t\n"
        "m.load()\n"
        "t.serve(m, t.graphs(0, False), False, 3)\n"
        "print(m.gsl_route_counts())\n")
    assert routes["ran_out"] > 0


def test_calls_keep_off_after_a_wait_that_ran_out():
    """Not every call pays for the wait: 16 take the general path at once, 32
    after the next wait that runs out, on each scratch by itself."""
    routes = run_without_patience(
        "import numpy as np, torch, graphgen, oracle, paper_2403_01261_amd as m\n"
        "g = graphgen.planted(30000, 300, 0.1, 30000, 3)\n"
        "ref = oracle.lpa(g).labels\n"
        "o, c = torch.from_numpy(g.offsets).cuda(), torch.from_numpy(g.cols).cuda()\n"
        "for k in range(1 + 16 + 1 + 32 + 1):\n"
        "    assert np.array_equal(m.gsl_lpa(o, c).cpu().numpy(), ref), k\n"
        "with m.Context() as ctx:\n"
        "    assert np.array_equal(ctx.lpa_graphs([(o, c)])[0][0].cpu().numpy(), ref)\n"
        "print(m.gsl_route_counts())\n")
    assert routes["ran_out"] == 4 and routes["held_back"] == 48 and routes["one_launch"] == 0
    routes = run_without_patience(
        "import paper_2403_01261_amd as m\n"
        "from tests import test_gpu_session_small as t\n"
        "m.load()\n"
        "t.serve(m, t.graphs(0, False), False, 1)\n"
        "print(m.gsl_route_counts())\n")
    assert 0 < routes["ran_out"] <= 3 and routes["held_back"] > 2 * routes["ran_out"]


@pytest.mark.parametrize("op", ["modularity", "split", "disconnected"])
def test_every_entry_point_counts_as_a_call_in_flight(gsl, op):
    """A graph of more than a quarter of the device's workgroups is not taken in
    one launch beside another call, whichever that is."""
    big = planted(1000000)
    off, cols, w = to_device(big)
    raw = gsl.gsl_lpa_ex(off, cols, w, split=False)[0]
    other = {"modularity": lambda: gsl.gsl_modularity(off, cols, w, raw), "split": lambda: gsl.gsl_split(off, cols, raw),
             "disconnected": lambda: gsl.gsl_disconnected(off, cols, raw)}[op]
    other()
    g = planted(60000)
    dev, ref = to_device(g), oracle.lpa(g).labels
    started, stop = threading.Event(), threading.Event()

    def beside():
        while not stop.is_set():
            other()
            started.set()

    th = threading.Thread(target=beside)
    with gsl.Context() as ctx:
        ctx.lpa_graphs([dev])
        th.start()
        started.wait()
        with Took(gsl) as t:
            for _ in range(60):
                lab = ctx.lpa_graphs([dev])[0][0]
                np.testing.assert_array_equal(lab.cpu().numpy(), ref)
        stop.set()
        th.join()
    say("beside %s: %s" % (op, t.routes))
    assert t.routes.get("busy", 0) > 0


@pytest.mark.parametrize("n,batch,windows", [(2500000, False, False), (5700000, False, False), (5800000, False, True),
                                             (5800000, True, False)])
def test_windows_are_for_large_graphs(gsl, n, batch, windows):
    """Single graphs below 11 * 2^19 vertices and batches below 2^23 sweep without windows."""
    g = test_gpu_near.band(n, (1, 2), 200, False)
    off, cols, w = to_device(g)
    say("windows n=%d batch=%s" % (n, batch))
    with Took(gsl) as t:
        if batch:
            ends = torch.tensor([[0, n], [0, g.nnz]], dtype=torch.int64, device="cuda")
            lab = gsl.gsl_lpa_batched(ends[0].contiguous(), ends[1].contiguous(), off, cols, None, 3, 0.0)[0]
        else:
            lab = gsl.gsl_lpa(off, cols, w, 3, 0.0)
    assert t.routes == ({"windows": 1} if windows else {})
    np.testing.assert_array_equal(lab.cpu().numpy(), oracle.lpa(g, 3, 0.0).labels)


def hubs(count, leaves, extra=0, fill=0):
    """`count` vertices with `leaves` neighbours of their own each -- half of all entries in rows of more than 64 --
    and `extra` edges among them (more than half then) or `fill` among the leaves (less)."""
    n = count * (leaves + 1)
    hub = np.arange(count) * (leaves + 1)
    edges = [(h, h + 1 + k) for h in hub for k in range(leaves)]
    edges += [(hub[k], hub[k + 1]) for k in range(extra)] + [(2 * k + 1, 2 * k + 2) for k in range(fill) if (2 * k + 2) % (leaves + 1)]
    perm = np.random.default_rng(n).permutation(n)
    return graphgen.from_undirected(n, [(int(perm[u]), int(perm[v])) for u, v in edges])


# one workgroup, workgroups that read each other's words, workgroups led by the first
@pytest.mark.parametrize("count,leaves", [(3, 70), (60, 90), (700, 80)])
def test_near_the_line_of_the_layout_rule(gsl, count, leaves):
    """Graphs with half of their entries in rows of more than 64 run in one launch, those with nearly all of them there
    (a clique) on the renumbered copy."""
    for extra, fill in ((0, 0), (1, 0), (0, 1)):
        g = hubs(count, leaves, extra, fill)
        deg = np.diff(g.offsets)
        say("line n=%d heavy %d of %d" % (g.n, deg[deg > 64].sum(), g.nnz))
        off, cols, w = to_device(g)
        with Took(gsl) as t:
            lab, st = gsl.gsl_lpa_ex(off, cols, w)
        assert t.routes == {"one_launch": 1}
        r = oracle.lpa(g)
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
        assert st["iterations"] == r.iterations and not st["renumbered"]
    g = graphgen.cliques([leaves] * count)
    off, cols, w = to_device(g)
    with Took(gsl) as t:
        lab, st = gsl.gsl_lpa_ex(off, cols, w)
    assert t.routes == {"declined": 1} and st["renumbered"]
    np.testing.assert_array_equal(lab.cpu().numpy(), oracle.lpa(g).labels)


def test_long_rows_are_seen_before_the_first_sweep_or_after_it(gsl):
    """One row of 2,049 beside many of 300 (which have more rows sampled), one beside short rows only (found by its
    window), and none above 2,048; weights, a batch, and the call that never allocates."""
    rng = np.random.default_rng(5)
    for n, heavy, longest, want in ((30000, 60, 2049, "declined"), (30000, 60, 2048, "one_launch"), (30000, 0, 2049, "declined"),
                                    (70000, 60, 2049, "declined")):
        u = np.concatenate([np.full(300, 200 * (k + 1)) for k in range(heavy)] + [np.zeros(longest, dtype=np.int64), np.arange(n // 2, n - 1)])
        v = np.concatenate([rng.choice(np.arange(n // 2, n), 300, replace=False) for _ in range(heavy)] +
                           [rng.choice(np.arange(n // 2, n), longest, replace=False), np.arange(n // 2 + 1, n)])
        g = graphgen.from_undirected(n, list(zip(u.tolist(), v.tolist())), rng.integers(1, 9, size=u.size) if heavy else None)
        assert np.diff(g.offsets).max() == longest
        say("long row n=%d heavy=%d longest=%d" % (n, heavy, longest))
        off, cols, w = to_device(g)
        ref = oracle.lpa(g).labels
        for call in (lambda: gsl.gsl_lpa_ex(off, cols, w, layout="original")[0], lambda: gsl.gsl_lpa_noalloc(off, cols, w),
                     lambda: gsl.gsl_lpa_graphs([(off, cols, w)])[0][0]):
            for _ in range(2):
                with Took(gsl) as t:
                    lab = call()
                assert t.routes == {want: 1}
                np.testing.assert_array_equal(lab.cpu().numpy(), ref)


def test_the_last_calls_variants(gsl):
    """The sweep variants that a call took where they are not the table's."""
    table = [v for _, v in gsl.gsl_get_tiers()]
    n = 300000
    v = np.arange(n, dtype=np.int64)

    def ring(reach):
        rows = np.concatenate([v] * (2 * reach))
        cols = np.concatenate([(v + h) % n for h in range(1, reach + 1)] + [(v - h) % n for h in range(1, reach + 1)])
        return to_device(graphgen.from_entries(n, rows, cols))

    for reach, want in ((3, {0: 0}), (8, {0: 15}), (16, {}), (20, {1: 18})):
        gsl.gsl_lpa(*ring(reach), max_iters=2)
        took, windows = gsl.gsl_last_variants()
        assert not windows and took == [want.get(k, x) for k, x in enumerate(table)], reach
    g = to_device(planted(3000))
    gsl.gsl_lpa(*g)
    assert gsl.gsl_last_variants() == ([-1] * 7, False)  # one launch
    test_gpu_near.test_batch(gsl)
    took, windows = gsl.gsl_last_variants()
    assert windows and took[0] == 16
    gsl.gsl_lpa_f32(g[0], g[1], torch.ones(g[1].numel(), device="cuda"))
    assert gsl.gsl_last_variants() == ([-1] * 7, False)


def test_batches_of_thousands_of_graphs(gsl):
    """Up to 4,096 graphs share one launch; thousands with weights count as larger."""
    b = graphgen.batched_planted(4096, 5, nmin=2, nmax=40, kmin=1, kmax=3)
    off, cols, _ = to_device(b)
    vb, eb = torch.from_numpy(b.vtx_base).cuda(), torch.from_numpy(b.edge_base).cuda()
    w = torch.ones_like(cols)
    say("batch of 4,096: %d vertices" % b.n)
    assert b.n + 16 * 4096 <= 1 << 17
    with Took(gsl) as t:
        plain = gsl.gsl_lpa_batched(vb, eb, off, cols)
        weighted = gsl.gsl_lpa_batched(vb, eb, off, cols, w)
    assert t.routes == {"one_launch": 2}
    n = (1 << 17) - 16 * 4096 + 4096  # vertices beyond the line for weights, 4,096 graphs
    size = n // 4096
    g = graphgen.cliques([size] * 4096)
    base = np.arange(4097, dtype=np.int64) * size
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    local = (g.cols - np.repeat(np.repeat(base[:-1], size), np.diff(g.offsets))).astype(np.int32)
    args = up(base), up(g.offsets[base]), up(g.offsets), up(local)
    with Took(gsl) as t:
        a = gsl.gsl_lpa_batched(*args, torch.ones(g.nnz, dtype=torch.int32, device="cuda"))
    assert t.routes == {}
    with Took(gsl) as t:
        c = gsl.gsl_lpa_batched(*args)
    assert t.routes == {"one_launch": 1}
    assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
    assert torch.equal(plain[0], weighted[0])
    for k in range(0, 4096, 97):
        r = oracle.lpa(b.subgraph(k))
        np.testing.assert_array_equal(plain[0][int(vb[k]):int(vb[k + 1])].cpu().numpy(), r.labels, err_msg="graph %d" % k)
        assert plain[1][k] == r.iterations


def test_few_graphs_that_keep_changing(gsl):
    """A workgroup's changes of one graph are counted together: graphs of many windows, of parts of one, and both."""
    sizes = [40000, 37, 200, 129, 100000, 64, 64, 1, 70000]
    gs = [graphgen.planted(n, max(1, n // 400), 0.02, n, 3 + n % 5) for n in sizes]
    dev = [to_device(g) for g in gs]
    with Took(gsl) as t:
        labels, sweeps, _ = gsl.gsl_lpa_graphs(dev, 20, 0.0)
    assert t.routes == {"one_launch": 1}
    for g, lab, ran in zip(gs, labels, sweeps):
        r = oracle.lpa(g, 20, 0.0)
        np.testing.assert_array_equal(lab.cpu().numpy(), r.labels)
        assert ran == r.iterations
