"""Steps of a session that run in one launch, against the oracle and beside
steps that cannot: small and larger arenas, rows too long for the launch, a
limited number of graphs collected per step, and waits that run out.  All
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


def star(n):
    return graphgen.from_undirected(n, [(0, k) for k in range(1, n)])


def graphs(wmax, large):
    gs = [graphgen.planted(n, max(1, n // 100), 0.1, n // 2, 3 + n, wmin=1 if wmax else 0, wmax=wmax)
          for n in (1, 2, 130, 900, 257, 5000, 12001, 300, 2500, 40, 7000)]
    if large:
        gs.insert(3, graphgen.planted(270000, 900, 0.05, 90000, 5, wmin=1 if wmax else 0, wmax=wmax))
    return gs


def serve(gsl, gs, weighted, sweeps, capacity=None):
    refs = [oracle.lpa(g, 20, 0.05) for g in gs]
    v, e = sum(g.n for g in gs), sum(g.nnz for g in gs)
    sess = gsl.Session(v, max(e, 1), max_graphs=len(gs), weighted=weighted)
    running, waiting, out = {}, list(range(len(gs))), {}
    while waiting or running:
        for t, st, lab in sess.add([to_device(gs[i]) for i in waiting[:3]]):
            assert st == gsl.GSL_OK
            i = waiting.pop(0)
            out[i] = lab
            if t < 0:
                assert gs[i].n == 0
            else:
                running[t] = i
        for t, ran in sess.step(sweeps, capacity):
            i = running.pop(t)
            assert ran == refs[i].iterations, (i, ran)
            np.testing.assert_array_equal(out[i].cpu().numpy(), refs[i].labels, err_msg="graph %d" % i)
    sess.close()


@pytest.mark.parametrize("sweeps", [1, 3, 16])
@pytest.mark.parametrize("wmax", [0, 9])
def test_steps(gsl, sweeps, wmax):
    say("session sweeps=%d wmax=%d" % (sweeps, wmax))
    serve(gsl, graphs(wmax, False), bool(wmax), sweeps)


def test_few_collected_per_step(gsl):
    serve(gsl, graphs(0, False), False, 16, capacity=2)


def test_large_arena_and_long_rows_between_small_steps(gsl):
    gs = graphs(0, True)
    gs.insert(6, star(2050))
    gs.insert(8, star(2049))
    serve(gsl, gs, False, 4)


def test_a_wait_that_runs_out_leaves_the_session_sound():
    """With no patience at all the launch of a step gives up, and the step runs
    kernel by kernel instead (a process of its own: the limit is read once)."""
    code = ("import paper_2403_01261_amd as m\n"
            "from tests import test_gpu_session_small as t\n"
            "m.load()\n"
            "t.serve(m, t.graphs(0, False), False, 3)\n"
            "print('same labels')\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=110,
                       env=dict(os.environ, GSL_SMALL_WAIT_TICKS="0"))
    assert r.returncode == 0 and "same labels" in r.stdout, r.stderr[-2000:]
