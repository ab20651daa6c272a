"""Separate graphs gathered tile by tile: tiles inside one graph and across
graphs, mixed weights, one entry out of range in the middle of a large graph
(that graph alone is rejected, its output untouched)."""
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


@pytest.mark.parametrize("at", [None, 0, 4095, 4096, 50000, -1])
def test_graphs(gsl, at):
    gs = [graphgen.planted(n, max(1, n // 100), 0.12, n // 2, 9 + n, wmin=w and 1, wmax=w)
          for n, w in ((300, 0), (9000, 7), (40, 3), (12000, 0), (700, 0))]
    dev = [to_device(g) for g in gs]
    if at is not None:
        dev[3][1][at] = gs[3].n if at % 2 else -1
    outs = [torch.full((g.n,), -7, dtype=torch.int32, device="cuda") for g in gs]
    say("gather at=%s" % at)
    _, sweeps, _, status = gsl.gsl_lpa_graphs([(*d, o) for d, o in zip(dev, outs)], 20, 0.05, return_status=True)
    for i, g in enumerate(gs):
        if at is not None and i == 3:
            assert status[i] != gsl.GSL_OK and (outs[i] == -7).all()
            continue
        r = oracle.lpa(g, 20, 0.05)
        assert status[i] == gsl.GSL_OK and sweeps[i] == r.iterations
        np.testing.assert_array_equal(outs[i].cpu().numpy(), r.labels)
