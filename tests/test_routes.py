"""The route counts on the host: a count per route of the header, none before
the first call, and no device work."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_count_per_route():
    import paper_2403_01261_amd as gsl
    if not os.path.exists(gsl.LIB_PATH):
        pytest.skip("libgsl_lpa.so not built")
    header = open(os.path.join(ROOT, "include", "gsl_lpa.h")).read()
    names = re.findall(r"GSL_ROUTE_([A-Z0-9_]+) = (\d+)", header)
    assert [int(v) for _, v in names] == list(range(len(names)))
    assert int(re.search(r"GSL_ROUTES = (\d+)", header).group(1)) == len(names)
    code = "import paper_2403_01261_amd as m; print(m.gsl_route_counts())"
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    assert eval(r.stdout) == {n.lower(): 0 for n, _ in names}
    assert gsl.load().gsl_route_counts(None) == gsl.GSL_EINVAL
