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


def test_kernel_names_of_the_variants():
    import paper_2403_01261_amd as gsl
    if not os.path.exists(gsl.LIB_PATH):
        pytest.skip("libgsl_lpa.so not built")
    assert gsl.gsl_last_variants() == ([-1] * 7, False)  # no call on this thread yet
    v = gsl.gsl_tier_variants()
    assert gsl.variant_kernel_name(v[16]) == "sweep_thread<32, false, true, true, false>"
    assert gsl.variant_kernel_name(v[16], windows=True) == "sweep_thread<32, false, true, true, true>"
    assert gsl.variant_kernel_name(v[0], True, 1 << 30) == "sweep_thread<8, true, false, true, false>"
    assert gsl.variant_kernel_name(v[6]) == "sweep_lds<16, 7, 256, 4>"
