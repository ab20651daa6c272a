"""The 16-byte row loads of the thread and small-graph kernels read no word
that holds no entry of the row: rows of every length a kernel may ask for, none
at all among them (a lane past its row's end), from every alignment, against
pages that may not be read.  The kernels' own code, built for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2403_01261_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2403_01261_amd.build import HIPCC
    out = str(tmp_path_factory.mktemp("host") / "row_loads")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", CSRC,
                        os.path.join(ROOT, "tests", "host", "row_loads.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


def test_only_words_of_the_row_are_read(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=60)
    tail = r.stdout.strip().split("\n")[-1]
    assert r.returncode == 0 and tail == "all rows", "ended with %d at: %s" % (r.returncode, tail)
