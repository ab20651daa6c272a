"""Workgroups of the one-launch kernel on devices of any size: they wait for
each other, so no launch asks for more than the device's CUs hold, nor do the
launches in flight together.  The header's own arithmetic, built for the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2403_01261_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "meeting.h"
using namespace gsl;
#define CHECK(x) do { if (!(x)) { printf("cus %d n %lld weighted %d batch %d: %s\n", cus, (long long)n, weighted, batch, #x); return 1; } } while (0)
int main() {
  for (int cus : {1, 2, 3, 32, 38, 64, 80, 128, 255, 256, 304})
    for (long long n : {1ll, 2ll, 128ll, 129ll, 256ll, 257ll, 4096ll, 32768ll, 32769ll, 65536ll, 65537ll, 131072ll, 262144ll, 1ll << 30})
      for (int weighted = 0; weighted < 2; ++weighted)
        for (int batch = 0; batch < 2; ++batch) {
          const int grid = small_grid(n, weighted, batch, cus), share = small_share(weighted);
          CHECK(grid >= 1 && grid <= kSmallGrid);
          CHECK(grid * share <= 2 * cus);
          CHECK(grid * share <= small_room(cus, true) || grid == 1);
          CHECK(small_room(cus, false) <= cus && small_room(cus, false) <= small_room(cus, true));
          CHECK(small_room(cus, true) <= 2 * cus && small_room(cus, true) <= kSmallGrid);
          CHECK(grid == 1 || (long long)(grid - 1) * kSmallWindow < n);  // no workgroup without a vertex
          if (n <= kSmallOne && !batch) CHECK(grid == 1);
          if (cus >= 256) {
            const long long want = n <= kSmallOne && !batch ? 1 : (n + 127) / 128, most = weighted ? 256 : 512;
            CHECK(grid == (want < most ? want : most));
            CHECK(small_room(cus, true) == 512 && small_room(cus, false) == 128);
          }
        }
  return 0;
}
"""


def test_launches_fit_the_device(tmp_path):
    src, out = str(tmp_path / "grid.cpp"), str(tmp_path / "grid")
    open(src, "w").write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", out], check=True)
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
