"""The arrival test of the grid barriers (csrc/grid_sync.h) on the host: whatever
solves went before, a block that has not arrived in this launch must not count
as arrived.  A solve clears the flags, then passes barriers in its reduction
and in its divide and conquer; the blocks that each joins go down and up, as
the live orders of a run do, over more than 2^16 solves, and the flags start
from zero or from anything at all.  No GPU."""
import subprocess

from paper_2503_18056_amd import build

SRC = r"""
#include <stdio.h>
#include <stdint.h>
#include "grid_sync.h"
using namespace tt;
static long long bad = 0;
static unsigned flag[SYNC_MAXP];

// P blocks pass nb barriers from ordinal base + 1 on: before a block stores an
// ordinal, its flag must not pass for it, and afterwards it must.
static void launch(unsigned base, int P, int nb) {
  unsigned ord = base;
  for (int k = 0; k < nb; ++k) {
    ++ord;
    for (int q = 0; q < P; ++q) {
      bad += grid_arrived(flag[q], ord);
      flag[q] = ord;
      bad += !grid_arrived(flag[q], ord);
    }
  }
}
static void solve(int Pr, int nr, int Pd, int nd) {
  for (int t = 0; t < 512; ++t) grid_clear(flag, t, 512);
  launch(GRID_ORD_REDUCE, Pr, nr);
  launch(GRID_ORD_DC, Pd, nd);
}

int main() {
  // narrow for `hold` solves, then wide
  const int hold[] = {0, 1, 100, 16384, 32767, 32768, 65535, 65536, 70000};
  for (int h : hold)
    for (unsigned first : {0u, 1u, 0x7fffffffu, 0x80000000u, 0xffffffffu}) {
      for (int q = 0; q < SYNC_MAXP; ++q) flag[q] = first;
      for (int i = 0; i < h; ++i) solve(16, 2, i % 2 ? 0 : 40, 3);
      solve(32, 3, 64, 8);
      solve(64, 3, 64, 8);
      solve(16, 3, 64, 8);
      solve(64, 1024, 64, 15);  // a barrier a column of the largest order
      solve(0, 0, 64, 15);      // the divide and conquer alone
      solve(64, 1024, 0, 0);
    }
  printf("%lld\n", bad);
  return bad != 0;
}
"""


def test_a_flag_of_an_earlier_launch_is_never_an_arrival(tmp_path):
    src = tmp_path / "grid_sync_test.hip"
    src.write_text(SRC)
    exe = tmp_path / "grid_sync_test"
    r = subprocess.run([build._hipcc(), "--cuda-host-only", "--offload-arch=" + build.ARCH, "-O2", "-std=c++17",
                        "-I" + build.CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, "early arrivals: " + r.stdout
