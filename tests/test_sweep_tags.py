"""Tags of the streaming fills' exchange words (CPU only: a small program built
from the kernels' own header).  From every count a workspace can hold, and
from counts at the ends of the integer range, a tag is in 1 .. tags and is not
used again before every other one was."""
import subprocess

import pytest

from paper_2311_17530_amd import build as B

PROGRAM = r"""
#include <stdint.h>
#include <stdio.h>
#include "msa_internal.h"
int main() {
  const int tags[2] = {msa::kSweepTags3, msa::kSweepTags};
  for (int t : tags) {
    for (int64_t first : {(int64_t)0, (int64_t)1, (int64_t)104, (int64_t)INT32_MAX,
                          (int64_t)INT32_MAX - 3, (int64_t)INT32_MIN, (int64_t)-1}) {
      int32_t c = msa::next_sweep((int32_t)first, 0);
      int last[16];
      for (int &x : last) x = -1000;
      for (int n = 0; n < 400; ++n) {
        const int g = msa::sweep_tag(c, t);
        if (c < 0 || g < 1 || g > t || n - last[g] < t) {
          printf("start %lld step %d count %d tag %d of %d\n", (long long)first, n, c, g, t);
          return 1;
        }
        last[g] = n;
        if (msa::next_sweep(c, 0) != c) return 2;  // a launch without a streaming fill
        c = msa::next_sweep(c, 1);
      }
    }
    for (int32_t c : {INT32_MAX, INT32_MIN, -1})  // counts no workspace holds
      if (msa::sweep_tag(c, t) < 1 || msa::sweep_tag(c, t) > t) return 3;
  }
  puts("ok");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("tags")
    (d / "t.hip").write_text(PROGRAM)
    r = subprocess.run([B.HIPCC, *B.COMMON, "-I", str(B.CSRC), "-o", str(d / "t"), str(d / "t.hip")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return d / "t"


def test_tags_go_round(program):
    r = subprocess.run([str(program)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout)
