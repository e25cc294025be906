"""The batched step's pinned staging is allocated once over the calls a program
makes on one set of clusters (an evaluation of a(x0), then steps).  A small host
program evaluates the library's own sizes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "scf_plan.h"
#include <cstdio>
int main() {
  const long long cases[][4] = {  // units, clusters, particles, units of the plan at most
      {1024, 10, 1200000, 1034}, {700, 48, 150000, 1072}, {1, 1, 100, 1025}, {1024, 2000, 4000000, 3024},
      {1024, 1 << 20, 1 << 21, 1 << 20}};
  for (auto& c : cases) {
    const long long nblk = (c[2] + 255) / 256 + c[1];
    const size_t bound = BatchUpload(c[3], (int)c[1], nblk, kCentreRows).total;
    auto need = [&](long long rows) {
      return BatchUpload(c[0], (int)c[1], nblk, 1).tab + (size_t)rows * c[1] * 9 * sizeof(double);
    };
    size_t cap = 0;
    printf("%lld", c[1]);
    for (long long steps : {0, 5, 200}) {
      int grown = need(steps + 1) > cap;
      if (grown) cap = staging_capacity(need(steps + 1), bound);
      printf(" %d", grown);
      if (cap < need(steps + 1)) return 1;
      if (cap > need(steps + 1) + (1u << 20) && grown) return 2;
    }
    // a long run grows it once more, and a somewhat longer one does not
    cap = staging_capacity(need(1001), bound);
    printf(" %d %d\n", cap < need(1001), cap < need(1400));
  }
  return 0;
}
"""


def test_one_allocation_over_the_calls_of_a_program(tmp_path):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("no hipcc")
    src = tmp_path / "staging.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "staging"
    csrc = os.path.join(ROOT, "paper_2602_13385_amd", "csrc")
    subprocess.check_call([HIPCC, "-std=c++17", "-O1", "-x", "hip", "--offload-host-only",
                           "--offload-arch=gfx950", "-I", csrc, "-I", os.path.join(ROOT, "include"),
                           str(src), "-o", str(exe)], stderr=subprocess.DEVNULL)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out
    lines = [l.split() for l in out.stdout.splitlines()]
    # one allocation for calls of 0, 5 and 200 steps (clusters by the million excepted)
    assert [l[1:4] for l in lines[:3]] == [["1", "0", "0"]] * 3
    assert [l[4:] for l in lines] == [["0", "0"]] * 5
