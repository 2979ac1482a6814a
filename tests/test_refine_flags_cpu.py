"""The words that the launches of a mixed-precision refinement hand on (no GPU):
every block of a sweep's solve takes the stop test, so that launch must read only
what earlier launches wrote and write only what later ones read."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "internal.h"
using namespace bte;
int main() {
  int status[4] = {0, 0, 0, 0};
  double resid = 0, E[3] = {}, n0x[3] = {};
  unsigned long long r[6], b[6], x[6];
  DevOps d;
  d.nx_total = 3, d.status = status, d.resid = &resid, d.E = E, d.n0x = n0x;
  d.rmax = r, d.bmax = b, d.xmax = x;
  int bad = 0;
  const int* written = nullptr;   // the done flag of the sweep before
  for (int k = 0; k < 8; ++k) {
    const RefineCheck c = refine_check(d, k & 1, 1e-14, k);
    bad += c.done == c.done1;                              // read and written by one launch
    bad += c.done1 == status || c.done1 == status + 2;     // the status bits, the sweeps
    bad += k > 0 && c.done != written;                     // the chain of the sweeps
    bad += c.r == c.r1 || c.b == c.b1 || c.x == c.x1;      // maxima read, and cleared for the next sweep
    bad += c.done < status || c.done >= status + 4 || c.done1 >= status + 4;
    written = c.done1;
  }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_a_sweep_reads_only_what_earlier_launches_wrote(tmp_path):
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no host compiler or HIP headers")
    src = tmp_path / "flags.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "flags"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{os.path.join(ROOT, 'paper_2502_16555_amd', 'csrc')}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip() == "0"
