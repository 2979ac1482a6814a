"""The dispatch of the trailing update (no GPU): a request that no kernel serves is
refused before anything is launched, never left out."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2502_16555_amd")

PROGRAM = r"""
#include <cstdio>
#include <stdexcept>
#include "internal.h"
int main(int, char** argv) {
  int kind = 0, kd = 0;
  std::sscanf(argv[1], "%d", &kind), std::sscanf(argv[2], "%d", &kd);
  try {
    bte::launch_update(kind, nullptr, 1024, 0, 1, 1, 0, 1, false, nullptr, kd, 0, nullptr, nullptr);
  } catch (const std::logic_error&) {
    std::puts("refused");
    return 0;
  }
  std::puts("accepted");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no host compiler or HIP headers")
    from paper_2502_16555_amd import _lib
    _lib.load()
    d = tmp_path_factory.mktemp("update")
    src, exe = d / "u.cpp", d / "u"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{os.path.join(PKG, 'csrc')}", str(src), "-o", str(exe), os.path.join(PKG, "libbte.so"),
                    f"-Wl,-rpath,{PKG}", "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined"], check=True)
    return str(exe)


@pytest.mark.parametrize("kind,kd", [(0, 384), (0, 512), (1, 384), (1, 512), (0, 64), (1, 640)])
def test_updates_that_no_kernel_serves_are_refused(program, kind, kd):
    out = subprocess.run([program, str(kind), str(kd)], capture_output=True, text=True)
    assert out.stdout.strip() == "refused", (out.returncode, out.stdout, out.stderr)
