"""The host's rules for choosing a path, compiled from the library's own header.  CPU only."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cmath>
#include "gp_internal.h"
int main() {
  const float ms = 0.25f;
  // the locator stays where it is at least as fast, equal times included
  if (!gp::locator_kept(ms, ms)) return 1;
  if (!gp::locator_kept(std::nextafter(ms, 0.0f), ms)) return 2;
  if (gp::locator_kept(std::nextafter(ms, 1.0f), ms)) return 3;
  return 0;
}
"""


def test_equal_times_keep_the_locator(tmp_path):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_1403_0802_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + csrc, "-I" + os.path.join(ROOT, "include"), str(src), "-o",
                        str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert subprocess.run([str(exe)]).returncode == 0
