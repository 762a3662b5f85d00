"""32-bit positions of the gather kernel's chunks (positions.hpp), compiled for the host: the
lookups left of a chunk and its bag ends, at the edges of 32 bits and of the rebase distance,
and for offsets that decrease (against the contract), where a chunk must read nothing."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_01676_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")

MAIN = r"""
#include <cstdio>
#include "positions.hpp"
int main() {
  long long d;
  while (std::scanf("%lld", &d) == 1) std::printf("%d %d\n", embx::stretch(d), embx::rel32(d));
  return 0;
}
"""


def test_positions_at_the_edges(tmp_path):
    src = tmp_path / "positions.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "positions"
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    far = 1 << 30
    edges = [0, 1, far, 1 << 31, 1 << 32, 1 << 40, (1 << 63) - 2]
    ds = sorted({s * (e + k) for e in edges for k in (-1, 0, 1) for s in (-1, 1)})
    r = subprocess.run([str(exe)], input=" ".join(map(str, ds)), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    assert [tuple(map(int, ln.split())) for ln in r.stdout.splitlines()] == \
        [(min(max(d, 0), far), min(max(d, 0), (1 << 31) - 1)) for d in ds]
