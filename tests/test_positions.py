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
  int n;
  if (std::scanf("%d", &n) != 1) return 1;
  const int far = embx::far_of(n);
  std::printf("%d\n", far);
  while (std::scanf("%lld", &d) == 1) std::printf("%d %d\n", embx::stretch(d, far), embx::rel32(d));
  return 0;
}
"""


@pytest.mark.parametrize("steps", [12, 13, 16])
@pytest.mark.parametrize("lanes", [16, 32, 64])
@pytest.mark.parametrize("most", [None, 100])
def test_positions_at_the_edges(tmp_path, most, lanes, steps):
    src = tmp_path / "positions.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "positions"
    cmd = ["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", str(exe)]
    if most is not None:
        cmd.append(f"-DEMBX_FAR={most}")
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    n = 64 // lanes * steps
    far = (most or 1 << 30) // n * n   # whole steps
    edges = [0, 1, far, 1 << 30, 1 << 31, 1 << 32, 1 << 40, (1 << 63) - 2]
    ds = sorted({s * (e + k) for e in edges for k in (-1, 0, 1) for s in (-1, 1)})
    r = subprocess.run([str(exe)], input=" ".join(map(str, [n, *ds])), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    lines = r.stdout.splitlines()
    assert int(lines[0]) == far
    assert [tuple(map(int, ln.split())) for ln in lines[1:]] == \
        [(min(max(d, 0), far), min(max(d, 0), (1 << 31) - 1)) for d in ds]
