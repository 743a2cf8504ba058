"""The loader's cell index (pic_load_key), on the host: one to one over the cells
of ragged tiles, and within the keys the loader allocates where they exceed 2^31."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1503_00276_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <set>
#include "pic_kernels.h"
static GridDesc grid(int dim, int a, int b, int c, int ta, int tb, int tc) {
  GridDesc g{};
  const int nx[3] = {a, b, c}, t[3] = {ta, tb, tc};
  g.dim = dim;
  g.ntiles = 1;
  for (int d = 0; d < 3; d++) {
    g.nx[d] = nx[d];
    g.tile[d] = t[d];
    g.ntile[d] = (nx[d] + t[d] - 1) / t[d];
    g.ntiles *= g.ntile[d];
  }
  return g;
}
int main() {
  const GridDesc s = grid(3, 11, 9, 7, 4, 5, 3);
  const long long n = (long long)s.ntiles * 4 * 5 * 3;
  std::set<long long> seen;
  for (int z = 0; z < 7; z++)
    for (int y = 0; y < 9; y++)
      for (int x = 0; x < 11; x++) {
        const int c[3] = {x, y, z};
        const long long k = pic_load_key(s, c);
        if (k < 0 || k >= n || !seen.insert(k).second) return 1;
      }
  const GridDesc big = grid(3, 1021, 1021, 2045, 5, 5, 5);
  const int last[3] = {1020, 1020, 2044};
  const long long keys = (long long)big.ntiles * 125;
  printf("%lld of %lld\n", pic_load_key(big, last), keys);
  return pic_load_key(big, last) == keys - 125 + 0 + 5 * (0 + 5 * 4) ? 0 : 2;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"), reason="needs g++ and HIP")
def test_load_key(tmp_path):
    src = tmp_path / "key.cpp"
    src.write_text(SRC)
    exe = tmp_path / "key"
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src),
                           "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    last, keys = (int(v) for v in r.stdout.split(" of "))
    assert 2 ** 31 < last < keys
