"""Which item a workgroup takes: division by multiplication, and the items of a launch each taken exactly once."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2410_01485_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "lg_mask.h"
int main() {
  const int ds[] = {1, 2, 3, 5, 7, 8, 12, 63, 64, 65, 1000, 4097, 65535, 65536, 16777215, 715827883, 1073741824, 2147483646, 2147483647};
  for (int d : ds) {
    const LgDiv v = lg_make_div(d);
    std::vector<long long> ns = {0, 1, 2147483646, 2147483647};
    for (long long q = 1; q * d - 1 <= 2147483647LL && q < 4000; q = q < 50 ? q + 1 : q * 3 / 2)
      for (int e = -1; e <= 1; ++e) ns.push_back(q * d + e);
    for (long long q = 2147483647LL / d, k = 0; k < 50 && q - k > 0; ++k)
      for (int e = -1; e <= 1; ++e) ns.push_back((q - k) * d + e);
    for (long long n : ns) {
      if (n < 0 || n > 2147483647LL) continue;
      int rem, x = lg_divmod(v, (int)n, &rem);
      if (x != n / d || rem != n % d) { std::printf("%lld / %d = %d rest %d\n", n, d, x, rem); return 1; }
    }
  }
  const int shapes[][5] = {{1, 1, 1, 1, 1}, {2, 8, 2, 5, 3}, {3, 6, 6, 7, 16}, {1, 64, 8, 129, 1000}, {4, 4, 1, 2, 2}, {4, 16, 16, 8, 7}, {4, 32, 16, 2, 300}};
  for (auto& s : shapes) {
    const int B = s[0], Hq = s[1], Hkv = s[2], nqt = s[3], run = s[4], total = B * Hq * nqt;
    const LgItems w = lg_make_items(total, run, nqt, Hq, Hkv);
    std::vector<int> seen(total, 0);
    for (long long id = 0; id < lg_run_grid(total, run); ++id) {
      const int L = lg_item_of((int)id, w.run);
      if (L >= total) continue;
      const LgItem it = lg_item(w, L);
      if (it.b < 0 || it.b >= B || it.hq < 0 || it.hq >= Hq || it.x < 0 || it.x >= nqt || it.hk != it.hq / (Hq / Hkv)) return 2;
      ++seen[(it.b * Hq + it.hq) * nqt + it.x];
    }
    for (int x : seen)
      if (x != 1) return 3;
  }
  return 0;
}
"""


@pytest.mark.parametrize("opt", ["-O0", "-O2"])
def test_division_by_multiplication_and_items(tmp_path, opt):
    src, exe = tmp_path / "items.cpp", tmp_path / "items"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", opt, "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
