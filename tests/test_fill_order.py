"""The periodic fill's map from workgroups to planes, on the host with the
functions that the kernel uses: every pair of planes once, and the order by XCD
where it is asked for, group counts that are multiples of 8 among them."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1103_3373_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "fill_order.hpp"
using namespace hy;
int main() {
  for (unsigned cnt : {1u, 7u, 64u, 65u, 240u, 250u, 511u, 512u, 1728u, 4096u})
    for (unsigned H : {8u, 10u, 11u, 12u, 24u})
      for (bool by_xcd : {false, true}) {
        std::vector<int> seen(cnt * H);
        for (unsigned b = 0; b < fill_grid(cnt, H, by_xcd); ++b) {
          const FillItem i = fill_item(b, cnt, H, by_xcd);
          if (i.group >= cnt) continue;
          if (i.pair >= H) return printf("pair %u of %u\n", i.pair, H), 1;
          ++seen[i.group * H + i.pair];
          if (by_xcd && b % 8 != i.group / ((cnt + 7) / 8)) return printf("cnt %u: group %u on XCD %u\n", cnt, i.group, b % 8), 1;
        }
        for (int s : seen)
          if (s != 1) return printf("cnt %u H %u: a pair %d times\n", cnt, H, s), 1;
      }
  // boxes of 64 to 3,072 groups, with every ghost width of the schemes
  for (int g : {2, 3, 4})
    for (long long cnt : {64, 65, 240, 512, 1728, 3072})
      for (bool grouped : {false, true})
        if (!fill_by_xcd(cnt, 4, g, 8, grouped)) return printf("%lld groups, g %d: not by XCD\n", cnt, g), 1;
  return fill_by_xcd(63, 4, 3, 8, false) || fill_by_xcd(4096, 4, 4, 16, true) || !fill_by_xcd(4096, 4, 3, 16, false);
}
"""


def test_fill_order(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
