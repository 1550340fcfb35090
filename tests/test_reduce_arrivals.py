"""The arrival counters of the one-launch reductions, simulated on the host with
the functions that the kernel uses: launches one after another finish with their
last workgroup, and launches that overlapped leave the counters in order."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1103_3373_amd", "csrc")
PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "arrivals.hpp"
using namespace hy;
unsigned set[kDoneSet];
bool add(unsigned i, unsigned w, unsigned sum) { const unsigned old = set[i]; set[i] += w; return arrival_completes(old, w, sum); }
bool arrive(unsigned b, unsigned P) { return add(arrival_leaf(b), arrival_weight(b, P), kLeafSum) && add(0, 1, kDoneLeaves); }
int main() {
  std::mt19937 rng(1);
  for (unsigned start : {0u, 0u - 4 * kLeafSum})  // also across the counters' wrap
    for (int trial = 0; trial < 300; ++trial) {
      for (unsigned& c : set) c = start;
      const int together = trial % 4;  // launches that overlap (0: none)
      std::vector<std::pair<unsigned, unsigned>> q;
      for (int l = 0; l < together; ++l) {
        const unsigned P = kDoneLeaves + rng() % (kReduceMax + 1 - kDoneLeaves);
        for (unsigned b = 0; b < P; ++b) q.push_back({b, P});
      }
      std::shuffle(q.begin(), q.end(), rng);
      int finishers = 0;
      for (auto [b, P] : q) finishers += arrive(b, P);
      if (finishers != together) return printf("%d launches together, %d finishers\n", together, finishers), 1;
      for (unsigned P : {16u, 17u, 31u, 500u, 1023u, 1024u, 16u}) {  // then one after another
        std::vector<unsigned> o(P);
        for (unsigned b = 0; b < P; ++b) o[b] = b;
        std::shuffle(o.begin(), o.end(), rng);
        for (unsigned k = 0; k < P; ++k)
          if (arrive(o[k], P) != (k + 1 == P)) return printf("after %d together: P %u, arrival %u\n", together, P, k), 1;
      }
    }
  return 0;
}
"""


def test_arrival_counters(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
