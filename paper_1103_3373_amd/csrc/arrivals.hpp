// How the workgroups of a one-launch reduction find out which of them finishes
// last.  Plain C++ (also compiled by the host tests).
#pragma once

namespace hy {

// Workgroup b adds to counter b mod 16 (a leaf), whoever completes a leaf adds
// one to the main counter: increments of one address take about 10 ns each, one
// after another.  Every launch, whatever its size, adds exactly kLeafSum to each
// leaf and kDoneLeaves to the main counter (the first workgroup of a leaf adds
// for the missing ones), and completion is the step over a multiple of that
// sum.  The counters are therefore never reset, and launches that overlap on one
// set, although they spoil each other's results, leave it in order: a limit of
// the launch's own (atomicInc) would leave it between two multiples, and the
// launches after it would finish early or not at all.
constexpr unsigned kReduceMax = 1024;                      // workgroups of a launch, at least kDoneLeaves
constexpr unsigned kDoneLeaves = 16, kDoneStride = 16;     // 64 bytes for each counter (128: no faster)
constexpr unsigned kDoneSet = (kDoneLeaves + 1) * kDoneStride;  // the main counter, then the leaves
constexpr unsigned kLeafSum = kReduceMax / kDoneLeaves;
static_assert((kLeafSum & (kLeafSum - 1)) == 0 && (kDoneLeaves & (kDoneLeaves - 1)) == 0, "the counters wrap at 2^32");

constexpr unsigned arrival_leaf(unsigned b) { return (b % kDoneLeaves + 1) * kDoneStride; }
// What workgroup b of P adds to its leaf.
constexpr unsigned arrival_weight(unsigned b, unsigned P) {
  return b < kDoneLeaves ? kLeafSum + 1 - (P / kDoneLeaves + (b < P % kDoneLeaves ? 1 : 0)) : 1;
}
// Whether adding w to a counter that was `old` steps over a multiple of `sum`.
constexpr bool arrival_completes(unsigned old, unsigned w, unsigned sum) { return ((old ^ (old + w)) & ~(sum - 1)) != 0; }

}  // namespace hy
