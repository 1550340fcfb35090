// Which group and planes a workgroup of the periodic ghost fill takes.  Plain C++
// (also compiled by the host tests).
#pragma once

namespace hy {

// A workgroup fills a pair of planes of one group (H pairs a group, cnt groups).
// Workgroups are dispatched to the 8 XCDs round-robin.  By XCD, XCD x takes the
// x-th eighth of the groups, whose neighbours then share its L2; otherwise the
// pairs of all groups follow one another.
struct FillItem {
  unsigned group, pair;  // no group if group >= cnt
};
constexpr unsigned fill_grid(unsigned cnt, unsigned H, bool by_xcd) { return (by_xcd ? (cnt + 7) / 8 * 8 : cnt) * H; }
constexpr FillItem fill_item(unsigned block, unsigned cnt, unsigned H, bool by_xcd) {
  const unsigned w = by_xcd ? block / 8 : block;
  return {w / H + (by_xcd ? block % 8 * ((cnt + 7) / 8) : 0u), w % H};
}

// Where the order by XCD pays, us by XCD and otherwise (FP32, g = 3, plain box /
// grouped source unless noted):
//     64 groups  5.0 / 5.7  and  5.5 / 6.1     240 groups  13 / 14  and  21 / 18
//    512         25 / 26         44 / 35      1,728        79 / 84      197 / 169
//  4,096        322 / 319       372 / 313     8,000       652 / 661     896 / 759
// 3,072 groups, g = 4: 184 / 168 and 229 / 225; 4,096: - / 427 and - / 347.
// The source is read 1.4 to 3.4 times, from the 256 MB cache behind the L2s where
// it fits in there: by XCD always.  Where it does not, eight streams far apart
// cost the memory more, the more ghost cells are written: up to 18% at g = 4.
// At g = 3 they still pay for a plain box, and for groups unless their rows are
// multiples of 8, which puts neighbours on one XCD in either order.  Below 64
// groups (4 us) nothing is gained; wider ghosts (no scheme has them) gain or lose
// up to 1.4 times.
constexpr bool fill_by_xcd(long long cnt, int elem_bytes, int g, int ngx, bool grouped) {
  return cnt >= 64 && g <= 5 &&
         (cnt * 5 * 4096 * elem_bytes <= 256LL << 20 || g == 2 || (g == 3 && (!grouped || ngx % 8 != 0)));
}

}  // namespace hy
