// How the k-steps of the weight gradient's large tiles are dealt to workgroups (gemm_wgrad.hip).  Plain C++, so that the host can check it by itself.
#pragma once
#include <stdint.h>

namespace sste {

// `members` tiles, one from each of as many equal runs of `groups` tiles, make a group, whose k-steps laid end to end are cut at
// bound[0 .. parts] and worked off by `parts` workgroups.  One member: splits of the token axis.
// Several: the number of workgroups per tile is a fraction, so that 100 tiles keep 250 of 256 CUs busy (five workgroups for every two)
// where two each would keep 200.  A workgroup whose part crosses from one member into the next does two segments; the segments of a
// member are summed in k order.  Workgroups of the same part number run next to each other and read the same k-steps, as with splits.
// On 180 random problems that the plan deals so, the whole weight gradient against splits: 6.4 % faster on the geometric mean, 5 % slower at
// worst, eight by more than 1 %.  The plan deals one random layer of 2048 tokens and more in 140 so, and every layer of 5120 x 1280.  32768 x 5120 x 1280 e4m3: product
// 127 -> 114.5 us, the sum of three partials per tile for two 13 -> 17; 16384 x 1280 x 5120 bf16: 134 -> 121 and 13 -> 18.  Inside a training step,
// where the chip holds a lower clock, half of that is left.  The kernel pays for it with scalar registers: the loop over segments keeps 17 ... 23 of them in lanes of
// a vector register, read back inside the main loop, and needs 250 ... 253 vector registers for the 227 of the plain form.  Groups
// of five to eight tiles lose the shared reads again (seventeen workgroups for seven tiles: up to 10 % slower).  Adding a tile's segments
// up in the workgroup that ends last instead would leave the reading to one CU per tile, at an eighth of what all of them draw.
constexpr int DEAL_MEMBERS = 4, DEAL_PARTS = 32, DEAL_SHORTEST = 4;      // shortest segment, k-steps
struct WgradDeal {
  int members, parts, groups;
  uint32_t segments;                      // of member m: bits 4 m .. 4 m + 3 (one member: not used, it has `parts`)
  int bound[DEAL_PARTS + 1];
  int first[DEAL_MEMBERS];                // the part that holds a member's first k-step
};

// A group of `members` tiles dealt to `parts` workgroups so that each takes the same time, a segment costing F and its k-steps; false
// where a workgroup would have nothing to do or a segment would be too short to be worth its F.  The kernel relies on it: a part
// without k-steps would store to a plane in front of the partial sums.
inline bool deal_group(WgradDeal& d, double f, double step, int64_t steps, int members, int parts, int groups) {
  d = WgradDeal{};
  d.members = members;
  d.parts = parts;
  d.groups = groups;
  const double share = ((double)(members * steps) * step + (double)(parts + members - 1) * f) / (double)parts;
  double at = 0.0;
  for (int c = 0; c < parts; c++) {
    double left = share;
    while (left > f + DEAL_SHORTEST * step && at < (double)(members * steps)) {
      const double member_end = (double)steps * (double)((int64_t)(at / (double)steps) + 1), take = (left - f) / step;
      if (at + take > member_end - DEAL_SHORTEST) {           // up to the member's end
        left -= f + (member_end - at) * step;
        at = member_end;
      } else {
        at = (double)(int64_t)(at + take + 0.5);
        left = 0.0;
      }
    }
    d.bound[c + 1] = (int)at;
  }
  d.bound[parts] = (int)(members * steps);
  for (int c = 0; c < parts; c++)
    if (d.bound[c] >= d.bound[c + 1]) return false;
  for (int m = 0; m < members; m++) {
    int segments = 0;
    for (int c = 0; c < parts; c++) {
      const int64_t a = m * steps > d.bound[c] ? m * steps : d.bound[c], b = (m + 1) * steps < d.bound[c + 1] ? (m + 1) * steps : d.bound[c + 1];
      if (a >= b) continue;
      if (b - a < DEAL_SHORTEST) return false;
      if (!segments) d.first[m] = c;
      segments++;
    }
    if (segments > 15) return false;
    d.segments |= (uint32_t)segments << (4 * m);
  }
  return true;
}

inline int most_segments(const WgradDeal& d) {
  int most = 0;
  for (int m = 0; m < d.members; m++) most = (int)((d.segments >> (4 * m)) & 15u) > most ? (int)((d.segments >> (4 * m)) & 15u) : most;
  return most;
}

}  // namespace sste
