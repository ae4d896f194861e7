// Order of the 256 x 256 tiles of a product with a packed weight.  Plain C++, so that the host can check it by itself.
#pragma once
#include <stdint.h>

namespace sste {

// `runs` runs of weight tiles (of 256 channels or features), each with all of its
// token tiles before the next run's; inside a run the weight's tiles run fastest.  A run of about ten where the weight has 18 tiles or more: an
// XCD goes through the tiles of a run again in every round, and half of a weight 5120 wide stays in its 4 MB of L2 (or more of it
// does) where the whole does not.  Random products of 256 x 256 tiles, against one run, geometric mean (worst): 18 ... 20 tiles and more than a
// round of them, forward 8-bit 4.1 % faster (1.5 % faster), bf16 equal (1.1 % slower), input gradient 0.8 / 1.2 % faster (0.5 % slower); 42 ...
// 73 tiles 4.6 % faster (0.4 % slower), 74 ... 256 tiles 5.6 % faster (0.3 % slower).  Below 18 tiles two runs gain nothing, below 10 they lose up to
// 14 %, a round's tiles then being far from square.  32768 x 5120 x 1280 e4m3 forward 153.4 -> 146.3 us, 16384 x 1280 x 5120 bf16 input gradient
// 181.3 -> 177.9.  Fetched from memory by a forward product of a block of width 1280 (mean of its four): e4m3, 32768 tokens 200 -> 145 MB, bf16, 16384
// tokens 277 -> 230 MB.
// Up to 73 tiles there are at most four runs, of up to 18 tiles: runs of ten are as fast on the mean and up to 2.5 % slower on 8-bit products of few
// k-steps.  Four for every weight, of up to 64 tiles, lost beyond (3.7 % slower than one run at worst, 3000 x 65536 x 5120 bf16 forward 1119 us against
// 988).  More than 256 tiles are not measured; from 64 runs on they get wider, which keeps the products below in 32 bits.
struct TileOrder {
  int m_tiles, n_tiles, runs;
};
constexpr TileOrder tile_order(int64_t m_tiles, int64_t n_tiles) {
  const int64_t runs = m_tiles >= 18 && m_tiles * n_tiles > 256 ? (m_tiles + 2) / 10 : 1, most = m_tiles <= 73 ? 4 : 64;
  return {(int)m_tiles, (int)n_tiles, (int)(runs < most ? runs : most)};
}
// One run needs one division, several need five, which a workgroup does before its first load: 5888 x 688 x 2944 e4m3 input gradient (296 workgroups)
// 25.6 us with the one, 26.2 with the five.
constexpr void tile_at(const TileOrder& o, int logical, int& tm, int& tn) {
  if (o.runs == 1) {
    tm = logical % o.m_tiles;
    tn = logical / o.m_tiles;
    return;
  }
  const int b = ((logical / o.n_tiles + 1) * o.runs - 1) / o.m_tiles;     // run b: weight tiles first .. first + width - 1
  const int first = b * o.m_tiles / o.runs, width = (b + 1) * o.m_tiles / o.runs - first;
  const int r = logical - first * o.n_tiles;
  tm = first + r % width;
  tn = r / width;
}

}  // namespace sste
