// Tile shapes of the matrix-core contraction (k_cgemm.hip) and the choice among
// them. Plain C++17 with no HIP dependency, so the host test suite can compile
// it with g++ and see which shape a layer takes.
#pragma once

#include <algorithm>
#include <cmath>

namespace oaa {

constexpr int kMfmaSlice = 16;  // reduction depth of one LDS slice

// Rows and columns of a tile, and the tiles a CU holds by LDS and registers
// (32 x 32 by LDS: its registers leave five).
struct MfmaTileShape {
  int tm, tn, occ;
};
constexpr MfmaTileShape kMfmaTiles[] = {
    {16, 64, 5}, {16, 128, 2}, {64, 16, 5}, {32, 32, 6},  {32, 64, 4},  {64, 32, 4},  {64, 64, 3},
    {96, 64, 2}, {64, 96, 2},  {128, 64, 2}, {96, 96, 2}, {128, 96, 1}, {96, 128, 1}, {128, 128, 1},
};

// Estimated time (ns) of F contractions of M x N results over Kr, in nsplit
// ranges of kchunk, on tiles of one shape: the larger of
//  * a CU's work on its tiles (matrix products of the slices; the split of the
//    operands, 12 vector instructions per element; a barrier per slice; the
//    result stores);
//  * the chain of one tile (a load's latency per slice, its products and
//    stores), times the rounds of resident tiles on 256 CUs.
// The rates are a fixed calibration against sweeps over the tile shapes: the
// large-kernel layer, 128 channels at 56 x 56, and layers of 5 to 138 channels.
// Within it the shapes rank as they measured, in us with the launch: 64 x 144 x
// 64 over 130 bins, 64 x 32 tiles 9.4 (estimated 6.0), 64 x 64 9.5 (7.5),
// 64 x 96 11.9 (8.9), 128 x 64 13.4 (10.3); 48 x 64 x 64 over 514 bins, 64 x 64
// 12 (8.2), 32 x 64 13 (9.5), 96 x 64 18 (11.6); 256 x 288 x 96 over 2050 bins,
// 128 x 96 779 (730), 128 x 64 814 (842), 96 x 96 821 (834), 64 x 64 1030 (917).
inline double mfma_estimate(int M, int N, int Kr, int kchunk, int nsplit, int F, const MfmaTileShape& s) {
  const int TM = s.tm, TN = s.tn, occ = s.occ;
  const double tiles = double((M + TM - 1) / TM) * ((N + TN - 1) / TN) * nsplit * F;
  const double slices = (std::min(Kr, kchunk) + kMfmaSlice - 1) / kMfmaSlice;
  const double area = double(TM) * TN;
  const double work = slices * (0.149 * area + 1.3 * (TM + TN) + 60) + 0.15 * area + 100;
  // 512 lanes (a CU to themselves) have half the products and stores per wave,
  // and part of a round is half as good for them
  const double lane = occ == 1 ? 0.5 * area : area;
  const double chain = slices * (0.1 * lane + 900) + 0.3 * lane + 1000;
  const double rounds = occ == 1 ? 0.5 * (tiles / 256 + std::ceil(tiles / 256)) : tiles / 256;
  return std::max(std::max(1.0, rounds) * work, std::ceil(tiles / (256 * occ)) * chain);
}

// Index of the shape with the least estimated time.
inline int mfma_tile_choice(int M, int N, int Kr, int kchunk, int nsplit, int F) {
  int best = 0, i = 0;
  double least = 0;
  for (const MfmaTileShape& s : kMfmaTiles) {
    const double t = mfma_estimate(M, N, Kr, kchunk, nsplit, F, s);
    if (i == 0 || t < least) {
      best = i;
      least = t;
    }
    ++i;
  }
  return best;
}

}  // namespace oaa
