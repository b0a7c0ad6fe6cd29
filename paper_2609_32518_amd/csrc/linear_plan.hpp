// Which kernel and output tile a projection y = x W^T takes (host arithmetic only, no HIP, so that the
// CPU tests exercise it).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace unstep {

constexpr int kLinearBK = 64;              // k per step

// The output tile is bn columns of y (rows of W) by bm rows of y; staged: the register-staged kernel of
// 256 threads, else the direct-to-LDS one of 512.
struct LinearTile {
  int bn, bm;
  bool staged;
  int32_t tiles_n, tiles_m;
  bool fits;                               // the launch's work-items are fewer than 2^32
};

inline LinearTile linear_tile(int32_t M, int32_t N, int bn, int bm, bool staged) {
  const int64_t tn = (int64_t(N) + bn - 1) / bn, tm = (int64_t(M) + bm - 1) / bm;
  return {bn, bm, staged, int32_t(tn), int32_t(tm), tn * tm <= int64_t(UINT32_MAX) / (staged ? 256 : 512)};
}

// Time of one 64-wide k step over the whole launch (us): every round of 256 work-groups takes at least
// `step` and the operand bytes of all tiles move at `tbps` together.
inline double linear_step_us(const LinearTile& t, double step, double tbps) {
  const double tiles = double(t.tiles_n) * double(t.tiles_m);
  return std::max(std::ceil(tiles / 256) * step, tiles * (t.bn + t.bm) * (kLinearBK * 2) / (tbps * 1e6));
}

// While 32-bit offsets address a tile's rows: the direct-to-LDS kernel, with the tile size that the
// measured rates put first (fixed costs of ~3 us are the same for all, so K only scales the
// comparison) among those whose launch fits.  Otherwise (longer rows, or none of them fits) the
// register-staged kernel; `fits` is false when that does not fit either.
inline LinearTile linear_plan(int32_t M, int32_t N, int32_t K) {
  LinearTile best = linear_tile(M, N, 128, 128, true);
  if (int64_t(256) * K * 2 >= (int64_t(1) << 31)) return best;
  struct {
    int bn, bm;
    double step, tbps;
  } const sizes[] = {{128, 256, 0.63, 12.3}, {128, 128, 0.31, 12.0}, {64, 128, 0.23, 14.5}, {64, 64, 0.155, 18.5}};
  double best_us = INFINITY;
  for (const auto& s : sizes) {
    const LinearTile t = linear_tile(M, N, s.bn, s.bm, false);
    const double us = linear_step_us(t, s.step, s.tbps);
    if (!t.fits || us >= best_us) continue;
    best = t;
    best_us = us;
  }
  return best;
}

}  // namespace unstep
