// Rules of the matrix-core kernel that depend on numbers alone (host only; no
// HIP header, so that they compile for the CPU by themselves).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace mbtp {

constexpr int kMxStepChans = 64;   // channels of a step: four cells
constexpr int kMxMaxSteps = 8;     // most steps that share a partial sum

// Steps of all partial sums of ns steps; channels past the last are padding.
inline int mx_padded_steps(int C, int ns) {
  const int G = kMxStepChans * ns;
  return (C + G - 1) / G * ns;
}

// Delay spread of 16 adjacent DMs, in samples a channel.  The delays of the
// first DM are common to all rows (staging follows them), so a DM range that
// starts high spreads no more than one from zero.
inline double mx_spread(const int32_t* delays, int ndms, int C) {
  if (ndms < 2) return 0.0;
  const int32_t* last = delays + (int64_t)(ndms - 1) * C;
  int32_t m = 0;
  for (int c = 0; c < C; ++c) m = std::max(m, last[c] - delays[c]);
  return 16.0 * m / (ndms - 1) / C;
}

// Steps that share one partial sum.  A step's products grow with its shifts,
// which grow with the channels' distance from the partial sum's middle;
// collecting a partial sum through LDS costs the same whatever it spans (about
// three shifts' products, and half as much again for the extra barrier of
// single steps).  With the spread s, a step takes about 4.4 + 0.22 s (channels
// of the partial sum) shifts: within 0.2 of the counted 6.4, 8.5 and 13.0 for
// 1, 2 and 4 steps of the 1024-channel beam.  Beside that a step stages its
// channels and waits for them, as much as some 20 shifts, whether it holds
// channels or padding: 28 channels x 39 DMs x 67796 outputs of equal delays
// take 20, 29, 44 and 75 us in partial sums of 1, 2, 4 and 8 steps; 847 x 864 x
// 44838: 405, 356, 423 and 449 us.  Over 480 shapes of 48 to 4096 channels the
// choice is 0.6 % slower than the best one on average (without the 20: 2.2 %,
// and up to 1.47 times).  The first DM's delays left out: 6 % less over 89
// shapes that start at DM 20 or 100 (1219 channels x 5 DMs x 41962 outputs from
// DM 100: 54.9 -> 48.3 us).
inline int mx_steps(double s, int C) {
  int best = 1;
  double cost = 1e30;
  for (int ns = 1; ns <= kMxMaxSteps; ns *= 2) {
    const double shifts = std::max(4.0, 4.4 + 0.22 * s * kMxStepChans * ns);
    const double c = (20.0 + shifts + (ns == 1 ? 4.7 : 3.2 / ns)) * mx_padded_steps(C, ns);
    if (c < cost) best = ns, cost = c;
  }
  return best;
}

// Whether a launch of ndms DMs and nout outputs is faster on this kernel, in
// tiles of mx_bd DMs and mx_bt outputs, than on the packed-add kernel in tiles
// of u8_bd and u8_bt, with `units` tiles at a time on the GPU.  In us, fitted to
// both kernels' times: a tile costs this kernel its steps, full or not (about
// 4.1 us each, and 8 to start and end), the other one its channels (0.13 us
// each for a few DMs, 0.23 for whole blocks).  So a step needs some 30 channels
// to pay: 13 channels x 1 DM x 1143 samples 10.5 us here and 5.8 there, 20 x
// 505 x 28403 40.1 and 32.5, 66 x 3 x 1346 17.7 and 16.2, 64 x 1 x 6786 10.3
// and 12.6, 93 x 19 x 9081 16.0 and 20.4.  Over 810 launches of 4 to 4096
// channels, 1 to 2048 DMs and 100 to 130000 outputs the choice is 0.6 % slower
// than the better kernel on average, and more than 3 % slower than the
// packed-add kernel twice (8 and 6 %).
inline bool mx_pays(int C, int ndms, int64_t nout, int ns, int mx_bd, int mx_bt, int u8_bd, int u8_bt, int units) {
  auto rounds = [&](int bd, int bt) {
    const int64_t tiles = (int64_t)((ndms + bd - 1) / bd) * ((nout + bt - 1) / bt);
    return (double)((tiles + units - 1) / units);
  };
  const double steps = mx_padded_steps(C, ns), full = std::min(ndms, u8_bd) / (double)u8_bd;
  const double mx = 8.0 + 4.1 * steps + (rounds(mx_bd, mx_bt) - 1) * (5.0 + 3.0 * steps);
  const double u8 = 5.0 + C * (0.13 + 0.10 * full) + (rounds(u8_bd, u8_bt) - 1) * (3.0 + 0.20 * C);
  return mx < u8;
}

}  // namespace mbtp
