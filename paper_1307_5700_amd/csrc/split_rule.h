// Which launches the split kernel takes from the tiled one: numbers alone (host
// only; no HIP header, so that it compiles for the CPU by itself).
#pragma once

#include <stdint.h>

namespace mbtp {

// Whether a launch of C channels and ndms DMs is faster on the split kernel, in
// `split` of its tiles, than on the tiled one, in `tiles` of bd DMs, on `units`
// compute units.  bytes: of a sample; ring: with ring samples.
//
// Tiles that leave units without work take as long as one tile, 0.32 us a channel
// for 48 DMs and 0.20 to 0.25 for a few of them or for the narrower tiles that
// wide spreads leave.  The split kernel's time grows with its tiles: 0.06 us a
// channel for each per unit, 0.08 to 0.1 with ring samples or a wide spread.  So
// at most four per unit (1024 channels x 120 DMs x 16384 samples, 3.5 a unit: 228
// against 323 us; 1024 x 200, 5.7: 357 against 330), three with ring samples (768
// x 100, 3.25, cleaned: 253 against 279; 1024 x 240, 3.75: 377 against 376), two
// for narrower tiles (1024 x 240 at 1 DM a step, 1.2: 114 against 194).
//
// A row is staged once per 8 DMs here and once per 48 there, which up to 32 DMs
// of f32 or f16 rows makes three per unit the most (865 x 11 x 107108 in f32,
// 3.3: 229 against 189 us; 3438 x 10 x 83000 in f16, 2.5: 511 against 731), two
// up to 160 channels, whose workgroups are small (132 x 12 x 76106, 2.3: 40 against
// 36; 2.0 at most: 0.98 or less of the tiled time).  8-bit rows keep four (910 x
// 11 x 103585, 3.2, cleaned: 194 against 263).
//
// One or two channel groups leave nothing to split (32 channels: 17 against 11
// us; 64: 18 either way; 128: 16 against 35) and a third that is half empty
// little: up to 80 channels one tile per unit with ring samples or few DMs (73 x
// 214 x 5464, 2.3: 44 against 37 us; 71 x 15 x 101048, 3.1: 31 against 27).
//
// Over 1400 launches of 65 to 4096 channels and 1 to 500 DMs one is more than 2 %
// slower than the tiled kernel (4 %).
inline bool split_pays(int C, int ndms, int bytes, bool ring, int bd, int64_t tiles, int64_t split, int units) {
  if (C <= 64 || tiles > units) return false;
  const bool thin = ndms <= 32 && bytes > 1;
  int per_unit = bd < 48 ? 2 : (ring ? 3 : 4);
  if (!ring && thin && bd >= 48) per_unit = C <= 160 ? 2 : 3;
  if (C <= 80 && (ring || thin)) per_unit = 1;
  return split <= (int64_t)per_unit * units;
}

}  // namespace mbtp
