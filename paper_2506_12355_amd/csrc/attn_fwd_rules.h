// Which instance of the attention kernel a call runs, from its shape, type and mask
// and the device's CU count: host code only.
#pragma once

#include <limits.h>

#include "attn_fwd_launch.h"

namespace qm {

// Key groups of a workgroup (1, 2 or 4) that a call runs with on a device of
// `cus` CUs.  A function of the shape, type and mask alone: not of tile_rows or
// layout, on which results do not depend.  (They do depend on the groups, whose
// sums are taken apart: a sequence's bytes in a small batch and in a large one, or
// on devices with other CU counts, differ within the rounding of the sums.)
inline int key_groups(const AttnArgs& a, int cus) {
  if (a.d == 192) return 1;
  // Workgroups of query blocks of `rows` rows, causal ones in pairs where they
  // are too many to stay single: from N = 4096 on (us, unsplit -> split, N = 4096
  // H = 16 and N = 8192 H = 8: d = 128 75.9 -> 74.4, 137 -> 133; d = 64 52.2 -> 47.5,
  // 92.1 -> 82.6; FP8 47.9 -> 46.8, 83.7 -> 80.7).  Up to N = 2048 pairs lose
  // (d = 128 N = 1000 H = 64 24.8 -> 28.4, N = 2048 H = 24 35.9 -> 37.3, FP8
  // 25.5 -> 29.1); between the two they would gain 0-4% (d = 128 N = 3000 H = 16
  // 49.7 -> 47.6) to 15% (d = 64 40.5 -> 35.2).
  const auto fits = [&](int rows) {
    const long long nq = (a.N + rows - 1) / rows;
    const long long heads = (long long)a.B * a.H;
    return nq * heads <= cus || (a.causal && a.N >= 4096 && (nq + 1) / 2 * heads <= cus);
  };
  // All query blocks in one round of one workgroup per CU: in two rounds the
  // split loses to two unsplit workgroups per CU (0.6-0.9x).  Below these
  // lengths the merge (about 1 us) outweighs the steps saved; each line lies
  // between the sizes named (us, unsplit -> split, B = 1, unmasked unless
  // causal is said):
  //   four groups: d = 64 N = 256 H = 8 6.05 -> 6.57, N = 512 8.31 -> 7.93;
  //   FP8 N = 256 7.05 -> 7.67, N = 512 9.20 -> 8.91;
  //   two groups, d = 64: N = 512 H = 64 9.07 -> 9.76, N = 1024 H = 32
  //   13.5 -> 13.0; causal N = 512 H = 64 10.3 -> 10.5, N = 1000 H = 32
  //   15.3 -> 13.8;
  //   two groups, d = 128: N = 1024 H = 16 17.5 -> 17.8, N = 2048 H = 8
  //   29.2 -> 27.0 (causal calls would gain a little sooner: N = 512 H = 32
  //   13.3 -> 13.7, N = 1000 H = 16 18.6 -> 17.9, H = 32 19.7 -> 19.5).
  if ((a.d == 64 || a.dtype == 2) && a.N >= 384 && fits(64)) return 4;
  if (a.N >= (a.d == 64 ? 768 : 1536) && fits(128)) return 2;
  return 1;
}

// Eight waves keep K/V tiles in LDS for the most rows; four let one workgroup's
// prologue and epilogue run beside another's key loop, which wins where
// workgroups are short, and where the 256-row tiles, dealt out in rounds over
// the CUs, would leave too many of them idle.
inline int choose_waves(const AttnArgs& a, int cus) {
  const auto tiles = [&](int rows) {
    const long long nq = (a.N + rows - 1) / rows;
    return (a.causal ? (nq + 1) / 2 : nq) * a.B * a.H;
  };
  // 192-wide keys run one workgroup of either size per CU: four waves where all
  // of theirs run at once (H = 16 N = 4096 causal 104.8 -> 85.6 us; in two
  // rounds, H = 8 N = 8192 unmasked, 270 -> 300).  Short causal pairs gain
  // nothing (H = 128 N = 512 23.5 -> 23.9), single query blocks do.
  if (a.d == 192) {
    const long long blocks = (long long)((a.N + 127) / 128) * a.B * a.H;
    return blocks <= cus || (a.N >= 768 && tiles(128) <= cus) ? 4 : 8;
  }
  // Short sequences, us, 256 -> 128 rows at a full grid: d = 128 bf16 N = 1024
  // 133 -> 131, N = 2048 233 -> 238, causal 145 -> 142, N = 4096 440 -> 457 and
  // 247 -> 247; d = 64 N = 2048 146 -> 138, N = 4096 274 -> 267, causal
  // 156 -> 150; FP8 N = 4096 282 -> 280, causal 165 -> 161.
  if (a.N <= (a.d == 64 || a.dtype == 2 ? 4096 : a.causal ? 2048 : 1024)) return 4;
  // Longer ones: a 256-row tile takes its CU 20 units of time, two 128-row
  // tiles side by side 21, a 128-row tile that has a CU to itself 14.  (B=3 H=32
  // N=3000: 392 -> 375 us, causal 257 -> 233; B=1 H=24 N=4096 causal, whose
  // 192 tiles of 256 rows fill 192 CUs: 104 us with them, 109 with 384 halves.)
  // (Where these costs say 1.05, two 128-row tiles for one of 256, 672 shapes beyond
  // N = 4096 took 0.97-1.16 times as long: in the mean 1.06 at d = 128, 1.09 at d = 64,
  // 1.03 with FP8.)
  // An odd number of causal query blocks leaves each head's middle one without a
  // partner, half a tile.  Where the tiles past the last whole round are such ones only
  // (the last of an XCD's whole heads), that round takes half as long.  H = 8 N = 8256,
  // 264 tiles of 128 rows: 256 -> 128 rows, d = 128 163.8 -> 142.8 us, d = 64
  // 118.6 -> 93.7, FP8 126.4 -> 87.8; H = 24 N = 5376, 264 tiles of 256 rows: FP8
  // 140.1 -> 97.2.  After a round of two 128-row tiles beside one another that holds at
  // d = 64 only, where a third fits beside them: H = 8 N = 16500, 264 and 520 tiles,
  // d = 64 311 -> 299, but d = 128 502 -> 530, FP8 296 -> 311.
  const auto half_units = [&](int rows, int alone, int beside) {   // beside: two on a CU
    const long long n = tiles(rows), left = n % cus, full = n / cus;
    const bool singles = a.causal && (a.N + rows - 1) / rows % 2 &&
                         (long long)a.B * a.H % kXcds == 0 && left <= kXcds &&
                         (rows == 256 || full % 2 || a.d == 64);
    const long long last = left == 0 ? 0 : full % 2 ? beside - alone : alone;
    return 2 * (full / 2 * beside + full % 2 * alone) + (singles ? last : 2 * last);
  };
  return half_units(128, 14, 21) < half_units(256, 20, 40) ? 4 : 8;
}

// Workgroups of a launch over `total` tiles: as many as are `resident` at once, each
// walking tiles in turn (rounds of `resident` tiles), or one per tile.
//
// Persistent workgroups save their set-up, but a CU keeps the tiles it was dealt.  With
// one workgroup per tile the CU that is free first takes the next, which evens out what
// two FP8 workgroups side by side make of their shares; only where the last round has at
// most one tile to a CU, that gives some CUs two of them and others none.  us, persistent
// -> one per tile, two per CU: last round above one per CU, N = 4096 H = 104 unmasked
// 468 -> 447, N = 2048 H = 120 144.0 -> 139.7, causal N = 3582 H = 136 268.9 -> 256.9;
// at most one, N = 4096 H = 64 unmasked 274 -> 272 but causal N = 1536 H = 211
// 87.5 -> 92.4, N = 2560 H = 112 119.9 -> 124.9.  Short tiles are bound by their set-up
// (N = 256 H = 496 20.8 -> 22.8), and one workgroup per CU gains 2-3% from staying.
inline int tile_grid(int total, int resident, int cus, int per_cu, int threads, int dtype, int N) {
  if (resident < kXcds || total <= resident) return total;
  const int last = total % resident;
  if (dtype == 2 && per_cu > 1 && N > 1000 && (last == 0 || last > cus) &&
      total <= INT_MAX / threads)   // as many as a grid takes
    return total;
  return resident;
}

}  // namespace qm
