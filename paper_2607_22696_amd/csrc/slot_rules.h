// Where the query-owned kernels take a tile's points by distinct voxels (dsa3d_slots.h) and where
// they load every corner: the rules of the dispatch, by row size, points and rows.
//
// Plain C++ (no HIP types), so that a host test can ask which code a call takes.
#pragma once

#include <stdint.h>

namespace dsa3d {

constexpr int kSlotQueries = 4;  // queries per wave, neighbours along x
constexpr int kSlotLanes = 16;   // lanes (points of a round) per query

// Whether the slots are built for rows of D channels: 128 or 256 bytes, 8 or 16 lanes of a load.
constexpr bool slot_rows_ok(int D, bool bf16) {
  return D * (bf16 ? 2 : 4) == 128 || D * (bf16 ? 2 : 4) == 256;
}

// Rounds that a kernel instance numbers together (0: every tile gathers) for rows of P points.
// Numbering costs a wave the same for 9 points as for 16, which a 1x3x3 kernel does not earn
// back: forward, 24 heads, gathering / by slots: 64 bf16 channels, 16x34x60 0.63 / 0.90 ms; 128
// channels, 16x34x60 1.14 / 1.06, 3x21x96 (2 heads) 19 / 24 us.  A grid of few rows waits for one
// wave's sweeps, which are a longer chain than the points' (4x14x21, 2 heads, forward: 64 fp32
// channels 3x3x3 57 / 82 us, 3x5x5 119 / 144; 64 bf16 3x3x3 39 / 64, 3x7x7 122 / 194) except for
// rows of 32 fp32 channels, eight to a load (4x8x8, 3x3x3 17 / 11), and many points of 128 bf16
// channels (4x14x21, 3x7x7 238 / 207).
constexpr int64_t kSlotRows = 16384;

constexpr bool few_rows(int D, bool bf16, int64_t rows, int P) {
  return D > 32 && !(bf16 && D == 128 && P > 2 * kSlotLanes) && rows < kSlotRows;
}

// The predicted-weights variant reads V only, half of what sharing saves: 64 bf16 channels, 64x34x60,
// 16 heads, 3x3x3: 2.40 ms gathering, 2.45 by slots.
constexpr int forward_rounds(int D, bool bf16, int64_t rows, int P, bool pw) {
  if (!slot_rows_ok(D, bf16) || P < kSlotLanes || few_rows(D, bf16, rows, P)) return 0;
  if (pw && bf16 && D == 64 && P <= 2 * kSlotLanes) return 0;
  return P <= 2 * kSlotLanes ? 2 : 5;
}

// The backward sweeps the slots three times and counts the compact tiles on their own, so it needs
// larger rows or more points.  V pass + K pass, gathering and by slots, N(0, 1) offsets: 128 bf16
// channels, 16x34x60, 24 heads: 1x3x3 1.92 / 2.49 ms, 3x3x3 4.58 / 3.90, 3x5x5 11.9 / 8.5, 3x7x7
// 22.9 / 18.0; 64 bf16 channels, 16 heads: 3x5x5 5.14 / 5.10, 3x7x7 10.2 / 11.1; 64 fp32
// channels, 9x33x47, 6 heads: 3x3x3 0.84 / 0.84 (two batch items), 3x5x5 1.14 / 0.93, 3x7x7 2.28 /
// 2.03.
constexpr int backward_rounds(int D, bool bf16, int64_t rows, int P) {
  if (!slot_rows_ok(D, bf16) || (bf16 && D == 64) || few_rows(D, bf16, rows, P)) return 0;
  if (P <= 2 * kSlotLanes) return bf16 && P >= kSlotLanes ? 2 : 0;
  return 5;
}

// Spread of a compact tile (compact_tile).  Offsets U[-3, 3] span about 700 voxels at 3x3x3 and 1090
// at 3x5x5, U[-4, 4] 1250 and 1770.  16x34x60 (fp32: 9x33x47), gathering / by slots.  Forward: 24 x
// 128 bf16, 3x3x3 U[-4, 4] 2.88 / 2.34 ms, 3x5x5 U[-3, 3] 7.32 / 4.64, U[-4, 4] 7.48 / 7.13; 16 x 64
// bf16, 3x3x3 U[-3, 3] 1.02 / 1.05, U[-4, 4] 1.07 / 1.21; 6 x 64 fp32, 3x3x3 U[-4, 4] 0.30 / 0.37.
// Backward, V pass + K pass: 24 x 128 bf16, 3x3x3 U[-3, 3] 4.68 / 4.50, U[-4, 4] 4.62 / 5.21, 3x5x5
// U[-3, 3] 12.0 / 12.0, U[-4, 4] 12.0 / 13.0.
// 16 x 64 bf16, 3x7x7 N(0, 1) by slots: 3.68 ms with 1000, 3.36 with 1500.
constexpr int forward_box(int D, bool bf16, int rounds) {
  return (bf16 && D == 128) || rounds > 2 ? 1500 : 1000;
}
constexpr int kBackwardBox = 1000;

}  // namespace dsa3d
