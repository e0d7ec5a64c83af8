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
// many points of 128 bf16 channels (forward, 3x5x5 and 3x7x7: 2x6x6, 1 head 52 / 23 and 98 / 40 us,
// 4x8x8, 2 heads 54 / 23 and 101 / 44, 4x14x21, 2 heads 116 / 46 and 221 / 87) and for rows of 32
// fp32 channels, eight to a load (3x3x3, 3x5x5 and 3x7x7: 2x6x6, 1 head 16.5 / 13.1, 39 / 19 and 73 /
// 32, 4x8x8, 2 heads 17.1 / 13.0, 40 / 19 and 73 / 34, 4x14x21, 2 heads 17.6 / 20.8, 40 / 36 and 74 /
// 69, 6x16x16, 4 heads 29.5 / 27.2, 74 / 48 and 140 / 93); of these, up to 32 points gather from
// kFewRows32 to kSlotRows32 rows (3x12x20, 2 heads 17.4 / 21.8).
constexpr int64_t kSlotRows = 16384;
constexpr int64_t kFewRows32 = 1024, kSlotRows32 = 4096;

constexpr bool few_rows(int D, bool bf16, int64_t rows, int P) {
  if (D <= 32) return P <= 2 * kSlotLanes && rows >= kFewRows32 && rows < kSlotRows32;
  return !(bf16 && D == 128 && P > 2 * kSlotLanes) && rows < kSlotRows;
}

// The predicted-weights variant reads V only, half of what sharing saves: 64 bf16 channels, 64x34x60,
// 16 heads, 3x3x3: 2.40 ms gathering, 2.45 by slots.  (The kernels that a rule never selects are not
// built.)
constexpr bool pw_two_rounds_ok(int D, bool bf16) { return slot_rows_ok(D, bf16) && !(bf16 && D == 64); }

constexpr int forward_rounds(int D, bool bf16, int64_t rows, int P, bool pw) {
  if (!slot_rows_ok(D, bf16) || P < kSlotLanes || few_rows(D, bf16, rows, P)) return 0;
  if (pw && P <= 2 * kSlotLanes && !pw_two_rounds_ok(D, bf16)) return 0;
  return P <= 2 * kSlotLanes ? 2 : 5;
}

// The backward sweeps the slots three times and counts the compact tiles on their own, so it needs
// larger rows or more points.  V pass + K pass, gathering and by slots, N(0, 1) offsets: 128 bf16
// channels, 16x34x60, 24 heads: 1x3x3 1.92 / 2.49 ms, 3x3x3 4.58 / 3.90, 3x5x5 11.9 / 8.5, 3x7x7
// 22.9 / 18.0; 64 bf16 channels, 16 heads: 3x5x5 5.14 / 5.10, 3x7x7 10.2 / 11.1; 64 fp32
// channels, 9x33x47, 6 heads: 3x3x3 0.84 / 0.84 (two batch items), 3x5x5 1.14 / 0.93, 3x7x7 2.28 /
// 2.03.
constexpr bool backward_slots_ok(int D, bool bf16) { return slot_rows_ok(D, bf16) && !(bf16 && D == 64); }

constexpr int backward_rounds(int D, bool bf16, int64_t rows, int P) {
  if (!backward_slots_ok(D, bf16) || few_rows(D, bf16, rows, P)) return 0;
  if (P <= 2 * kSlotLanes) return bf16 && P >= kSlotLanes ? 2 : 0;
  return 5;
}

// Spread of a compact wave (compact_wave): the largest box of voxels that the points of one of its
// queries may span.  Offsets N(0, 1) span about 440 voxels at 3x3x3, 800 at 3x5x5 and 1100 at 3x7x7
// (the largest of four queries), U[-2, 2] 340, 570 and 850, U[-3, 3] 730, 1090 and 1500, U[-4, 4]
// 1250, 1860 and 2480; beside the grid's faces less.
// Where the points of most waves span about that much, ms gathering / by slots (grids 16x34x60 with
// 24 heads x 128 bf16, 16x32x32 with 8 x 64 bf16, 2 x 9x33x47 with 6 heads of 64 or 32 fp32):
//   forward        3x3x3 U[-3, 3]   3x3x3 U[-4, 4]   3x5x5 U[-3, 3]   3x7x7 U[-3, 3]
//   128 bf16       2.84 / 2.00      2.84 / 2.43      7.32 / 5.03      14.2 / 11.3
//   64 fp32        0.547 / 0.551    0.542 / 0.623    1.56 / 1.29      3.09 / 2.97
//   64 bf16        0.236 / 0.283    0.236 / 0.280    0.620 / 0.658    1.30 / 1.50
//   32 fp32        0.307 / 0.337    0.304 / 0.335    0.830 / 0.809    1.80 / 1.84
//   backward (all phases)
//   128 bf16       6.53 / 6.40      6.44 / 6.59      17.1 / 16.2      32.5 / 32.3
//   64 fp32                                          3.93 / 4.21      7.78 / 8.92
// and N(0, 1): forward 128 bf16 2.85 / 1.51, 7.28 / 3.26 and 14.1 / 6.67 (3x3x3, 3x5x5, 3x7x7), 64
// bf16 0.236 / 0.231, 0.618 / 0.454 and 1.30 / 0.94; backward 128 bf16 6.57 / 5.64, 17.3 / 13.4 and
// 32.5 / 27.2, 64 fp32 4.02 / 3.64 (3x5x5) and 8.03 / 7.46.  At U[-8, 8] every wave gathers.
constexpr int forward_box(int D, bool bf16, int P) {
  const bool small = D * (bf16 ? 2 : 4) == 128;  // 128-byte rows
  if (P <= 2 * kSlotLanes) return small ? 550 : bf16 ? 1500 : 700;
  return P <= 5 * kSlotLanes ? (small ? 1000 : bf16 ? 1600 : 1350) : small ? 1300 : 1600;
}
constexpr int backward_box(bool bf16, int P) {
  if (P <= 2 * kSlotLanes) return 1000;
  return P <= 5 * kSlotLanes ? (bf16 ? 1150 : 900) : bf16 ? 1350 : 1200;
}

}  // namespace dsa3d
