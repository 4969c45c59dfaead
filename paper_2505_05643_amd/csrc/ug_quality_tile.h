// Shape of the image-quality kernel's wave tile and the LDS places of its
// column sums, as plain constant expressions (no device code), so that the
// host can check every access against the array.
#pragma once

namespace ug {

constexpr int kQRad = 5, kQWin = 2 * kQRad + 1;
constexpr int kQCols = 64;                // input columns of a strip (a wave's lanes)
constexpr int kQOut = kQCols - 2 * kQRad; // output columns per strip
constexpr int kQRows = 4;                 // rows per step
constexpr int kQPer = 4;                  // neighbouring outputs per lane of the row pass
constexpr int kQPairs = (kQWin + kQPer - 1) / 2;  // pairs of column sums those outputs need
constexpr int kQPitch = 68;               // doubles per row of column sums in LDS

// LDS place of a pair of columns: the pairs of columns 32 and up swap with
// their neighbours, so that lanes eight groups of four apart read 16 bytes
// from different banks.
constexpr int q_pair(int pair) { return pair ^ ((pair >> 4) & 1); }

// The j-th pair (j < kQPairs) read by group og of kQPer outputs.  The groups
// behind the last output read the last group's pairs (their outputs are not
// kept): the highest pair read is 32, the row's 33rd.
constexpr int kQLastGroup = (kQOut - 1) / kQPer;
constexpr int q_read_pair(int og, int j) { return q_pair(2 * (og < kQLastGroup ? og : kQLastGroup) + j); }
static_assert(kQPitch % 2 == 0 && q_read_pair(64 / kQRows - 1, kQPairs - 1) < kQPitch / 2, "reads stay in the row");

}  // namespace ug
