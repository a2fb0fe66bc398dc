// Score rows as the scoring kernels stage them in LDS: bytes of a row's planes and from row to row.  (Plain C++: a test compiles it too.)
#pragma once

namespace laq {

// A 128-bit read of 64 lanes is worked off 16 lanes at a time, over 64 banks of 4 bytes: lanes 0 .. 3, 12 .. 15 and 20 .. 27 of each half wave together, then the
// others.  What a row has beside its planes keeps these 16 pieces in different banks:
//   tiles of 32 x 32: lane l reads row l % 32, piece l / 32: an odd number of 16 bytes from row to row
//   tiles of 16 x 16: lane l reads row l % 16, piece l / 16: an odd number of 32 bytes (with 16, piece 1 of row 11 lies in the banks of piece 0 of row 12: 4 cycles
//     more for each read of 8; SQ_LDS_BANK_CONFLICT of the first two-pass kernel, 67 heads x 2042 keys, 128 rows, 549 000 : 0)
constexpr int ROW32_PAD = 16, ROW16_PAD = 32;

// bytes of d bf16 in whole steps of 16, 32 elements
constexpr int plane_bytes(int d) { return (d + 15) / 16 * 32; }
constexpr int plane16_bytes(int d) { return (d + 31) / 32 * 64; }
// `planes` of them (a float has three) and the rest
constexpr int staged_row(int d, int planes) { return planes * plane_bytes(d) + ROW32_PAD; }
constexpr int staged_row16(int d, int planes) { return planes * plane16_bytes(d) + ROW16_PAD; }

}  // namespace laq
