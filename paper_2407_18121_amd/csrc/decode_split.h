// How a generation step's (batch, head) pairs are divided over workgroups.  Without HIP, so that the rules can be tested by themselves.
#pragma once

#include <algorithm>

#include "chip.h"

namespace ec {

// Workgroups of a divided launch per share: workgroups are handed to the XCDs in turn, and those of one pair have to meet.
constexpr int split_stride(int BH) { return (BH + kXcds - 1) / kXcds * kXcds; }

// Lines of a pair: its XCD's from first_line(row) on, one for each share but the owner's; row: number of the pair's output row, counted over
// all of memory.  The pairs of a launch that meet on one XCD have numbers eight apart, and their lines follow each other.
constexpr int kLines = 256;  // of every XCD
constexpr unsigned first_line(unsigned long long row, int splits) { return (unsigned)(row / kXcds) * (unsigned)(splits - 1) % kLines; }

// Workgroups that one (batch, head) is divided over when the caller leaves the choice to the library: as many as its XCD has
// compute units for, where that saves more than the exchange costs (2.6 us against 1 us per 54 KB of one (batch, head)'s rows).
// Measured, divided against one workgroup, % of the time, at KB of K and V of one pair (graph replay; bf16 D128, f32 D128, bf16 D64, f32 D64):
//   B*H =  8 (8 shares)   240 KB  +4  0  0 -5    260  -4 -8 -7 -10    300 -10 -15 -13 -17      4096 rows of bf16 D128 39 -> 10.7 us
//   B*H = 40 (6)          240 KB  +6 +3 +2  0    260  -2 -3 -4  -6    300  -7  -8  -8 -11
//   B*H = 48 (5)          240 KB  +6 +4 +5 +1    280   0 -4 -2  -6    300  -3  -6  -4  -9
//   B*H = 64 (4)          300 KB  +4 +2 +1  0    320   0 -3 -5  -5    360  -4  -6  -7  -9      4096 rows 43 -> 25
//   B*H = 72 (3)          320 KB  +3 +1 -1 -1    350  +1 -3 -1  -3    380  -1  -5  -3  -5
//   B*H = 80 (3)          350 KB  +5  0 +1 -1    380   0 -2 -1  -3    420  -2  -5  -6  -6
//   B*H = 84 (2)          420 KB  -2 -3 -4 -5    480  -5 -6 -6  -9    540  -7  -9  -8 -10      4400 rows 48 -> 35
//   B*H = 96 (2)          420 KB   0  0 +1 -2    480  -2 -3 -3  -5    512  -6  -6  -5  -9      4096 rows 51 -> 35
//   B*H = 128 (2)         700 KB  +4 +2 +3  0    850  +3 +2  0   0    960   0  +1 -2  -1      4096 rows 51 -> 47
// So from 240 KB on (bf16 D128: 256), and 3 KB more for every pair beyond 36, as there are fewer shares then; four shares not below 320
// KB, two 32 KB later, and beyond 96 pairs from 960.  The same kernel's divided launches differ by up to 5 % from one loading of the library to
// the next (B*H 8 and 16 most), undivided ones do not.
// All workgroups of a pair are on one XCD, so the fullest XCD sets the number: ceil(B*H / 8) pairs share its 32 compute units.  As many
// shares as the chip has units per pair, 256 / (B*H), put up to 36 workgroups there (45 with sixteen shares), and the last ones wait
// for a unit.  bf16 D128, so / by the fullest XCD / undivided:
//   B*H = 33: 2000 rows 13.0 / 11.1 / 21.2    4400 21.6 / 16.9 / 43.1    B*H = 41: 1030 rows 10.8 / 9.5 / 12.8    4400 24.5 / 19.4 / 43.8
//   B*H = 49: 1030 rows 11.6 / 10.3 / 13.0    4400 28.4 / 21.9 / 44.4    B*H = 84: 1030 rows 15.7 / 13.1 / 13.9   4400 46.5 / 34.7 / 47.8
//   B*H = 20: 3100 rows 13.1 / 11.2 / 30.7    4400 15.7 / 12.9 / 42.0    B*H = 28: 3100 rows 15.2 / 12.8 / 31.0   4400 19.0 / 15.5 / 42.8
// Sixteen shares instead of eight where an XCD has room for them: B*H = 8, bf16 1200 rows 8.3 / 8.8, 4096 rows (2 MB) 11.7 / 10.7, f32 4096 rows
// 16.5 / 13.0; ten, where three pairs share an XCD, are no better than eight: B*H = 24, 3100 rows 12.4 / 11.8.
inline int decode_auto_splits(int BH, int n_rows, int row_bytes, bool half)
{
    const long long bytes = 2LL * n_rows * row_bytes;
    const int room = kXcdUnits / (split_stride(BH) / kXcds);
    const int splits = std::min(room, room >= 16 && bytes >= 3 << 19 ? 16 : 8);
    const int least = half && row_bytes >= 256 ? 256 : 240;
    const int pays = BH > 96 ? 960 : std::max(splits == 4 ? 320 : 0, least + 3 * std::max(BH - 36, 0) + (splits == 2 ? 32 : 0));  // KB
    return splits >= 2 && bytes >= pays * 1024LL ? splits : 1;
}

}  // namespace ec
