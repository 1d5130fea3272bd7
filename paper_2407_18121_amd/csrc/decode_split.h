// How a generation step's (batch, head) pairs are divided over workgroups.  Without HIP, so that the rules can be tested by themselves.
#pragma once

#include <algorithm>

#include "chip.h"

namespace ec {

// Workgroups of a divided launch per share: workgroups are handed to the XCDs in turn, and those of one pair have to meet.
constexpr int split_stride(int BH) { return (BH + kXcds - 1) / kXcds * kXcds; }

// Workgroups that one (batch, head) is divided over when the caller leaves the choice to the library: as many as its XCD has
// compute units for, where that saves more than the exchange costs (2.6 us against 1 us per 54 KB of one (batch, head)'s rows).
// Measured, us per launch (graph replay, D128, one workgroup / divided; crossover):
//   bf16, B*H =  8:  450 rows 7.1 / 7.1     550 8.0 / 7.6   4096 39.3 / 10.7     f32  220 rows 6.7 / 6.7   260  7.7 / 7.1   4096 75.0 / 13.0
//   bf16, B*H = 32:  500 rows 7.7 / 7.8     640 9.2 / 8.1   4096 40.6 / 15.9     f32  230 rows 7.4 / 7.3   260  8.0 / 7.7   4096 77.8 / 25.1
//   bf16, B*H = 64:  600 rows 9.1 / 9.4     700 10.0 / 9.8  4096 42.7 / 25.2     f32  250 rows 8.3 / 8.8   300  9.8 / 9.3
//   bf16, B*H = 96:  800 rows 11.6 / 12.2  1200 16.0 / 14.9 4096 51.0 / 35.3     f32  550 rows 14.8 / 14.6
//   bf16, B*H = 128: 1600 rows 22.9 / 22.4 2400 33.1 / 31.2 4096 51.0 / 46.8     f32 1000 rows 28.0 / 26.5
// All workgroups of a pair are on one XCD, so the fullest XCD sets the number: ceil(B*H / 8) pairs share its 32 compute units.  As many
// shares as the chip has units per pair, 256 / (B*H), put up to 36 workgroups there (45 with sixteen shares), and the last ones wait
// for a unit.  bf16 D128, so / by the fullest XCD / undivided:
//   B*H = 33: 2000 rows 13.0 / 11.1 / 21.2    4400 21.6 / 16.9 / 43.1    B*H = 41: 1030 rows 10.8 / 9.5 / 12.8    4400 24.5 / 19.4 / 43.8
//   B*H = 49: 1030 rows 11.6 / 10.3 / 13.0    4400 28.4 / 21.9 / 44.4    B*H = 84: 1030 rows 15.7 / 13.1 / 13.9   4400 46.5 / 34.7 / 47.8
//   B*H = 20: 3100 rows 13.1 / 11.2 / 30.7    4400 15.7 / 12.9 / 42.0    B*H = 28: 3100 rows 15.2 / 12.8 / 31.0   4400 19.0 / 15.5 / 42.8
// Sixteen shares instead of eight where an XCD has room for them: B*H = 8, bf16 1200 rows 8.3 / 8.8, 4096 rows (2 MB) 11.7 / 10.7, f32 4096 rows
// 16.5 / 13.0; ten, where three pairs share an XCD, are no better than eight: B*H = 24, 3100 rows 12.4 / 11.8.
inline int decode_auto_splits(int BH, int n_rows, int row_bytes)
{
    const long long bytes = 2LL * n_rows * row_bytes;
    const int room = kXcdUnits / (split_stride(BH) / kXcds);
    const int splits = std::min(room, room >= 16 && bytes >= 3 << 19 ? 16 : 8);
    const int pays = splits >= 5 ? 240 << 10 : splits >= 3 ? 320 << 10 : BH <= 96 ? 512 << 10 : 960 << 10;
    return splits >= 2 && bytes >= pays ? splits : 1;
}

}  // namespace ec
