// Which kernels a scoring call runs on.  Host code without HIP, so that the rule can be tested by itself.
#pragma once

#include <stdint.h>

#include "../../include/ec.h"

namespace ec {

enum class ScoreRoute { kMfma = 0, kF32 = 1, kSimt = 2, kMfmaOffGrid = 3 };

// The matrix-core kernels move tiles through buffer descriptors, whose length and byte offsets have 32 bits and cover one
// head: all its rows and the ones that a prefetch asks for behind the last row (at most 384; the descriptor answers
// those, as long as the offset does not wrap around to the head's first rows).
constexpr long long kDescriptorBytes = 1LL << 32, kRowsBehind = 1024;

// rows: of one head's K and V, at least as many as Q has.  The vector kernels index with 64 bits and take the longer heads.
inline ScoreRoute score_route(int dt, int D, long long rows, const void* q, const void* k, const void* v, const void* out)
{
    const long long row_bytes = (long long)D * (dt == EC_F32 ? 4 : 2);
    if ((rows + kRowsBehind) * row_bytes > kDescriptorBytes) return ScoreRoute::kSimt;
    // Tiles go straight from memory into LDS, 16 bytes at a time.  Rows that do not lie on 16-byte boundaries pass through
    // registers in bf16, and take the vector kernels in fp32.
    const bool on_grid = (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v) & 15) == 0;
    if (dt == EC_BF16) return on_grid ? ScoreRoute::kMfma : ScoreRoute::kMfmaOffGrid;
    return on_grid && ((uintptr_t)out & 15) == 0 ? ScoreRoute::kF32 : ScoreRoute::kSimt;
}

// Pairs of tiles in the bf16 kernels: a workgroup takes two tiles of a head, the n-th from either end, so that all
// workgroups do the same work; alone, they come longest first and the chip evens out what is left.  Pairs save a
// workgroup's start and end, but run in rounds: 512 workgroups (two per compute unit) at a time, of equal length, so
// that a last round that is nearly empty costs as much as a full one, and an odd tile without a partner leaves a half.
// Measured at H8..40, B1..32, T100..8192 and for chunks over prefixes; the forward pass in pairs against single tiles, us of
// the whole call at D 128, D 64:
//   last round nearly empty    B1 H32 T4700, 608 pairs: +39 of 379, +39 of 262   B1 H40 T3500, 560 pairs: +18 of 288, +12 of 202
//   first round just exceeded  B1 H40 T3200, 520 pairs: -18 of 209, -13 of 145 (the eight run alone on their compute units)
//   full rounds                B2 H32 T2048, 512 pairs: -17 of 121, -14 of 85    B1 H32 T8192, 1024 pairs: -6 of 800, -20 of 513
//   few tiles, one is odd      B4 H32 T1100, 9 tiles: +9 of 110, +9 of 85        B16 H40 T640, 5 tiles: +7 of 180, +5 of 110
//   few tiles                  B4 H32 T768, 6 tiles: -4.6 of 55, +2.6 of 42; in one full round B8 H32 T512, 4 tiles: -2.9, -4.1
//   prefix longer than chunk   B4 H32 T512 P1500: +7 of 119, +11 of 84 (the tiles are nearly equally long)
constexpr long long kPairRound = 512;
constexpr long long kPairMin = 256;  // one per compute unit

// The rounds that `pairs` workgroups take are filled to `percent` on average.
inline bool rounds_filled(long long pairs, int percent)
{
    return pairs * 100 >= percent * kPairRound * ((pairs + kPairRound - 1) / kPairRound);
}

// Query tiles (128 rows) of the forward pass: D 64 has half the matrix work per tile and pairs pay only where nothing is lost.
inline bool pair_query_tiles(int D, long long tiles, long long heads, long long Tq, long long P)
{
    const long long pairs = (tiles + 1) / 2 * heads;
    if (tiles < 4 || pairs < kPairMin || P > Tq) return false;
    if (pairs <= kPairRound + kPairRound / 32)
        return D == 128 || pairs >= 480 || (tiles >= 8 && (pairs == kPairMin || pairs >= 304));
    if (tiles % 2 == 1) return tiles >= 13 && rounds_filled(pairs, D == 128 ? 60 : 93);
    return D == 128 ? rounds_filled(pairs, 60) : tiles >= 6 && rounds_filled(pairs, 70);
}

// Key tiles (256 rows) of the column pass.  Between 257 and 383 pairs some compute units hold two and most hold one:
// B1 H40 T3500 +15 of 288, +21 of 202.
// Five tiles: B4 H32 T1100 +4.4 of 110, +8.7 of 85.
inline bool pair_key_tiles(int D, long long tiles, long long heads, long long Tq, long long P)
{
    const long long pairs = (tiles + 1) / 2 * heads;
    if (tiles < 4 || tiles == 5 || pairs < kPairMin || 2 * P > Tq) return false;
    if (pairs <= kPairRound) return pairs == kPairMin || pairs >= 384;
    return D == 128 || rounds_filled(pairs, 70);
}

}  // namespace ec
