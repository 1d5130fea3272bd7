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

}  // namespace ec
