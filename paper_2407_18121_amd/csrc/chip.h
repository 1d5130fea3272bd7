// The chip as launches see it: numbers without HIP.
#pragma once

namespace ec {

constexpr int kXcds = 8;       // each with an L2 of its own; workgroups are handed to them round-robin by linear id
constexpr int kXcdUnits = 32;  // compute units of one
constexpr int kComputeUnits = kXcds * kXcdUnits;

}  // namespace ec
