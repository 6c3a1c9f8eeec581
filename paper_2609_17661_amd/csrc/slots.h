// Slot arithmetic of segments of up to 2^31 - 256 slots, in 32 bits (host and device).
#pragma once

#include <stdint.h>

namespace pic1d {

// Tiles of `tile` slots that n slots take.
constexpr int32_t tiles_of(int32_t n, int32_t tile) { return n / tile + (n % tile != 0 ? 1 : 0); }

// Whether a slot handed out by an allocation counter lies in its segment.  A step hands out
// at most 2^30 pairs, so the counter of a segment near 2^31 slots may pass 2^31, but not 2^32.
constexpr bool slot_in(int32_t slot, int32_t cap) { return (uint32_t)slot < (uint32_t)cap; }

// ... and whether all n slots from it do.
constexpr bool slots_in(int32_t slot, int32_t n, int32_t cap) { return (uint32_t)slot + (uint32_t)n <= (uint32_t)cap; }

}  // namespace pic1d
