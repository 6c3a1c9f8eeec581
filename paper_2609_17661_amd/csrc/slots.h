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

// Tag of a species' cell.  The tags of the particles sum to the counts times the tags (mod
// 2^32) if every cell holds as many particles as its count says; tags of neighbours are not
// related, so particles counted in another cell do not cancel.
constexpr uint32_t cell_tag(uint32_t cell, uint32_t species) {
    uint32_t x = (4u * cell + species + 1u) * 0x9E3779B1u;
    x ^= x >> 15;
    x *= 0x2C1B3C6Du;
    return x ^ (x >> 13);
}

}  // namespace pic1d
