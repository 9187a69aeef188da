// done_slots.hpp -- counting the finished workgroups of a launch that goes on in its last one.
//
// A launch counts in a slot of its own, out of a ring of kDoneSlots, and clears the next launch's, so every launch
// starts from zeros that the launch before it wrote, whatever became of the slot since its last use.  (A single slot
// that every launch leaves at zero works as long as launches on a handle are ordered; after two that overlap, it may
// keep a remainder for good, and no later launch finds its last workgroup.)
#pragma once

#include <stdint.h>

namespace lacache {

constexpr int kDoneCount = 9;               // words of a slot: workgroups done, 1 + x: those with index x modulo 8
constexpr int kDoneStride = 32;             // words from one to the next (a cache line each)
constexpr int kDoneSlotWords = kDoneCount * kDoneStride;
constexpr int kDoneSlots = 16;              // more than the launches of one handle that ever overlap by mistake
constexpr int kDoneWords = kDoneSlots * kDoneSlotWords;

// The slot of the launch with this ticket (0, 1, 2, ... in the order of the launches).
__host__ __device__ inline uint32_t* done_slot(uint32_t* done, uint32_t ticket) {
    return done + (ticket % kDoneSlots) * kDoneSlotWords;
}

// Counts workgroup `block` of `grid`; true for the one that counts last.  add(p) adds 1 to *p for the whole device and
// returns what it held.  By index modulo 8 (the XCD) first: 256 additions to one word would queue up.
template <class Add>
__host__ __device__ inline bool count_done(uint32_t* slot, uint32_t block, uint32_t grid, Add add) {
    const uint32_t x = block & 7u, of_x = (grid - x + 7u) / 8u, xs = grid < 8u ? grid : 8u;
    return add(&slot[(1 + x) * kDoneStride]) == of_x - 1 && add(&slot[0]) == xs - 1;
}

}  // namespace lacache
