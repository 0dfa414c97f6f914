// Blocks of 1024 positions of a head that a share of the losses adds up, and the register that holds each (alr.hip).
#pragma once
#include <stdint.h>

namespace l2kv {

// Share `share` of `shares` of a head of `blocks` blocks takes [first, end): at least one and at most kSlots, as long as
// shares <= blocks <= shares * kSlots.  Block e is in slot e % kSlots, so that the slot of a block known at compile time is known too.
template <uint32_t kSlots> struct PositionBlocks {
    uint32_t first, end;
    __host__ __device__ PositionBlocks(uint32_t blocks, uint32_t share, uint32_t shares)
        : first(share * blocks / shares), end((share + 1) * blocks / shares) {}
    // The block to fetch into a slot; slots that the share does not need repeat its first block, so nothing past the head is named.
    __host__ __device__ uint32_t in_slot(uint32_t slot) const {
        const uint32_t block = first + (slot + kSlots - first % kSlots) % kSlots;
        return block < end ? block : first;
    }
    __host__ __device__ bool has(uint32_t block) const { return block - first < end - first; }
};

}  // namespace l2kv
