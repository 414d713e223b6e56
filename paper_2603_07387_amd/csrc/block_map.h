// Which slot and which of its groups a scatter block takes.  Plain C++: also
// compiled on its own by the test of this map.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define TN_HOST_DEVICE __host__ __device__
#else
#define TN_HOST_DEVICE
#endif

namespace tn {

struct SlotBlock {
  uint32_t slot, group;  // slot = n: padding of the grid, no work
};

constexpr uint32_t kXcds = 8;  // block b runs on XCD b mod 8

// Blocks of a grid row of n slots with gx groups each.
TN_HOST_DEVICE constexpr uint32_t slot_blocks(uint32_t n, uint32_t gx) {
  return (n * gx + kXcds - 1) / kXcds * kXcds;
}

// Eight slots at a time are one per XCD, a slot's groups one after the other on
// its XCD, so that they share its entries in that L2.  The last n mod 8 slots
// go over all XCDs in turn: kept to one each they would leave the others idle
// (a triangle's three slots, 4096 samples of 64 x 64, m = 1024, FP32: 138 us per
// call on three XCDs, 86 on all; its two pairs of 256 x 256 matrices, 512
// samples, m = 65536: 1564 and 723 us).
TN_HOST_DEVICE constexpr SlotBlock slot_block(uint32_t b, uint32_t n, uint32_t gx) {
  const uint32_t rest = n % kXcds, whole = n - rest;
  if (b < whole * gx) {
    const uint32_t run = b / (kXcds * gx), at = b - run * (kXcds * gx);
    return SlotBlock{run * kXcds + at % kXcds, at / kXcds};
  }
  const uint32_t j = b - whole * gx;
  if (j >= rest * gx) return SlotBlock{n, 0};
  return SlotBlock{whole + j % rest, j / rest};
}

}  // namespace tn
