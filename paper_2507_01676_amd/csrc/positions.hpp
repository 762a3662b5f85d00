// 32-bit positions inside a chunk of the gather kernel's multi-lookup queue, from the 64-bit
// offsets of the batch.  Plain functions of numbers, so that the host can check them.
#pragma once

#include <cstdint>

#include "device_types.hpp"

namespace embx {

constexpr int kFar = 1 << 30;   // longest stretch of lookups between two rebases of a chunk

// Lookups to walk before the next rebase, of the d that are left: none where an end lies
// before its start (offsets that decrease break the contract; such a chunk reads nothing).
EMBX_HD inline int stretch(int64_t d) {
  const int hi = static_cast<int>(d >> 32);
  const uint32_t lo = static_cast<uint32_t>(d);
  if (hi < 0) return 0;
  return hi > 0 || lo > static_cast<uint32_t>(kFar) ? kFar : static_cast<int>(lo);
}

// A bag end d lookups past the base, as far as 32 bits go (one before the base ends at once).
EMBX_HD inline int rel32(int64_t d) {
  const int hi = static_cast<int>(d >> 32);
  const uint32_t lo = static_cast<uint32_t>(d);
  if (hi < 0) return 0;
  return hi > 0 || lo > static_cast<uint32_t>(INT32_MAX) ? INT32_MAX : static_cast<int>(lo);
}

}  // namespace embx
