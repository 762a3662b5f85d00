// 32-bit positions inside a chunk of the gather kernel's multi-lookup queue, from the 64-bit
// offsets of the batch.  Plain functions of numbers, so that the host can check them.
#pragma once

#include <cstdint>

#include "device_types.hpp"

// Most lookups between two rebases of a chunk (a small value in a test build makes ordinary
// batches rebase).
#ifndef EMBX_FAR
#define EMBX_FAR (1 << 30)
#endif

namespace embx {

// The stretch between rebases for steps of N lookups: whole steps, because a step shorter
// than N may only be a chunk's last (it ends every bag whose end lies inside N).
EMBX_HD constexpr int far_of(int N) { return EMBX_FAR / N * N; }
static_assert(EMBX_FAR >= 64 && EMBX_FAR <= (1 << 30), "a step at least, and positions and their differences fit 32 bits");

// Lookups to walk before the next rebase, of the d that are left: none where an end lies
// before its start (offsets that decrease break the contract; such a chunk reads nothing).
EMBX_HD inline int stretch(int64_t d, int far) {
  const int hi = static_cast<int>(d >> 32);
  const uint32_t lo = static_cast<uint32_t>(d);
  if (hi < 0) return 0;
  return hi > 0 || lo > static_cast<uint32_t>(far) ? far : static_cast<int>(lo);
}

// A bag end d lookups past the base, as far as 32 bits go (one before the base ends at once).
EMBX_HD inline int rel32(int64_t d) {
  const int hi = static_cast<int>(d >> 32);
  const uint32_t lo = static_cast<uint32_t>(d);
  if (hi < 0) return 0;
  return hi > 0 || lo > static_cast<uint32_t>(INT32_MAX) ? INT32_MAX : static_cast<int>(lo);
}

}  // namespace embx
