// Which head a workgroup of the decode launch takes (host and device code).
#pragma once

#include <stdint.h>

namespace hk {

// floor(2^32 / n) + 1 (2^32 - 1 for n = 1), never 0: its product with a turn below 2^16, shifted
// by 32, is the turn's quotient by n (one less for n = 1, which head_of makes up for).
constexpr uint32_t turn_magic(int n) {
  return n > 1 ? (uint32_t)((1ull << 32) / (uint32_t)n) + 1u : 0xffffffffu;
}

// (x + turn) % n for x < n, turn < 2^16 and magic = turn_magic(n)
constexpr int head_of(int x, int turn, int n, uint32_t magic) {
  const int s = x + turn - n * (int)(((uint64_t)(uint32_t)turn * magic) >> 32);
  return s >= n ? s - n : s;
}

}  // namespace hk
