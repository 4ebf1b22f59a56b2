// The 9-way searches of the partition's key range, eight trial keys a round.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ng {

// Trial keys x_t = a + floor((b - a)(t + 1) / 9), t < 8: at least a, below b.
__host__ __device__ inline uint32_t part_probe(uint32_t a, uint32_t b, uint32_t t) {
  return a + (uint32_t)((uint64_t)(b - a) * (t + 1) / 9);
}

// [a, b] after a round: f = the first t whose key is at or past the sought one,
// 8 if none is.  A search that has ended (a == b: its trial keys are b, f is 0
// or 8) stays as it is while another one goes on.  It ends at the smallest key of [a, b) at or past the sought
// one, at the first b if there is none.
__host__ __device__ inline void part_narrow(uint32_t& a, uint32_t& b, uint32_t f) {
  const bool open = a != b;
  const uint32_t na = f > 0 ? part_probe(a, b, f - 1) + 1 : a;
  if (f < 8) b = part_probe(a, b, f);
  if (open) a = na;
}

}  // namespace ng
