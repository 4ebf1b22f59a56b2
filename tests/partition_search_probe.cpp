// Test helper: the two key searches of a partition round on the host, side by
// side as the kernel runs them -- rounds until both have ended.
// Usage: probe; reads lines "a b first0 first1" (64-bit, a key x is past the
// sought one when x >= first) and prints "a0 b0 a1 b1 rounds" for each.
#include <cstdio>

#include "ng_search.h"

static uint32_t first_past(uint32_t a, uint32_t b, unsigned long long first) {
  uint32_t t = 0;
  while (t < 8 && ng::part_probe(a, b, t) < first) ++t;
  return t;
}

int main() {
  unsigned long long a, b, f0, f1;
  while (scanf("%llu %llu %llu %llu", &a, &b, &f0, &f1) == 4) {
    uint32_t a0 = (uint32_t)a, b0 = (uint32_t)b, a1 = a0, b1 = b0, rounds = 0;
    while ((a0 < b0 || a1 < b1) && ++rounds < 100) {
      const uint32_t t0 = first_past(a0, b0, f0), t1 = first_past(a1, b1, f1);
      ng::part_narrow(a0, b0, t0);
      ng::part_narrow(a1, b1, t1);
    }
    printf("%u %u %u %u %u\n", a0, b0, a1, b1, rounds);
  }
}
