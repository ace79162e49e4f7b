// Undoes call_number step by step for counts as a process has them: says "ok" if every count comes back, which no two counts
// with one number would, and only zero has the number zero.
#include <stdio.h>

#include <initializer_list>

#include "call_number.hpp"

static uint64_t unshift(uint64_t v, int by) {
  uint64_t x = v;
  for (int i = by; i < 64; i += by) x = v ^ (x >> by);
  return x;
}

static uint64_t inverse(uint64_t odd) {      // modulo 2^64, by Newton's iteration
  uint64_t x = odd;
  for (int i = 0; i < 6; ++i) x *= 2 - odd * x;
  return x;
}

static uint64_t count_of(uint64_t v) {
  v = unshift(v, 31) * inverse(0x94d049bb133111ebull);
  v = unshift(v, 27) * inverse(0xbf58476d1ce4e5b9ull);
  return unshift(v, 30);
}

int main() {
  int even = 0;
  for (uint64_t start : {uint64_t(1), uint64_t(123456789012345), uint64_t(1) << 62, ~uint64_t(0) - 100000})
    for (uint64_t c = start; c - start < 100000; ++c) {
      const uint64_t v = scmoe::call_number(c);
      if (v == 0 || count_of(v) != c) {
        printf("count %llu: number %llu, count %llu\n", (unsigned long long)c, (unsigned long long)v, (unsigned long long)count_of(v));
        return 1;
      }
      even += v % 2 == 0;
    }
  if (scmoe::call_number(0) != 0 || even < 190000 || even > 210000) {
    printf("%d even numbers of 400000\n", even);
    return 1;
  }
  printf("ok\n");
  return 0;
}
