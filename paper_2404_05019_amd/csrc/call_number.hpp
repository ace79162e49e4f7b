// Numbers that tell the launches of one layer call from every other call's.
#pragma once
#include <stdint.h>

namespace scmoe {

// Another number for every count, zero for zero alone: a permutation of the 64-bit numbers (each step can be undone), whose
// values look like random ones, so that what else lies in memory is taken for one of them with a probability of 2^-64.
inline uint64_t call_number(uint64_t count) {
  count = (count ^ (count >> 30)) * 0xbf58476d1ce4e5b9ull;
  count = (count ^ (count >> 27)) * 0x94d049bb133111ebull;
  return count ^ (count >> 31);
}

}  // namespace scmoe
