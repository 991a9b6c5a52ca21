// sample_table.h -- the hash table of a sample of particles: when it is used,
// its size and its hash (plain C++, so that they can be checked on the host).
#pragma once

#include <stdint.h>

namespace mpc {

// Entries - 1 (a power of two less one) of the table for m of a box's np
// particles, 0 < m <= np < 2^31; 0: the inverse of the index array instead.
// Two words an entry and 8 m to 16 m entries stay within the 4 np bytes of the
// inverse where 32 m <= np.
constexpr uint32_t sample_table_mask(uint64_t m, uint64_t np) {
  if (32 * m > np) return 0;
  uint32_t n = 8;
  while (n < 8 * m) n *= 2;
  return n - 1;
}

// The 32-bit finalizer of MurmurHash3 (A. Appleby): a bijection that spreads
// any stride of indices over all bits, so that every table size has a home
// slot for every entry.  (One product whose bits 7 to 31 were kept had 2^25
// home slots at most: with more samples than that, linear probing walked
// through millions of entries for each particle of the box.)
constexpr uint32_t sample_hash(uint32_t key, uint32_t mask) {
  key ^= key >> 16;
  key *= 0x85ebca6bu;
  key ^= key >> 13;
  key *= 0xc2b2ae35u;
  key ^= key >> 16;
  return key & mask;
}

}  // namespace mpc
