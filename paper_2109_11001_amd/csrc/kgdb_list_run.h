// A list rebuild's row masks and run of entries: a thread tests the candidates of a row into a mask, collects
// its list's 16-bit entries in LDS and stores them as 32-bit words.  Plain C++, so that a host build can
// check it.
#pragma once
#include <stdint.h>

namespace kgdb {

// Both views may alias: with plain integer types the compiler is free to read a word before the entries it
// holds have been written (g++ -O3 does, on the host).
typedef uint16_t __attribute__((may_alias)) RunEntry;
typedef uint32_t __attribute__((may_alias)) RunWord;

__host__ __device__ __forceinline__ void run_put(unsigned char* p, int v) { *(RunEntry*)p = (uint16_t)v; }
__host__ __device__ __forceinline__ uint32_t run_word(const unsigned char* p) { return *(const RunWord*)p; }

// A row's mask, candidate u in bit 31 - u, with the first n candidates; and without candidate u.  A row may be
// longer than a mask (its further candidates are tested one by one): defined for every n and u.
__host__ __device__ __forceinline__ uint32_t row_first(uint32_t mask, int n) {
  return n > 0 ? mask & (0xffffffffu << (32 - (n < 32 ? n : 32))) : 0u;
}
__host__ __device__ __forceinline__ uint32_t row_without(uint32_t mask, int u) {
  return u < 32 ? mask & ~(0x80000000u >> u) : mask;
}

}  // namespace kgdb
