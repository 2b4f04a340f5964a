// A list rebuild's run of entries: a thread collects its list's 16-bit entries in LDS and stores them as
// 32-bit words.  Plain C++, so that a host build can check it.
#pragma once
#include <stdint.h>

namespace kgdb {

// Both views may alias: with plain integer types the compiler is free to read a word before the entries it
// holds have been written (g++ -O3 does, on the host).
typedef uint16_t __attribute__((may_alias)) RunEntry;
typedef uint32_t __attribute__((may_alias)) RunWord;

__host__ __device__ __forceinline__ void run_put(unsigned char* p, int v) { *(RunEntry*)p = (uint16_t)v; }
__host__ __device__ __forceinline__ uint32_t run_word(const unsigned char* p) { return *(const RunWord*)p; }

}  // namespace kgdb
