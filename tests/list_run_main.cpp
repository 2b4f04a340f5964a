// Host check of csrc/kgdb_list_run.h, built by test_list_run.py with g++ -O3 (and the undefined-behaviour
// sanitizer): prints "ok", or what went wrong.
#include <cstdio>

#include "kgdb_list_run.h"

using namespace kgdb;

// a word, two entries into it, the word again
__attribute__((noinline)) static uint32_t reread(unsigned char* p, int a, int b) {
  const uint32_t before = run_word(p);
  run_put(p, a);
  run_put(p + 2, b);
  return run_word(p) - before;
}

int main() {
  alignas(4) unsigned char buf[4] = {0, 0, 0, 0};
  if (reread(buf, 3, 4) != 0x00040003u) { std::puts("an entry written is not read back"); return 1; }
  for (int n = -1; n <= 64; ++n) {  // rows of a dense melt hold up to 96 candidates
    uint32_t first = 0, without = 0xffffffffu;
    for (int u = 0; u < 32; ++u) {
      if (u < n) first |= 1u << (31 - u);
      if (u == n) without &= ~(1u << (31 - u));
    }
    if (row_first(0xffffffffu, n) != first || (n >= 0 && row_without(0xffffffffu, n) != without)) {
      std::printf("mask of a row of %d\n", n);
      return 1;
    }
  }
  std::puts("ok");
  return 0;
}
