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
  std::puts("ok");
  return 0;
}
