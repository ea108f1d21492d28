// Prints the number of row chunks and of blocks per chunk that the Gram
// products are split into, for every "M n ld single" line of standard input.
// Built with g++ by tests/test_native_gram.py.
#include <cstdio>

#include "../../paper_2203_07820_amd/csrc/internal.h"

int main() {
  long long M, ld;
  int n, single;
  while (std::scanf("%lld %d %lld %d", &M, &n, &ld, &single) == 4)
    std::printf("%d %d\n", chfsi::gram_chunks(M, n, ld, single != 0), chfsi::gram_blocks(n));
  return 0;
}
