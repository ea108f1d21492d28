// Host-only driver: the scaled 1D factors of the cell matrix (op_build.cpp) of
// the given degree, as chfsi_op_build() computes them, one hexadecimal value
// per line: (p + 1)^2 of the stiffness, (p + 1)^2 of the derivative and p + 1 of
// the mass.  Built with g++ by tests/test_native_tables_1d.py.
#include <cstdio>
#include <cstdlib>

#include "../../paper_2203_07820_amd/csrc/internal.h"

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  chfsi_system sys{};
  sys.p = std::atoi(argv[1]);
  sys.ncell = std::atoi(argv[2]);
  sys.L = std::atof(argv[3]);
  chfsi::HostTables t;
  if (!chfsi::build_tables(sys, t).empty()) return 1;
  for (const auto* v : {&t.ts_K, &t.ts_S, &t.ts_m})
    for (double x : *v) std::printf("%a\n", x);
  return 0;
}
