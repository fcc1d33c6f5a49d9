// Prints what the host rules of amh_kernels.h give for the arguments of a command line, for
// tests/test_host_rules.py (no GPU needed).
//   half_window <d> <L>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "amh_kernels.h"

int main(int argc, char** argv) {
  const auto num = [&](int i) { return std::atoll(i < argc ? argv[i] : "0"); };
  if (argc == 4 && !std::strcmp(argv[1], "half_window")) {
    std::printf("%d\n", amh::half_window((int)num(2), (int)num(3)));
    return 0;
  }
  return 2;
}
