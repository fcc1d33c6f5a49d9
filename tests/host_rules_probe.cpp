// Prints what the host rules of amh_kernels.h give for the arguments of a command line, for
// tests/test_host_rules.py (no GPU needed).
//   half_window <d> <L>
//   last_knot2 <d_min> <bin_w> <n_bins>
//   carry <G> <h> <L> <dev_max>
//   run_end <L> <global_every> <n_global> <anchor_every> <t> <end>
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
  if (argc == 5 && !std::strcmp(argv[1], "last_knot2")) {
    std::printf("%.9g\n", (double)amh::last_knot2(std::atof(argv[2]), std::atof(argv[3]), (int)num(4)));
    return 0;
  }
  if (argc == 6 && !std::strcmp(argv[1], "carry")) {
    const int G = (int)num(2), h = (int)num(3), L = (int)num(4);
    std::printf("%d %d\n", amh::carry_pays(G, h, L) ? 1 : 0, amh::carry_exact(h, L, (float)std::atof(argv[5])) ? 1 : 0);
    return 0;
  }
  if (argc == 8 && !std::strcmp(argv[1], "run_end")) {
    amh::SweepParams P{};
    P.L = (int)num(2);
    P.global_every = (int)num(3);
    P.n_global = (int)num(4);
    P.anchor_every = (int)num(5);
    std::printf("%lld\n", (long long)amh::run_end(P, num(6), num(7)));
    return 0;
  }
  return 2;
}
