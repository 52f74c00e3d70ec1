// Prints what the library's size rules (rules.hpp) choose.
//   rules_check store BYTES
//   rules_check fused ITEMS
//   rules_check middle ITEMS GRID2 FP64
//   rules_check adjoint POINTS GROUPS BINS
//   rules_check direct POINTS TILES THREADS FP64 DETECTORS CUS
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rules.hpp"

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "store")) std::printf("%d\n", fcas::store_policy(std::strtoull(argv[2], nullptr, 10)));
  else if (argc == 3 && !std::strcmp(argv[1], "fused")) std::printf("%d\n", fcas::fused_takes(std::atoi(argv[2])));
  else if (argc == 5 && !std::strcmp(argv[1], "middle"))
    std::printf("%d\n", fcas::middle_groups(std::atoll(argv[2]), std::atoi(argv[3]), std::atoi(argv[4])));
  else if (argc == 5 && !std::strcmp(argv[1], "adjoint"))
    std::printf("%d\n", fcas::adjoint_parts(std::atoi(argv[2]), std::atoi(argv[3]), std::atoll(argv[4])));
  else if (argc == 8 && !std::strcmp(argv[1], "direct"))
    std::printf("%d\n", fcas::direct_call(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]),
                                          std::atoi(argv[6]), std::atoi(argv[7])));
  else return 1;
  return 0;
}
