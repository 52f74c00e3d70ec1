// Prints what the library's size rules (rules.hpp) choose.
//   rules_check store BYTES
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rules.hpp"

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "store")) std::printf("%d\n", fcas::store_policy(std::strtoull(argv[2], nullptr, 10)));
  else return 1;
  return 0;
}
