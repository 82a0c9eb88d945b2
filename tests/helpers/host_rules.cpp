// host_rules.cpp -- host-only build of the library's dispatch rules (test
// infrastructure; built by tests/test_host_rules.py with the HIP compiler's
// host pass only).
//
//   host_rules blocks <samples>
//     Philox blocks of four samples of the semianalytical estimator.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "cp_internal.hpp"

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "blocks")) {
    std::printf("%d\n", cp::semi_blocks(std::atoi(argv[2])));
    return 0;
  }
  std::fprintf(stderr, "usage: see the head of this file\n");
  return 2;
}
