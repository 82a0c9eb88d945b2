// host_rules.cpp -- host-only build of the library's dispatch rules (test
// infrastructure; built by tests/test_host_rules.py with the HIP compiler's
// host pass only).
//
//   host_rules blocks <samples>
//     Philox blocks of four samples of the semianalytical estimator.
//   host_rules thread <samples> <bins> <bytes of an element> <vertices>
//     whether that estimator gives a vertex to a thread (1) or a wave (0).
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "cp_internal.hpp"

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "blocks")) {
    std::printf("%d\n", cp::semi_blocks(std::atoi(argv[2])));
    return 0;
  }
  if (argc == 6 && !std::strcmp(argv[1], "thread")) {
    std::printf("%d\n", cp::semi_by_thread(std::atoi(argv[2]), std::atoi(argv[3]), (size_t)std::atoi(argv[4]),
                                           std::atoll(argv[5])));
    return 0;
  }
  std::fprintf(stderr, "usage: see the head of this file\n");
  return 2;
}
