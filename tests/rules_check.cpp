// Prints the launch rules' decisions at the sizes given on the command line.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rules.hpp"

int main(int argc, char** argv) {
  if (argc == 5 && !std::strcmp(argv[1], "pull_streams"))
    std::printf("%d\n", adapm::pull_streams(std::atoll(argv[2]), std::atoll(argv[3]), std::atoi(argv[4])));
  else if (argc == 5 && !std::strcmp(argv[1], "pull_rows"))
    std::printf("%d\n", adapm::pull_rows(std::atoll(argv[2]), std::atoi(argv[3]), std::atoi(argv[4])));
  else if (argc == 4 && !std::strcmp(argv[1], "push_prepare_tiled_keys"))
    std::printf("%lld\n", (long long)adapm::push_prepare_tiled_keys(std::atoll(argv[2]), std::atoi(argv[3])));
  else if (argc == 7 && !std::strcmp(argv[1], "merge_streams"))
    std::printf("%d\n", adapm::merge_streams(std::atoll(argv[2]), std::atoll(argv[3]), std::atoi(argv[4]) != 0,
                                             std::atoi(argv[5]) != 0, std::atoi(argv[6]) != 0));
  else if (argc == 4 && !std::strcmp(argv[1], "kge_tiled_keys"))
    std::printf("%lld\n", (long long)adapm::kge_tiled_keys(std::atoll(argv[2]), std::atoll(argv[3])));
  else
    return 1;
  return 0;
}
