// Prints which kernel paper_2601_07891_amd/csrc/score_linear_rule.h gives an input to.
//
// usage: linear_form_check rows Dh H
#include <cstdio>
#include <cstdlib>

#include "score_linear_rule.h"

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  const char* const names[] = {"rows", "stream", "wide", "narrow", "short"};
  std::printf("%s\n", names[(int)kvzap::linear::form_of(std::atoll(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]))]);
  return 0;
}
