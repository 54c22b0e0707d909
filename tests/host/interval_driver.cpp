// Test driver of the score intervals: reads lines "c s wv" (float32 values) from
// stdin and prints x3_lower of each.
#include <cstdio>

#include "../../paper_2204_08988_amd/csrc/interval.hpp"

int main() {
  float c, s, wv;
  while (std::scanf("%f %f %f", &c, &s, &wv) == 3) std::printf("%.9g\n", dpmm::x3_lower(c, s, wv));
  return 0;
}
