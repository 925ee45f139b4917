// Host build of round_to_24_bits against the rounding to an fp32 word: prints
// the number of differing results over random doubles of the fp32 range, and
// the special values.
#define ADAPM_HD
#include <cmath>
#include <cstdio>
#include <random>

#include "fp64math.hpp"

int main() {
  std::mt19937_64 g(4321);
  long differ = 0;
  for (long i = 0; i < 4000000; ++i) {
    const double m = std::ldexp((double)(g() >> 11), -53) + 0.5;
    double p = std::ldexp(m, (int)(g() % 252) - 125);   // normal fp32 values, below the largest
    if (i % 3 == 0) p = std::ldexp((double)(g() >> 40), (int)(g() % 210) - 110);   // 24 bits: stays as it is
    if (i % 2) p = -p;
    differ += adapm::round_to_24_bits(p) != (double)(float)p;
  }
  const double tie = 1.0 + std::ldexp(1.0, -24);   // halfway between 1 and its neighbour above
  std::printf("%ld %d %d %d %d %d\n", differ, adapm::round_to_24_bits(0.0) == 0.0,
              std::signbit(adapm::round_to_24_bits(-0.0)) != 0, adapm::round_to_24_bits(INFINITY) == INFINITY,
              std::isnan(adapm::round_to_24_bits(NAN)), adapm::round_to_24_bits(tie) == 1.0 + std::ldexp(1.0, -23));
  return 0;
}
