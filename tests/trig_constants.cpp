// Host check of the DFT twiddle constants: sin and cos of every turn t / S that the in-register DFTs use are the
// doubles nearest to the long double values.
#include <cmath>
#include <cstdio>
#include <initializer_list>

#include "../paper_2406_10765_amd/csrc/fft_trig.hpp"

int main() {
  const long double pi = 3.14159265358979323846264338327950288L;
  long bad = 0, n = 0;
  for (int S : {1, 2, 3, 4, 6, 8, 9, 12, 16, 18, 24})
    for (int t = -S; t <= S; ++t) {
      // the angle reduced to one octant, so that the long double value keeps its 64 bits
      const double s = pw::turn_sin(t, S), c = pw::turn_cos(t, S);
      auto ref = [&](long num, long den) {  // sin(2 pi num / den), |num / den| <= 1 / 8 by symmetry
        num = (num % den + den) % den;
        long double sign = 1;
        if (2 * num > den) { num = den - num; sign = -1; }
        if (4 * num > den) { num = den - 2 * num; den *= 2; }
        return sign * (8 * num > den ? cosl(2 * pi * (den - 4 * num) / (4 * den)) : sinl(2 * pi * num / den));
      };
      n += 2;
      if (s != (double)ref(t, S)) ++bad;
      if (c != (double)ref(4L * t + S, 4L * S)) ++bad;
    }
  std::printf("%ld constants, %ld not the nearest double\n", n, bad);
  return bad ? 1 : 0;
}
