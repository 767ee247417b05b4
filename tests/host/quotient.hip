// quotient() of qa_wave.hpp on the CPU: over every exponent of d from the smallest normal number up, with numerators
// whose quotient and whose remainder are normal numbers, it is n / d correctly rounded; below, where 1 / d overflows, it
// is not finite although n / d is.
#include <cmath>
#include <cstdio>
#include <limits>
#include <random>

#include "qa_wave.hpp"

template <class T>
static long check(int emin, int emax, int digits) {
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> u(1.0, 2.0);
  long wrong = 0;
  for (int e = emin; e <= emax; e++)
    for (int i = 0; i < 400; i++) {
      const T d = std::ldexp(static_cast<T>(u(rng)), e);
      // exponent of n: the quotient's and the remainder's (n's less `digits`) stay normal, the quotient finite
      const int lo = std::max(emin + digits + 1, emin + e + 1), hi = std::min(emax - 1, emax + e - 1);
      if (hi < lo) continue;
      const int k = lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1));
      const T n = std::ldexp(static_cast<T>(u(rng)), k) * (i % 2 ? T(-1) : T(1));
      if (qa::quotient(n, d, T(1) / d) != n / d) wrong++;
    }
  return wrong;
}

template <class T>
static bool overflows_below() {
  const T d = std::numeric_limits<T>::min() / 16, n = std::numeric_limits<T>::min();
  return std::isfinite(n / d) && !std::isfinite(qa::quotient(n, d, T(1) / d));
}

int main() {
  const long w32 = check<float>(-126, 127, 24), w64 = check<double>(-1022, 1023, 53);
  std::printf("wrong32 %ld wrong64 %ld below32 %d below64 %d\n", w32, w64, overflows_below<float>() ? 1 : 0,
              overflows_below<double>() ? 1 : 0);
  return 0;
}
