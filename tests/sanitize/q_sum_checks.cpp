// The whole-number Q' block sums of the certified sampler (q_units, q_value)
// under AddressSanitizer and UndefinedBehaviorSanitizer, CPU only: the same
// bits in any order, no overflow (an undefined conversion would be reported),
// and the bound on the distance from the exact sum that the header states.
// Exit status 0 = every check held.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "lda_internal.h"

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
      return 1;                                                       \
    }                                                                 \
  } while (0)

int main() {
  std::mt19937_64 g(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  int fp64_order_matters = 0;
  for (int trial = 0; trial < 2000; ++trial) {
    // terms of any size down to 2^-70 of the largest; the word's Q' is their sum and a little more
    const int n = 1 + int(g() % (trial % 50 ? 400 : 32768));
    const double scale = std::ldexp(1.0, int(g() % 1800) - 900);
    std::vector<double> term(static_cast<size_t>(n));
    long double exact = 0.0L;
    for (double &t : term) {
      t = scale * std::ldexp(u(g), -int(g() % (trial % 3 ? 70 : 2)));
      exact += t;
    }
    const double qp = double(exact) * (1.0 + (trial % 4 ? u(g) : 0.0));
    const int ex = lda::q_exponent(qp);
    CHECK(qp < std::ldexp(1.0L, ex) && qp >= std::ldexp(0.5L, ex));
    auto whole = [&] {
      unsigned long long s = 0;
      for (double t : term) s += lda::q_units(t, ex);
      return s;
    };
    auto plain = [&] {
      double s = 0.0;
      for (double t : term) s += t;
      return s;
    };
    const unsigned long long first = whole();
    const double first_plain = plain();
    bool moved = false;
    for (int q = 0; q < 8; ++q) {
      std::shuffle(term.begin(), term.end(), g);
      CHECK(whole() == first);
      moved = moved || plain() != first_plain;
    }
    fp64_order_matters += moved;
    // half a unit of 2^(ex - 62) <= 2^-61 Q' per term, and the conversion back (2^-53 of the sum)
    const long double err = std::fabs((long double)(lda::q_value(first, ex)) - exact);
    CHECK(err <= n * std::ldexp((long double)qp, -62) + std::ldexp(exact, -53) + std::ldexp(exact, -60));
  }
  CHECK(fp64_order_matters > 1000);  // what the whole numbers are for
  // an underflown Q' and its terms, and the smallest numbers
  CHECK(lda::q_units(0.0, lda::q_exponent(0.0)) == 0);
  CHECK(lda::q_value(lda::q_units(4.9e-324, lda::q_exponent(4.9e-324)), lda::q_exponent(4.9e-324)) == 4.9e-324);
  std::printf("Q' sum checks passed\n");
  return 0;
}
