// Host build of the digit representation: sums of two products of zero,
// finite and not finite values, and of one beside an entry outside the
// series, by the rule of the convolutions (a term more than S digits below the
// largest is left out).  Lines: the four factors (z, f, n, i; m: outside), 1
// where the sum is a not-a-number.
#include "../paper_2301_12659_amd/csrc/digits.hpp"
#include <algorithm>
#include <cstdio>

using namespace mdk;

constexpr int L = 8, S = Digits<L>::S;

struct Num {
  double d[S];
  int rho;
};

static Num make(char kind) {
  double a[L] = {kind == 'f' ? 0x1.8p+1000 : kind == 'n' ? NAN : kind == 'i' ? INFINITY : 0.0};
  Num r{};
  tidy_limbs<L>(a);
  to_digits<L, S>(a, r.d, r.rho);
  if (kind == 'm') r.rho = DIGIT_MASK;
  return r;
}

int main() {
  const char *kinds = "zfnim";
  for (const char *a = kinds; *a != 'm'; ++a)
    for (const char *b = kinds; *b != 'm'; ++b)
      for (const char *c = kinds; *c; ++c)
        for (const char *e = kinds; *e; ++e) {
          const Num u[2] = {make(*a), make(*c)}, v[2] = {make(*b), make(*e)};
          int R = 2 * DIGIT_ZERO;
          for (int t = 0; t < 2; ++t) R = std::max(R, u[t].rho + v[t].rho);
          double z[S] = {0.0}, r[L];
          for (int t = 0; t < 2; ++t) {
            const int delta = R - u[t].rho - v[t].rho;
            for (int p = 0; p < S; ++p)
              for (int q = delta; p + q < S; ++q) z[p + q] += u[t].d[p] * v[t].d[q - delta];
          }
          from_digits<L, S>(z, R, r);
          printf("%c%c%c%c %d\n", *a, *b, *c, *e, r[0] != r[0] ? 1 : 0);
        }
}
