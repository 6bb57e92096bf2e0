// Host build of the digit representation: dot products of seeded multiple
// doubles (limb patterns as sums that cancel leave them, too) by digits, every
// operand and result limb printed exactly (hex floats) for an exact rational
// check in Python.  Lines: L n spread, then a and b of every term, the result.
#include "../paper_2301_12659_amd/csrc/digits.hpp"
#include <algorithm>
#include <cstdio>
#include <random>

using namespace mdk;

template <int L> void draw(std::mt19937_64 &g, int spread, int pattern, double (&a)[L]) {
  std::uniform_real_distribution<double> u(0.5, 1.0), s(-1.0, 1.0);
  a[0] = u(g) * (s(g) < 0 ? -1.0 : 1.0) * std::ldexp(1.0, (int)(s(g) * spread));
  for (int l = 1; l < L; ++l) a[l] = a[l - 1] * std::ldexp(s(g), -53);
  if (pattern == 1)  // a zero limb, the rest one place too early
    for (int l = L - 1; l >= 1; --l) a[l] = l == 1 ? 0.0 : a[l] * std::ldexp(1.0, 50);
  if (pattern == 2)
    for (int l = 1; l < L; ++l) a[l] *= std::ldexp(1.0, -17 * l);  // gaps
  if (pattern == 3 && L > 2) a[L - 1] = a[L - 2] = 0.0;
}

template <int L> void run(std::mt19937_64 &g, int n, int spread) {
  constexpr int S = Digits<L>::S;
  static double da[128][S], db[128][S];
  int ra[128], rb[128], R = 4 * DIGIT_ZERO;
  printf("%d %d %d", L, n, spread);
  for (int i = 0; i < n; ++i) {
    double a[L], b[L];
    draw<L>(g, spread, i % 4, a);
    draw<L>(g, spread, (i / 4) % 4, b);
    for (double v : a) printf(" %a", v);
    for (double v : b) printf(" %a", v);
    tidy_limbs<L>(a);
    tidy_limbs<L>(b);
    to_digits<L, S>(a, da[i], ra[i]);
    to_digits<L, S>(b, db[i], rb[i]);
    R = std::max(R, ra[i] + rb[i]);
  }
  double z[S] = {0.0}, r[L];
  for (int i = 0; i < n; ++i) {
    const int delta = R - ra[i] - rb[i];
    for (int p = 0; p < S; ++p)
      for (int q = delta; p + q < S; ++q) z[p + q] += da[i][p] * db[i][q - delta];
    if ((i + 1) % (504 / S) == 0) carry_digits<S>(z);
  }
  from_digits<L, S>(z, R, r);
  for (double v : r) printf(" %a", v);
  printf("\n");
}

int main() {
  std::mt19937_64 g(1);
  for (int t = 0; t < 12; ++t)
    for (int spread : {0, 3, 11, 40, 150})
      for (int n : {1, 2, 7, 24, 65, 128}) run<8>(g, n, spread);
  // a value that is not finite makes the product a not-a-number
  double a[8] = {INFINITY}, d[Digits<8>::S], z[Digits<8>::S], r[8];
  int rho;
  tidy_limbs<8>(a);
  to_digits<8, Digits<8>::S>(a, d, rho);
  for (int k = 0; k < Digits<8>::S; ++k) z[k] = d[k] * 2.0;
  from_digits<8, Digits<8>::S>(z, rho, r);
  printf("nonfinite %d\n", r[0] != r[0] ? 1 : 0);
}
