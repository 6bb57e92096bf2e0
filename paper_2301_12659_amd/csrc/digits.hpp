// Multiple doubles as digits in radix 2^23, for sums of products (the truncated
// convolutions): a = sum_p d_p 2^(23 (rho - p - 1)), p < S, with integer digits
// |d_p| <= 2^22 kept in doubles and an exponent rho of its own for every
// number.  The product of two digits and sums of up to 512 of them are exact in
// a double, so a multiply-add of two numbers is S (S + 1) / 2 plain fused
// multiply-adds on independent accumulators, without the error-free additions of
// the level sums (MD<L>::fma_lazy): 231 instructions in place of 960 for octo
// doubles (S = 21), and no dependent chain.
//
// Two terms of a sum whose products have different radix exponents are
// aligned by a shift of whole digits (delta), so that every sum is formed
// relative to its own largest term, as with the level sums, whatever the range
// of the operands.  The precision is S digits less the two leading ones, which
// may be short: 23 (S - 2) bits at worst, 437 for S = 21, with up to
// S products of the last level and beyond dropped (about 2^4.5 units there).
// Not-a-numbers and infinities give not-a-numbers, times a zero too.
#pragma once
#include "md.hpp"

namespace mdk {

constexpr int DIGIT_BITS = 23;
constexpr double DIGIT_BASE = 8388608.0;       // 2^23
constexpr double DIGIT_INV = 1.0 / 8388608.0;  // 2^-23
// exponent of a zero: far below any other, so that its terms count as masked
constexpr int DIGIT_ZERO = -100000;
// exponent of a value that is not finite: so far above any other that its product
// with a zero, a not-a-number, is above those of finite values
constexpr int DIGIT_NAN = 200000;
// exponent of an entry outside a series: its sum with any other, DIGIT_NAN among
// them, is below that of two zeros
constexpr int DIGIT_MASK = 8 * DIGIT_ZERO;

template <int L> struct Digits;
template <> struct Digits<8> { static constexpr int S = 21; };

// Limbs in order of size without overlap, their sum unchanged.  A sum whose
// leading limbs cancel (x + dx, say) can leave a zero limb followed by limbs
// larger than their place allows.
template <int L>
MD_INLINE void tidy_limbs(double (&a)[L]) {
#pragma unroll
  for (int j = 0; j < L - 1; ++j) {  // limb j: the sum of what remains, its rounding errors remain
    double s = a[L - 1];
#pragma unroll
    for (int q = L - 2; q >= j; --q) {
      double t;
      md::two_sum(a[q], s, t, a[q + 1]);
      s = t;
    }
    a[j] = s;
  }
}

// The digits of a, tidy (limb by limb: the next limb joins the remainder, exactly,
// where its bits begin) and its exponent rho.
template <int L, int S>
MD_INLINE void to_digits(const double (&a)[L], double (&d)[S], int &rho) {
  const double top = __builtin_fabs(a[0]);
  int e = 0;
#if defined(__HIP_DEVICE_COMPILE__)
  e = __builtin_amdgcn_frexp_exp(top);
#else
  (void)std::frexp(top, &e);
#endif
  rho = (e + DIGIT_BITS + DIGIT_BITS * 100) / DIGIT_BITS - 100;  // |a| <= 2^(23 rho - 1)
  const bool finite = top <= 0x1.fffffffffffffp+1023;
  if (!finite) rho = DIGIT_NAN;
  const int sh = DIGIT_BITS * (1 - rho);
  // what remains is r + pend + tail, each the rounding error of the one before;
  // bits move up as the digits leave r
  double r = __builtin_ldexp(a[0], sh), pend = 0.0, tail = 0.0;
#pragma unroll
  for (int p = 0; p < S; ++p) {
    if (p > 0) {
      double s, t;
      md::fast_two_sum(r * DIGIT_BASE, pend * DIGIT_BASE, s, t);
      r = s;
      md::fast_two_sum(t, tail * DIGIT_BASE, pend, tail);
    }
#pragma unroll
    for (int l = 1; l < L; ++l)
      if ((53 * l) / DIGIT_BITS == p) {
        double s, e, t;
        md::two_sum(r, __builtin_ldexp(a[l], sh + DIGIT_BITS * p), s, e);
        r = s;
        md::two_sum(pend, e, s, t);
        pend = s;
        tail += t;
      }
    d[p] = __builtin_rint(r);
    r -= d[p];
  }
  if (top == 0.0) rho = DIGIT_ZERO;
}

// Carries from the last accumulator up: every z_k, k > 0, becomes a digit.
template <int S>
MD_INLINE void carry_digits(double (&z)[S]) {
#pragma unroll
  for (int k = S - 1; k > 0; --k) {
    const double c = __builtin_rint(z[k] * DIGIT_INV);
    z[k] = __builtin_fma(c, -DIGIT_BASE, z[k]);
    z[k - 1] += c;
  }
}

// a = sum_k z_k 2^(23 (R - k - 2)) rounded to L limbs (z: accumulators of
// products, up to 2^53).  The digits are paired (46 bits, exact) and the pairs,
// which do not overlap, summed from the last to the first once for every limb,
// each sum's rounding errors being what remains for the next.
template <int L, int S>
MD_INLINE void from_digits(double (&z)[S], int R, double (&a)[L]) {
  constexpr int m = S / 2 + 1;  // the first alone, the others in pairs
  static_assert(m >= L, "as many pairs as limbs");
  carry_digits<S>(z);
  double y[m];
  y[0] = z[0];  // at most 2^52 (a digit's carries included)
  double w = 1.0;
#pragma unroll
  for (int q = 1; q < m; ++q) {
    w *= DIGIT_INV * DIGIT_INV;
    y[q] = w * __builtin_fma(z[2 * q - 1], DIGIT_BASE, 2 * q < S ? z[2 * q < S ? 2 * q : 0] : 0.0);
  }
#pragma unroll
  for (int j = 0; j < L; ++j) {  // limb j: the sum of what remains, its rounding errors remain
    double s = y[m - 1];
#pragma unroll
    for (int q = m - 2; q >= j; --q) {
      double t;
      md::fast_two_sum(y[q], s, t, y[q + 1]);
      s = t;
    }
    y[j] = s;
  }
  const int sh = DIGIT_BITS * (R - 2);
#pragma unroll
  for (int l = 0; l < L; ++l) a[l] = __builtin_ldexp(y[l], sh);
}

}  // namespace mdk
