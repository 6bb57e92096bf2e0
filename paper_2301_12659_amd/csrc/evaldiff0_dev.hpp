// Device routine of the coefficient-0 derivatives, shared by the pre-pass of
// the evaluation (evaldiff.hip) and the small systems' M (prepass.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace mdk {

// Coefficient 0 of every derivative product (the entries of A_0), one
// thread per monomial, for supports of at most EVAL0_MAXK variables.  The
// same products as evaldiff_kernel restricted to the constant coefficients,
// which are plain multiple-double products: f_0 = c * CF(0), forward
// products f_j = f_{j-1} x_{v_j}(0) kept in registers, then the backward
// products b formed on the way back, d/dx_{v_j} = a_j f_{j-1} b_{k-j}.  The
// loads of the k constant coefficients are issued before the products, so
// the thread waits for memory once.
constexpr int EVAL0_MAXK = 8;

// (t: the monomial, or past the last; wait: called by every thread once its
// tables' loads are issued, false: give up)
template <int L, class Wait>
__device__ __forceinline__ bool eval0_monomial(const EvalArgs &a, int t, const Wait &wait) {
  // the monomial's support, exponents and coefficient do not depend on x:
  // their loads are issued before any wait for x
  const bool live = t < a.m;
  const int mono = live ? t : 0;
  int e0 = 0, k = 0;
  int vv[EVAL0_MAXK], ex[EVAL0_MAXK];
  double f[EVAL0_MAXK][L];  // f[j] = f_j for j < k (f_0 = c CF)
  if (live) {
    e0 = a.mon_ptr[mono];
    k = a.mon_ptr[mono + 1] - e0;
    ld<L>(a.cff, a.m, mono, f[0]);
  }
#pragma unroll
  for (int j = 0; j < EVAL0_MAXK; ++j) {
    vv[j] = 0;
    ex[j] = 1;
    if (j < k) {
      vv[j] = a.var[e0 + j];
      ex[j] = a.exp[e0 + j];
    }
  }
  if (!wait()) return false;
  if (!live || k == 0) return true;  // k == 0: no derivatives
  const size_t nD = (size_t)a.n * a.D, zD = (size_t)a.nnz * a.D;
  double xs[EVAL0_MAXK][L];
#pragma unroll
  for (int j = 0; j < EVAL0_MAXK; ++j) {
    md::zero<L>(xs[j]);
    if (j < k) {
      if (a.wait_ctr) ld_agent<L>(a.x, nD, (size_t)vv[j] * a.D, xs[j]);
      else ld<L>(a.x, nD, (size_t)vv[j] * a.D, xs[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < EVAL0_MAXK; ++j) {  // common factor: x^(a-1) for exponents >= 2
    if (j < k)
      for (int p = 1; p < ex[j]; ++p) {
        double r[L];
        MD<L>::mul(f[0], xs[j], r);
        md::copy<L>(r, f[0]);
      }
  }
#pragma unroll
  for (int j = 1; j < EVAL0_MAXK; ++j)
    if (j < k) MD<L>::mul(f[j - 1], xs[j - 1], f[j]);
  double b[L];  // backward product b_{k-j}, b_0 = 1
  md::zero<L>(b);
  b[0] = 1.0;
#pragma unroll
  for (int j = EVAL0_MAXK; j >= 1; --j) {
    if (j > k) continue;
    double d[L];
    if (j == k) md::copy<L>(f[j - 1], d);
    else MD<L>::mul(f[j - 1], b, d);
    md::mul_int<L>(d, ex[j - 1]);
#pragma unroll
    for (int l = 0; l < L; ++l) a.der[(size_t)l * zD + (size_t)(e0 + j - 1) * a.D] = d[l];
    if (j > 1) {
      double r[L];
      if (j == k) md::copy<L>(xs[j - 1], r);
      else MD<L>::mul(b, xs[j - 1], r);
      md::copy<L>(r, b);
    }
  }
  return true;
}

// Wait of a whole workgroup for x written by a launch on another stream (see
// EvalArgs); true at once where x is complete.
__device__ __forceinline__ bool eval0_wait(const EvalArgs &a) {
  if (!a.wait_ctr) return true;
  __shared__ int ok;
  if (threadIdx.x == 0) ok = wait_count(a.wait_ctr, a.wait_target, a.wait_status) ? 1 : 0;
  __syncthreads();
  return ok != 0;
}

}  // namespace mdk
