// M = A_0^{-1} for the Newton step without a multiple-double factorization on
// its critical path: the inverse X of A_0's leading limbs in doubles
// (inv64_kernel), then every column of M by iterative refinement,
//     x := x + X (e_j - A_0 x),
// with the residual formed in multiple-double arithmetic (refine_kernel).  A
// pass gains about 53 - log2(n cond(A_0)) bits, so a quad-double row of a
// well conditioned A_0 takes four passes, all of them matrix-vector products,
// where the Householder factorization of [A_0 | I] is a chain of n dependent
// reflectors.  The rows are independent of each other: one workgroup per
// row, no hand-over between workgroups.
//
// The refinement is taken only where it is as good as the factorization.
// inv64_kernel raises *need when A_0 has no pivot, a non-finite entry or
// ||A_0||_F ||X||_F >= 2^40, and refine_kernel when a row's residual does
// not contract; the launches of the factorization that follow on the stream
// return at once unless *need is set.  Below that bound no diagonal entry of
// R can be under the singularity threshold of the factorization
// (|R_ii| >= sigma_min >= 1/||X||_F, |R_jj| <= ||A_0||_F), so that the same
// matrices are reported singular as by the factorization alone.  A matrix that
// does not suit pays for the attempt: a step of one coefficient at cond(A_0) = 1e13
// takes 288 us instead of 249 with the factorization alone (double double, n =
// 64; 529 and 488 in quad double).  The bound is on A_0 as it is: rows of
// scales 2^40 apart take that way, too, however well conditioned otherwise.
#include "inverse_dev.hpp"
#include "kernels.hpp"

namespace mdk {

template <int RW, int NB, int NW>
__global__ void __launch_bounds__(64 * NW) inv64_kernel(int n, const double *a, double *x, int *need) {
  // on the chain of the step, beside the evaluation: raised issue priority
  __builtin_amdgcn_s_setprio(3);
  inv64_matrix<RW, NB, NW>(n, a, x, need);
}

template <int L>
__global__ void __launch_bounds__(RefineThreads<L>::value, RefineThreads<L>::waves)
    refine_kernel(int n, int S, const double *a, const double *x0, double *M, int *need) {
  extern __shared__ double lds[];
  __builtin_amdgcn_s_setprio(3);
  refine_row<L>(n, S, blockIdx.x, a, x0, M, need, lds);
}

// Where the refinement replaces the factorization: at least two limbs, and
// the matrix of doubles in the registers of one workgroup.  From 129 columns on
// they have no room for the factors of a panel (7.5 us a column), and in double
// doubles the factorization is faster: a step of n = 150, 16 coefficients, takes 806 us with it and 1292
// with the refinement (n = 128: 647 and 287).  In quad doubles the refinement
// stays the faster (the complex step of 2 n = 160: 2051 and 1804 us; a real one:
// launch_inverse's callers), in octo doubles by far (n = 150: 9568 and 3272).
bool inverse_refined(int L, int n) { return L >= 2 && n <= (L == 2 ? 128 : 192); }

template <int L>
static void launch_refine(int n, const double *a, const double *x0, double *M, int *need, hipStream_t st) {
  const int blocks = (n + 63) / 64, S = refine_parts<L>(n);
  hipLaunchKernelGGL(refine_kernel<L>, dim3(n), dim3(64 * blocks * S), refine_lds<L>(n, S), st, n, S, a, x0, M, need);
}

hipError_t launch_inverse(int L, int n, const double *a, double *x0, double *M, int *need, hipStream_t st) {
  if (!inverse_refined(L, n)) return hipErrorInvalidValue;
  if (n <= 8) hipLaunchKernelGGL((inv64_kernel<1, 8, 1>), dim3(1), dim3(64), 0, st, n, a, x0, need);
  else if (n <= 32) hipLaunchKernelGGL((inv64_kernel<1, 8, 4>), dim3(1), dim3(256), 0, st, n, a, x0, need);
  else if (n <= 64) hipLaunchKernelGGL((inv64_kernel<1, 8, 8>), dim3(1), dim3(512), 0, st, n, a, x0, need);
  else if (n <= 128) hipLaunchKernelGGL((inv64_kernel<2, 8, 16>), dim3(1), dim3(1024), 0, st, n, a, x0, need);
  else hipLaunchKernelGGL((inv64_kernel<3, 12, 16>), dim3(1), dim3(1024), 0, st, n, a, x0, need);
  if (L == 2) launch_refine<2>(n, a, x0, M, need, st);
  else if (L == 4) launch_refine<4>(n, a, x0, M, need, st);
  else launch_refine<8>(n, a, x0, M, need, st);
  return hipGetLastError();
}

}  // namespace mdk
