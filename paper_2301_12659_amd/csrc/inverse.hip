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
// ||A_0||_F ||X||_F >= 2^40, also once the scales of its rows and columns are taken
// out (powers of two, exact), and refine_kernel when a row's residual does
// not contract; the launches of the factorization that follow on the stream
// return at once unless *need is set.  No diagonal entry of R is then under the
// singularity threshold of the factorization (|R_ii| >= sigma_min >= 1/||X||_F,
// |R_jj| <= ||A_0||_F, and ||A_0||_F ||X||_F < 2^(53 L - 8) / n for a scaled
// matrix, too), so that the same matrices are reported singular as by the
// factorization alone.  A matrix that does not suit pays for the attempt: a step of
// one coefficient at cond(A_0) = 1e13 takes 291 us instead of 250 with the
// factorization alone (double double, n = 64; 533 and 488 in quad double).  One
// whose rows differ in scale by 2^50 does not: the medium quad-double system, every
// other polynomial times 2^-50, 462 us a step, 860 factorized after a first attempt
// and 735 without.
#include "inverse_dev.hpp"
#include "kernels.hpp"

namespace mdk {

template <int L, int RW, int NB, int NW>
__global__ void __launch_bounds__(64 * NW) inv64_kernel(int n, const double *a, double *x, int *need) {
  // on the chain of the step, beside the evaluation: raised issue priority
  __builtin_amdgcn_s_setprio(3);
  inv64_matrix<L, RW, NB, NW>(n, a, x, need);
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

template <int L>
static void launch_inv64(int n, const double *a, double *x0, int *need, hipStream_t st) {
  if (n <= 8) hipLaunchKernelGGL((inv64_kernel<L, 1, 8, 1>), dim3(1), dim3(64), 0, st, n, a, x0, need);
  else if (n <= 32) hipLaunchKernelGGL((inv64_kernel<L, 1, 8, 4>), dim3(1), dim3(256), 0, st, n, a, x0, need);
  else if (n <= 64) hipLaunchKernelGGL((inv64_kernel<L, 1, 8, 8>), dim3(1), dim3(512), 0, st, n, a, x0, need);
  else if (n <= 128) hipLaunchKernelGGL((inv64_kernel<L, 2, 8, 16>), dim3(1), dim3(1024), 0, st, n, a, x0, need);
  else if constexpr (L > 2)  // (inverse_refined)
    hipLaunchKernelGGL((inv64_kernel<L, 3, 12, 16>), dim3(1), dim3(1024), 0, st, n, a, x0, need);
}

hipError_t launch_inverse(int L, int n, const double *a, double *x0, double *M, int *need, hipStream_t st) {
  if (!inverse_refined(L, n)) return hipErrorInvalidValue;
  auto run = [&](auto tag) {
    constexpr int LL = decltype(tag)::value;
    launch_inv64<LL>(n, a, x0, need, st);
    launch_refine<LL>(n, a, x0, M, need, st);
  };
  if (L == 2) run(std::integral_constant<int, 2>{});
  else if (L == 4) run(std::integral_constant<int, 4>{});
  else run(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

}  // namespace mdk
