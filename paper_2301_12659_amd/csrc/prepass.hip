// M = A_0^{-1} of a small system from coefficient 0 of the iterate, in one
// launch of one workgroup: the coefficient-0 derivatives (evaldiff0_dev.hpp),
// the assembly of A_0, the inverse in doubles and its refinement
// (inverse_dev.hpp), and the factorization where that does not suit A_0
// (factor_dev.hpp).  As launches of their own these are seven of a step's
// twelve, none of them longer than a few microseconds: the step was bound by
// the host's launches.  Four pipelined steps of 8 variables, 64 monomials, 16
// coefficients in double doubles: 230 us with the launches apart, 171 in one
// (24 us beside the rest of a step).
#include "evaldiff0_dev.hpp"
#include "factor_dev.hpp"
#include "inverse_dev.hpp"

namespace mdk {

constexpr int PREPASS_NT = 256, PREPASS_MAXN = 16;

// Row j of M as refine_row forms it, for n <= 16 and by one wavefront: lane
// 16 s + v has the terms i = s, s + 4, ... of column v; A_0 (as [L][n][n]) and
// the inverse in doubles (x0 [n][n]) in LDS.  False where it does not contract.
template <int L>
__device__ bool refine_row_small(int n, int j, const double *as, const double *x0, double *M) {
  constexpr int LX = L + 1;
  const int lane = threadIdx.x & 63, v = lane & 15, s = lane >> 4, nn = n * n;
  const bool col = v < n;
  const int vv = col ? v : 0;
  double y[LX];
  md::zero<LX>(y);
  y[0] = col ? x0[j * n + vv] : 0.0;
  const double done = ldexp(1.0, -53 * L);
  double prev = 1.0, rho = 0.0;
  int limbs = 1;  // of the residual before
  for (int pass = 0;; ++pass) {
    const bool last = pass > 0 && (prev * rho * rho * 1024.0 <= done || prev <= refine_floor(L));
    double e = 0.0, t = 0.0;
    auto form = [&](auto tag) {
      constexpr int P = decltype(tag)::value, LA = P > L ? L : P;
      double u[P], r[P], q[P];
      md::zero<P>(u);
      t = 0.0;
      for (int i0 = 0; i0 < n; i0 += 4) {
        const int i = i0 + s, ii = min(i, n - 1);
        double av[LA], yv[P];
#pragma unroll
        for (int l = 0; l < LA; ++l) av[l] = i < n ? as[l * nn + ii * n + vv] : 0.0;
#pragma unroll
        for (int l = 0; l < P; ++l) yv[l] = -__shfl(y[l], ii, 64);
        t = __builtin_fma(fabs(av[0]), fabs(yv[0]), t);
        if constexpr (LA == P) MD<P>::fma_lazy(u, av, yv);
        else MD<P>::fma_lazy_h(u, av, yv);
      }
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {
        double o[P];
#pragma unroll
        for (int l = 0; l < P; ++l) o[l] = __shfl_xor(u[l], off, 64);
        MD<P>::add_lazy(u, o);
        t += __shfl_xor(t, off, 64);
      }
      if (v == j) {
        double one[P];
        md::zero<P>(one);
        one[0] = 1.0;
        MD<P>::add_lazy(u, one);
      }
      MD<P>::renorm(u, r);
      MD<P>::renorm(r, q);
      e = q[0];
    };
    if (pass == 0) form(std::integral_constant<int, 2>{});
    else if (last) form(std::integral_constant<int, LX>{});
    else form(std::integral_constant<int, L>{});
    double om = 0.0;
    if (col) {
      const double o = e == 0.0 ? 0.0 : fabs(e) / t;
      om = o >= 0.0 ? o : INFINITY;  // a NaN counts as infinite
    }
    for (int off = 8; off > 0; off >>= 1) om = fmax(om, __shfl_xor(om, off, 64));
    om = __shfl(om, 0, 64);
    double c = 0.0;  // the correction (e_j - y A_0) X
    for (int i0 = 0; i0 < n; i0 += 4) {
      const int i = i0 + s, ii = min(i, n - 1);
      const double ei = __shfl(e, ii, 64);
      c = __builtin_fma(i < n ? ei : 0.0, x0[ii * n + vv], c);
    }
    c += __shfl_xor(c, 16, 64);
    c += __shfl_xor(c, 32, 64);
    double cv[LX], r[LX];
    md::zero<LX>(cv);
    cv[0] = c;
    MD<LX>::add(y, cv, r);
    md::copy<LX>(r, y);
    if (pass == 0 || !(om <= refine_floor(limbs))) rho = fmax(rho, om / fmax(prev, refine_floor(limbs)));
    if (last && om * fmax(rho, 0x1p-53) * 64.0 <= done) break;
    prev = om;
    limbs = pass == 0 ? 2 : last ? LX : L;
    if (!(rho <= 0x1p-8) || pass >= 8 * L) return false;  // not contracting (or not finite)
  }
  if (col && s == 0) {
#pragma unroll
    for (int l = 0; l < L; ++l) M[(size_t)l * nn + j * n + v] = y[l];
  }
  return true;
}

template <int L>
__global__ void __launch_bounds__(PREPASS_NT) prepass_small_kernel(EvalArgs a, const int32_t *asm_ptr,
                                                                 const int32_t *asm_ent, double *a0, double *x0,
                                                                 double *invd, double *M, int32_t *status, int *done) {
  // on the chain of the step, beside the evaluation: raised issue priority
  __builtin_amdgcn_s_setprio(3);
  constexpr int NN = PREPASS_MAXN * PREPASS_MAXN;
  __shared__ double as[L * NN], xs[NN], shr[8 * 8 + 16];
  __shared__ int need, sing;
  const int n = a.n, nn = n * n, tid = threadIdx.x;
  if (tid == 0 && a.reset_status) *a.reset_status = MD_OK;
  for (int t0 = 0; t0 < a.m; t0 += PREPASS_NT) {
    const bool ok = eval0_monomial<L>(a, t0 + tid, [&] { return t0 > 0 || eval0_wait(a); });
    if (!ok) return;  // (the whole workgroup)
  }
  __syncthreads();
  // A_0, summed in the order of the assembly of A
  const size_t zD = (size_t)a.nnz * a.D;
  for (int ij = tid; ij < nn; ij += PREPASS_NT) {
    const int lo = asm_ptr[ij], hi = asm_ptr[ij + 1];
    double acc[L];
    md::zero<L>(acc);
    for (int t = lo; t < hi; ++t) {
      double y[L], r[L];
      ld<L>(a.der, zD, (size_t)asm_ent[t] * a.D, y);
      if (t == lo) {
        md::copy<L>(y, acc);
      } else {
        MD<L>::add(acc, y, r);
        md::copy<L>(r, acc);
      }
    }
    st<L>(a0, nn, ij, acc);
#pragma unroll
    for (int l = 0; l < L; ++l) as[l * nn + ij] = acc[l];
  }
  __syncthreads();
  inv64_matrix<L, 1, 8, PREPASS_NT / 64>(n, as, xs, &need);
  __syncthreads();
  if (!need) {
    __syncthreads();  // (need was read)
    for (int j = tid >> 6; j < n; j += PREPASS_NT / 64)
      if (!refine_row_small<L>(n, j, as, xs, M)) need = 1;
    __syncthreads();
  }
  if (need) {
    factor_matrix<L>(n, 8, a0, x0, invd, M, shr, sing);
    __syncthreads();
    if (tid == 0 && sing) set_status(status, MD_ESINGULAR);
  }
  if (done) {  // a reader on another stream polls *done, n counts
    __syncthreads();
    for (int e = tid; e < nn; e += PREPASS_NT) {
      double y[L];
      ld<L>(M, nn, e, y);
      st_agent<L>(M, nn, e, y);
    }
    wait_vm();
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(done, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Systems that one workgroup takes in about the time of two launches: the
// registers of the coefficient-0 products, a few rounds of monomials, and rows
// that four wavefronts refine in two (quad double) or four rounds.
bool prepass_small(int L, int n, int m, int maxk) {
  return m > 0 && m <= 2 * PREPASS_NT && maxk <= evaldiff0_max_support(L) && ((L == 2 && n <= 16) || (L == 4 && n <= 8));
}

hipError_t launch_prepass_small(int L, const EvalArgs &a, const int32_t *asm_ptr, const int32_t *asm_ent, double *a0,
                                double *x0, double *invd, double *M, int32_t *status, int *done, hipStream_t st) {
  if (L == 2)
    hipLaunchKernelGGL(prepass_small_kernel<2>, dim3(1), dim3(PREPASS_NT), 0, st, a, asm_ptr, asm_ent, a0, x0, invd, M,
                       status, done);
  else if (L == 4)
    hipLaunchKernelGGL(prepass_small_kernel<4>, dim3(1), dim3(PREPASS_NT), 0, st, a, asm_ptr, asm_ent, a0, x0, invd, M,
                       status, done);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mdk
