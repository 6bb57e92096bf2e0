// Evaluation and differentiation of a polynomial system at a power series
// (Section 5.1: reverse mode of algorithmic differentiation with power-series
// products; Section 6: operands staged through shared memory into registers).
// The sums into b(t) = -p(x(t)) and the Jacobian series A(t) are in
// assemble.hip.
//
// Work decomposition.  Two teams of lanes per monomial (evaldiff_team_kernel);
// beside a running QR, where monomials are short, one "worker", a group of G
// lanes of one wavefront, which evaluates and differentiates one whole
// monomial, product after product, with three series buffers in LDS.  In a
// truncated product c_s = sum_{i<=s} a_i b_{s-i} the outputs are paired, s and
// D-1-s, so every pair has exactly D+1 multiply-adds: the triangular work is
// balanced without the zero padding of the paper's kernels (which pad to D^2
// multiplications, Section 5.1).  A worker splits each pair over S = 2 lanes
// (S = 1 when D > 64) that take the first and second half of its D+1 terms; the
// halves of the second output are added at the end.  G = S * (smallest power of
// two >= ceil(D/2)).  Each lane accumulates its terms as multiple-double level
// sums and renormalizes once per output.
//
// Per monomial c * prod_j x_{v_j}^{a_j} with support v_1 < ... < v_k:
//   common factor   CF = prod_{a_j >= 2} x_{v_j}^{a_j - 1}   (the paper's systems
//                   have exponent one only; this reading keeps every derivative a
//                   single cross product), f_0 = c * CF (or the scalar c);
//   backward        b_1 = x_{v_k}, b_q = b_{q-1} * x_{v_{k-q+1}}, q = 2..k-1;
//   forward         f_j = f_{j-1} * x_{v_j}, j = 1..k, value = f_k;
//   cross           d/dx_{v_j} = a_j f_{j-1} * b_{k-j} (j < k), d/dx_{v_k} = a_k f_{k-1}.
// With exponents one and a scalar f_0 this is the paper's 3k-5 convolutions.
// The backward products are parked in the derivative slots of the entries
// that consume them, so no extra memory is needed.
#include "evaldiff0_dev.hpp"
#include "evaldiff_dev.hpp"

namespace mdk {

template <int L, int G2>
__global__ void __launch_bounds__((8 * G2 > 64 ? 8 * G2 : 64), L == 8 ? 2 : 4) evaldiff_team_kernel(EvalArgs a) {
  extern __shared__ __align__(16) double lds[];
  if constexpr (8 * G2 >= 64) {
    eval_monomial_team<L, G2>(a, __builtin_amdgcn_readfirstlane(a.order[blockIdx.x]), threadIdx.x, lds);
  } else {  // several monomials per wavefront
    const int lanes = a.values_only ? 4 * G2 : 8 * G2, per = blockDim.x / lanes;
    const int w = threadIdx.x / lanes, idx = blockIdx.x * per + w;
    if (idx >= a.m) return;
    eval_monomial_team<L, G2>(a, a.order[idx], threadIdx.x - w * lanes, lds + (size_t)w * team_doubles<L, G2>());
  }
}

template <int L>
__global__ void __launch_bounds__(256, (L == 8) ? 1 : 2) evaldiff_kernel(EvalArgs a) {
  extern __shared__ double lds[];
  const int G = worker_lanes(a.Dc);
  const int wpb = blockDim.x / G;  // workers per block
  const int wid = threadIdx.x / G, lane = threadIdx.x - wid * G;
  const int widx = blockIdx.x * wpb + wid;
  if (widx >= a.m) return;  // whole worker exits together
  eval_monomial<L>(a, a.order[widx], lane, lds + (size_t)wid * 3 * L * (a.Dc + 1));
}

template <int L>
__global__ void __launch_bounds__(256) evaldiff0_kernel(EvalArgs a) {
  // it opens the factorization's chain, which runs beside the staged solve
  // and the evaluation: the highest issue priority on a shared CU
  __builtin_amdgcn_s_setprio(3);
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  // the step's status word, reset by its first launch (every launch that can
  // report into it comes later in stream order; no evaluation kernel does)
  if (t == 0 && a.reset_status) *a.reset_status = MD_OK;
  (void)eval0_monomial<L>(a, t, [&] { return eval0_wait(a); });
}

hipError_t launch_evaldiff0(int L, const EvalArgs &a, hipStream_t st) {
  // one wavefront per workgroup: the few thousand monomials spread over as
  // many CUs as possible (each thread is a chain of dependent products)
  const dim3 grid((a.m + 63) / 64);
  switch (L) {
    case 1: hipLaunchKernelGGL(evaldiff0_kernel<1>, grid, dim3(64), 0, st, a); break;
    case 2: hipLaunchKernelGGL(evaldiff0_kernel<2>, grid, dim3(64), 0, st, a); break;
    case 4: hipLaunchKernelGGL(evaldiff0_kernel<4>, grid, dim3(64), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The same for supports of any size, and for octo doubles, whose registers the
// kernel above would spill: W lanes (a power of two) per monomial, each with a
// few consecutive variables.  The products of the variables ahead of a lane and
// behind it come from scans over the lanes, log2 W steps instead of a chain
// of 2k - 2 products; a lane then goes through its own variables.  Bound by the
// chain; measured in octo doubles: 160 monomials of 1 to 160 variables 1531 us
// as a chain of products.
template <int L>
__global__ void __launch_bounds__(64, L == 8 ? 1 : 2) evaldiff0_scan_kernel(EvalArgs a, int W) {
  const int lane = threadIdx.x, t = lane & (W - 1);
  const int idx = blockIdx.x * (64 / W) + lane / W;
  const bool live = idx < a.m;
  const int mono = live ? idx : 0;
  const int e0 = a.mon_ptr[mono], k = live ? a.mon_ptr[mono + 1] - e0 : 0;
  const int C = (k + W - 1) / W, j0 = min(t * C, k), j1 = min(j0 + C, k);
  const size_t nD = (size_t)a.n * a.D, zD = (size_t)a.nnz * a.D;
  auto load_x = [&](int j, double (&r)[L]) { ld<L>(a.x, nD, (size_t)a.var[e0 + j] * a.D, r); };
  auto der = [&](int j) { return (size_t)(e0 + j) * a.D; };
  auto times = [&](double (&f)[L], const double (&y)[L]) {
    double r[L];
    MD<L>::mul(f, y, r);
    md::copy<L>(r, f);
  };
  auto one = [&](double (&r)[L]) {
    md::zero<L>(r);
    r[0] = 1.0;
  };
  // the lane's products of its variables and of their common factors
  double pre[L], suf[L], cf[L];
  one(pre);
  one(cf);
  bool factors = false;
  for (int j = j0; j < j1; ++j) {
    double xv[L];
    load_x(j, xv);
    if (j == j0) md::copy<L>(xv, pre);
    else times(pre, xv);
    for (int p = 1; p < a.exp[e0 + j]; ++p) {
      factors = true;
      times(cf, xv);
    }
  }
  md::copy<L>(pre, suf);
  const bool any = __any(factors);
  for (int off = 1; off < W; off <<= 1) {
    double up[L], down[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      up[l] = __shfl_up(pre[l], off, W);
      down[l] = __shfl_down(suf[l], off, W);
    }
    if (t >= off) times(pre, up);
    if (t + off < W) times(suf, down);
    if (any) {
      double o[L];
#pragma unroll
      for (int l = 0; l < L; ++l) o[l] = __shfl_xor(cf[l], off, W);
      times(cf, o);
    }
  }
  {  // of the lanes ahead and behind, without the lane itself
    double up[L], down[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      up[l] = __shfl_up(pre[l], 1, W);
      down[l] = __shfl_down(suf[l], 1, W);
    }
    ld<L>(a.cff, a.m, mono, pre);
    if (any) times(pre, cf);  // f_0 = c CF
    if (t > 0) times(pre, up);
    if (t + 1 < W) md::copy<L>(down, suf);
    else one(suf);
  }
  for (int j = j1 - 1; j > j0; --j) {  // behind each of the lane's variables, parked in its slot
    double xv[L];
    st<L>(a.der, zD, der(j), suf);
    load_x(j, xv);
    times(suf, xv);
  }
  for (int j = j0; j < j1; ++j) {  // a_j (f_0 x_{v_1} .. x_{v_{j-1}}) (x_{v_{j+1}} .. x_{v_k})
    double d[L], xv[L];
    if (j > j0) ld<L>(a.der, zD, der(j), suf);
    MD<L>::mul(pre, suf, d);
    md::mul_int<L>(d, a.exp[e0 + j]);
    st<L>(a.der, zD, der(j), d);
    if (j + 1 < j1) {
      load_x(j, xv);
      times(pre, xv);
    }
  }
}

hipError_t launch_evaldiff0_scan(int L, const EvalArgs &a, int maxk, hipStream_t st) {
  int W = 1;
  while (W < maxk && W < 64) W <<= 1;
  const dim3 grid((a.m + 64 / W - 1) / (64 / W));
  if (a.m <= 0) return hipSuccess;
  MD_DISPATCH(L, hipLaunchKernelGGL(evaldiff0_scan_kernel<LL>, grid, dim3(64), 0, st, a, W));
  return hipGetLastError();
}

// Larger supports, and octo doubles, take the scans.
int evaldiff0_max_support(int L) { return L <= 4 ? EVAL0_MAXK : 0; }

// Powers x_v^p, p = 2..maxexp-1, for the common factors of exponents >= 3.
template <int L>
__global__ void __launch_bounds__(256, (L == 8) ? 1 : 2) power_kernel(int n, int D, int Dc, int maxp, const double *x, double *pw) {
  extern __shared__ double lds[];
  const int G = worker_lanes(Dc);
  const int wpb = blockDim.x / G;
  const int wid = threadIdx.x / G, lane = threadIdx.x - wid * G;
  const int v = blockIdx.x * wpb + wid;
  if (v >= n) return;
  double *U = lds + (size_t)wid * 3 * L * (Dc + 1), *X = U + L * (Dc + 1), *W = X + L * (Dc + 1);
  zero_pads(U, L, Dc, lane, G);
  const size_t nD = (size_t)n * D;
  load_series_t<L>(X, x, nD, (size_t)v * D, Dc, lane, G);
  load_series_t<L>(U, x, nD, (size_t)v * D, Dc, lane, G);
  wave_sync();
  for (int p = 2; p <= maxp; ++p) {
    conv_any<L>(U, X, W, Dc, lane, 1);
    wave_sync();
    store_series_t<L>(pw + (size_t)(p - 2) * L * nD, nD, (size_t)v * D, W, Dc, lane, G);
    double *t = U;
    U = W;
    W = t;
    wave_sync();
  }
}

// ------------------------------------------------------------------ launchers

template <int L, int G2>
static void launch_team(const EvalArgs &a, hipStream_t st) {
  const int lanes = a.values_only ? 4 * G2 : 8 * G2, per = 8 * G2 < 64 ? 64 / lanes : 1;
  const size_t lds = per * team_doubles<L, G2>() * sizeof(double);
  hipLaunchKernelGGL((evaldiff_team_kernel<L, G2>), dim3((a.m + per - 1) / per), dim3(per * lanes), lds, st,
                     a);
}

template <int L>
hipError_t launch_evaldiff_T(const EvalArgs &a, int maxexp, double *pw_mut, hipStream_t st) {
  const int G = worker_lanes(a.Dc);
  const int wpb = 256 / G;
  const size_t lds = (size_t)wpb * 3 * L * (a.Dc + 1) * sizeof(double);
  static bool attr_set = false;
  if (!attr_set) {  // dynamic LDS above 64 KB needs the attribute
    (void)hipFuncSetAttribute((const void *)power_kernel<L>, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
    (void)hipFuncSetAttribute((const void *)evaldiff_kernel<L>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              150 * 1024);
    (void)hipGetLastError();  // an attribute the runtime refuses must not be reported by the launch
    attr_set = true;
  }
  if (maxexp >= 3) {
    const int blocks = (a.n + wpb - 1) / wpb;
    hipLaunchKernelGGL(power_kernel<L>, dim3(blocks), dim3(256), lds, st, a.n, a.D, a.Dc, maxexp - 1, a.x, pw_mut);
  }
  if (evaldiff_on_digits(L, a.Dc)) return launch_evaldiff_digits(L, a, st);
  if (a.m > 0) {
    if (!a.beside_qr) {  // (one worker per monomial leaves a QR's wavefronts more issue slots)
      const int G2 = pair_lanes(a.Dc);
      if constexpr (L < 8) {  // (octo doubles: on digits from order 17 on)
        if (G2 == 16) launch_team<L, 16>(a, st);
        if (G2 == 32) launch_team<L, 32>(a, st);
        if (G2 == 64) launch_team<L, 64>(a, st);
      }
      switch (G2) {
        case 1: launch_team<L, 1>(a, st); break;
        case 2: launch_team<L, 2>(a, st); break;
        case 4: launch_team<L, 4>(a, st); break;
        case 8: launch_team<L, 8>(a, st); break;
      }
    } else {
      const int blocks = (a.m + wpb - 1) / wpb;
      hipLaunchKernelGGL(evaldiff_kernel<L>, dim3(blocks), dim3(256), lds, st, a);
    }
  }
  return hipGetLastError();
}

hipError_t launch_evaldiff(int L, const EvalArgs &a, int maxexp, double *pw, hipStream_t st) {
  switch (L) {
    case 1: return launch_evaldiff_T<1>(a, maxexp, pw, st);
    case 2: return launch_evaldiff_T<2>(a, maxexp, pw, st);
    case 4: return launch_evaldiff_T<4>(a, maxexp, pw, st);
    case 8: return launch_evaldiff_T<8>(a, maxexp, pw, st);
  }
  return hipErrorInvalidValue;
}

int evaldiff_workers_per_block(int D) { return pair_lanes(D) < 8 ? 8 / pair_lanes(D) : 1; }

}  // namespace mdk
