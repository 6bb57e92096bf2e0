// Evaluation and differentiation of a polynomial system at a power series
// (Section 5.1: reverse mode of algorithmic differentiation with power-series
// products; Section 6: operands staged through shared memory into registers).
// The sums into b(t) = -p(x(t)) and the Jacobian series A(t) are in
// assemble.hip.
//
// Work decomposition.  Two teams of lanes per monomial (evaldiff_team_kernel);
// beside a running QR, and in the batched step, one "worker", a group of G
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
#include "evaldiff_dev.hpp"

namespace mdk {

// Two teams of lanes per monomial.  Team B forms the backward chain while team
// A forms the common factor; then at every forward step A forms f_j = f_{j-1} *
// x_{v_j} while B forms the cross product f_{j-1} * b_{k-j} of the same f_{j-1},
// so the chain of dependent products shortens from 3k - 5 to about 2k - 2
// (values only: team A alone).
//
// Within a product the outputs are paired, o1 = p and o2 = D-1-p, and the D+1
// terms of a pair, those of o2 first, are split over four lanes (quarters) of
// the team's 4 G2, G2 = pair_lanes: the chain of a product is a quarter of a
// pair's terms, and only the last two quarters change from o2 to o1.  The
// quarters' level sums are added pairwise; the lanes of quarter 0 (o2) and
// quarter 3 (o1) finish one coefficient each, which they keep in registers
// from product to product.  U (the f of the forward chain, B's chain ahead of
// it) and V are in LDS, a stride known at compile time apart, with entry D
// zero for masked terms.
//
// Orders up to 8 leave room for several monomials in a wavefront.
//
// Bound by the FP64 issue rate (quad double, 2048 monomials, order 64: 230 us,
// 128 for the multiply-adds alone) and, in small systems, by the longest
// monomial's chain.  Against one wavefront per team (orders 33 and up) and one
// worker per monomial (below), in us: quad double 2048 monomials of order 64
// 243 -> 230, 1463 of order 51 150 -> 101, 1024 of order 32 130 -> 49, 2048
// of order 1 54 -> 25; double double 2048 of order 64 97 -> 52, 64 of order 16
// 14 -> 8.
template <int G2> struct TeamLane {
  int D, quarter, p, o1, o2;
  int own;     // the coefficient the lane finishes, or -1
  int t0, t1;  // the lane's terms
};

template <int G2>
__device__ __forceinline__ TeamLane<G2> team_lane(int D, int tl) {
  TeamLane<G2> q;
  q.D = D;
  q.quarter = tl / G2;
  q.p = tl - q.quarter * G2;
  q.o1 = min(q.p, (D - 1) / 2);  // (lanes without a pair repeat the last one)
  q.o2 = D - 1 - q.o1;
  q.own = q.p > q.o1 ? -1 : q.quarter == 0 ? q.o2 : (q.quarter == 3 && q.o2 > q.o1) ? q.o1 : -1;
  // o2 has at least half = ceil((D + 1) / 2) terms
  const int half = (D + 2) / 2, h0 = (half + 1) / 2, h1 = half + (D + 2 - half) / 2;
  q.t0 = q.quarter == 0 ? 0 : q.quarter == 1 ? h0 : q.quarter == 2 ? half : h1;
  q.t1 = q.quarter == 0 ? h0 : q.quarter == 1 ? half : q.quarter == 2 ? h1 : D + 1;
  return q;
}

// Workgroup barrier; one wavefront needs none of its own.
template <bool WIDE>
__device__ __forceinline__ void team_sync() {
  if constexpr (WIDE) __syncthreads();
  else wave_sync();
}

// The level sums of the lane's terms of U V: part2 of output o2, part1 of o1.
template <int L, int G2>
__device__ __forceinline__ void team_conv(const double *U, const double *V, const TeamLane<G2> &q, double (&part1)[L],
                                          double (&part2)[L]) {
  constexpr int Dp = 2 * G2 + 1;
  double acc[L], parked[L];
  md::zero<L>(acc);
  md::zero<L>(parked);
  const int H = ((q.D + 2) / 2 + 1) / 2;  // terms of quarter 0; the others have as many or one less
  const bool ahead = q.t0 <= q.o2;
  const int i0 = ahead ? q.t0 : q.t0 - q.o2 - 1;
  const double *pu = U + i0, *pv = V + ((ahead ? q.o2 : q.o1) - i0), *const pv1 = V + q.o1;
  auto term = [&] {
    double u[L], v[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      u[l] = pu[l * Dp];
      v[l] = pv[l * Dp];
    }
    MD<L>::fma_lazy(acc, u, v);
  };
  const int park = q.o2 - q.t0;  // o2's last term
  auto advance = [&](int tt) {
    const bool change = tt == park;
    pu = change ? U : pu + 1;
    pv = change ? pv1 : pv - 1;
    if (__any(change)) {
      if (change) {
        md::copy<L>(acc, parked);
        md::zero<L>(acc);
      }
    }
  };
  int tt = 0;
  for (; tt + 2 < H; tt += 2) {
    term();
    advance(tt);
    term();
    advance(tt + 1);
  }
  if (tt + 1 < H) {
    term();
    advance(tt);
  }
  if (q.t1 - q.t0 < H) {
    pu = U + q.D;
    pv = V;
  }
  term();
  const bool changed = park < H - 1;  // the lane ended on o1
#pragma unroll
  for (int l = 0; l < L; ++l) {
    part2[l] = changed ? parked[l] : acc[l];
    part1[l] = changed ? acc[l] : 0.0;
  }
}

// LDS of one monomial: U and V of both teams, then per team the exchange of
// partial sums.
template <int L, int G2>
constexpr size_t team_doubles() {
  return (size_t)(4 * (2 * G2 + 1) + 2 * (G2 > 32 ? 4 : G2 > 16 ? 1 : 0) * G2) * L;
}

template <int L, int G2>
__device__ void eval_monomial_team(const EvalArgs &a, int mono, int tid, double *lds) {
  constexpr int TL = 4 * G2, Dp = 2 * G2 + 1;
  constexpr bool WIDE = 2 * TL > 64, ALONE = 2 * TL >= 64;  // ALONE: one monomial per workgroup
  const int Dc = a.Dc, D = a.D;
  const bool derivs = a.values_only == 0;
  const bool isA = tid < TL;
  const int team = isA ? 0 : 1, tl = tid - team * TL;
  const TeamLane<G2> q = team_lane<G2>(Dc, tl);
  const bool owner = q.own >= 0;
  const int s = owner ? q.own : 0;
  double *UA = lds;
  double *Uown = lds + team * 2 * L * Dp, *V = Uown + L * Dp;
  double *X = lds + 4 * L * Dp + team * (G2 > 32 ? 4 : 1) * G2 * L;
  for (int r = tl; r < 4 * L; r += TL) lds[r * Dp + Dc] = 0.0;
  int e0 = a.mon_ptr[mono], e1 = a.mon_ptr[mono + 1];
  if constexpr (ALONE) {
    e0 = __builtin_amdgcn_readfirstlane(e0);
    e1 = __builtin_amdgcn_readfirstlane(e1);
  }
  const int k = e1 - e0;
  const size_t nD = (size_t)a.n * D, mD = (size_t)a.m * D, zD = (size_t)a.nnz * D;
  const size_t xls = a.x_ls ? a.x_ls : nD;
  double c[L];
  ld<L>(a.cff, a.cff_ls ? a.cff_ls : (size_t)a.m, mono, c);
  if (k == 0) {  // constant monomial (all of its lanes leave)
    if (isA && owner) {
#pragma unroll
      for (int l = 0; l < L; ++l) a.val[(size_t)l * mD + (size_t)mono * D + s] = (s == 0) ? c[l] : 0.0;
      if (a.vsize) a.vsize[(size_t)mono * D + s] = (s == 0) ? fabs(c[0]) : 0.0;
    }
    return;
  }
  // this lane's coefficient of a series in memory; zero for lanes without one
  auto load = [&](const double *g, size_t ls, size_t off, double (&r)[L]) {
    md::zero<L>(r);
    if (owner) ld<L>(g, ls, off + s, r);
  };
  auto load_x = [&](int e, double (&r)[L]) { load(a.x, xls, (size_t)a.var[e0 + e] * D, r); };
  auto put = [&](double *W, const double (&r)[L]) {
    if (owner) {
#pragma unroll
      for (int l = 0; l < L; ++l) W[l * Dp + s] = r[l];
    }
  };
  auto store_der = [&](int e, const double (&r)[L]) {
    if (owner) st<L>(a.der, zD, (size_t)(e0 + e) * D + s, r);
  };

  int nbig = 0;
  for (int j = 0; j < k; ++j) nbig += a.exp[e0 + j] >= 2 ? 1 : 0;
  const bool f0_scalar = nbig == 0;
  // steps: the common factor CF = prod x^(a-1) (A) beside the backward chain
  // b_q, q = 2..k-1, parked in the slot of entry k-q-1 (B), then the forward
  // chain (A) beside the cross products (B)
  const int steps_a = max(nbig - 1, 0), steps_b = derivs ? max(k - 2, 0) : 0;
  const int start = max(steps_a, steps_b), total = start + k;
  double f[L];  // f_j (A), b_q (B)
  md::zero<L>(f);
  int next = 0;  // entry of the next factor of CF
  auto load_cf = [&](double (&w)[L]) {
    while (a.exp[e0 + next] < 2) ++next;
    const int p = a.exp[e0 + next] - 1, v = a.var[e0 + next];
    ++next;
    if (p == 1) load(a.x, xls, (size_t)v * D, w);
    else load(a.pw + (size_t)(p - 2) * L * nD, nD, (size_t)v * D, w);
  };
  if (isA && !f0_scalar) load_cf(f);
  if (!isA && steps_b > 0) load_x(k - 1, f);  // b_1
  const bool track = a.vsize != nullptr;
  double vmax = 0.0;
  for (int t = 0; t < total; ++t) {
    const int j = t - start + 1;  // forward step (from 1), else an earlier one
    const int ej = j - 1, aj = j >= 1 ? a.exp[e0 + ej] : 1;
    if (j == 1 && isA) {  // f_0 = c CF (c in coefficient 0 without a common factor)
      if (!f0_scalar) {
        double w[L];
        MD<L>::mul(c, f, w);
        md::copy<L>(w, f);
      } else {
#pragma unroll
        for (int l = 0; l < L; ++l) f[l] = s == 0 ? c[l] : 0.0;
      }
      vmax = fabs(f[0]);
    }
    const bool scalar = f0_scalar && j == 1;
    const bool run = j < 1 ? t < (isA ? steps_a : steps_b) : (isA || j < k);
    double r[L];
    if (run) {  // the operand V
      double w[L];
      if (j < 1) {
        if (isA) load_cf(w);
        else load_x(k - 2 - t, w);  // x_{v_{k-q+1}}, q - 2 = t
      } else if (isA) {
        load_x(ej, w);
      } else if (k - j == 1) {
        load_x(k - 1, w);  // b_1 = x_{v_k}
      } else {
        load(a.der, zD, (size_t)(e0 + ej) * D, w);  // b_{k-j}, which this lane stored
      }
      if (scalar) MD<L>::mul(c, w, r);
      else put(V, w);
      if ((isA || j < 1) && !scalar) put(Uown, f);
    }
    if (isA && derivs && j == k) {  // d/dx_{v_k} = a_k f_{k-1}
      double w[L];
      md::copy<L>(f, w);
      md::mul_int<L>(w, aj);
      store_der(ej, w);
    }
    if (!scalar) {  // r = U V, this lane's coefficient; U and V are free afterwards
      team_sync<WIDE>();
      double mine[L], send[L];
      if (run) {
        team_conv<L, G2>(j < 1 ? Uown : UA, V, q, send, mine);
        // quarters 0, 1, 2 go on with o2, quarter 3 with o1
#pragma unroll
        for (int l = 0; l < L; ++l) {
          const double p1 = send[l], p2 = mine[l];
          mine[l] = q.quarter == 3 ? p1 : p2;
          send[l] = q.quarter == 2 ? p1 : p2;
        }
      } else {
        md::zero<L>(mine);
        md::zero<L>(send);
      }
      double o[L];
      if constexpr (G2 <= 32) {
#pragma unroll
        for (int l = 0; l < L; ++l) o[l] = __shfl_xor(send[l], G2, 64);
      } else {
        if (q.quarter > 0) {
#pragma unroll
          for (int l = 0; l < L; ++l) X[(q.quarter * L + l) * G2 + q.p] = send[l];
        }
        team_sync<WIDE>();
#pragma unroll
        for (int l = 0; l < L; ++l) o[l] = q.quarter == 1 ? 0.0 : X[((q.quarter ^ 1) * L + l) * G2 + q.p];
      }
      MD<L>::add_lazy(mine, o);
      if constexpr (G2 <= 16) {
#pragma unroll
        for (int l = 0; l < L; ++l) o[l] = __shfl_xor(mine[l], 2 * G2, 64);
        team_sync<WIDE>();
      } else {
        if (q.quarter == 2) {
#pragma unroll
          for (int l = 0; l < L; ++l) X[l * G2 + q.p] = mine[l];
        }
        team_sync<WIDE>();
#pragma unroll
        for (int l = 0; l < L; ++l) o[l] = X[l * G2 + q.p];
      }
      if (q.quarter == 0) MD<L>::add_lazy(mine, o);
      MD<L>::renorm(mine, r);
    }
    if (isA) {
      if (run) md::copy<L>(r, f);
      if (j >= 1) vmax = fmax(vmax, fabs(f[0]));
    } else if (run) {
      if (j < 1) {
        md::copy<L>(r, f);
        store_der(k - 3 - t, r);
      } else {
        md::mul_int<L>(r, aj);
        store_der(ej, r);
      }
    }
  }
  if (isA && owner) {
    st<L>(a.val, mD, (size_t)mono * D + s, f);
    if (track) a.vsize[(size_t)mono * D + s] = vmax;
  }
}

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

// Coefficient 0 of every derivative product (the entries of A_0), one
// thread per monomial, for supports of at most EVAL0_MAXK variables.  The
// same products as evaldiff_kernel restricted to the constant coefficients,
// which are plain multiple-double products: f_0 = c * CF(0), forward
// products f_j = f_{j-1} x_{v_j}(0) kept in registers, then the backward
// products b formed on the way back, d/dx_{v_j} = a_j f_{j-1} b_{k-j}.  The
// loads of the k constant coefficients are issued before the products, so
// the thread waits for memory once.
constexpr int EVAL0_MAXK = 8;

template <int L>
__global__ void __launch_bounds__(256) evaldiff0_kernel(EvalArgs a) {
  // it opens the factorization's chain, which runs beside the staged solve
  // and the evaluation: the highest issue priority on a shared CU
  __builtin_amdgcn_s_setprio(3);
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  // the step's status word, reset by its first launch (every launch that can
  // report into it comes later in stream order; no evaluation kernel does)
  if (t == 0 && a.reset_status) *a.reset_status = MD_OK;
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
  if (a.wait_ctr) {
    __shared__ int ok;
    if (threadIdx.x == 0) ok = wait_count(a.wait_ctr, a.wait_target, a.wait_status) ? 1 : 0;
    __syncthreads();
    if (!ok) return;
  }
  if (!live || k == 0) return;  // k == 0: no derivatives
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

// Octo doubles would spill the registers of this kernel: they take the
// general kernel with one coefficient.
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
