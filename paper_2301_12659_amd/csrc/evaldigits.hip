// Evaluation and differentiation by convolutions on digits (digits.hpp): the
// products of evaldiff.hip (forward, backward and cross products, common
// factors) with every truncated product formed as plain fused multiply-adds of
// digits instead of multiple-double level sums.
//
// Work decomposition.  One workgroup per monomial, two teams of TL = 2 G2 lanes
// (G2 = pair_lanes: 16, 32, 64 for orders up to 32, 64, 128).  They share the
// products of the common factor and of the backward chain; then at every forward
// step A forms f_j = f_{j-1} x_{v_j} while B forms the cross product
// f_{j-1} b_{k-j} of the same f_{j-1} (values only: team A alone).  Within a
// product the outputs are paired, o1 = p and o2 = D-1-p, so that every pair has
// D+1 terms, split over lanes p (half 0: the first part of o2) and p + G2 (half
// 1: the rest of o2, then o1) in chunks of four terms, so that the change from
// o2 to o1 sits at a chunk's edge.  Lane p then finishes output o2, lane p + G2
// output o1:
// every lane owns one coefficient of every series, which it loads, rounds to
// limbs, stores and writes back as digits.
//
// LDS: the digits of three series (the operand U, which the teams share or use
// in turn, and each team's V), [S][TL + 1] doubles (a stride known at compile
// time) with entry D zero for masked terms and, ahead of V, PAD rows of zeros:
// a term whose exponents are delta digits below the sum's largest reads V's
// digits delta rows further up.  A product that meets a larger delta is formed
// again with the row index clamped at the first zero row.
//
// Bound by the FP64 issue rate: 231 (octo double) or 78 (quad double) fused
// multiply-adds per term on independent accumulators, against 960 and 112
// dependent instructions for the level sums.  The next term's digits are
// loaded into the registers that the current term's rows leave.  Three series
// instead of four (the common factor beside the backward chain) leave room for
// two workgroups per CU at order 128 in octo doubles.  Measured (octo double, 8192
// monomials, order 128; 43.9 ms by level sums): 17.9 ms with
// the single products formed by one team while the other waits, 13.7 shared.
#include "digits.hpp"
#include "evaldiff_dev.hpp"

namespace mdk {

constexpr int DIGIT_PAD = 3;

// A series in LDS: digit p of coefficient s at d[p * Dp + s], its exponent r[s],
// DIGIT_MASK for four entries ahead of the first and behind the last.
struct DigitSeries {
  double *d;
  int *r;
};

// Lane-wise constants of the products of order D (G2 = pair_lanes(D)).
struct DigitLane {
  int D, half, p, o1, o2;
  bool act;   // the lane's pair exists
  int own;    // the coefficient the lane finishes, or -1
  int chunks; // chunks of four terms per half
  int nc2, c0;  // chunks of o2; first chunk of the lane's half
};

template <int G2>
__device__ __forceinline__ DigitLane digit_lane(int D, int tl) {
  DigitLane q;
  q.D = D;
  q.half = tl >= G2 ? 1 : 0;
  q.p = tl - q.half * G2;
  q.act = q.p < (D + 1) / 2;
  q.o1 = q.p;
  q.o2 = D - 1 - q.p;
  q.own = !q.act ? -1 : (q.half == 0 ? q.o2 : (q.o2 > q.o1 ? q.o1 : -1));
  int nc = 0;
  for (int b = 0; b < 4 && b < (D + 1) / 2; ++b) nc = max(nc, (b + 4) / 4 + (D - b + 3) / 4);
  q.chunks = (nc + 1) / 2;
  q.nc2 = (q.o2 + 4) >> 2;
  q.c0 = q.half ? min(q.chunks, q.nc2) : 0;
  return q;
}

// The chunks of a lane: chunk c of its half is chunk c0 + c of the pair, four
// terms i = i0 .. i0 + 3 of output o2 (before chunk nc2) or o1.
struct DigitChunk {
  int i0, o;
  bool second;
};
__device__ __forceinline__ DigitChunk digit_chunk(const DigitLane &q, int c) {
  const int cc = q.c0 + c;
  DigitChunk t;
  t.second = cc < q.nc2;
  t.i0 = 4 * (t.second ? cc : cc - q.nc2);
  t.o = t.second ? q.o2 : q.o1;
  // nothing to do: past the end of o1, o1 == o2, half 0 beyond o2, no pair
  if (t.i0 > t.o || !q.act || (!t.second && (!q.half || q.o2 <= q.o1))) {
    t.i0 = 0;
    t.o = -4;  // the terms' V entry is ahead of the first
  }
  return t;
}

// Sums of the exponents of a chunk's terms; masked terms (past the output)
// fall on the entries that hold DIGIT_MASK, below any sum of two exponents.
__device__ __forceinline__ void chunk_exponents(const DigitSeries &U, const DigitSeries &V, const DigitChunk &t,
                                                int (&sum)[4]) {
  const int *u = U.r + t.i0, *v = V.r + max(t.o - t.i0, -1);
#pragma unroll
  for (int e = 0; e < 4; ++e) sum[e] = u[e] + v[t.o < 0 ? 0 : -e];
}

// The largest exponents R1, R2 of the terms of outputs o1 and o2 in chunks
// cbeg .. cend - 1 of the lane's half.
__device__ __forceinline__ void digit_exponents(const DigitSeries &U, const DigitSeries &V, const DigitLane &q, int &R1,
                                                int &R2, int cbeg, int cend) {
  R1 = R2 = 2 * DIGIT_ZERO;
#pragma unroll 2
  for (int c = cbeg; c < cend; ++c) {
    const DigitChunk t = digit_chunk(q, c);
    int s[4];
    chunk_exponents(U, V, t, s);
    const int m = max(max(s[0], s[1]), max(s[2], s[3]));
    if (t.second) R2 = max(R2, m);
    else R1 = max(R1, m);
  }
}

// Accumulators of the lane's own output of U * V (z, exponent R: the value is
// sum_k z_k 2^(23 (R - k - 2))) less what the lane of the other half holds of
// it.  Half 0 has only terms of o2, with the same i in all lanes (U is read as
// a broadcast), and so does half 1 until its lanes turn to o1 one after the
// other.  Half 0 finishes o2 and half 1 o1; half 1's part of o2 is parked in
// other, as digits.  Chunks cbeg .. cend - 1 of the half: the others are another
// team's, whose z and other add to these.  Returns false where a term needed
// more than DIGIT_PAD rows of shift (WIDE: never).
template <int S, int Dp, bool WIDE>
__device__ __forceinline__ bool conv_digits(const DigitSeries &U, const DigitSeries &V, const DigitLane &q, int R1,
                                            int R2, int cbeg, int cend, double (&z)[S], double (&other)[S]) {
  bool far = false;
  const double *up, *vp;
  int vrow = 0;  // WIDE: -delta
  // the current and the next chunk: indices and shifts
  DigitChunk t, tn;
  int d[4], dn[4];
  auto fetch = [&](int c) {
    tn = digit_chunk(q, c);
    chunk_exponents(U, V, tn, dn);
    const int R = tn.second ? R2 : R1;
#pragma unroll
    for (int e = 0; e < 4; ++e) dn[e] = R - dn[e];
  };
  // the addresses of a term's digits (U's zero entry if masked)
  auto locate = [&](const DigitChunk &c, int shift, int e) {
    const bool on = shift < S;
    int delta = on ? shift : 0;
    if (!WIDE) {
      far = far || delta > DIGIT_PAD;
      delta = min(delta, DIGIT_PAD);
    }
    up = U.d + (on ? c.i0 + e : q.D);
    vp = V.d + (on ? c.o - c.i0 - e : 0);
    if (WIDE) vrow = -delta;
    else vp -= delta * Dp;
  };
  auto ldv = [&](int k) -> double {
    if constexpr (WIDE) return vp[max(k + vrow, -1) * Dp];
    else return vp[k * Dp];
  };
  double acc[S], u[S], v[S];
#pragma unroll
  for (int k = 0; k < S; ++k) acc[k] = other[k] = 0.0;
  fetch(cbeg);
  locate(tn, dn[0], 0);
#pragma unroll
  for (int k = 0; k < S; ++k) {
    u[k] = up[k * Dp];
    v[k] = ldv(k);
  }
  constexpr int FLUSH = 504 / S / 4;  // chunks between carries: sums of at most 504 products
  int since = 0;
#pragma unroll 1
  for (int c = cbeg; c < cend; ++c) {
    if (q.c0 + c == q.nc2 && q.half) {  // o2 complete
#pragma unroll
      for (int k = 0; k < S; ++k) {
        other[k] = acc[k];
        acc[k] = 0.0;
      }
    }
    t = tn;
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = dn[e];
    fetch(c + 1);  // past the last chunk: another part's or masked, unused
#pragma unroll(S <= 12 && !WIDE ? 4 : 1)
    for (int e = 0; e < 4; ++e) {
      // the next term's digits arrive while this one's rows run
      const int en = (e + 1) & 3;
      const int sh = e == 0 ? d[1] : e == 1 ? d[2] : e == 2 ? d[3] : dn[0];
      locate(e < 3 ? t : tn, sh, en);
#pragma unroll
      for (int a = 0; a < S; ++a) {
        // the highest digit last: its successor was loaded last
#pragma unroll
        for (int b = S - 1 - a; b >= 0; --b) acc[a + b] = __builtin_fma(u[a], v[b], acc[a + b]);
        if (a & 1) {  // two rows' operands are free: pairs of loads
          u[a - 1] = up[(a - 1) * Dp];
          u[a] = up[a * Dp];
          v[S - 1 - a] = ldv(S - 1 - a);
          v[S - a] = ldv(S - a);
        } else if (a == S - 1) {
          u[a] = up[a * Dp];
          v[0] = ldv(0);
        }
      }
    }
    if (++since == FLUSH) {
      since = 0;
      carry_digits<S>(acc);
    }
  }
  if (q.c0 + cend <= q.nc2 && q.half) {  // all of it o2
#pragma unroll
    for (int k = 0; k < S; ++k) {
      other[k] = acc[k];
      acc[k] = 0.0;
    }
  }
  carry_digits<S>(other);
#pragma unroll
  for (int k = 0; k < S; ++k) z[k] = acc[k];
  return !far;
}

// Barrier of the workgroup: one wavefront needs none of its own.
struct DigitSync {
  bool wide;
  __device__ __forceinline__ void operator()() const {
    if (wide) __syncthreads();
    else wave_sync();
  }
};

template <int L, int G2>
__device__ void eval_monomial_digits(const EvalArgs &a, int mono, char *lds) {
  constexpr int S = Digits<L>::S, TL = 2 * G2, Dp = TL + 1, RP = TL + 8;  // RP: exponents of a series with their pads
  const int Dc = a.Dc, D = a.D;
  const bool derivs = a.values_only == 0;
  const int tid = threadIdx.x;
  const bool isA = tid < TL;
  const int tl = isA ? tid : tid - TL;
  const DigitSync sync{blockDim.x > 64};
  const DigitLane q = digit_lane<G2>(Dc, tl);
  const bool owner = q.own >= 0;
  const int s = owner ? q.own : 0;
  // LDS: U [S][Dp], per team V [PAD + S][Dp], the exponents of each, the
  // exchange of the largest exponents
  const size_t ud = (size_t)S * Dp, vd = (size_t)(S + DIGIT_PAD) * Dp;
  double *base = reinterpret_cast<double *>(lds);
  const int teams = derivs ? 2 : 1, team = isA ? 0 : 1;
  int *rbase = reinterpret_cast<int *>(base + ud + teams * vd);
  const DigitSeries U{base, rbase + 4};
  const DigitSeries V{base + ud + team * vd + (size_t)DIGIT_PAD * Dp, rbase + (1 + team) * RP + 4};
  const DigitSeries VA{base + ud + (size_t)DIGIT_PAD * Dp, rbase + RP + 4};
  int *rx = rbase + (1 + teams) * RP;  // [team][2 TL]
  for (int k = tl; k < DIGIT_PAD * Dp; k += TL) V.d[k - DIGIT_PAD * Dp] = 0.0;
  for (int k = tid; k < (1 + teams) * RP; k += blockDim.x) rbase[k] = DIGIT_MASK;
  if (isA && tl < S) U.d[tl * Dp + Dc] = 0.0;
  sync();
  const int e0 = __builtin_amdgcn_readfirstlane(a.mon_ptr[mono]);
  const int k = __builtin_amdgcn_readfirstlane(a.mon_ptr[mono + 1]) - e0;
  const size_t nD = (size_t)a.n * D, mD = (size_t)a.m * D, zD = (size_t)a.nnz * D;
  const size_t xls = a.x_ls ? a.x_ls : nD;
  double c[L];
  ld<L>(a.cff, a.cff_ls ? a.cff_ls : (size_t)a.m, mono, c);
  if (k == 0) {  // constant monomial (the whole workgroup leaves)
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
  auto put = [&](const DigitSeries &W, const double (&r)[L]) {
    double d[S], w[L];
    int rho;
    md::copy<L>(r, w);
    tidy_limbs<L>(w);
    to_digits<L, S>(w, d, rho);
    if (owner) {
#pragma unroll
      for (int p = 0; p < S; ++p) W.d[p * Dp + s] = d[p];
      W.r[s] = rho;
    }
  };
  auto store_der = [&](int e, const double (&r)[L]) {
    if (owner) st<L>(a.der, zD, (size_t)(e0 + e) * D + s, r);
  };

  int nbig = 0;
  for (int j = 0; j < k; ++j) nbig += a.exp[e0 + j] >= 2 ? 1 : 0;
  const bool f0_scalar = nbig == 0;
  // steps with a product: the common factor CF = prod x^(a-1), the backward
  // chain b_q, q = 2..k-1, parked in the slot of entry k-q-1, then the forward
  // chain (A) beside the cross products (B).  Where there is one product only
  // (before the forward chain, and its last step) the teams share it: each
  // takes half of the chunks, A finishes.
  const int steps_a = max(nbig - 1, 0), steps_b = derivs ? max(k - 2, 0) : 0;
  double f[L], r[L];
  md::zero<L>(f);
  md::zero<L>(r);
  int next = 0;  // entry of the next factor of CF
  auto load_cf = [&](double (&w)[L]) {
    while (a.exp[e0 + next] < 2) ++next;
    const int p = a.exp[e0 + next] - 1, v = a.var[e0 + next];
    ++next;
    if (p == 1) load(a.x, xls, (size_t)v * D, w);
    else load(a.pw + (size_t)(p - 2) * L * nD, nD, (size_t)v * D, w);
  };
  if (!f0_scalar) load_cf(f);
  const bool track = a.vsize != nullptr;
  double vmax = 0.0;
  const int start = steps_a + steps_b, total = start + k;
  for (int t = 0; t < total; ++t) {
    const int j = t - start + 1;  // forward step (from 1), else an earlier one
    const int ej = j - 1, aj = j >= 1 ? a.exp[e0 + ej] : 1;
    if (j == 1 && steps_b > 0) sync();  // team B reads the parked products, which A stored
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
    const bool first = t < steps_a, back = !first && j < 1, scalar = f0_scalar && j == 1;
    const bool single = first || back || j == k;  // one product only
    const bool joint = single && teams == 2 && !scalar;
    const bool takes_v = joint ? !isA : (isA || !single);  // loads the operand V
    if (takes_v) {
      double w[L];
      if (first) load_cf(w);
      else if (back) load_x(k - 2 - (t - steps_a), w);  // x_{v_{k-q+1}}, q - 2 = t - steps_a
      else if (isA || j == k) load_x(ej, w);
      else if (k - j == 1) load_x(k - 1, w);  // b_1 = x_{v_k}
      else load(a.der, zD, (size_t)(e0 + ej) * D, w);  // b_{k-j}
      if (scalar) {  // times the coefficient
        if (derivs && j == k) {  // (team A) d/dx_{v_k} = a_k f_{k-1}
          md::copy<L>(f, r);
          md::mul_int<L>(r, aj);
          store_der(ej, r);
        }
        MD<L>::mul(c, w, r);
      } else {
        put(joint ? VA : V, w);
      }
    } else if (first) {
      int skip = next;  // (both teams count the factors)
      while (a.exp[e0 + skip] < 2) ++skip;
      next = skip + 1;
    }
    if (!scalar) {  // r = U V, this lane's coefficient; U and V are free afterwards
      if (isA) {
        if (derivs && j == k) {  // d/dx_{v_k} = a_k f_{k-1}
          md::copy<L>(f, r);
          md::mul_int<L>(r, aj);
          store_der(ej, r);
        }
        if (!back) md::copy<L>(f, r);
        else if (t == steps_a) load_x(k - 1, r);  // b_1
        put(U, r);
      }
      sync();
      const bool run = joint || takes_v;
      const DigitSeries W = joint ? VA : V;
      const int part = (q.chunks + 1) / 2;
      const int cbeg = joint && !isA ? part : 0, cend = joint && isA ? part : q.chunks;
      double z[S], other[S];
      int R1 = 0, R2 = 0;
      if (run) digit_exponents(U, W, q, R1, R2, cbeg, cend);
      if (G2 < 64 && !joint) {
        R1 = max(R1, __shfl_xor(R1, G2, 64));
        R2 = max(R2, __shfl_xor(R2, G2, 64));
      } else {
        rx[(team * TL + tl) * 2] = R1;
        rx[(team * TL + tl) * 2 + 1] = R2;
        sync();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int other_team = joint ? (e >> 1) : team;
          const int o = other_team * TL + ((e & 1) ? tl ^ G2 : tl);
          R1 = max(R1, rx[2 * o]);
          R2 = max(R2, rx[2 * o + 1]);
        }
      }
      if (run) {
        if (!__all(conv_digits<S, Dp, false>(U, W, q, R1, R2, cbeg, cend, z, other)))
          conv_digits<S, Dp, true>(U, W, q, R1, R2, cbeg, cend, z, other);
      } else {
#pragma unroll
        for (int p = 0; p < S; ++p) z[p] = other[p] = 0.0;
      }
      // half 1's part of o2 to the lane of half 0, team B's share to team A
      if (G2 < 64 && !joint) {
#pragma unroll
        for (int p = 0; p < S; ++p) {
          const double o = __shfl_xor(other[p], G2, 64);
          if (!q.half) z[p] += o;
        }
        sync();
      } else {  // through V
        sync();
        const bool send = joint && !isA;
        if (run && q.half) {
#pragma unroll
          for (int p = 0; p < S; ++p) W.d[p * Dp + q.p + (send ? G2 : 0)] = other[p];
        }
        if (joint) {
          carry_digits<S>(z);
          if (send) {
#pragma unroll
            for (int p = 0; p < S; ++p) V.d[p * Dp + tl] = z[p];
          }
        }
        sync();
        if (run && !send) {
          if (!q.half) {
#pragma unroll
            for (int p = 0; p < S; ++p) z[p] += W.d[p * Dp + q.p];
          }
          if (joint) {
            const double *zb = base + ud + vd + (size_t)DIGIT_PAD * Dp;
#pragma unroll
            for (int p = 0; p < S; ++p) {
              if (!q.half) z[p] += W.d[p * Dp + q.p + G2];
              z[p] += zb[p * Dp + tl];
            }
          }
        }
        sync();
      }
      if (run && !(joint && !isA)) from_digits<L, S>(z, q.half ? R1 : R2, r);
    }
    if (isA) {
      if (back) {
        store_der(k - 3 - (t - steps_a), r);
      } else {
        md::copy<L>(r, f);
        if (j >= 1) vmax = fmax(vmax, fabs(f[0]));
      }
    } else if (!single) {
      md::mul_int<L>(r, aj);
      store_der(ej, r);
    }
  }
  if (isA && owner) {
    st<L>(a.val, mD, (size_t)mono * D + s, f);
    if (track) a.vsize[(size_t)mono * D + s] = vmax;
  }
}

template <int L, int G2>
__global__ void __launch_bounds__(4 * G2, 2) evaldiff_digits_kernel(EvalArgs a) {
  extern __shared__ __align__(16) char ldsc[];
  eval_monomial_digits<L, G2>(a, __builtin_amdgcn_readfirstlane(a.order[blockIdx.x]), ldsc);
}

// Orders whose products fill a team of at least 32 lanes; measured in octo
// doubles at order 41: 537 us by level sums, 279 on digits.  Quad doubles stay with the
// level sums: 112 instructions per term against 78, and the digits' alignment
// and rounding cost more than that saves (order 64: 243 us against 316).
bool evaldiff_on_digits(int L, int Dc) { return L == 8 && Dc > 16; }

template <int L, int G2>
static hipError_t launch_T(const EvalArgs &a, hipStream_t st) {
  constexpr int S = Digits<L>::S, Dp = 2 * G2 + 1;
  const int teams = a.values_only ? 1 : 2;
  const size_t lds = ((size_t)S + teams * (S + DIGIT_PAD)) * Dp * sizeof(double) +
                     ((1 + teams) * (2 * G2 + 8) + teams * 4 * G2) * sizeof(int);
  static const bool large = [] {
    (void)hipFuncSetAttribute((const void *)evaldiff_digits_kernel<L, G2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              150 * 1024);
    (void)hipGetLastError();  // an attribute the runtime refuses must not be reported by the launch
    return true;
  }();
  (void)large;
  hipLaunchKernelGGL((evaldiff_digits_kernel<L, G2>), dim3(a.m), dim3(teams * 2 * G2), lds, st, a);
  return hipGetLastError();
}

template <int L>
static hipError_t launch_L(const EvalArgs &a, hipStream_t st) {
  switch (pair_lanes(a.Dc)) {
    case 16: return launch_T<L, 16>(a, st);
    case 32: return launch_T<L, 32>(a, st);
    case 64: return launch_T<L, 64>(a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_evaldiff_digits(int L, const EvalArgs &a, hipStream_t st) {
  if (a.m <= 0) return hipSuccess;
  if (!evaldiff_on_digits(L, a.Dc)) return hipErrorInvalidValue;
  return launch_L<8>(a, st);
}

}  // namespace mdk
