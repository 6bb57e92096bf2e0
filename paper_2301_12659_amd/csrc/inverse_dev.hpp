// Device routines of the inverse by refinement, shared by the single-system
// launches (inverse.hip, which describes the method) and the batched step.
#pragma once
#include <type_traits>

#include "common.hpp"

namespace mdk {

// Lane i's double, uniform over the wavefront (i uniform).
__device__ __forceinline__ double lane_f64(double x, int i) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, i);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), i);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sum of a double over `width` consecutive lanes (a power of two <= 64), in
// every lane of the team (the pairing of team_sum).
__device__ __forceinline__ double team_sum_f64(double v, int width) {
  if (width >= 2) v += dpp_f64<DPP_XOR1>(v);
  if (width >= 4) v += dpp_f64<DPP_XOR2>(v);
  if (width >= 8) v += dpp_f64<DPP_HALF_MIRROR>(v);
  if (width >= 16) v += dpp_f64<DPP_MIRROR>(v);
  if (width >= 32) v += __shfl_xor(v, 16, 64);
  if (width >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}

// Largest of a value over the wavefront, uniform.
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, DPP_XOR1, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, DPP_XOR2, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, DPP_HALF_MIRROR, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, DPP_MIRROR, 0xF, 0xF, false));
  const unsigned a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
  const unsigned c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
  return max(max(a, b), max(c, d));
}

// Exponents of the largest entries of a's rows (re) and, these taken out, of its
// columns (ce), by one workgroup of at least n threads; whether they differ by more
// than a few powers of two (uniform).
__device__ inline bool scale_exponents(int n, const double *a, int *re, int *ce) {
  constexpr int NONE = -(1 << 20);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, nw = blockDim.x >> 6;
  auto exponent = [&](int i, int j) {
    const double e = fabs(a[(size_t)i * n + j]);
    return e > 0.0 ? __builtin_amdgcn_frexp_exp(e) : NONE;
  };
  if (tid < n) ce[tid] = NONE;
  for (int i = w; i < n; i += nw) {
    int m = NONE;
    for (int j = lane; j < n; j += 64) m = max(m, exponent(i, j));
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, 64));
    if (lane == 0) re[i] = m;
  }
  __syncthreads();
  for (int j = lane; j < n; j += 64) {
    int m = NONE;
    for (int i = w; i < n; i += nw) m = max(m, exponent(i, j) - re[i]);
    atomicMax(&ce[j], m);
  }
  __syncthreads();
  return __syncthreads_or(tid < n && (abs(re[tid] - re[0]) >= 4 || abs(ce[tid] - ce[0]) >= 4)) != 0;
}

// In-place Gauss-Jordan inversion of the leading limbs of a ([n][n]
// row-major) by one workgroup of NW wavefronts, the matrix in registers: wavefront
// w owns the panel of NB columns from NB w on, lane i the rows i + 64 s of
// them.  The owner of a panel eliminates it alone, column by column, with
// partial pivoting (the largest entry among the rows not yet used, to 12
// bits of mantissa; rows are not moved), without barriers or LDS; it then
// leaves the panel in LDS, and with W[i][m] its entry in row i and p_m its
// pivot rows, every other column takes one update of rank NB,
//     a_i := (i a pivot row of the panel ? 0 : a_i) + sum_m W[i][m] a_{p_m}.
// One workgroup barrier per panel (the panels alternate between two
// buffers); every wavefront returns after the same one.  Bound by the chain of
// the panel owners, 0.6 (n = 64) to 1 us (n = 128) per column (a maximum over the
// lanes, lane reads, one division), where one column per barrier with the rows
// spread over the wavefronts took 1.1 us (n = 64); with three rows a lane it is
// 7.5 us (n = 160: 1.2 ms), the factors read from LDS for every entry.
//
// *need becomes 1 where a is not regular or ||a||_F ||x||_F is 2^40 or more, else
// 0.  Before it says so, a matrix whose rows or columns differ in scale is inverted
// once more with their powers of two taken out, which the refinement does not
// notice: it is exact in them.  Then the bound is on the scaled matrix, and on a
// itself the one below which the factorization to L limbs would not have found
// a singular (inverse.hip).
template <int L, int RW, int NB, int NW>
__device__ void inv64_matrix(int n, const double *a, double *x, int *need) {
  constexpr int ROWS = 64 * RW;
  __shared__ double panel[2][NB][ROWS];
  __shared__ int perm[NB * NW], where[ROWS], bad[2];
  __shared__ double red[2][NW];
  __shared__ int re[ROWS], ce[ROWS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = w * NB;
  // product of the squares of two norms, summed over the workgroup (uniform; the
  // last bits of the sums are the same in every wavefront)
  auto norms = [&](double na, double nx) {
    na = team_sum_f64(na, 64);
    nx = team_sum_f64(nx, 64);
    if (lane == 0) {
      red[0][w] = na;
      red[1][w] = nx;
    }
    __syncthreads();
    double sa = 0.0, sx = 0.0;
    for (int q = 0; q < NW; ++q) {
      sa += red[0][q];
      sx += red[1][q];
    }
    return sa * sx;
  };
  double v[RW][NB];
  for (bool scaled = false;; scaled = true) {
    double na = 0.0;
#pragma unroll
    for (int s = 0; s < RW; ++s)
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const int i = lane + 64 * s, j = c0 + c;
        v[s][c] = (i < n && j < n) ? a[(size_t)i * n + j] : 0.0;
        if (scaled && i < n && j < n) v[s][c] = ldexp(v[s][c], -(re[i] + ce[j]));
        na = __builtin_fma(v[s][c], v[s][c], na);
      }
    bool used[RW];  // own rows that were pivots
#pragma unroll
    for (int s = 0; s < RW; ++s) used[s] = lane + 64 * s >= n;
    // entry of column c in row p (uniform), uniform
    auto entry = [&](int c, int p) {
      double e = v[0][c];
#pragma unroll
      for (int s = 1; s < RW; ++s) e = (p >> 6) == s ? v[s][c] : e;
      return lane_f64(e, p & 63);
    };
    __syncthreads();
    bool regular = true;
    const int panels = (n + NB - 1) / NB;
    for (int q = 0; q < panels; ++q) {
      const int buf = q & 1;
      // the next panel's owner is on the chain, the other updates beside it not
      if (w == q + 1 || w == q) __builtin_amdgcn_s_setprio(3);
      else __builtin_amdgcn_s_setprio(1);
      if (w == q) {
        bool ok = true;
#pragma unroll
        for (int m = 0; m < NB; ++m) {
          if (c0 + m < n) {
            unsigned key = 0;
#pragma unroll
            for (int s = 0; s < RW; ++s) {
              const unsigned h = (unsigned)(__double_as_longlong(v[s][m]) >> 32) & 0x7fffff00u;
              const unsigned ks = used[s] || h == 0 ? 0u : (h | (unsigned)(lane + 64 * s));
              key = max(key, ks);
            }
            key = wave_max_u32(key);
            ok = ok && key != 0;
            const int p = (int)(key & 255u);
            double row[NB];
#pragma unroll
            for (int c = 0; c < NB; ++c) row[c] = entry(c, p);
            const double inv = 1.0 / row[m];
#pragma unroll
            for (int c = 0; c < NB; ++c) row[c] *= inv;
            row[m] = inv;
#pragma unroll
            for (int s = 0; s < RW; ++s) {
              const bool piv = lane + 64 * s == p;
              const double f = -v[s][m];
              v[s][m] = 0.0;
#pragma unroll
              for (int c = 0; c < NB; ++c) v[s][c] = piv ? row[c] : __builtin_fma(f, row[c], v[s][c]);
              used[s] = used[s] || piv;
            }
            if (lane == 0) {
              perm[c0 + m] = p;
              where[p] = c0 + m;
            }
          }
        }
        if (lane == 0) bad[buf] = ok ? 0 : 1;
#pragma unroll
        for (int s = 0; s < RW; ++s)
#pragma unroll
          for (int m = 0; m < NB; ++m) panel[buf][m][lane + 64 * s] = v[s][m];
      }
      __syncthreads();
      // no pivot: the same decision in every wavefront, since the word alternates
      // like the panels (the next owner may be done before the last wavefront
      // reads this one; the one after next waits for the next barrier)
      if (bad[buf]) {
        regular = false;
        break;
      }
      if (w != q && c0 < n) {
        int pr[NB];
        double wt[RW][NB];
        const int width = min(NB, n - q * NB);
#pragma unroll
        for (int m = 0; m < NB; ++m) {
          pr[m] = m < width ? __builtin_amdgcn_readfirstlane(perm[q * NB + m]) : 0;
#pragma unroll
          for (int s = 0; s < RW; ++s)
            wt[s][m] = RW < 3 && m < width ? panel[buf][m][lane + 64 * s] : 0.0;
        }
        bool in[RW];
#pragma unroll
        for (int s = 0; s < RW; ++s) {
          in[s] = false;
#pragma unroll
          for (int m = 0; m < NB; ++m) in[s] = in[s] || (m < width && lane + 64 * s == pr[m]);
          used[s] = used[s] || in[s];
        }
#pragma unroll
        for (int c = 0; c < NB; ++c) {
          double y[NB];
#pragma unroll
          for (int m = 0; m < NB; ++m) y[m] = entry(c, pr[m]);
#pragma unroll
          for (int s = 0; s < RW; ++s) {
            double t = in[s] ? 0.0 : v[s][c];
            if constexpr (RW < 3) {
#pragma unroll
              for (int m = 0; m < NB; ++m) t = __builtin_fma(wt[s][m], y[m], t);
            } else {  // W stays in LDS: with three rows a lane its registers are full
#pragma unroll
              for (int m = 0; m < NB; ++m)
                if (m < width) t = __builtin_fma(panel[buf][m][lane + 64 * s], y[m], t);
            }
            v[s][c] = t;
          }
          if constexpr (RW == 3) asm volatile("" ::: "memory");
        }
      }
    }
    bool good = false;
    if (regular) {
      double nx = 0.0;
#pragma unroll
      for (int s = 0; s < RW; ++s)
#pragma unroll
        for (int c = 0; c < NB; ++c) nx = __builtin_fma(v[s][c], v[s][c], nx);
      good = norms(na, nx) < 0x1p80;  // not when a norm is not finite
      // entry (k, perm[m]) of the inverse is in row perm[k], column m
      na = nx = 0.0;
#pragma unroll
      for (int s = 0; s < RW; ++s)
#pragma unroll
        for (int c = 0; c < NB; ++c) {
          const int i = lane + 64 * s, j = c0 + c;
          if (i < n && j < n) {
            double e = v[s][c];
            if (scaled) {
              e = ldexp(e, -(ce[where[i]] + re[perm[j]]));
              const double b = a[(size_t)i * n + j];
              na = __builtin_fma(b, b, na);
              nx = __builtin_fma(e, e, nx);
            }
            x[(size_t)where[i] * n + perm[j]] = e;
          }
        }
      if (scaled) {
        __syncthreads();  // (red was read)
        good = good && norms(na, nx) < ldexp(1.0, 106 * L - 16) / ((double)n * n);
      }
    }
    if (good || scaled || !scale_exponents(n, a, re, ce)) {
      if (tid == 0) *need = good ? 0 : 1;
      return;
    }
  }
}

// Lane-wise level sums of the terms i0 <= i < i1 of column v of -y A_0 (y
// [L + 1][n] in LDS, P of its limbs; LA limbs of A_0: P, or P - 1 where A_0 has
// no more), and in t the sum of |y(i)| |A_0(i,v)|.
template <int P, int LA = P>
__device__ __forceinline__ void residual_terms(int n, int v, int i0, int i1, const double *a, const double *ys,
                                               double (&u)[P], double &t) {
  const size_t nn = (size_t)n * n;
  double next[LA];
  md::zero<LA>(next);
  if (LA < 8 && i0 < i1) ld<LA>(a, nn, (size_t)i0 * n + v, next);
#pragma unroll 1
  for (int i = i0; i < i1; ++i) {
    double av[LA], yv[P];
    if constexpr (LA < 8) {  // the next entry's loads travel while this one is multiplied
      md::copy<LA>(next, av);
      if (i + 1 < i1) ld<LA>(a, nn, (size_t)(i + 1) * n + v, next);
    } else {
      ld<LA>(a, nn, (size_t)i * n + v, av);
    }
#pragma unroll
    for (int l = 0; l < P; ++l) yv[l] = -ys[l * n + i];
    t = __builtin_fma(fabs(av[0]), fabs(yv[0]), t);
    if constexpr (LA == P) MD<P>::fma_lazy(u, av, yv);
    else MD<P>::fma_lazy_h(u, av, yv);
  }
}

// Entry v of the residual e_j - y A_0: the level sums of all parts of the
// terms (in part, LDS), the unit entry added where diag, renormalized twice:
// after the cancellation the first pass can leave a zero limb ahead of
// significant ones.
template <int P>
__device__ __forceinline__ double residual_entry(int n, int v, int parts, bool diag, const double *part, double &t) {
  double u[P], r[P], s[P];
#pragma unroll
  for (int l = 0; l < P; ++l) u[l] = part[l * n + v];
  t = part[P * n + v];
#pragma unroll 1
  for (int q = 1; q < parts; ++q) {
    const double *pq = part + (size_t)q * (P + 1) * n;
    double o[P];
#pragma unroll
    for (int l = 0; l < P; ++l) o[l] = pq[l * n + v];
    MD<P>::add_lazy(u, o);
    t += pq[P * n + v];
  }
  if (diag) {
    double one[P];
    md::zero<P>(one);
    one[0] = 1.0;
    MD<P>::add_lazy(u, one);
  }
  MD<P>::renorm(u, r);
  MD<P>::renorm(r, s);
  return s[0];
}

// What a residual of `limbs` limbs cannot tell from zero, relative to the size of
// its terms: neither an omega below it measures the contraction to the next, nor
// the next one the contraction from it.  (The rounding errors of level sums grow
// from level to level: 2^-401 in 8 limbs with n = 130.)
__device__ __forceinline__ double refine_floor(int limbs) { return ldexp(1.0, 16 - 51 * limbs); }

// Row j of M, y, by iterative refinement y += (e_j - y A_0) X from
// the inverse X (x0) in doubles.  Rows, not columns: lane v then reads column v
// of A_0 and X, row after row, coalesced.  blockDim.x = 64 ceil(n / 64) S: the
// wavefronts split the n terms of a sum into S parts, added through LDS.  With
// omega the largest entry of the residual relative to the size of its terms
// and rho the contraction seen so far, this pass's omega over the one before
// among it, the row is done once omega rho is safely below the working
// precision: the correction just added was then the last one that counts.  (The
// first omega alone says nothing of the contraction: it is about 2^-53
// whatever the conditioning.  Ended on it, double-double rows were up to five
// digits behind the factorization at cond(A_0) = 1e12.)  An omega below the floor
// of the residual before is that one's rounding error and no contraction: counted
// as one, octo-double rows went on until they did not contract any more.  Early passes form the
// residual with only the limbs they need; the last one takes one limb more than
// the working precision (and y carries one more), so that M is A_0^{-1} rounded
// to L limbs, without the rounding errors of a residual at L limbs, which
// cond(A_0) would multiply.  A row that stops contracting raises *need.
// (waves: wavefronts a SIMD that the row's registers leave; a few registers more
// and a quad-double batch takes a fifth longer)
template <int L>
struct RefineThreads {
  static constexpr int value = L == 8 ? 256 : 512, waves = L == 2 ? 5 : L == 4 ? 3 : 1;
};
template <int L>
__device__ void refine_row(int n, int S, int j, const double *a, const double *x0, double *M, int *need, double *lds) {
  constexpr int LX = L + 1;  // limbs of y
  double *ys = lds, *es = lds + (size_t)LX * n, *part = es + n;  // part [S][LX + 1][n]
  __shared__ double red[2][8];
  __shared__ int stop;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nw = blockDim.x >> 6, blocks = nw / S;
  const int split = w / blocks, v = (w - split * blocks) * 64 + lane;
  const bool col = v < n, lead = split == 0 && col;
  const int vv = col ? v : 0;
  const int i0 = split * n / S, i1 = (split + 1) * n / S;
  // read once: other rows' workgroups may raise the word meanwhile
  if (tid == 0) stop = *need;
  for (int q = tid; q < LX * n; q += blockDim.x) ys[q] = q < n ? x0[(size_t)j * n + q] : 0.0;
  __syncthreads();
  if (stop != 0) return;
  const double done = ldexp(1.0, -53 * L);
  double prev = 1.0, rho = 0.0;
  int limbs = 1;  // of the residual before
  for (int pass = 0;; ++pass) {
    // the last pass that counts, if it contracts as those before it
    const bool last = pass > 0 && (prev * rho * rho * 1024.0 <= done || prev <= refine_floor(L));
    double om = 0.0, e = 0.0, t = 0.0;
    // level sums of this wavefront's part of the terms at P limbs, then the
    // entries by the wavefronts of part 0
    auto form = [&](auto tag) {
      constexpr int P = decltype(tag)::value, LA = P > L ? L : P;
      double u[P], tt = 0.0;
      md::zero<P>(u);
      residual_terms<P, LA>(n, vv, i0, i1, a, ys, u, tt);
      if (col) {
        double *pq = part + (size_t)split * (P + 1) * n;
#pragma unroll
        for (int l = 0; l < P; ++l) pq[l * n + v] = u[l];
        pq[P * n + v] = tt;
      }
      __syncthreads();
      if (lead) e = residual_entry<P>(n, v, S, v == j, part, t);
    };
    if (pass == 0) form(std::integral_constant<int, 2>{});
    else if (last) form(std::integral_constant<int, LX>{});
    else if (L == 8 && pass <= 2) form(std::integral_constant<int, (L < 4 ? L : 4)>{});
    else form(std::integral_constant<int, L>{});
    if (lead) {
      const double o = e == 0.0 ? 0.0 : fabs(e) / t;
      om = o >= 0.0 ? o : INFINITY;  // a NaN counts as infinite
      es[v] = e;
    }
    for (int off = 32; off > 0; off >>= 1) om = fmax(om, __shfl_xor(om, off, 64));
    if (lane == 0) red[pass & 1][w] = om;
    __syncthreads();
    om = red[pass & 1][0];
    for (int q = 1; q < blocks; ++q) om = fmax(om, red[pass & 1][q]);
    // the correction (e_j - y A_0) X
    double c = 0.0;
    for (int i = i0; i < i1; ++i) c = __builtin_fma(es[i], x0[(size_t)i * n + vv], c);
    if (split > 0 && col) part[(size_t)split * n + v] = c;
    __syncthreads();
    if (lead) {
      for (int q = 1; q < S; ++q) c += part[(size_t)q * n + v];
      double yv[LX], cv[LX], s[LX];
      md::zero<LX>(cv);
      cv[0] = c;
#pragma unroll
      for (int l = 0; l < LX; ++l) yv[l] = ys[l * n + v];
      MD<LX>::add(yv, cv, s);
#pragma unroll
      for (int l = 0; l < LX; ++l) ys[l * n + v] = s[l];
    }
    __syncthreads();
    if (pass == 0 || !(om <= refine_floor(limbs))) rho = fmax(rho, om / fmax(prev, refine_floor(limbs)));
    if (last && om * fmax(rho, 0x1p-53) * 64.0 <= done) break;
    prev = om;
    limbs = pass == 0 ? 2 : last ? LX : L == 8 && pass <= 2 ? 4 : L;
    if (!(rho <= 0x1p-8) || pass >= 8 * L) {  // not contracting (or not finite)
      if (tid == 0) atomicOr(need, 1);
      return;
    }
  }
  if (lead) {
    const size_t nn = (size_t)n * n;
#pragma unroll
    for (int l = 0; l < L; ++l) M[(size_t)l * nn + (size_t)j * n + v] = ys[l * n + v];
  }
}

// Parts of the terms: at most four, as many as the workgroup has threads for
// (256 threads for 64 columns find room beside the evaluation's wavefronts);
// LDS of a row.
template <int L>
inline int refine_parts(int n) {
  const int p = RefineThreads<L>::value / (64 * ((n + 63) / 64));
  return p < 4 ? p : 4;
}
template <int L>
inline size_t refine_lds(int n, int S) {
  return ((size_t)(L + 2) * n + (size_t)S * (L + 2) * n) * sizeof(double);
}

}  // namespace mdk
