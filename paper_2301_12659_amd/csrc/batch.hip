// Newton steps for a batch of independent polynomial systems ("paths") of
// uneven size.  The paper tracks many solution paths of a homotopy (Section 1);
// each path is one system p(x; c) = 0 with its own n, truncation degree d and
// monomials, and one step of every path is the Newton step of Section 2.
//
// Work decomposition.  Every phase of a step is one launch over all paths of a
// chunk: a path's work is spread over the chip, and the paths' tails overlap.
//   evaluation and differentiation, one launch per width of a monomial's
//     teams of lanes (evaldiff_dev.hpp), the monomials longest first;
//   assembly of b(t) and of the Jacobian series (coefficient-major, A_k
//     contiguous);
//   M = A_0^{-1} by refinement from an inverse in doubles, one workgroup per
//     path and then per row (inverse_dev.hpp); the Householder QR of A_0 with
//     Q^T and M = R^{-1} Q^T for the paths it does not suit;
//   N = M A_1;
//   the stages dx_k = M r_k - N dx_{k-1}, r_m -= A_{m-k} dx_k in blocks of
//     four: the stages of a block by one workgroup per path, the later
//     right-hand sides by the whole grid;
//   x := x + dx, norms and status.
// The workspace is G times the largest path's intermediates (2 per CU, more of
// small ones); paths that do not fit it together are run in chunks.
// Measured (quad double, 1024 paths of n = 16..96, 16, 32 or 64 coefficients, 8
// to 32 monomials per polynomial): 126 ms with the whole step of a path in one
// workgroup, where the largest path, on its own at the end, was the bound;
// 68 ms in phases: evaluation 29, updates 16, refinement 11, stages 5, assembly
// 4.5, N 2.2.
//
// Mixed precision (Section 1): the residual and the update at L limbs, the
// Jacobian, the QR and the stages at Ls <= L limbs (the leading limb planes
// of x, cff and b).
//
// Tiles.  The multiply-add reductions of the QR updates, N and the stages
// use teams of T lanes per dot product, T in {4, 8, 16} chosen per size
// bucket of (n, D) by md_batch_autotune (default 8).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "batch_tiles.hpp"
#include "evaldiff_dev.hpp"
#include "factor_dev.hpp"
#include "inverse_dev.hpp"

namespace mdk {

struct PathMeta {
  int n, D, m, nnz;
  int poly_off, mon_off, ent_off, asm_off, asment_off;  // offsets into the packed tables
  long long x_off, cff_off;                              // offsets within a limb plane of x (cst) and cff
  int bucket;
};

struct BatchArgs {
  const PathMeta *meta;
  const int32_t *order;
  const long long *off;                    // per entry of order: its path's bytes in slots
  const int32_t *poly_ptr, *mon_ptr, *var, *exp, *asm_ptr, *asm_ent;
  const int32_t *tile;                     // team lanes per bucket
  const double *cff, *cst;
  double *x;
  size_t x_ls, cff_ls;                     // limb strides of x (cst) and cff
  int32_t *status;                         // per path
  double *norms;                           // per path: max |b|, max |dx|
  char *slots;
};

// The intermediates of one path.
template <int L, int Ls> struct PathSlot {
  double *val, *der, *b, *At, *qr, *qt, *tau, *invd, *M, *N, *r, *dx;
};
template <int L, int Ls>
__device__ __forceinline__ PathSlot<L, Ls> path_slot(const PathMeta &pm, double *slot) {
  const size_t n = pm.n, D = pm.D, nn = n * n, nD = n * D, nnD = nn * D;
  auto take = [&](size_t cnt) {
    double *q = slot;
    slot += (cnt + 31) & ~(size_t)31;
    return q;
  };
  PathSlot<L, Ls> w;
  w.val = take((size_t)L * pm.m * D);
  w.der = take((size_t)L * pm.nnz * D);
  w.b = take((size_t)L * nD);
  w.At = take((size_t)Ls * nnD);
  w.qr = take((size_t)Ls * nn);
  w.qt = take((size_t)Ls * nn);
  w.tau = take((size_t)Ls * n);
  w.invd = take((size_t)Ls * n);
  w.M = take((size_t)Ls * nn);
  w.N = take((size_t)Ls * nn);
  w.r = take((size_t)Ls * nD);
  w.dx = take((size_t)Ls * nD);
  return w;
}

// 1. Evaluation and differentiation of the monomials work[0 .. count) =
// (entry of order, monomial) of the paths whose order has G2 = pair_lanes,
// teams of lanes as in evaldiff.hip.  LIMBS = L: the values, with the
// derivatives when Ls == L; LIMBS = Ls < L: the derivatives alone.
template <int L, int Ls, int LIMBS, int G2>
__global__ void __launch_bounds__((8 * G2 > 64 ? 8 * G2 : 64), 4) batch_eval_kernel(BatchArgs B, const int2 *work,
                                                                                    int count) {
  extern __shared__ __align__(16) double lds[];
  constexpr bool VALUES = LIMBS == L, DERIVS = LIMBS == Ls;
  constexpr int lanes = (DERIVS ? 8 : 4) * G2, per = 8 * G2 < 64 ? 64 / lanes : 1;
  const int w = per == 1 ? 0 : threadIdx.x / lanes, idx = blockIdx.x * per + w;
  if (idx >= count) return;
  int pos = work[idx].x, mono = work[idx].y;
  if constexpr (per == 1) {
    pos = __builtin_amdgcn_readfirstlane(pos);
    mono = __builtin_amdgcn_readfirstlane(mono);
  }
  const PathMeta pm = B.meta[B.order[pos]];
  const PathSlot<L, Ls> s = path_slot<L, Ls>(pm, reinterpret_cast<double *>(B.slots + B.off[pos]));
  EvalArgs a;
  a.n = pm.n;
  a.D = pm.D;
  a.Dc = pm.D;
  a.m = pm.m;
  a.nnz = pm.nnz;
  a.mon_ptr = B.mon_ptr + pm.mon_off;
  a.var = B.var + pm.ent_off;
  a.exp = B.exp + pm.ent_off;
  a.order = nullptr;  // not read: monomials are addressed directly
  a.cff = B.cff + pm.cff_off;
  a.x = B.x + pm.x_off;
  a.pw = a.x;  // not read: batched paths have exponents of at most 2, no power table
  a.val = VALUES ? s.val : nullptr;
  a.der = s.der;
  a.x_ls = B.x_ls;
  a.cff_ls = B.cff_ls;
  a.values_only = DERIVS ? 0 : 1;
  eval_monomial_team<LIMBS, G2>(a, mono, threadIdx.x - w * lanes, lds + (size_t)w * team_doubles<LIMBS, G2>());
}

constexpr int BATCH_NT = 256;
constexpr int BATCH_MAXN = 128;  // rows per lane <= 2 in the back substitution

__host__ __device__ inline int size_bucket(int n, int D) {
  const int bn = n <= 32 ? 0 : (n <= 64 ? 1 : 2);
  const int bd = D <= 16 ? 0 : (D <= 32 ? 1 : 2);
  return bn * 3 + bd;
}
constexpr int BATCH_BUCKETS = 9;

// Blocks of a launch over paths: blockIdx.x is the entry of order, blockIdx.y
// and gridDim.y split the path's work.
template <int L, int Ls>
__device__ __forceinline__ PathSlot<L, Ls> block_path(const BatchArgs &B, PathMeta &pm) {
  pm = B.meta[B.order[blockIdx.x]];
  return path_slot<L, Ls>(pm, reinterpret_cast<double *>(B.slots + B.off[blockIdx.x]));
}

// 2. Assembly: b = -(c_0 + sum of the row's monomial values) at L limbs and
// its coefficient-major leading limbs r[k][i]; the Jacobian series,
// coefficient-major At[k][i][j], and A_0 once more for a factorization.  A
// unit is a tile of `tile_rows` entries (i, j) with all their coefficients,
// turned through LDS so that both sides move whole cache lines, or 256
// entries of b.  Bound by HBM.
__host__ __device__ inline int assemble_tiles(int n, int D) { return (n * n + tile_rows(D) - 1) / tile_rows(D); }
__host__ __device__ inline int assemble_units(int n, int D) {
  return assemble_tiles(n, D) + (n * D + BATCH_NT - 1) / BATCH_NT;
}

template <int L, int Ls>
__global__ void __launch_bounds__(BATCH_NT) batch_assemble_kernel(BatchArgs B) {
  extern __shared__ double lds[];
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  constexpr int NT = BATCH_NT;
  const int tid = threadIdx.x;
  const int n = pm.n, D = pm.D, m = pm.m, nnz = pm.nnz, R = tile_rows(D);
  const size_t nn = (size_t)n * n, nD = (size_t)n * D, nnD = nn * D;
  const int32_t *poly_ptr = B.poly_ptr + pm.poly_off, *asm_ptr = B.asm_ptr + pm.asm_off;
  const int32_t *asm_ent = B.asm_ent + pm.asment_off;
  const double *cst = B.cst + pm.x_off;
  const int tiles = assemble_tiles(n, D), units = assemble_units(n, D);
  for (int unit = blockIdx.y; unit < units; unit += gridDim.y) {
    if (unit < tiles) {
      const int ij0 = unit * R, rows = min(R, (int)nn - ij0);
      for (int q = tid; q < rows * D; q += NT) {
        const int row = q / D, s = q - row * D, ij = ij0 + row;
        double acc[Ls];
        md::zero<Ls>(acc);
        const int lo = asm_ptr[ij], hi = asm_ptr[ij + 1];
        if (lo < hi) {
          ld<Ls>(w.der, (size_t)nnz * D, (size_t)asm_ent[lo] * D + s, acc);
          for (int t = lo + 1; t < hi; ++t) {
            double v[Ls], y[Ls];
            ld<Ls>(w.der, (size_t)nnz * D, (size_t)asm_ent[t] * D + s, v);
            MD<Ls>::add(acc, v, y);
            md::copy<Ls>(y, acc);
          }
        }
#pragma unroll
        for (int l = 0; l < Ls; ++l) lds[tile_index(D, l, s, row)] = acc[l];
        if (s == 0) st<Ls>(w.qr, nn, ij, acc);
      }
      __syncthreads();
      for (int q = tid; q < R * D; q += NT) {
        const int s = q / R, row = q - s * R;
        if (row < rows)
#pragma unroll
          for (int l = 0; l < Ls; ++l) w.At[(size_t)l * nnD + (size_t)s * nn + ij0 + row] = lds[tile_index(D, l, s, row)];
      }
      __syncthreads();
    } else {
      const int q = (unit - tiles) * NT + tid;
      if (q < (int)nD) {
        const int i = q / D, s = q - i * D;
        double acc[L];
        ld<L>(cst, B.x_ls, (size_t)q, acc);
        for (int mj = poly_ptr[i]; mj < poly_ptr[i + 1]; ++mj) {
          double v[L], y[L];
          ld<L>(w.val, (size_t)m * D, (size_t)mj * D + s, v);
          MD<L>::add(acc, v, y);
          md::copy<L>(y, acc);
        }
        md::neg<L>(acc, acc);
        st<L>(w.b, nD, q, acc);
#pragma unroll
        for (int l = 0; l < Ls; ++l) w.r[(size_t)l * nD + (size_t)s * n + i] = acc[l];
      }
    }
  }
}

// 3. M = A_0^{-1} by refinement from an inverse in doubles (inverse.hip):
// the inverse X goes into the space of Q^T, the word that asks for the
// factorization into that of tau.
template <int L, int Ls>
__device__ __forceinline__ int *path_need(const PathSlot<L, Ls> &w) {
  return reinterpret_cast<int *>(w.tau);
}
template <int L, int Ls, int RW, int NB, int NW>
__global__ void __launch_bounds__(64 * NW) batch_inv64_kernel(BatchArgs B, int lo) {
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  if (pm.n <= lo || pm.n > NB * NW) return;
  inv64_matrix<Ls, RW, NB, NW>(pm.n, w.qr, w.qt, path_need(w));
}
// (sizes lo < n <= hi; grid.y: rows)
template <int L, int Ls>
__global__ void __launch_bounds__(RefineThreads<Ls>::value, Ls == 4 ? 3 : 2)
    batch_refine_kernel(BatchArgs B, int lo, int hi, int S) {
  extern __shared__ double lds[];
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  if (pm.n <= lo || pm.n > hi || (int)blockIdx.y >= pm.n) return;
  refine_row<Ls>(pm.n, S, blockIdx.y, w.qr, w.qt, w.M, path_need(w), lds);
}

// The same by a factorization, for the paths whose A_0 asked for it; sing: A_0
// is singular to working precision.
template <int L, int Ls>
__global__ void __launch_bounds__(BATCH_NT) batch_factor_kernel(BatchArgs B) {
  __shared__ double shr[8 * 8 + 16];
  __shared__ int sh_sing;
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  const int tid = threadIdx.x, n = pm.n;
  int *flags = path_need(w);
  const bool needed = flags[0] != 0;
  __syncthreads();
  if (tid == 0) flags[1] = 0;
  if (!needed) return;
  factor_matrix<Ls>(n, B.tile[pm.bucket], w.qr, w.qt, w.invd, w.M, shr, sh_sing);
  if (tid == 0) flags[1] = sh_sing;
}

// 4. N = M A_1.
template <int L, int Ls>
__device__ __forceinline__ void form_n(const BatchArgs &B, const PathMeta &pm, const PathSlot<L, Ls> &w) {
  if (pm.D <= 1) return;
  const int n = pm.n, T = B.tile[pm.bucket], nteams = blockDim.x / T, tl = threadIdx.x % T;
  const size_t nn = (size_t)n * n, nnD = nn * pm.D;
  for (int task = blockIdx.y * nteams + threadIdx.x / T; task < (int)nn; task += gridDim.y * nteams) {
    const int i = task / n, j = task - i * n;
    double acc[Ls], s2[Ls];
    md::zero<Ls>(acc);
    for (int v = tl; v < n; v += T) {
      double mv[Ls], av[Ls];
      ld<Ls>(w.M, nn, (size_t)i * n + v, mv);
      ld<Ls>(w.At, nnD, nn + (size_t)v * n + j, av);
      MD<Ls>::fma_lazy(acc, mv, av);
    }
    team_sum_lazy<Ls>(acc, T);
    MD<Ls>::renorm(acc, s2);
    if (tl == 0) st<Ls>(w.N, nn, (size_t)i * n + j, s2);
  }
}
template <int L, int Ls>
__global__ void __launch_bounds__(BATCH_NT) batch_n_kernel(BatchArgs B) {
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  form_n<L, Ls>(B, pm, w);
}

// 5. Stages in blocks of BATCH_BLOCK: the block's own stages by one workgroup
// per path, dx_k = M r_k - N dx_{k-1} and r_m -= A_{m-k} dx_k for the later m of
// the block (the term m = k + 1 is N dx_k) ...
constexpr int BATCH_BLOCK = 4;

template <int L, int Ls>
__device__ __forceinline__ void solve_stages(const BatchArgs &B, const PathMeta &pm, const PathSlot<L, Ls> &w, int kb,
                                             int kend) {
  const int n = pm.n, D = pm.D;
  const int T = B.tile[pm.bucket], nteams = blockDim.x / T, team = threadIdx.x / T, tl = threadIdx.x % T;
  const size_t nn = (size_t)n * n, nD = (size_t)n * D, nnD = nn * D;
  for (int k = kb; k < kend; ++k) {
    for (int i = team; i < n; i += nteams) {
      double acc[Ls], s2[Ls];
      md::zero<Ls>(acc);
      for (int v = tl; v < n; v += T) {
        double mv[Ls], rv[Ls];
        ld<Ls>(w.M, nn, (size_t)i * n + v, mv);
        ld<Ls>(w.r, nD, (size_t)k * n + v, rv);
        MD<Ls>::fma_lazy(acc, mv, rv);
        if (k > 0) {
          double nv[Ls], xv[Ls];
          ld<Ls>(w.N, nn, (size_t)i * n + v, nv);
          md::neg<Ls>(nv, nv);
          ld<Ls>(w.dx, nD, (size_t)(k - 1) * n + v, xv);
          MD<Ls>::fma_lazy(acc, nv, xv);
        }
      }
      team_sum_lazy<Ls>(acc, T);
      MD<Ls>::renorm(acc, s2);
      if (tl == 0) st<Ls>(w.dx, nD, (size_t)k * n + i, s2);
    }
    __syncthreads();
    const int ntask = (kend - k - 2) * n;
    if (ntask <= 0) continue;
    for (int task = team; task < ntask; task += nteams) {
      const int mm = k + 2 + task / n, i = task % n;
      double acc[Ls], s2[Ls];
      md::zero<Ls>(acc);
      for (int v = tl; v < n; v += T) {
        double av[Ls], xv[Ls];
        ld<Ls>(w.At, nnD, (size_t)(mm - k) * nn + (size_t)i * n + v, av);
        ld<Ls>(w.dx, nD, (size_t)k * n + v, xv);
        MD<Ls>::fma_lazy(acc, av, xv);
      }
      team_sum_lazy<Ls>(acc, T);
      MD<Ls>::renorm(acc, s2);
      if (tl == 0) {
        double rv[Ls], t2[Ls];
        ld<Ls>(w.r, nD, (size_t)mm * n + i, rv);
        MD<Ls>::sub(rv, s2, t2);
        st<Ls>(w.r, nD, (size_t)mm * n + i, t2);
      }
    }
    __syncthreads();
  }
}

template <int L, int Ls>
__global__ void __launch_bounds__(512) batch_stages_kernel(BatchArgs B, int kb) {
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  if (kb < pm.D) solve_stages<L, Ls>(B, pm, w, kb, min(kb + BATCH_BLOCK, pm.D));
}

// ... then all later right-hand sides, r_m -= sum over the block's stages k of
// A_{m-k} dx_k, by the whole grid.  A task is a row of BATCH_BLOCK neighbouring
// r_m: it reads 7 entries of A for 16 multiply-adds.
__host__ __device__ inline int update_tasks(int n, int D, int kb) {
  const int first = kb + BATCH_BLOCK;
  return first < D ? n * ((D - first + BATCH_BLOCK - 1) / BATCH_BLOCK) : 0;
}

template <int L, int Ls>
__global__ void __launch_bounds__(BATCH_NT) batch_update_kernel(BatchArgs B, int kb) {
  constexpr int K = BATCH_BLOCK;
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  const int n = pm.n, D = pm.D, first = kb + K;
  if (first >= D) return;
  const int T = B.tile[pm.bucket], nteams = blockDim.x / T, tl = threadIdx.x % T;
  const size_t nn = (size_t)n * n, nD = (size_t)n * D, nnD = nn * D;
  const int ntask = update_tasks(n, D, kb);
  for (int task = blockIdx.y * nteams + threadIdx.x / T; task < ntask; task += gridDim.y * nteams) {
    const int g = task / n, i = task - g * n, m0 = first + K * g, a0 = m0 - kb - (K - 1);
    double acc[K][Ls];
#pragma unroll
    for (int q = 0; q < K; ++q) md::zero<Ls>(acc[q]);
    for (int v = tl; v < n; v += T) {
      double dv[K][Ls];
#pragma unroll
      for (int q = 0; q < K; ++q) ld<Ls>(w.dx, nD, (size_t)(kb + q) * n + v, dv[q]);
#pragma unroll
      for (int a = 0; a < 2 * K - 1; ++a) {
        const int ai = a0 + a;  // 1: in N
        double av[Ls];
        md::zero<Ls>(av);
        if (ai > 1 && ai < D) ld<Ls>(w.At, nnD, (size_t)ai * nn + (size_t)i * n + v, av);
#pragma unroll
        for (int q = 0; q < K; ++q) {
          const int s = q + K - 1 - a;  // stage of the block
          if (s >= 0 && s < K) MD<Ls>::fma_lazy(acc[q], av, dv[s]);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < K; ++q) {
      double s2[Ls];
      team_sum_lazy<Ls>(acc[q], T);
      MD<Ls>::renorm(acc[q], s2);
      if (tl == 0 && m0 + q < D) {
        double rv[Ls], t2[Ls];
        ld<Ls>(w.r, nD, (size_t)(m0 + q) * n + i, rv);
        MD<Ls>::sub(rv, s2, t2);
        st<Ls>(w.r, nD, (size_t)(m0 + q) * n + i, t2);
      }
    }
  }
}

// 6. x := x + dx, norms and status.
template <int L, int Ls>
__device__ __forceinline__ void finish_path(const BatchArgs &B, const PathMeta &pm, const PathSlot<L, Ls> &w,
                                            double *shr) {
  const int tid = threadIdx.x, NT = blockDim.x, n = pm.n, D = pm.D, p = B.order[blockIdx.x];
  const size_t nD = (size_t)n * D;
  double *x = B.x + pm.x_off;
  const double *b = w.b, *dx = w.dx;
  double nb = 0.0, nx = 0.0;
  bool finite = true;
  for (int q = tid; q < (int)nD; q += NT) {
    const int i = q / D, s = q - i * D;
    double xv[L], d[Ls], dw[L], t[L];
    ld<L>(x, B.x_ls, (size_t)q, xv);
#pragma unroll
    for (int l = 0; l < Ls; ++l) d[l] = dx[(size_t)l * nD + (size_t)s * n + i];
    md::widen<Ls>(d, dw);
    MD<L>::add(xv, dw, t);
    st<L>(x, B.x_ls, (size_t)q, t);
    const double bq = b[q];
    finite = finite && isfinite(bq) && isfinite(d[0]);
    nb = fmax(nb, fabs(bq));
    nx = fmax(nx, fabs(d[0]));
  }
  nb = block_max(nb, shr);
  nx = block_max(nx, shr);
  const double fin = block_max(finite ? 0.0 : 1.0, shr);
  if (tid == 0) {
    B.norms[2 * (size_t)p] = nb;
    B.norms[2 * (size_t)p + 1] = nx;
    B.status[p] = path_need(w)[1] ? MD_ESINGULAR : (fin > 0.0 ? MD_ENONFINITE : MD_OK);
  }
}
template <int L, int Ls>
__global__ void __launch_bounds__(BATCH_NT) batch_finish_kernel(BatchArgs B) {
  __shared__ double shr[BATCH_NT / 64];
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  finish_path<L, Ls>(B, pm, w, shr);
}

// 4., 5. and 6. of small systems with few coefficients in one launch, a
// workgroup per path: as launches they take 4 to 5 us each, however little there
// is to do (64 paths of n = 2, 16 coefficients, double double: 68 us a step, 80
// with them apart; two of n = 4, 16 coefficients, quad double: 157 and 141).
template <int L, int Ls>
__global__ void __launch_bounds__(BATCH_NT) batch_small_kernel(BatchArgs B) {
  __shared__ double shr[BATCH_NT / 64];
  PathMeta pm;
  const PathSlot<L, Ls> w = block_path<L, Ls>(B, pm);
  form_n<L, Ls>(B, pm, w);
  __syncthreads();
  solve_stages<L, Ls>(B, pm, w, 0, pm.D);
  __syncthreads();
  finish_path<L, Ls>(B, pm, w, shr);
}
bool batch_small(int n, int D) { return D <= 8 ? n <= 8 : D <= 16 && n <= 3; }

template <int L, int Ls, int LIMBS, int G2>
void launch_batch_eval(const BatchArgs &A, const int2 *work, int count, hipStream_t st) {
  constexpr int lanes = (LIMBS == Ls ? 8 : 4) * G2, per = 8 * G2 < 64 ? 64 / lanes : 1;
  const size_t lds = per * team_doubles<LIMBS, G2>() * sizeof(double);
  hipLaunchKernelGGL((batch_eval_kernel<L, Ls, LIMBS, G2>), dim3((count + per - 1) / per), dim3(per * lanes), lds, st,
                     A, work, count);
}

// cls = log2 G2
template <int L, int Ls, int LIMBS>
void launch_batch_eval(int cls, const BatchArgs &A, const int2 *work, int count, hipStream_t st) {
  switch (cls) {
    case 0: return launch_batch_eval<L, Ls, LIMBS, 1>(A, work, count, st);
    case 1: return launch_batch_eval<L, Ls, LIMBS, 2>(A, work, count, st);
    case 2: return launch_batch_eval<L, Ls, LIMBS, 4>(A, work, count, st);
    case 3: return launch_batch_eval<L, Ls, LIMBS, 8>(A, work, count, st);
    case 4: return launch_batch_eval<L, Ls, LIMBS, 16>(A, work, count, st);
    case 5: return launch_batch_eval<L, Ls, LIMBS, 32>(A, work, count, st);
    case 6: return launch_batch_eval<L, Ls, LIMBS, 64>(A, work, count, st);
  }
}

}  // namespace mdk

// ------------------------------------------------------------------ host API

constexpr int BATCH_CLASSES = 7;  // pair_lanes 1 .. 64

// A run over a list of paths: chunks whose intermediates fit the workspace
// together, and the monomials of a chunk by evaluation kernel, longest first.
struct BatchRun {
  struct Chunk {
    int first, count;  // entries of order
    int maxn, maxD;
    int tile;          // doubles of LDS per limb of the assembly's tiles
    int asm_units, update_tasks;  // the most of a path: units of the assembly, rows of the first update
    int work[BATCH_CLASSES], works[BATCH_CLASSES];  // first, number
  };
  std::vector<Chunk> chunks;
  void *d = nullptr;
  const long long *off = nullptr;
  const int2 *work = nullptr;
  const int32_t *order = nullptr;
};

struct md_batch {
  int L, P, G;
  int maxn, maxD;
  std::vector<mdk::PathMeta> meta;
  std::vector<int32_t> order;             // all paths, most expensive first
  std::vector<double> cost;
  int32_t tile[mdk::BATCH_BUCKETS];
  long long x_total, cff_total;
  size_t slot_bytes;
  mdk::PathMeta *d_meta = nullptr;
  int32_t *d_tables = nullptr, *d_tile = nullptr;
  std::vector<int32_t> mon_ptr;           // host copy of the packed table
  BatchRun run;                           // over all paths
  const int32_t *d_poly_ptr = nullptr, *d_mon_ptr = nullptr, *d_var = nullptr, *d_exp = nullptr;
  const int32_t *d_asm_ptr = nullptr, *d_asm_ent = nullptr;
  // one captured step (graph) for a fixed set of arguments
  hipStream_t cap = nullptr;
  hipGraphExec_t exec = nullptr;
  const void *key[8] = {nullptr};
  int key_prec = 0;
  bool seen = false;
};

namespace {

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t slot_doubles(int L, int Ls, int n, int D, int m, int nnz) {
  auto r = [](size_t c) { return (c + 31) & ~(size_t)31; };
  const size_t nn = (size_t)n * n, nD = (size_t)n * D;
  return r((size_t)L * m * D) + r((size_t)L * nnz * D) + r((size_t)L * nD) + r((size_t)Ls * nn * D) +
         3 * r((size_t)Ls * nn) + 2 * r((size_t)Ls * n) + r((size_t)Ls * nn) + 2 * r((size_t)Ls * nD);
}

// workspace: the intermediates of a chunk of paths, G times the largest path's
size_t batch_ws_bytes(const md_batch *b) { return (size_t)b->G * b->slot_bytes; }

// The chunks and work lists of a run over `list`, on the device.
hipError_t build_run(const md_batch *b, const std::vector<int32_t> &list, BatchRun &run) {
  const size_t budget = (size_t)b->G * b->slot_bytes;
  std::vector<long long> off(list.size());
  std::vector<int2> work;
  size_t used = budget;  // the first path opens a chunk
  auto cls = [&](int p) {
    int c = 0;
    while ((1 << c) < mdk::pair_lanes(b->meta[p].D)) ++c;
    return c;
  };
  run.chunks.clear();
  for (size_t q = 0; q < list.size(); ++q) {
    const mdk::PathMeta &pm = b->meta[list[q]];
    const size_t bytes = align256(slot_doubles(b->L, b->L, pm.n, pm.D, pm.m, pm.nnz) * sizeof(double));
    if (used + bytes > budget) {
      run.chunks.push_back({(int)q, 0, 0, 0, 0, 0, 0, {}, {}});
      used = 0;
    }
    off[q] = (long long)used;
    used += bytes;
    BatchRun::Chunk &ch = run.chunks.back();
    ch.count++;
    ch.maxn = std::max(ch.maxn, pm.n);
    ch.maxD = std::max(ch.maxD, pm.D);
    ch.tile = mdk::tile_doubles(ch.tile, pm.D);
    ch.asm_units = std::max(ch.asm_units, mdk::assemble_units(pm.n, pm.D));
    ch.update_tasks = std::max(ch.update_tasks, mdk::update_tasks(pm.n, pm.D, 0));
  }
  for (BatchRun::Chunk &ch : run.chunks)
    for (int c = 0; c < BATCH_CLASSES; ++c) {
      std::vector<std::vector<int2>> by_k(mdk::BATCH_MAXN + 1);  // by support size
      for (int q = ch.first; q < ch.first + ch.count; ++q) {
        if (cls(list[q]) != c) continue;
        const mdk::PathMeta &pm = b->meta[list[q]];
        const int32_t *mp = b->mon_ptr.data() + pm.mon_off;
        for (int j = 0; j < pm.m; ++j) by_k[mp[j + 1] - mp[j]].push_back(make_int2(q, j));
      }
      ch.work[c] = (int)work.size();
      for (int k = mdk::BATCH_MAXN; k >= 0; --k) work.insert(work.end(), by_k[k].begin(), by_k[k].end());
      ch.works[c] = (int)work.size() - ch.work[c];
    }
  const size_t no = off.size() * sizeof(long long), nw = work.size() * sizeof(int2), nl = list.size() * sizeof(int32_t);
  hipError_t e = hipMalloc(&run.d, no + nw + nl);
  if (e != hipSuccess) return e;
  char *d = static_cast<char *>(run.d);
  if ((e = hipMemcpy(d, off.data(), no, hipMemcpyHostToDevice)) != hipSuccess ||
      (nw && (e = hipMemcpy(d + no, work.data(), nw, hipMemcpyHostToDevice)) != hipSuccess) ||
      (e = hipMemcpy(d + no + nw, list.data(), nl, hipMemcpyHostToDevice)) != hipSuccess) {
    (void)hipFree(run.d);
    run.d = nullptr;
    return e;
  }
  run.off = reinterpret_cast<const long long *>(d);
  run.work = reinterpret_cast<const int2 *>(d + no);
  run.order = reinterpret_cast<const int32_t *>(d + no + nw);
  return hipSuccess;
}

template <int L, int Ls>
void launch_chunk(const mdk::BatchArgs &A, const BatchRun::Chunk &ch, const int2 *work, hipStream_t st) {
  for (int c = BATCH_CLASSES - 1; c >= 0; --c) {
    if (!ch.works[c]) continue;
    mdk::launch_batch_eval<L, Ls, L>(c, A, work + ch.work[c], ch.works[c], st);
    if constexpr (Ls != L) mdk::launch_batch_eval<L, Ls, Ls>(c, A, work + ch.work[c], ch.works[c], st);
  }
  using namespace mdk;
  BatchArgs B = A;
  B.order = A.order + ch.first;
  B.off = A.off + ch.first;
  const int P = ch.count, maxn = ch.maxn, maxD = ch.maxD;
  // workgroups per path: enough to spread a chunk of few paths over the chip,
  // few enough that small paths' empty workgroups do not count
  const int Y = std::max(16, std::min(256, 2048 / P));
  const dim3 NT(BATCH_NT), one(P);
  // (and no more than the largest path has work for)
  auto split = [&](int most) { return dim3(P, std::max(1, std::min(Y, most))); };
  constexpr int TEAMS = BATCH_NT / 16;  // (16 lanes a team, the widest tile)
  const size_t tile = (size_t)Ls * ch.tile * sizeof(double);
  hipLaunchKernelGGL((batch_assemble_kernel<L, Ls>), split(ch.asm_units), NT, tile, st, B);
  hipLaunchKernelGGL((batch_inv64_kernel<L, Ls, 1, 8, 4>), one, dim3(256), 0, st, B, 0);
  if (maxn > 32) hipLaunchKernelGGL((batch_inv64_kernel<L, Ls, 1, 8, 8>), one, dim3(512), 0, st, B, 32);
  if (maxn > 64) hipLaunchKernelGGL((batch_inv64_kernel<L, Ls, 2, 8, 16>), one, dim3(1024), 0, st, B, 64);
  auto refine = [&](int lo, int hi) {
    const int n = std::min(hi, maxn);
    // rows enough to fill the chip without splitting a row's sums (1024 paths:
    // 16.5 ms in four parts, 11.0 in one), or short sums, where parts are wavefronts
    // that do not find room at once (512 paths of n = 4, double double: 25 us in
    // four parts, 9 in one)
    const long long rows = (long long)P * n;
    int S = rows >= 4096 ? 1 : refine_parts<Ls>(n);
    if (n < 16) S = std::max(1, std::min(S, (int)(1024 * (Ls == 4 ? 3 : 2) / rows)));
    hipLaunchKernelGGL((batch_refine_kernel<L, Ls>), dim3(P, n), dim3(64 * ((n + 63) / 64) * S), refine_lds<Ls>(n, S), st,
                       B, lo, hi, S);
  };
  refine(0, 64);
  if (maxn > 64) refine(64, 128);
  hipLaunchKernelGGL((batch_factor_kernel<L, Ls>), one, NT, 0, st, B);
  // a stage's rows by one workgroup: no more wavefronts than rows of 16 lanes
  // (512 paths of n = 4, 8 coefficients, quad double: 46 us with 512 threads, 25 with 64)
  auto rows = [&](int most) { return dim3(std::min(most, (maxn * 16 + 63) / 64 * 64)); };
  if (batch_small(maxn, maxD)) {
    hipLaunchKernelGGL((batch_small_kernel<L, Ls>), one, rows(BATCH_NT), 0, st, B);
    return;
  }
  if (maxD > 1) hipLaunchKernelGGL((batch_n_kernel<L, Ls>), split((maxn * maxn + TEAMS - 1) / TEAMS), NT, 0, st, B);
  for (int kb = 0; kb < maxD; kb += BATCH_BLOCK) {
    hipLaunchKernelGGL((batch_stages_kernel<L, Ls>), one, rows(512), 0, st, B, kb);
    if (kb + BATCH_BLOCK < maxD)
      hipLaunchKernelGGL((batch_update_kernel<L, Ls>), split((ch.update_tasks + TEAMS - 1) / TEAMS), NT, 0, st, B, kb);
  }
  hipLaunchKernelGGL((batch_finish_kernel<L, Ls>), one, NT, 0, st, B);
}

hipError_t launch_step(const md_batch *b, int Ls, const BatchRun &run, const double *cff, const double *cst, double *x,
                       int32_t *status, double *norms, void *ws, hipStream_t st) {
  mdk::BatchArgs A;
  A.meta = b->d_meta;
  A.order = run.order;
  A.off = run.off;
  A.poly_ptr = b->d_poly_ptr;
  A.mon_ptr = b->d_mon_ptr;
  A.var = b->d_var;
  A.exp = b->d_exp;
  A.asm_ptr = b->d_asm_ptr;
  A.asm_ent = b->d_asm_ent;
  A.tile = b->d_tile;
  A.cff = cff;
  A.cst = cst;
  A.x = x;
  A.x_ls = (size_t)b->x_total;
  A.cff_ls = (size_t)b->cff_total;
  A.status = status;
  A.norms = norms;
  A.slots = static_cast<char *>(ws);
  for (const BatchRun::Chunk &ch : run.chunks) {
    if (b->L == 2) launch_chunk<2, 2>(A, ch, run.work, st);
    else if (Ls == 4) launch_chunk<4, 4>(A, ch, run.work, st);
    else launch_chunk<4, 2>(A, ch, run.work, st);
  }
  return hipGetLastError();
}

}  // namespace

extern "C" {

int md_batch_create(int prec, int npaths, const int32_t *n, const int32_t *d, const int32_t *m,
                    const int32_t *poly_ptr, const int32_t *mon_ptr, const int32_t *var, const int32_t *exp,
                    md_batch **out) {
  if (!out) return mdk::api_fail(MD_EINVAL, "NULL argument");
  *out = nullptr;
  if (prec != MD_DD && prec != MD_QD) return mdk::api_fail(MD_EINVAL, "batches run in double or quad double");
  if (npaths < 1 || !n || !d || !m || !poly_ptr || !mon_ptr) return mdk::api_fail(MD_EINVAL, "bad batch description");
  md_batch *b = new md_batch();
  b->L = prec;
  b->P = npaths;
  b->maxn = b->maxD = 0;
  std::vector<int32_t> tab_poly, tab_mon, tab_var, tab_exp, tab_asm, tab_asment;
  long long xo = 0, co = 0;
  size_t poly_o = 0, mon_o = 0, ent_o = 0;
  for (int p = 0; p < npaths; ++p) {
    const int np = n[p], Dp = d[p] + 1, mp = m[p];
    if (np < 1 || np > mdk::BATCH_MAXN || d[p] < 0 || Dp > MD_MAX_COEFFS || mp < 0) {
      delete b;
      return mdk::api_fail(MD_EINVAL, "path size out of range (1 <= n <= 128, 0 <= d < 128)");
    }
    const int32_t *pp = poly_ptr + poly_o, *mpt = mon_ptr + mon_o;
    if (pp[0] != 0 || pp[np] != mp || mpt[0] != 0) {
      delete b;
      return mdk::api_fail(MD_EINVAL, "poly_ptr / mon_ptr of a path must start at 0 and cover its monomials");
    }
    for (int i = 0; i < np; ++i)
      if (pp[i + 1] < pp[i]) {
        delete b;
        return mdk::api_fail(MD_EINVAL, "poly_ptr must be nondecreasing");
      }
    const int nnz = mpt[mp];
    if (nnz < 0 || (nnz > 0 && (!var || !exp))) {
      delete b;
      return mdk::api_fail(MD_EINVAL, "bad monomial supports");
    }
    std::vector<int32_t> cnt((size_t)np * np + 1, 0);
    double cost = 0.0;
    for (int j = 0; j < mp; ++j) {
      if (mpt[j + 1] < mpt[j]) {
        delete b;
        return mdk::api_fail(MD_EINVAL, "mon_ptr must be nondecreasing");
      }
      const int k = mpt[j + 1] - mpt[j];
      cost += (double)std::max(1, 3 * k - 5) * Dp * Dp;
      for (int q = mpt[j]; q < mpt[j + 1]; ++q) {
        const int v = var[ent_o + q], e = exp[ent_o + q];
        if (v < 0 || v >= np || (q > mpt[j] && v <= var[ent_o + q - 1])) {
          delete b;
          return mdk::api_fail(MD_EINVAL, "variables must be in range and strictly increasing per monomial");
        }
        if (e < 1 || e > 2) {
          delete b;
          return mdk::api_fail(MD_EINVAL, "batched paths take exponents 1 and 2");
        }
      }
    }
    // assembly lists of the path: entries contributing to (row i, column v), monomial order
    std::vector<int32_t> rowof(mp, 0);
    for (int i = 0; i < np; ++i)
      for (int j = pp[i]; j < pp[i + 1]; ++j) rowof[j] = i;
    std::vector<std::vector<int32_t>> lists((size_t)np * np);
    for (int j = 0; j < mp; ++j)
      for (int q = mpt[j]; q < mpt[j + 1]; ++q) lists[(size_t)rowof[j] * np + var[ent_o + q]].push_back(q);
    mdk::PathMeta pm;
    pm.n = np;
    pm.D = Dp;
    pm.m = mp;
    pm.nnz = nnz;
    pm.poly_off = (int)tab_poly.size();
    pm.mon_off = (int)tab_mon.size();
    pm.ent_off = (int)tab_var.size();
    pm.asm_off = (int)tab_asm.size();
    pm.asment_off = (int)tab_asment.size();
    pm.x_off = xo;
    pm.cff_off = co;
    pm.bucket = mdk::size_bucket(np, Dp);
    tab_poly.insert(tab_poly.end(), pp, pp + np + 1);
    tab_mon.insert(tab_mon.end(), mpt, mpt + mp + 1);
    tab_var.insert(tab_var.end(), var + ent_o, var + ent_o + nnz);
    tab_exp.insert(tab_exp.end(), exp + ent_o, exp + ent_o + nnz);
    int32_t acc = 0;
    for (size_t ij = 0; ij < (size_t)np * np; ++ij) {
      tab_asm.push_back(acc);
      for (int32_t e : lists[ij]) tab_asment.push_back(e);
      acc += (int32_t)lists[ij].size();
    }
    tab_asm.push_back(acc);
    b->meta.push_back(pm);
    cost += (double)np * np * Dp * Dp / 2 + (double)np * np * np;
    b->cost.push_back(cost);
    b->maxn = std::max(b->maxn, np);
    b->maxD = std::max(b->maxD, Dp);
    xo += (long long)np * Dp;
    co += mp;
    poly_o += np + 1;
    mon_o += mp + 1;
    ent_o += nnz;
  }
  b->x_total = xo;
  b->cff_total = co;
  b->mon_ptr = tab_mon;
  b->order.resize(npaths);
  std::iota(b->order.begin(), b->order.end(), 0);
  std::stable_sort(b->order.begin(), b->order.end(), [&](int a2, int b2) { return b->cost[a2] > b->cost[b2]; });
  for (int q = 0; q < mdk::BATCH_BUCKETS; ++q) b->tile[q] = 8;
  size_t slot = 0;
  for (const auto &pm : b->meta)
    slot = std::max(slot, slot_doubles(b->L, b->L, pm.n, pm.D, pm.m, pm.nnz) * sizeof(double));
  b->slot_bytes = align256(slot);
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) {
    delete b;
    return mdk::api_hip_fail(e, "device query");
  }
  // two of the largest paths per compute unit fill the chip; of smaller ones, as
  // many as 256 MB hold, since every chunk is a pass over all launches (8192
  // paths of n = 4, 8 coefficients, double double: 1373 us in 16 chunks with 16
  // workgroups a path throughout, 524 in one with as many as there is work for)
  const size_t fit = ((size_t)256 << 20) / b->slot_bytes;
  b->G = (int)std::min<size_t>(npaths, std::max<size_t>(2 * std::max(cus, 1), fit));
  // device tables: meta, order, tile, then the int tables
  const size_t nt = tab_poly.size() + tab_mon.size() + tab_var.size() + tab_exp.size() + tab_asm.size() +
                    tab_asment.size();
  std::vector<int32_t> all;
  all.reserve(nt + mdk::BATCH_BUCKETS);
  auto seg = [&](const std::vector<int32_t> &v) {
    size_t o = all.size();
    all.insert(all.end(), v.begin(), v.end());
    return o;
  };
  const size_t o_poly = seg(tab_poly), o_mon = seg(tab_mon), o_var = seg(tab_var), o_exp = seg(tab_exp),
               o_asm = seg(tab_asm), o_ase = seg(tab_asment);
  std::vector<int32_t> tl(b->tile, b->tile + mdk::BATCH_BUCKETS);
  const size_t o_tile = seg(tl);
  if ((e = hipMalloc((void **)&b->d_tables, std::max<size_t>(all.size(), 1) * sizeof(int32_t))) != hipSuccess ||
      (e = hipMemcpy(b->d_tables, all.data(), all.size() * sizeof(int32_t), hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMalloc((void **)&b->d_meta, b->meta.size() * sizeof(mdk::PathMeta))) != hipSuccess ||
      (e = hipMemcpy(b->d_meta, b->meta.data(), b->meta.size() * sizeof(mdk::PathMeta), hipMemcpyHostToDevice)) !=
          hipSuccess ||
      (e = build_run(b, b->order, b->run)) != hipSuccess ||
      (e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking)) != hipSuccess) {
    if (b->run.d) (void)hipFree(b->run.d);
    if (b->d_tables) (void)hipFree(b->d_tables);
    if (b->d_meta) (void)hipFree(b->d_meta);
    delete b;
    return mdk::api_hip_fail(e, "batch setup");
  }
  b->d_poly_ptr = b->d_tables + o_poly;
  b->d_mon_ptr = b->d_tables + o_mon;
  b->d_var = b->d_tables + o_var;
  b->d_exp = b->d_tables + o_exp;
  b->d_asm_ptr = b->d_tables + o_asm;
  b->d_asm_ent = b->d_tables + o_ase;
  b->d_tile = b->d_tables + o_tile;
  *out = b;
  return MD_OK;
}

int md_batch_destroy(md_batch *b) {
  if (!b) return MD_OK;
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->cap) (void)hipStreamDestroy(b->cap);
  if (b->run.d) (void)hipFree(b->run.d);
  if (b->d_tables) (void)hipFree(b->d_tables);
  if (b->d_meta) (void)hipFree(b->d_meta);
  delete b;
  return MD_OK;
}

int md_batch_offsets(const md_batch *b, int64_t *x_off, int64_t *cff_off, int64_t *x_total, int64_t *cff_total) {
  if (!b) return mdk::api_fail(MD_EINVAL, "NULL batch");
  for (int p = 0; p < b->P; ++p) {
    if (x_off) x_off[p] = b->meta[p].x_off;
    if (cff_off) cff_off[p] = b->meta[p].cff_off;
  }
  if (x_total) *x_total = b->x_total;
  if (cff_total) *cff_total = b->cff_total;
  return MD_OK;
}

int md_batch_workspace_size(const md_batch *b, size_t *bytes) {
  if (!b || !bytes) return mdk::api_fail(MD_EINVAL, "NULL argument");
  *bytes = batch_ws_bytes(b);
  return MD_OK;
}

int md_batch_newton_step(md_batch *b, int prec_solve, const double *cff, const double *cst, double *x,
                         int32_t *dev_status, double *dev_norms, void *ws, size_t ws_bytes, hipStream_t st) {
  if (!b || !cff || !cst || !x || !dev_status || !dev_norms) return mdk::api_fail(MD_EINVAL, "NULL argument");
  if (!(prec_solve == b->L || (b->L == MD_QD && prec_solve == MD_DD)))
    return mdk::api_fail(MD_EINVAL, "solve precision: the batch's, or double double under quad double");
  if (!ws || ws_bytes < batch_ws_bytes(b)) return mdk::api_fail(MD_ENOSPACE, "workspace too small");
  // the step's launches, some forty for paths of 64 coefficients, are replayed from
  // a captured graph while the arguments stay the same (captured on the second
  // call with them)
  const void *key[8] = {cff, cst, x, dev_status, dev_norms, ws, nullptr, nullptr};
  bool same = b->key_prec == prec_solve;
  for (int q = 0; q < 8; ++q) same = same && key[q] == b->key[q];
  hipError_t e;
  if (same && b->exec) {
    e = hipGraphLaunch(b->exec, st);
    return e == hipSuccess ? MD_OK : mdk::api_hip_fail(e, "graph launch");
  }
  if (same && b->seen && !mdk::api_timing_enabled()) {
    hipGraph_t g = nullptr;
    if ((e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal)) != hipSuccess)
      return mdk::api_hip_fail(e, "capture");
    hipError_t le = launch_step(b, prec_solve, b->run, cff, cst, x, dev_status, dev_norms, ws, b->cap);
    e = hipStreamEndCapture(b->cap, &g);
    if (le != hipSuccess || e != hipSuccess) {
      if (g) (void)hipGraphDestroy(g);
      return mdk::api_hip_fail(le != hipSuccess ? le : e, "capture");
    }
    e = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
      b->exec = nullptr;
      return mdk::api_hip_fail(e, "graph instantiate");
    }
    e = hipGraphLaunch(b->exec, st);
    return e == hipSuccess ? MD_OK : mdk::api_hip_fail(e, "graph launch");
  }
  if (b->exec) {
    (void)hipGraphExecDestroy(b->exec);
    b->exec = nullptr;
  }
  for (int q = 0; q < 8; ++q) b->key[q] = key[q];
  b->key_prec = prec_solve;
  b->seen = true;
  e = launch_step(b, prec_solve, b->run, cff, cst, x, dev_status, dev_norms, ws, st);
  return e == hipSuccess ? MD_OK : mdk::api_hip_fail(e, "batched step");
}

int md_batch_autotune(md_batch *b, int prec_solve, const double *cff, const double *cst, const double *x,
                      double *x_scratch, int32_t *dev_status, double *dev_norms, void *ws, size_t ws_bytes,
                      hipStream_t st, int32_t *chosen) {
  if (!b || !cff || !cst || !x || !x_scratch || !dev_status || !dev_norms) return mdk::api_fail(MD_EINVAL, "NULL argument");
  if (!(prec_solve == b->L || (b->L == MD_QD && prec_solve == MD_DD)))
    return mdk::api_fail(MD_EINVAL, "solve precision: the batch's, or double double under quad double");
  if (!ws || ws_bytes < batch_ws_bytes(b)) return mdk::api_fail(MD_ENOSPACE, "workspace too small");
  static const int cand[3] = {4, 8, 16};
  const size_t xbytes = (size_t)b->L * b->x_total * sizeof(double);
  hipError_t e;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess)
    return mdk::api_hip_fail(e, "autotune setup");
  for (int bk = 0; bk < mdk::BATCH_BUCKETS; ++bk) {
    std::vector<int32_t> list;
    for (int32_t p : b->order)
      if (b->meta[p].bucket == bk) list.push_back(p);
    if (list.empty()) continue;
    BatchRun run;
    if ((e = build_run(b, list, run)) != hipSuccess) break;
    float best = 0.0f;
    int best_t = b->tile[bk];
    for (int c = 0; c < 3 && e == hipSuccess; ++c) {
      b->tile[bk] = cand[c];
      if ((e = hipMemcpy(const_cast<int32_t *>(b->d_tile), b->tile, sizeof(b->tile), hipMemcpyHostToDevice)) !=
          hipSuccess)
        break;
      float ms = 0.0f;
      for (int rep = 0; rep < 2 && e == hipSuccess; ++rep) {  // the first run warms up
        if ((e = hipMemcpyAsync(x_scratch, x, xbytes, hipMemcpyDeviceToDevice, st)) != hipSuccess) break;
        if ((e = hipEventRecord(e0, st)) != hipSuccess) break;
        if ((e = launch_step(b, prec_solve, run, cff, cst, x_scratch, dev_status, dev_norms, ws, st)) != hipSuccess)
          break;
        if ((e = hipEventRecord(e1, st)) != hipSuccess || (e = hipEventSynchronize(e1)) != hipSuccess) break;
        if ((e = hipEventElapsedTime(&ms, e0, e1)) != hipSuccess) break;
      }
      if (e == hipSuccess && (c == 0 || ms < best)) {
        best = ms;
        best_t = cand[c];
      }
    }
    b->tile[bk] = best_t;
    (void)hipStreamSynchronize(st);  // (a failed launch may leave others behind)
    (void)hipFree(run.d);
  }
  if (e == hipSuccess)
    e = hipMemcpy(const_cast<int32_t *>(b->d_tile), b->tile, sizeof(b->tile), hipMemcpyHostToDevice);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (e != hipSuccess) return mdk::api_hip_fail(e, "autotune");
  if (chosen)
    for (int q = 0; q < mdk::BATCH_BUCKETS; ++q) chosen[q] = b->tile[q];
  if (b->exec) {  // a captured step holds the old launch; capture again
    (void)hipGraphExecDestroy(b->exec);
    b->exec = nullptr;
    b->seen = false;
  }
  return MD_OK;
}

int md_batch_set_tiles(md_batch *b, const int32_t *tiles) {
  if (!b || !tiles) return mdk::api_fail(MD_EINVAL, "NULL argument");
  for (int q = 0; q < mdk::BATCH_BUCKETS; ++q)
    if (tiles[q] != 4 && tiles[q] != 8 && tiles[q] != 16) return mdk::api_fail(MD_EINVAL, "tiles are 4, 8 or 16 lanes");
  std::memcpy(b->tile, tiles, sizeof(b->tile));
  hipError_t e = hipMemcpy(const_cast<int32_t *>(b->d_tile), b->tile, sizeof(b->tile), hipMemcpyHostToDevice);
  if (e != hipSuccess) return mdk::api_hip_fail(e, "tiles");
  if (b->exec) {
    (void)hipGraphExecDestroy(b->exec);
    b->exec = nullptr;
    b->seen = false;
  }
  return MD_OK;
}

}  // extern "C"
