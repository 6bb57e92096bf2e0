// M = A_0^{-1} by Householder QR with Q^T and back substitution, all of it in
// one workgroup: the batched step and the small systems where the refinement
// of an inverse in doubles does not suit A_0.
#pragma once
#include "common.hpp"

namespace mdk {

// Sum of an accumulator over the whole workgroup (four wavefronts), the
// renormalized total in every thread.
template <int L>
__device__ void block_sum_lazy(double (&u)[L], double (&r)[L], double *sh) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  team_sum_lazy<L>(u, 64);
  __syncthreads();  // sh may still be read from the previous call
  if (lane == 0)
#pragma unroll
    for (int l = 0; l < L; ++l) sh[wv * L + l] = u[l];
  __syncthreads();
  double t[L];
#pragma unroll
  for (int l = 0; l < L; ++l) t[l] = sh[l];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
    double o[L];
#pragma unroll
    for (int l = 0; l < L; ++l) o[l] = sh[w * L + l];
    MD<L>::add_lazy(t, o);
  }
  MD<L>::renorm(t, r);
}

__device__ inline double block_max(double v, double *sh) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  __syncthreads();
  if (lane == 0) sh[wv] = v;
  __syncthreads();
  double r = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, sh[w]);
  return r;
}

// qr [L][n][n] holds A_0 (row-major; overwritten), qt and M [L][n][n], invd [L][n]
// are the results' and scratch memory, n <= 128; T (4, 8 or 16) lanes a dot
// product.  shr: 80 doubles of LDS; sh_sing becomes 1 where A_0 is singular to
// working precision.
template <int Ls>
__device__ void factor_matrix(int n, int T, double *qr, double *qt, double *invd, double *M, double *shr, int &sh_sing) {
  const int tid = threadIdx.x, NT = blockDim.x;
  const int team = tid / T, tl = tid % T, nteams = NT / T;
  const size_t nn = (size_t)n * n;
  if (tid == 0) sh_sing = 0;
  for (int q = tid; q < (int)nn; q += NT) {
    const int i = q / n, j = q - i * n;
#pragma unroll
    for (int l = 0; l < Ls; ++l) qt[(size_t)l * nn + q] = (l == 0 && i == j) ? 1.0 : 0.0;
  }
  __syncthreads();
  // Householder QR of A_0 (row-major, in place) with Q^T
  for (int c = 0; c < n; ++c) {
    double u[Ls], nrm2[Ls];
    md::zero<Ls>(u);
    for (int i = c + tid; i < n; i += NT) {
      double xi[Ls];
      ld<Ls>(qr, nn, (size_t)i * n + c, xi);
      MD<Ls>::fma_lazy(u, xi, xi);
    }
    block_sum_lazy<Ls>(u, nrm2, shr);
    if (tid == 0) {
      double x0[Ls], beta[Ls], tc[Ls], inv[Ls];
      ld<Ls>(qr, nn, (size_t)c * n + c, x0);
      if (!(nrm2[0] > 0.0)) {
        md::copy<Ls>(x0, beta);
        md::zero<Ls>(tc);
        md::zero<Ls>(inv);
        sh_sing = 1;
      } else {
        double y[Ls], alpha[Ls], v0[Ls];
        md::rsqrt_newton<Ls>(nrm2, y);
        MD<Ls>::mul(nrm2, y, alpha);
        const bool nonneg = x0[0] >= 0.0;
        if (nonneg) md::neg<Ls>(alpha, beta);
        else md::copy<Ls>(alpha, beta);
        MD<Ls>::sub(x0, beta, v0);
        MD<Ls>::mul(v0, y, tc);
        if (!nonneg) md::neg<Ls>(tc, tc);
        md::recip_newton<Ls>(v0, inv);
      }
#pragma unroll
      for (int l = 0; l < Ls; ++l) {
        shr[8 * 8 + l] = inv[l];
        shr[8 * 8 + 8 + l] = tc[l];
      }
      st<Ls>(qr, nn, (size_t)c * n + c, beta);
    }
    __syncthreads();
    double inv[Ls], tc[Ls];
#pragma unroll
    for (int l = 0; l < Ls; ++l) {
      inv[l] = shr[8 * 8 + l];
      tc[l] = shr[8 * 8 + 8 + l];
    }
    for (int i = c + 1 + tid; i < n; i += NT) {  // v below the diagonal
      double xi[Ls], vi[Ls];
      ld<Ls>(qr, nn, (size_t)i * n + c, xi);
      MD<Ls>::mul(xi, inv, vi);
      st<Ls>(qr, nn, (size_t)i * n + c, vi);
    }
    __syncthreads();
    // apply H_c to the trailing columns of A_0 and to every column of Q^T
    const int na = n - 1 - c;
    for (int col = team; col < na + n; col += nteams) {
      double *base = col < na ? qr : qt;
      const int j = col < na ? c + 1 + col : col - na;
      double acc[Ls], dot[Ls], w[Ls];
      md::zero<Ls>(acc);
      for (int i = c + tl; i < n; i += T) {
        double vi[Ls], xv[Ls];
        if (i == c) {
          md::zero<Ls>(vi);
          vi[0] = 1.0;
        } else {
          ld<Ls>(qr, nn, (size_t)i * n + c, vi);
        }
        ld<Ls>(base, nn, (size_t)i * n + j, xv);
        MD<Ls>::fma_lazy(acc, vi, xv);
      }
      team_sum_lazy<Ls>(acc, T);
      MD<Ls>::renorm(acc, dot);
      MD<Ls>::mul(dot, tc, w);
      for (int i = c + tl; i < n; i += T) {
        double vi[Ls], xv[Ls];
        if (i == c) {
          md::zero<Ls>(vi);
          vi[0] = 1.0;
        } else {
          ld<Ls>(qr, nn, (size_t)i * n + c, vi);
        }
        ld<Ls>(base, nn, (size_t)i * n + j, xv);
        MD<Ls>::fms(xv, vi, w);
        st<Ls>(base, nn, (size_t)i * n + j, xv);
      }
    }
    __syncthreads();
  }
  // reciprocals of diag(R), with the singularity test of the single-system path
  {
    double dmax = 0.0;
    for (int i = tid; i < n; i += NT) dmax = fmax(dmax, fabs(qr[(size_t)i * n + i]));
    dmax = block_max(dmax, shr);
    for (int i = tid; i < n; i += NT) {
      double rii[Ls], q[Ls];
      ld<Ls>(qr, nn, (size_t)i * n + i, rii);
      if (!(fabs(rii[0]) > ldexp((double)n, -53 * Ls) * dmax)) {
        md::zero<Ls>(q);
        sh_sing = 1;
      } else {
        md::recip_newton<Ls>(rii, q);
      }
      st<Ls>(invd, n, i, q);
    }
  }
  __syncthreads();
  // M = R^{-1} Q^T: one wavefront per column, rows in lanes (p and p + 64)
  {
    const int lane = tid & 63, wv = tid >> 6, nw = NT >> 6;
    for (int c = wv; c < n; c += nw) {
      double y0[Ls], y1[Ls];
      md::zero<Ls>(y0);
      md::zero<Ls>(y1);
      if (lane < n) ld<Ls>(qt, nn, (size_t)lane * n + c, y0);
      if (lane + 64 < n) ld<Ls>(qt, nn, (size_t)(lane + 64) * n + c, y1);
      for (int i = n - 1; i >= 0; --i) {
        double z[Ls], zi[Ls];
        md::zero<Ls>(z);
        const bool hi = i >= 64;
        const int src = hi ? i - 64 : i;
        if (lane == src) {
          double d[Ls];
          ld<Ls>(invd, n, i, d);
          if (hi) {
            MD<Ls>::mul(y1, d, z);
            md::copy<Ls>(z, y1);
          } else {
            MD<Ls>::mul(y0, d, z);
            md::copy<Ls>(z, y0);
          }
        }
#pragma unroll
        for (int l = 0; l < Ls; ++l) zi[l] = __shfl(z[l], src, 64);
        if (lane < i) {
          double rp[Ls];
          ld<Ls>(qr, nn, (size_t)lane * n + i, rp);
          MD<Ls>::fms(y0, rp, zi);
        }
        if (lane + 64 < i) {
          double rp[Ls];
          ld<Ls>(qr, nn, (size_t)(lane + 64) * n + i, rp);
          MD<Ls>::fms(y1, rp, zi);
        }
      }
      if (lane < n) st<Ls>(M, nn, (size_t)lane * n + c, y0);
      if (lane + 64 < n) st<Ls>(M, nn, (size_t)(lane + 64) * n + c, y1);
    }
  }
  __syncthreads();
}

}  // namespace mdk
