// dcdl_dict.h -- kernels of the dictionary update (Sec. 4.2, eq. dict_update).
//
// With the sufficient statistics phi (K, K, 2L-1...) and psi (K, P, L...) of
// eq. phi, the data term of eq. dict_update and its gradient are
//   F(D)      = 1/2 ||X||^2 - <D, psi> + 1/2 <D, Q(D)>
//   grad F(D) = Q(D) - psi,   Q(D)_{k,p}[t] = sum_{k'} sum_{t'} phi[k, k', t - t'] D_{k',p}[t']
// (Q is the quadratic form's matrix applied to D; the signal size does not
// enter).  Everything here runs in FP64: the problem is K P |Theta| values.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dcdl_kernels.h"

namespace dcdl {

constexpr int kDictMaxTaps = 2048;  // |Theta| of the dictionary update

// Partial sums of Q = phi applied to D: part[s][k][p][t] is the sum over the
// s-th range of kc atoms k'.  One wave per (k, s), block of 64 NT tiles and p:
// for each k' it stages the row phi[k, k', :] and the atom D[k', p, :] in LDS
// and slides them past each other.
//
// A matrix of n^2 K^2 multiply-adds over K^2 m values of phi (16x16 atoms, K =
// 25: 41 million, 2 us at the FP64 vector rate) needs many waves and few LDS
// reads.  One workgroup per (k, p) with one output per thread and two LDS reads
// per multiply-add used K P of the 256 CUs and took 298 us there.  Here the k'
// are split until the chip is full, and a lane holds TW neighbouring outputs
// of a row: one new value of phi and one (broadcast) of D serve TW of them.
template <int TW, int NT>
__global__ __launch_bounds__(64) void phi_matvec(Geom g, int S, int kc, const double *__restrict__ phi,
                                                 const double *__restrict__ D, double *__restrict__ part) {
  extern __shared__ double dsm[];
  const int n = g.L1 * g.L2, m = g.U1 * g.U2;
  const int L2p = (g.L2 + TW - 1) / TW * TW, tw = L2p / TW, tiles = g.L1 * tw;
  // a padded atom row meets zeros of D; the phi it reads there lies in the
  // rows beside, or in the TW - 1 values before and after them
  double *const sp = dsm + TW - 1, *const sd = sp + m + TW - 1;
  const int k = blockIdx.x / S, s = blockIdx.x - k * S, p = blockIdx.z, lane = threadIdx.x;
  const int tile0 = blockIdx.y * 64 * NT + lane;
  double acc[NT][TW];
  int t1[NT], t2[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int t = tile0 + 64 * i < tiles ? tile0 + 64 * i : 0;
    t1[i] = t / tw;
    t2[i] = (t - t1[i] * tw) * TW;
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = 0.0;
  }
  for (int i = lane; i < TW - 1; i += 64) dsm[i] = sp[m + i] = 0.0;
  for (int i = lane; i < g.L1 * L2p; i += 64) sd[i] = 0.0;
  const int ke = min(g.K, (s + 1) * kc);
  for (int kk = s * kc; kk < ke; ++kk) {
    __syncthreads();
    for (int i = lane; i < n; i += 64) sd[i / g.L2 * L2p + i % g.L2] = D[((long long)kk * g.P + p) * n + i];
    for (int i = lane; i < m; i += 64) sp[i] = phi[((long long)k * g.K + kk) * m + i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (tile0 - lane + 64 * i >= tiles) break;
      for (int u1 = 0; u1 < g.L1; ++u1) {
        const double *const prow = sp + (t1[i] - u1 + g.L1 - 1) * g.U2 + t2[i] + g.L2 - 1;
        const double *const drow = sd + u1 * L2p;
        double w[TW];  // prow[j - u2] for j = 1 ... TW - 1 of the step to come
#pragma unroll
        for (int j = 1; j < TW; ++j) w[j] = prow[j];
        for (int u2 = 0; u2 < L2p; u2 += TW) {
#pragma unroll
          for (int q = 0; q < TW; ++q) {
            const double d = drow[u2 + q];
            double v[TW];
            v[0] = prow[-(u2 + q)];
#pragma unroll
            for (int j = 1; j < TW; ++j) v[j] = w[j];
#pragma unroll
            for (int j = 0; j < TW; ++j) acc[i][j] += v[j] * d;
#pragma unroll
            for (int j = 1; j < TW; ++j) w[j] = v[j - 1];
          }
        }
      }
    }
  }
  double *const out = part + (((long long)s * g.K + k) * g.P + p) * n;
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    if (tile0 + 64 * i >= tiles) break;
#pragma unroll
    for (int j = 0; j < TW; ++j)
      if (t2[i] + j < g.L2) out[t1[i] * g.L2 + t2[i] + j] = acc[i][j];
  }
}

// One projected-gradient trial: Dn = Proj(D - step G), one workgroup per atom.
// Proj scales an atom whose norm exceeds 1 back to the unit sphere.
// sums, when given, are three values set to 0 for the kernels that follow.
__global__ __launch_bounds__(256) void pgd_trial(int per_atom, const double *__restrict__ D,
                                                 const double *__restrict__ G, double step, double *__restrict__ Dn,
                                                 double *sums) {
  __shared__ double sh[4];
  if (sums && blockIdx.x == 0 && threadIdx.x < 3) sums[threadIdx.x] = 0.0;
  const long long base = (long long)blockIdx.x * per_atom;
  double a = 0.0;
  for (int i = threadIdx.x; i < per_atom; i += 256) {
    const double v = D[base + i] - step * G[base + i];
    Dn[base + i] = v;
    a += v * v;
  }
  a = block_sum<256>(a, sh);
  if (a > 1.0) {
    const double s = 1.0 / sqrt(a);
    for (int i = threadIdx.x; i < per_atom; i += 256) Dn[base + i] *= s;
  }
}

// Qn = the sum of the S partial results of phi_matvec, in order, and
// out[0] += <Dn, psi>, out[1] += <Dn, Qn>, out[2] += <G, Dn - D> (D, G may be NULL).
__global__ __launch_bounds__(256) void trial_dots(long long n, int S, const double *__restrict__ part,
                                                  const double *__restrict__ Dn, const double *__restrict__ D,
                                                  const double *__restrict__ psi, double *__restrict__ Qn,
                                                  const double *__restrict__ G, double *out) {
  __shared__ double sh[4];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
    double q = 0.0;
#pragma unroll 8
    for (int s = 0; s < S; ++s) q += part[s * n + i];
    Qn[i] = q;
    const double d = Dn[i];
    a0 += d * psi[i];
    a1 += d * q;
    if (G) a2 += G[i] * (d - D[i]);
  }
  a0 = block_sum<256>(a0, sh);
  a1 = block_sum<256>(a1, sh);
  a2 = block_sum<256>(a2, sh);
  if (threadIdx.x == 0) {
    atomic_add_f64(out, a0);
    atomic_add_f64(out + 1, a1);
    atomic_add_f64(out + 2, a2);
  }
}

// G = Q - psi.
__global__ __launch_bounds__(256) void grad_from_q(long long n, const double *__restrict__ Q,
                                                   const double *__restrict__ psi, double *__restrict__ G) {
  for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256) G[i] = Q[i] - psi[i];
}

// out = max_k sum_{k', tau} |phi[k, k', tau]|: an upper bound of every row sum
// of the quadratic form's matrix, hence of its largest eigenvalue (Gershgorin).
__global__ __launch_bounds__(256) void phi_row_bound(int K, int m, const double *__restrict__ phi, double *out) {
  __shared__ double sh[4];
  const int k = blockIdx.x;
  double a = 0.0;
  for (long long i = threadIdx.x; i < (long long)K * m; i += 256) a += fabs(phi[(long long)k * K * m + i]);
  a = block_sum<256>(a, sh);
  if (threadIdx.x == 0) atomic_max_nonneg(out, a);
}

}  // namespace dcdl
