// Reverse pass of the rank-m Krylov kernel: gradients of a scalar L(K delta)
// with respect to delta, gamma, W and the expansion-point spin Hamiltonians.
//
// Krylov part (Sec. II.G). The forward builds v_1 = f~/|f~|, f~_k = A v_k with
// A = K0 (R - I) (R the response, q1 = R v), v_{k+1} = the normalized part of
// f~_k orthogonal to v_1..v_k, and x = V c with c solving (F~^T F~) c = F~^T f~.
// Its reverse, given x_bar:
//   c_bar = V^T x_bar, V_bar = x_bar c^T, z = O^-1 c_bar, f~_bar = F~ z,
//   F~_bar = r z^T - F~ z c^T with r = f~ - F~ c (least-squares adjoint);
//   then for k = rank..1: the adjoint of the orthonormalization that made
//   v_{k+1} from f~_k (w_bar = (I - v v^T) v_bar_{k+1} / rho_k,
//   F~_bar_k += (I - V_k V_k^T) w_bar, V_bar_j -= w_bar h_j + f~_k p_j),
//   lambda_k = F~_bar_k, y_k = K0^T lambda_k and v_bar_k += A^T lambda_k
//   = R^T y_k - y_k.
// The response is self-adjoint in the metric Gamma = diag(gamma, W I):
// R = M chi M Gamma with chi the symmetric potential-space response and
// M = [[I, I], [I, -I]], so R^T y = Gamma g with g = M chi M y, the response
// to the potentials (y_q + y_m, y_q - y_m) with identity coupling.
// Parameter gradients: gamma_bar += g_q v_q^T, W_bar += g_m . v_m, and
// dL/dH^sigma from the change of chi with the expansion point.
//
// Expansion-point part (Sec. II.C). With a = M y_k and b = M Gamma v_k,
// s_k = a^T chi b = sum_sigma sum_ij F_ij Xa_ij Xb_ij + Wsum dmu_a dmu_b,
// Xa = C^T H1[a] C. Under a symmetric change E of H^sigma (E' = C^T E C in the
// eigenbasis) the levels move by E'_ii, the eigenvectors rotate by
// E'_ij / (eps_j - eps_i) and mu follows the electron count. Summed over k:
//   E'_bar_ij = ((K - K^T)_ij + (w_i - w_j) D_ij) / (eps_i - eps_j),  i != j,
//     K = sum_k Y0_b Xa + Y0_a Xb (Y0 = F o X),  D = sum_k dmu_b Xa + dmu_a Xb,
//   E'_bar_ii = g_i - w_i / Wsum sum_sigma,j g_j,
//     g_i = sum_k sum_j 2 f[e_i, e_i, e_j] Xa_ij Xb_ij
//           + w'_i (Xa_ii dmu_b + Xb_ii dmu_a - dmu_a dmu_b),
// with f[.,.,.] the second divided difference of the Fermi function and
// w' = -f''. Pairs closer than tau = 1e-3 kT take the same sum written with
// second divided differences, sum_l f[e_i, e_j, e_l] (Xb_il Xa_lj + Xa_il Xb_lj),
// which has no small denominator. Finally dL/dH^sigma = C E'_bar C^T.
#pragma once

#include <hip/hip_runtime.h>

#include "kk_gemm.hpp"
#include "kk_kernels.hpp"

namespace kk {

// Second and fourth derivatives of f(x) = 1/(1+exp(beta(x - mu))).
__device__ __forceinline__ void fermi_d2_d4(double x, double mu, double beta, double* d2, double* d4) {
  const double f = occ(x, mu, beta), fc = occ(-x, -mu, beta), g = f * fc, b2 = beta * beta;
  *d2 = b2 * g * (fc - f);
  *d4 = b2 * b2 * g * (fc - f) * (1.0 - 12.0 * g);
}

// f[x, y, z] for nodes with known f and 1 - f. Nodes spread less than tau:
// expansion about their mean c, f''(c)/2 + f''''(c) h2 / 24 with h2 = 1/2 sum
// of squared deviations (the first-order term vanishes about the mean); else
// (f[b, c] - f[a, b]) / (c - a) over the widest pair of the sorted nodes.
__device__ __forceinline__ double fermi_dd2(double x, double fx, double fcx, double y, double fy, double fcy,
                                            double z, double fz, double fcz, double mu, double beta,
                                            double tau) {
#define KK_SWAP3(p, q)                              \
  if (p > q) {                                      \
    double t_ = p; p = q; q = t_;                   \
    t_ = f##p; f##p = f##q; f##q = t_;              \
    t_ = fc##p; fc##p = fc##q; fc##q = t_;          \
  }
  KK_SWAP3(x, y)
  KK_SWAP3(y, z)
  KK_SWAP3(x, y)
#undef KK_SWAP3
  if (z - x < tau) {
    const double c = (x + y + z) / 3.0;
    const double dx = x - c, dy = y - c, dz = z - c;
    const double h2 = 0.5 * (dx * dx + dy * dy + dz * dz);
    double d2, d4;
    fermi_d2_d4(c, mu, beta, &d2, &d4);
    return 0.5 * d2 + d4 * h2 / 24.0;
  }
  const double f_yz = fermi_divided_difference(y, fy, fcy, z, fz, fcz, beta);
  const double f_xy = fermi_divided_difference(x, fx, fcx, y, fy, fcy, beta);
  return (f_yz - f_xy) / (z - x);
}

// (w_i - w_j)/(e_i - e_j) with w = -f', for |e_i - e_j| < tau: -(f''(m) + f''''(m) h^2 / 6).
__device__ __forceinline__ double w_dd_close(double ei, double ej, double mu, double beta) {
  const double m = 0.5 * (ei + ej), h = 0.5 * (ei - ej);
  double d2, d4;
  fermi_d2_d4(m, mu, beta, &d2, &d4);
  return -(d2 + d4 * h * h / 6.0);
}

// One spin of a group of directions: X of their items (a up, a dn, b up, b dn), np2 apart.
struct AdjSpin {
  const double *Xa, *Xb;           // np x np, direction 0; the next direction's stride apart
  const double *eps, *f, *fc, *w;  // np
  double* D;                       // np x np accumulator
  double* gdiag;                   // np accumulator
};
struct AdjSpins {
  AdjSpin s[2];
  size_t stride;
  int directions;
};

// Reverse-pass state of the Krylov loop on the device.
//   Vbar, Fbar: MAX_RANK x n2, bbar: n2.
// One block of 1024 threads; n2 <= 8192.
__global__ void __launch_bounds__(1024) adj_init(const double* __restrict__ V, const double* __restrict__ Ft,
                                                 const double* __restrict__ ftilde, int n2,
                                                 const KrylovState* __restrict__ st,
                                                 const double* __restrict__ xbar, double* __restrict__ Vbar,
                                                 double* __restrict__ Fbar, double* __restrict__ bbar) {
  __shared__ double O[MAX_RANK][MAX_RANK + 1];
  __shared__ double c[MAX_RANK], z[MAX_RANK];
  __shared__ int ok;
  const int r = st->rank;
  // O = F~^T F~ (lower triangle), F~^T f~ and V^T x_bar, one wave each
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, npairs = r * (r + 1) / 2;
  for (int p = wave; p < npairs + 2 * r; p += blockDim.x / WAVE) {
    int a, b = 0;
    const double *x, *y;
    if (p < npairs) {
      a = 0;
      while ((a + 1) * (a + 2) / 2 <= p) ++a;
      b = p - a * (a + 1) / 2;
      x = Ft + (size_t)a * n2;
      y = Ft + (size_t)b * n2;
    } else {
      a = (p - npairs) >> 1;
      x = ((p - npairs) & 1 ? V : Ft) + (size_t)a * n2;
      y = (p - npairs) & 1 ? xbar : ftilde;
    }
    double d = 0.0;
    for (int i = lane; i < n2; i += WAVE) d += x[i] * y[i];
    d = wave_sum_dpp(d);
    if (lane == 0) {
      if (p < npairs) O[a][b] = d;
      else ((p - npairs) & 1 ? z : c)[a] = d;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    ok = 1;
    for (int j = 0; j < r && ok; ++j) {
      double dj = O[j][j];
      for (int k = 0; k < j; ++k) dj -= O[j][k] * O[j][k];
      if (!(dj > 0.0)) { ok = 0; break; }
      const double ljj = sqrt(dj);
      O[j][j] = ljj;
      for (int i = j + 1; i < r; ++i) {
        double s = O[i][j];
        for (int k = 0; k < j; ++k) s -= O[i][k] * O[j][k];
        O[i][j] = s / ljj;
      }
    }
    for (int pass = 0; pass < 2 && ok; ++pass) {  // c = O^-1 F~^T f~, z = O^-1 V^T x_bar
      double* x = pass ? z : c;
      for (int i = 0; i < r; ++i) {
        double s = x[i];
        for (int k = 0; k < i; ++k) s -= O[i][k] * x[k];
        x[i] = s / O[i][i];
      }
      for (int i = r - 1; i >= 0; --i) {
        double s = x[i];
        for (int k = i + 1; k < r; ++k) s -= O[k][i] * x[k];
        x[i] = s / O[i][i];
      }
    }
    if (!ok)
      for (int i = 0; i < r; ++i) { c[i] = 0.0; z[i] = 0.0; }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n2; i += blockDim.x) {
    double res = ftilde[i], fz = 0.0;
    for (int a = 0; a < r; ++a) {
      const double fa = Ft[(size_t)a * n2 + i];
      res -= c[a] * fa;
      fz += z[a] * fa;
    }
    bbar[i] = fz;
    const double xb = xbar[i];
    for (int a = 0; a < r; ++a) {
      Fbar[(size_t)a * n2 + i] = res * z[a] - fz * c[a];
      Vbar[(size_t)a * n2 + i] = xb * c[a];
    }
  }
}

// Reverse of the orthonormalization that produced v_{k+1} from f~_k (skipped
// for the last direction), then y = -lambda_k (K0 = -I) or lambda_k (the host
// applies K0^T). With u given (K0 = -I) the potentials of a = M y follow, on every orbital. One
// block of 1024 threads, PER >= n2 / 1024 entries each; the 2 (k + 1) dot products run NJ rows of V
// at a time, so that a reduction (all of this kernel's time) serves as many rows.
template <int PER, int NJ>
__global__ void __launch_bounds__(1024) adj_gs(const double* __restrict__ V, const double* __restrict__ Ft, int n2,
                                               int k, int last, double* __restrict__ Vbar,
                                               double* __restrict__ Fbar, double* __restrict__ y, int negate,
                                               const int* __restrict__ offsets, int np, double* __restrict__ u) {
  constexpr int NW = 16;
  __shared__ double part[2][NW][2 * NJ];
  __shared__ double hh[MAX_RANK], pp[MAX_RANK];
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  int buf = 0;
  // sums of N values over the block into sum[], the same bits in every thread; one barrier
  auto reduce = [&](auto& v, auto& sum) __attribute__((always_inline)) {
    constexpr int N = sizeof(v) / sizeof(double);
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const double t = wave_sum_dpp(v[q]);
      if (lane == 0) part[buf][wave][q] = t;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) sum[q] = wave_sum_dpp(lane < nw ? part[buf][lane][q] : 0.0);
    buf ^= 1;
  };
  double* fb = Fbar + (size_t)k * n2;
  if (!last) {
    const double* vn = V + (size_t)(k + 1) * n2;
    const double* fk = Ft + (size_t)k * n2;
    const double* vb = Vbar + (size_t)(k + 1) * n2;
    double first[2] = {}, rt[2], wb[PER];
    for (int i = threadIdx.x; i < n2; i += blockDim.x) {
      first[0] += vn[i] * fk[i];
      first[1] += vn[i] * vb[i];
    }
    reduce(first, rt);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = threadIdx.x + e * blockDim.x;
      wb[e] = i < n2 ? (vb[i] - vn[i] * rt[1]) / rt[0] : 0.0;
    }
    for (int j0 = 0; j0 <= k; j0 += NJ) {
      double d[2 * NJ] = {}, sum[2 * NJ];
#pragma unroll
      for (int q = 0; q < NJ; ++q) {
        if (j0 + q > k) break;
        const double* vj = V + (size_t)(j0 + q) * n2;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          const int i = threadIdx.x + e * blockDim.x;
          const double v = i < n2 ? vj[i] : 0.0;
          d[2 * q] += v * (i < n2 ? fk[i] : 0.0);
          d[2 * q + 1] += v * wb[e];
        }
      }
      reduce(d, sum);
      if (threadIdx.x == 0)
        for (int q = 0; q < NJ && j0 + q <= k; ++q) {
          hh[j0 + q] = sum[2 * q];
          pp[j0 + q] = sum[2 * q + 1];
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = threadIdx.x + e * blockDim.x;
      if (i >= n2) continue;
      double proj = 0.0;
      for (int j = 0; j <= k; ++j) {
        const double vji = V[(size_t)j * n2 + i];
        proj += vji * pp[j];
        Vbar[(size_t)j * n2 + i] -= wb[e] * hh[j] + fk[i] * pp[j];
      }
      fb[i] += wb[e] - proj;
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < n2; i += blockDim.x) y[i] = negate ? -fb[i] : fb[i];
  if (u == nullptr) return;
  __syncthreads();
  const int N = n2 / 2;
  for (int a = threadIdx.x; a < N; a += blockDim.x) {
    const double up = y[a] + y[N + a], dn = y[a] - y[N + a];
    for (int i = offsets[a]; i < offsets[a + 1]; ++i) {
      u[i] = up;
      u[np + i] = dn;
    }
  }
}

// y = A^T x for a row-major n x n A (one thread per output; coalesced over columns).
__global__ void gemv_t(const double* __restrict__ A, const double* __restrict__ x, int n, double* __restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int j = 0; j < n; ++j) s += A[(size_t)j * n + i] * x[j];
  y[i] = s;
}

// Chemical-potential shifts of the pairs of items (2 p, 2 p + 1) = (up, dn) of xdiag. One block each.
__global__ void adj_dmu(const double* __restrict__ xdiag, int nb, int np, const double* __restrict__ w0,
                        const double* __restrict__ w1, const double* __restrict__ wsum_p, double* __restrict__ dmu) {
  __shared__ double sh[17];
  const int p = blockIdx.x;
  const double* x0 = xdiag + (size_t)(2 * p) * np;
  const double* x1 = xdiag + (size_t)(2 * p + 1) * np;
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) s += w0[i] * x0[i] + w1[i] * x1[i];
  s = block_sum(s, sh);
  const double wsum = *wsum_p;
  if (threadIdx.x == 0) dmu[p] = wsum > 0.0 ? s / wsum : 0.0;
}

// Row i of spin blockIdx.y over all directions k of the group (dmu[2 k] of a, dmu[2 k + 1] of b):
// D_ij += sum_k dmu_b Xa_ij + dmu_a Xb_ij and
// g_i += sum_k (sum_j 2 f[e_i, e_i, e_j] Xa_ij Xb_ij + w'_i (Xa_ii dmu_b + Xb_ii dmu_a - dmu_a dmu_b)).
// The divided difference is formed once per element and D is updated once, whatever the directions
// (128 atoms, 8 directions: 8 x 21 us -> 78 us).
__global__ void adj_rows(AdjSpins sp, int nb, int np, const double* __restrict__ dmu, const double* __restrict__ mu_p,
                         double beta, double tau) {
  __shared__ double sh[17];
  const AdjSpin& s = sp.s[blockIdx.y];
  const int i = blockIdx.x, nd = sp.directions;
  const double mu = *mu_p;
  const double ei = s.eps[i], fi = s.f[i], fci = s.fc[i];
  const double* xa = s.Xa + (size_t)i * np;
  const double* xb = s.Xb + (size_t)i * np;
  double* d = s.D + (size_t)i * np;
  double acc = 0.0;
  for (int j = threadIdx.x; j < nb; j += blockDim.x) {
    double dj = d[j], ab = 0.0;
    for (int k = 0; k < nd; ++k) {
      const double a = xa[k * sp.stride + j], b = xb[k * sp.stride + j];
      dj += dmu[2 * k + 1] * a + dmu[2 * k] * b;
      ab += a * b;
    }
    d[j] = dj;
    acc += 2.0 * fermi_dd2(ei, fi, fci, ei, fi, fci, s.eps[j], s.f[j], s.fc[j], mu, beta, tau) * ab;
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) {
    double d2, d4;
    fermi_d2_d4(ei, mu, beta, &d2, &d4);
    double t = 0.0;
    for (int k = 0; k < nd; ++k) {
      const double da = dmu[2 * k], db = dmu[2 * k + 1];
      t += xa[k * sp.stride + i] * db + xb[k * sp.stride + i] * da - da * db;
    }
    s.gdiag[i] += acc - d2 * t;
  }
}

// Near-degenerate pairs: pk[p] += sum_k sum_l f[e_i, e_j, e_l] (Xb_il Xa_jl + Xa_il Xb_jl)
// (X symmetric). pairs[p] = (i, j) for p < n0 in spin 0, then spin 1. One block per pair.
__global__ void adj_pairs(AdjSpins sp, const int2* __restrict__ pairs, int n0, int nb, int np,
                          const double* __restrict__ mu_p, double beta, double tau, double* __restrict__ pk) {
  __shared__ double sh[17];
  const int p = blockIdx.x;
  const AdjSpin& s = sp.s[p < n0 ? 0 : 1];
  const int i = pairs[p].x, j = pairs[p].y;
  const double mu = *mu_p;
  const double ei = s.eps[i], fi = s.f[i], fci = s.fc[i], ej = s.eps[j], fj = s.f[j], fcj = s.fc[j];
  const double *xai = s.Xa + (size_t)i * np, *xbi = s.Xb + (size_t)i * np;
  const double *xaj = s.Xa + (size_t)j * np, *xbj = s.Xb + (size_t)j * np;
  double acc = 0.0;
  for (int l = threadIdx.x; l < nb; l += blockDim.x) {
    double x = 0.0;
    for (int k = 0; k < sp.directions; ++k) {
      const size_t o = k * sp.stride + l;
      x += xbi[o] * xaj[o] + xai[o] * xbj[o];
    }
    acc += fermi_dd2(ei, fi, fci, ej, fj, fcj, s.eps[l], s.f[l], s.fc[l], mu, beta, tau) * x;
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) pk[p] += acc;
}

// E'_bar in the eigenbasis (see the header), spin blockIdx.z, 32 x 32 tiles; pairs closer than tau
// are left at 0 for adj_pair_final. K of a spin is the sum of `chunks` partial sums, 2 np^2 apart.
struct AdjFinal {
  const double *K, *D;  // [chunks][2][np][np], [2][np][np]
  const double *eps[2], *w[2], *gdiag[2];
  double* Ep;           // [2][np][np]
};
__global__ void adj_final(const AdjFinal a, int chunks, const double* __restrict__ gtot_p,
                          const double* __restrict__ wsum_p, int nb, int np, double tau) {
  const int z = blockIdx.z;
  const size_t np2 = (size_t)np * np;
  const double *K = a.K + z * np2, *D = a.D + z * np2, *eps = a.eps[z], *w = a.w[z], *gdiag = a.gdiag[z];
  double* Ep = a.Ep + z * np2;
  auto k_at = [&](size_t o) {
    double v = K[o];
    for (int c = 1; c < chunks; ++c) v += K[o + 2 * c * np2];
    return v;
  };
  __shared__ double kt[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
  for (int r = ty; r < 32; r += 8) kt[r][tx] = k_at((size_t)(bx + r) * np + by + tx);  // K^T tile
  __syncthreads();
  const double wsum = *wsum_p, gtot = *gtot_p;
  for (int r = ty; r < 32; r += 8) {
    const int i = by + r, j = bx + tx;
    double v = 0.0;
    if (i < nb && j < nb) {
      if (i == j) {
        v = gdiag[i] - (wsum > 0.0 ? w[i] / wsum * gtot : 0.0);
      } else {
        const double gap = eps[i] - eps[j];
        if (fabs(gap) >= tau) {
          const size_t ij = (size_t)i * np + j;
          v = ((k_at(ij) - kt[tx][r]) + (w[i] - w[j]) * D[ij]) / gap;
        }
      }
    }
    Ep[(size_t)i * np + j] = v;
  }
}

__global__ void adj_pair_final(const int2* __restrict__ pairs, int n0, int npairs, const double* __restrict__ pk,
                               const double* __restrict__ D0, const double* __restrict__ D1,
                               const double* __restrict__ e0, const double* __restrict__ e1,
                               const double* __restrict__ mu_p, double beta, int np, double* __restrict__ Ep0,
                               double* __restrict__ Ep1) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npairs) return;
  const bool s1 = p >= n0;
  const double* D = s1 ? D1 : D0;
  const double* e = s1 ? e1 : e0;
  double* Ep = s1 ? Ep1 : Ep0;
  const int i = pairs[p].x, j = pairs[p].y;
  const double v = pk[p] + w_dd_close(e[i], e[j], *mu_p, beta) * D[(size_t)i * np + j];
  Ep[(size_t)i * np + j] = v;
  Ep[(size_t)j * np + i] = v;
}

// v_bar_k += Gamma g - y; one wave per atom row.
__global__ void adj_apply(const double* __restrict__ gamma, int N, double W, const double* __restrict__ g,
                          const double* __restrict__ y, double* __restrict__ vbar) {
  const int a = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int lane = threadIdx.x & (WAVE - 1);
  if (a >= N) return;
  const double* gr = gamma + (size_t)a * N;
  double s = 0.0;
  for (int j = lane; j < N; j += WAVE) s += gr[j] * g[j];
  s = wave_sum(s);
  if (lane == 0) {
    vbar[a] += s - y[a];
    vbar[N + a] += W * g[N + a] - y[N + a];
  }
}

// The parameter gradients of all directions at once (g and V: rank x 2N), directions in the
// sweep's order: gamma_bar_ij = sum_k g_q,i v_q,j, one block per row i, and W_bar = sum_k g_m . v_m
// in block N.
__global__ void adj_params(const double* __restrict__ g, const double* __restrict__ V, int N, int rank,
                           double* __restrict__ gamma_bar, double* __restrict__ wbar) {
  __shared__ double sh[17];
  const int i = blockIdx.x;
  const size_t n2 = 2 * (size_t)N;
  if (i < N) {
    for (int j = threadIdx.x; j < N; j += blockDim.x) {
      double s = 0.0;
      for (int k = rank - 1; k >= 0; --k) s += g[k * n2 + i] * V[k * n2 + j];
      gamma_bar[(size_t)i * N + j] = s;
    }
    return;
  }
  double w = 0.0;
  for (int k = rank - 1; k >= 0; --k) {
    double s = 0.0;
    for (int j = threadIdx.x; j < N; j += blockDim.x) s += g[k * n2 + N + j] * V[k * n2 + N + j];
    w += block_sum(s, sh);
  }
  if (threadIdx.x == 0) *wbar = w;
}

// f~_bar += reverse of v_1 = f~ / |f~|; out = -f~_bar (K0 = -I) or f~_bar. One block.
__global__ void __launch_bounds__(1024) adj_finish(const double* __restrict__ V, const double* __restrict__ Vbar,
                                                   const double* __restrict__ ftilde, int n2,
                                                   const double* __restrict__ bbar, double* __restrict__ out,
                                                   int negate) {
  __shared__ double sh[17];
  double t = 0.0, nn = 0.0;
  for (int i = threadIdx.x; i < n2; i += blockDim.x) {
    t += V[i] * Vbar[i];
    nn += ftilde[i] * ftilde[i];
  }
  t = block_sum(t, sh);
  const double nrm = sqrt(block_sum(nn, sh));
  for (int i = threadIdx.x; i < n2; i += blockDim.x) {
    const double b = bbar[i] + (nrm > 0.0 ? (Vbar[i] - V[i] * t) / nrm : 0.0);
    out[i] = negate ? -b : b;
  }
}

// dst (nb x nb) = src (np x np) without the padding, for both spins (blockIdx.y; src np^2 apart).
__global__ void unpad_copy(const double* __restrict__ src2, int np, double* __restrict__ dst0,
                           double* __restrict__ dst1, int nb) {
  const double* src = src2 + (size_t)blockIdx.y * np * np;
  double* dst = blockIdx.y ? dst1 : dst0;
  const size_t n = (size_t)nb * nb;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
    const size_t i = e / nb, j = e - i * nb;
    dst[e] = src[i * np + j];
  }
}

}  // namespace kk
