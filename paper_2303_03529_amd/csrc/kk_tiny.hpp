// FP64 responses of the smallest systems, whose Krylov step is a chain of launches each not much
// longer than an empty one (about 4 us, 1 us apart). Two launches transform, one reduces:
//   tiny_forward   X = C^T U~ G + its transpose over both operand pairs, the Fermi factors and both
//                  triangles of Y, one workgroup per 32 x 32 tile pair and spin;
//   tiny_back      P = C Y and its Mulliken row sums, one workgroup per 32 x 32 tile and spin;
//   combine_block  the Mulliken sums, the chemical-potential shift and the preconditioned
//                  derivative, by every block of the launch that needs them next
//                  (orth_potentials of the next direction, or the solve).
// A tile's contraction is cut over the eight waves of its workgroup and summed through LDS, so
// nothing of a split contraction goes through memory: against 64 x 64 tiles cut into chunks
// that are launch items of their own, no symmetrizing pass, and a sixth of the Mulliken partial
// rows. Operands go from L2 to registers without LDS (every wave reads rows of its own), as pairs
// of columns: lane lc of a matrix fragment holds columns 2 lc and 2 lc + 1, the first in the
// fragment of even columns, the second in that of odd ones.
#pragma once

#include <hip/hip_runtime.h>

#include "kk_gemm.hpp"
#include "kk_kernels.hpp"

namespace kk {

constexpr int TINY_TILE = 32, TINY_WAVES = 8, TINY_THREADS = TINY_WAVES * WAVE;
// Contraction steps (4 rows each) that a wave has in flight, the kernels' U: of these the one that
// leaves the fewest of the wave's `steps` over, then the largest. A load past the end is one of
// the last step again, and costs as much: 8 atoms (3 steps) 80 us an update with U = 3 or 4 and 92 us with 6,
// 37 atoms (11 steps) 190 us with 6, 200 us with 4 and 214 us with 5. Sixteen waves with half the steps
// each were 1-17 % slower.
constexpr int TINY_FORWARD_U[] = {6, 5, 4, 3}, TINY_BACK_U[] = {8, 6, 5, 3};
template <int N>
inline int tiny_batch(const int (&candidates)[N], int steps) {
  int best = candidates[0], waste = 1 << 30;
  for (int u : candidates) {
    const int w = (steps + u - 1) / u * u - steps;
    if (w < waste) {
      waste = w;
      best = u;
    }
  }
  return best;
}

struct TinyArgs {
  struct Item {
    const double *C, *G, *CT, *u;
    const double *eps, *f, *fc, *w;
    double *Y, *xdiag, *part;
  } item[2];         // by spin
  int n, kc, tiles;  // row stride; contraction length (a multiple of 32); tiles of 32 that cover it
  double beta;
  const int* stop;
};

__device__ __forceinline__ d2 tiny_load(const double* p) { return *reinterpret_cast<const d2*>(p); }

// Grid (tile pairs, 2 spins); TEST: one block more in each spin, the first of which runs test.
template <int U, bool TEST>
__global__ __launch_bounds__(TINY_THREADS) void tiny_forward(const TinyArgs a, const ResidualTest test) {
  constexpr int T = TINY_TILE;
  __shared__ double red[TINY_WAVES][T * T];
  __shared__ double yt[T][T + 1];
  static_assert(TINY_WAVES * T * T >= solve_lds(RESIDUAL_TEST_MAX_RANK), "the test's LDS");
  if (TEST && blockIdx.x == 0) {
    if (blockIdx.y == 0) residual_test(test, &red[0][0]);
    return;
  }
  const int stopped = *a.stop;
  const TinyArgs::Item& it = a.item[blockIdx.y];
  int I = 0, rem = TEST ? blockIdx.x - 1 : blockIdx.x;
  while (rem >= a.tiles - I) {
    rem -= a.tiles - I;
    ++I;
  }
  const int m0 = I * T, n0 = (I + rem) * T, n = a.n;
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, lr = lane >> 4, lc = lane & 15;
  const int total = a.kc / 4;  // steps of the contraction; this wave's are wave, wave + TINY_WAVES, ...
  d4 acc[2][2] = {};
  const size_t row0 = (size_t)lr;
  const double *cm = it.C + row0 * n + m0 + 2 * lc, *gm = it.G + row0 * n + m0 + 2 * lc;
  const double *cn = it.C + row0 * n + n0 + 2 * lc, *gn = it.G + row0 * n + n0 + 2 * lc;
  const double* up = it.u + row0;
  const size_t stride = (size_t)4 * n;
  // the spectrum at this thread's elements of the reduced tile, loaded ahead of the contraction
  constexpr int EPT = T * T / TINY_THREADS;
  double em[EPT], fm[EPT], fcm[EPT], en[EPT], fn[EPT], fcn[EPT];
#pragma unroll
  for (int h = 0; h < EPT; ++h) {
    const int e = threadIdx.x + h * TINY_THREADS, q = e / WAVE, l = e & (WAVE - 1);
    const int m = m0 + 2 * ((l >> 4) + 4 * (q & 3)) + (q >> 3), c = n0 + 2 * (l & 15) + ((q >> 2) & 1);
    em[h] = it.eps[m]; fm[h] = it.f[m]; fcm[h] = it.fc[m];
    en[h] = it.eps[c]; fn[h] = it.f[c]; fcn[h] = it.fc[c];
  }
  for (int s0 = wave; s0 < total; s0 += U * TINY_WAVES) {
    d2 vcm[U], vgm[U], vcn[U], vgn[U];
    double vu[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const size_t s = min(s0 + q * TINY_WAVES, total - 1);
      vcm[q] = tiny_load(cm + s * stride);
      vgn[q] = tiny_load(gn + s * stride);
      vgm[q] = tiny_load(gm + s * stride);
      vcn[q] = tiny_load(cn + s * stride);
      vu[q] = up[s * 4];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const double u = s0 + q * TINY_WAVES < total ? vu[q] : 0.0;
      const d2 a0 = u * vcm[q], a1 = u * vgm[q];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[i], vgn[q][j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[i], vcn[q][j], acc[i][j], 0, 0, 0);
    }
  }
  if (stopped) return;  // the same value in every thread, tested once the loads are under way
  // element r of fragment (i, j): row 2 (lr + 4 r) + i and column 2 lc + j of the tile
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][((i * 2 + j) * 4 + r) * WAVE + lane] = acc[i][j][r];
  __syncthreads();
#pragma unroll
  for (int h = 0; h < T * T / TINY_THREADS; ++h) {
    const int e = threadIdx.x + h * TINY_THREADS, q = e / WAVE, l = e & (WAVE - 1);
    const int tm = 2 * ((l >> 4) + 4 * (q & 3)) + (q >> 3), tn = 2 * (l & 15) + ((q >> 2) & 1);
    const int m = m0 + tm, c = n0 + tn;
    if (m > c) continue;  // below the diagonal of a diagonal tile: the mirror of an element above
    double x = red[0][e];
#pragma unroll
    for (int w = 1; w < TINY_WAVES; ++w) x += red[w][e];
    x *= 0.5;
    double y;
    if (m == c) {
      it.xdiag[m] = x;
      y = -it.w[m] * x;
    } else {
      y = fermi_divided_difference(em[h], fm[h], fcm[h], en[h], fn[h], fcn[h], a.beta) * x;
    }
    yt[tm][tn] = y;
    if (m0 == n0) yt[tn][tm] = y;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < T * T / TINY_THREADS; ++h) {
    const int e = threadIdx.x + h * TINY_THREADS, r = e / T, c = e % T;
    it.Y[(size_t)(m0 + r) * n + n0 + c] = yt[r][c];
    if (m0 != n0) it.Y[(size_t)(n0 + r) * n + m0 + c] = yt[c][r];
  }
}

template <int U>
__global__ __launch_bounds__(TINY_THREADS) void tiny_back(const TinyArgs a) {
  constexpr int T = TINY_TILE;
  __shared__ double rs[TINY_WAVES][T];
  const int stopped = *a.stop;
  const TinyArgs::Item& it = a.item[blockIdx.y];
  const int tm = blockIdx.x / a.tiles, tn = blockIdx.x - tm * a.tiles;
  const int m0 = tm * T, n0 = tn * T, n = a.n;
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, lr = lane >> 4, lc = lane & 15;
  const int total = a.kc / 4;
  const size_t row0 = (size_t)lr, stride = (size_t)4 * n;
  const double *cp = it.CT + row0 * n + m0 + 2 * lc, *yp = it.Y + row0 * n + n0 + 2 * lc;
  d2 g[2][4];  // G at the accumulator's elements, loaded ahead of the contraction
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) g[i][r] = tiny_load(it.G + (size_t)(m0 + 2 * (lr + 4 * r) + i) * n + n0 + 2 * lc);
  d4 acc[2][2] = {};
  for (int s0 = wave; s0 < total; s0 += U * TINY_WAVES) {
    d2 vc[U], vy[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const size_t s = min(s0 + q * TINY_WAVES, total - 1);
      vc[q] = tiny_load(cp + s * stride);
      vy[q] = tiny_load(yp + s * stride);
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const d2 c = s0 + q * TINY_WAVES < total ? vc[q] : d2{0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[i], vy[q][j], acc[i][j], 0, 0, 0);
    }
  }
  if (stopped) return;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double s = acc[i][0][r] * g[i][r][0] + acc[i][1][r] * g[i][r][1];
      s = row16_sum(s);
      if (lc == 0) rs[wave][2 * (lr + 4 * r) + i] = s;
    }
  __syncthreads();
  if (threadIdx.x < T) {
    double s = rs[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < TINY_WAVES; ++w) s += rs[w][threadIdx.x];
    it.part[(size_t)tn * n + m0 + threadIdx.x] = s;
  }
}

// What combine_small does, and with K0 (DENSE) precondition after it, for every atom of the
// system in one block of COMBINE_BLOCK threads: f~ = K0 (q1 - v), or -(q1 - v), of the direction v into
// ft_lds (2 natoms doubles). The block that `write`s also stores it and q1. Two rounds of loads (K0's
// rows, the orbital ranges and the terms of the shift, then the partial rows, an atom a wave), whose
// latency is most of what this costs. SPLIT: the sums in combine_small's order, to the same bits, which
// the split products, and so their rounding, go on from. natoms <= COMBINE_BLOCK_ATOMS.
struct CombineArgs {
  const double *xdiag, *part, *w_up, *w_dn, *wsum, *t, *v, *K0;
  const int* offsets;
  double *q1, *ft;
  int nparts, nb, np, natoms, split;
};
constexpr int COMBINE_BLOCK = 1024, COMBINE_BLOCK_ATOMS = 64;
template <bool SPLIT, bool DENSE>
__device__ __forceinline__ void combine_block(const CombineArgs& c, double* ft_lds, bool write) {
  constexpr int NW = COMBINE_BLOCK / WAVE, LOADS = SPLIT ? 6 : 3, N2MAX = 2 * COMBINE_BLOCK_ATOMS;
  constexpr int SUM_THREADS = SPLIT ? COMBINE_THREADS : COMBINE_BLOCK;
  constexpr int ROWS = DENSE ? N2MAX / NW : 1, COLS = DENSE ? N2MAX / WAVE : 1;
  __shared__ double psum[SUM_THREADS / WAVE], dl[DENSE ? N2MAX : 1];
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, N = c.natoms, n2 = 2 * N;
  auto sum = [](double x) __attribute__((always_inline)) { return SPLIT ? wave_sum(x) : wave_sum_dpp(x); };
  double kr[ROWS][COLS];
  if constexpr (DENSE) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
      for (int k = 0; k < COLS; ++k) {
        const int row = wave + r * NW, j = lane + k * WAVE;
        kr[r][k] = row < n2 && j < n2 ? c.K0[(size_t)row * n2 + j] : 0.0;
      }
  }
  const double wsum = *c.wsum;
  if (threadIdx.x < SUM_THREADS) {
    double s = 0.0;
    for (int i = threadIdx.x; i < c.nb; i += SUM_THREADS) s += c.w_up[i] * c.xdiag[i] + c.w_dn[i] * c.xdiag[c.np + i];
    s = sum(s);
    if (lane == 0) psum[wave] = s;
  }
  double* const dn = DENSE ? dl : ft_lds;  // the atoms' Mulliken sums of both spins first
  for (int a = wave; a < N; a += NW) {
    const int i0 = c.offsets[a], norb = c.offsets[a + 1] - i0, tot = c.nparts * norb;
    const double *p0 = c.part + i0, *p1 = p0 + (size_t)c.nparts * c.np;
    double a0 = 0.0, a1 = 0.0;
    for (int base = 0; base < tot; base += LOADS * WAVE) {
      double v0[LOADS], v1[LOADS];
#pragma unroll
      for (int k = 0; k < LOADS; ++k) {
        const int e = base + lane + k * WAVE;
        const bool ok = e < tot;
        const int p = ok ? e / norb : 0;
        const size_t o = (size_t)p * c.np + (e - p * norb);
        v0[k] = ok ? p0[o] : 0.0;
        v1[k] = ok ? p1[o] : 0.0;
      }
#pragma unroll
      for (int k = 0; k < LOADS; ++k) {
        a0 += v0[k];
        a1 += v1[k];
      }
    }
    a0 = sum(a0);
    a1 = sum(a1);
    if (lane == 0) {
      dn[a] = a0;
      dn[N + a] = a1;
    }
  }
  __syncthreads();
  double top = 0.0;
  if constexpr (SPLIT) {
    top = wave_sum(lane < SUM_THREADS / WAVE ? psum[lane] : 0.0);
  } else {
    for (int q = 0; q < NW; ++q) top += psum[q];
  }
  const double dmu = wsum > 0.0 ? top / wsum : 0.0;
  for (int a = threadIdx.x; a < N; a += COMBINE_BLOCK) {
    const double d0 = dn[a] + dmu * c.t[a], d1 = dn[N + a] + dmu * c.t[N + a];
    const double qa = d0 + d1, ma = d0 - d1;
    const double fa = DENSE ? qa - c.v[a] : -(qa - c.v[a]), fm = DENSE ? ma - c.v[N + a] : -(ma - c.v[N + a]);
    dn[a] = fa;
    dn[N + a] = fm;
    if (write) {
      c.q1[a] = qa;
      c.q1[N + a] = ma;
      if constexpr (!DENSE) {
        c.ft[a] = fa;
        c.ft[N + a] = fm;
      }
    }
  }
  __syncthreads();
  if constexpr (DENSE) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int row = wave + r * NW;  // wave-uniform
      if (row >= n2) break;
      double f = 0.0;
#pragma unroll
      for (int k = 0; k < COLS; ++k) {
        const int j = lane + k * WAVE;
        if (j < n2) f += kr[r][k] * dl[j];
      }
      f = wave_sum(f);
      if (lane == 0) {
        ft_lds[row] = f;
        if (write) c.ft[row] = f;
      }
    }
    __syncthreads();
  }
}

}  // namespace kk
