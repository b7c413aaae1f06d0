// Vector, reduction and setup kernels of the spin-charge response and the
// Krylov loop. All reductions use a fixed order, so results are bitwise
// reproducible run to run.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "kk_gemm.hpp"

namespace kk {

constexpr int WAVE = 64;
constexpr double BREAKDOWN_TOL = 1e-13;
constexpr int MAX_RANK = 64;

// Sum over the wave by exchanges with lane ^ 32, 16, 8, 4, 2, 1 in turn, the same bits in every lane.
// (After the first three steps values repeat every 8 lanes, so a rotation by 4 is the exchange
// with lane ^ 4.)
__device__ __forceinline__ double row_sum(double v) {  // of a row of 16 lanes
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  return v;
}
__device__ __forceinline__ double wave_sum(double v) { return row_sum(add_xor<16>(add_xor<32>(v))); }
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, lane_xor<32>(v));
  v = fmax(v, lane_xor<16>(v));
  v = fmax(v, dpp_f64<0x128>(v));
  v = fmax(v, dpp_f64<0x124>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  return fmax(v, dpp_f64<0xB1>(v));
}

// Wave-wide sum of a double in another fixed order, the same bits in every lane, for serial
// reduction chains (the orthonormalization, the m x m solve): within each row of 16 lanes by DPP moves
// (rotate by 8 and 4, then exchange with lane ^ 2 and lane ^ 1: every step adds two values
// that the partner lane adds in the other order, so all 16 lanes end with the same bits),
// then the four row sums read from lanes 0, 16, 32 and 48 and added as (r0 + r1) + (r2 + r3).
__device__ __forceinline__ double lane_f64(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

// Sum over a block of up to 1024 threads (multiple of 64); every thread gets
// thread 0's total. sh must hold at least 17 doubles.
__device__ double block_sum(double v, double* sh) {
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
  const int nw = blockDim.x / WAVE;
  v = wave_sum(v);
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  if (wave == 0) {
    double t = (lane < nw) ? sh[lane] : 0.0;
    t = wave_sum(t);
    if (lane == 0) sh[16] = t;
  }
  __syncthreads();
  const double r = sh[16];
  __syncthreads();
  return r;
}

// The padded copies of a prepare in one launch, blockIdx.z choosing the matrix: 0 S, 1 Z
// (transposed), 2 and 3 Q of each spin, each dst (np x np, zero padded) = src (nb x nb) in
// 32 x 32 tiles; 4 gamma (contiguous). As launches of their own they cost a small prepare about
// 4 us each; together 3.4 us at 16 atoms.
struct SetupCopies {
  const double* src[4];
  double* dst[4];
  const double* gamma;
  double* gamma_dst;
  size_t gamma_n;
  int nb, np;
};
constexpr int SETUP_COPIES_Z = 5, SETUP_TRANSPOSED = 1;
__global__ void setup_copies(const SetupCopies c) {
  if (blockIdx.z == 4) {
    const size_t step = (size_t)gridDim.x * gridDim.y * blockDim.x;
    for (size_t i = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < c.gamma_n; i += step)
      c.gamma_dst[i] = c.gamma[i];
    return;
  }
  __shared__ double t[32][33];
  const bool transpose = blockIdx.z == SETUP_TRANSPOSED;
  const double* __restrict__ src = c.src[blockIdx.z];
  double* __restrict__ dst = c.dst[blockIdx.z];
  const int nb = c.nb, np = c.np;
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    // read source rows coalesced: source tile origin is (by, bx) if plain, (bx, by) if transposed
    const int k = ty + 8 * q;
    const int sr = (transpose ? bx : by) + k, sc = (transpose ? by : bx) + tx;
    t[k][tx] = (sr < nb && sc < nb) ? src[(size_t)sr * nb + sc] : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = ty + 8 * q;
    dst[(size_t)(by + k) * np + bx + tx] = transpose ? t[tx][k] : t[k][tx];
  }
}

// dst = src^T of up to four np x np matrices, one per blockIdx.z (32 x 32 tiles).
struct TransposeArgs {
  const double* src[4];
  double* dst[4];
};
__global__ void transpose_sq(const TransposeArgs a, int np) {
  __shared__ double t[32][33];
  const double* __restrict__ src = a.src[blockIdx.z];
  double* __restrict__ dst = a.dst[blockIdx.z];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int q = 0; q < 4; ++q) t[ty + 8 * q][tx] = src[(size_t)(bx + ty + 8 * q) * np + by + tx];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) dst[(size_t)(by + ty + 8 * q) * np + bx + tx] = t[tx][ty + 8 * q];
}

// From 40 kT below mu on it rounds to one, and a wave of such levels (most of them, in order) is
// spared the exponential and the division.
__device__ __forceinline__ double occ(double e, double mu, double beta) {
  const double x = beta * (e - mu);
  if (x < -40.0) return 1.0;
  return 1.0 / (1.0 + exp(x));
}

// Sec. II.C: the spectrum of a prepared expansion point in one launch of one block. One
// chemical potential for both spins with sum_sigma sum_k f(eps_k) = N_e, then per level (padded
// to np with zeros) eps, f = 1/(1+exp(beta(e-mu))), fc = 1 - f (computed as f of the mirrored
// argument) and w = beta f fc, and wsum = the sum of both spins' w.
// mu is where the bisection of [min eps - 40 kT, max eps + 40 kT] down to 1e-15 ends, polished by
// Newton steps where its count is still off. What the kernel costs is its number of counts, all of
// it reduction latency, so the halvings whose outcome is known are not counted: Newton's
// iteration (with its own sums, ordered for speed) first finds the root to the count's rounding,
// and the bisection then counts only at midpoints within SPECTRUM_NOISE N_e / (dN/dmu) of it,
// where rounding could decide. A count too flat there to tell (that distance reaches
// 0.1 kT: a gap many kT wide at N_e) leaves every halving to a count of its own, as does a
// Newton iteration that does not settle. The count is monotone and its slope changes by at most a
// factor e per kT, so farther out its sign is that of the midpoint's side: mu has the same bits
// either way. Against 57 counts, and with the occupations and the sum as launches of their own:
// 16 atoms 65 + 14 -> 30 us, 128 atoms 89 + 14 -> 37 us, 1024 atoms 393 + 20 -> 123 us. Of what was left
// much was instructions that every wave repeats, so the sums take one barrier and half the final
// exchanges, the known halvings are one wave's, and the block has 256 or 512 threads where those
// hold the levels; the window tables are a launch of their own where they are used: with
// tables 31 us at 16 and 43 us at 128 atoms, now 14.5 and 28 us (tables 10 us at 200 atoms). The counts
// with both midpoints that can follow, two halvings a reduction, cost more exponentials
// than the reductions they spared (8.0 against 5.3 us at 16 atoms).
struct SpectrumArgs {
  const double* e[2];                    // levels of each spin, nb
  double *eps[2], *f[2], *fc[2], *w[2];  // np each
  double *mu, *wsum;
  int nb, np;
  double n_e, beta;
  // Window tables (kk_gemm.hpp): act, range and tiles of each spin, count of both. tiles_in: the
  // forward tile list in launch order, ntiles of bm x bn blocks. cut: with ref the largest of
  // the w and |F| between the outermost levels, blocks are active from |F| >= cut ref (exact_cut
  // 0) or from beta cut (exact_cut 1).
  unsigned char* act[2];
  int2* range[2];
  int2* tiles[2];
  int* count;
  const int2* tiles_in;
  int ntiles, bm, bn, exact_cut;
  double cut;
};
constexpr double SPECTRUM_NOISE = 2e-14;
// Which blocks of Y are left out (Window). Within a block pair |F_ij| = beta f_lo (1 - f_hi)
// phi <= beta max f max(1 - f) min(1, 1 / (beta gap)) over the pair's levels, the lower factor
// from the block that can hold the lower level.
//   FP64, BF16: below 2^-60 of ref, a lower bound of the largest |F|, 2^7 below FP64's rounding
//   of the products' sums.
//   FP16 x 3: below 2^-42 beta, where s_Y |Y| <= 2^14 |F| / (beta / 4) < 2^-25 rounds to zero in
//   both pieces of Y, so leaving the block out changes no bit of the products.
constexpr double WIN_CUT = 0x1p-60, WIN_CUT_F16 = 0x1p-42;
constexpr int WIN_MAX_BLOCKS = 1024;  // Nb <= 65536
constexpr int SPECTRUM_MAX_THREADS = 1024;

// Sums of N values over the block, the same bits in every thread, with one barrier: buf alternates
// between calls, so a wave still reading one call's partial sums never sees the next call's.
// EXACT: to block_sum's bits (those of a block of 1024 threads too, if only the first T hold levels).
template <int NW, int N, bool EXACT>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*sh)[NW][2], int& buf) {
  static_assert(N <= 2, "sh");
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
#pragma unroll
  for (int q = 0; q < N; ++q) v[q] = EXACT ? wave_sum(v[q]) : wave_sum_dpp(v[q]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < N; ++q) sh[buf][wave][q] = v[q];
  __syncthreads();
  // (block_sum's first two exchanges here would add zeros: the waves' sums fill one row)
  static_assert(NW <= 16, "a row");
#pragma unroll
  for (int q = 0; q < N; ++q) v[q] = row_sum((lane & 15) < NW ? sh[buf][lane & 15][q] : 0.0);
  buf ^= 1;
}

// T: threads, 256 or 512 where they hold a level of each spin each (fewer waves repeat what every
// wave computes alike), else 1024. PER: levels per thread and spin kept in registers.
template <int T, int PER>
__global__ void __launch_bounds__(T) spectrum(const SpectrumArgs a) {
  constexpr int NW = T / WAVE;
  __shared__ double sums[2][NW][2], ends[3];
  __shared__ double smin[NW], smax[NW];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE, nb = a.nb;
  const double beta = a.beta, n_e = a.n_e, kT = 1.0 / beta;
  int buf = 0;
  double e0[PER], e1[PER];
  double lo = 1e300, hi = -1e300;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = tid + k * T;
    e0[k] = i < nb ? a.e[0][i] : 0.0;
    e1[k] = i < nb ? a.e[1][i] : 0.0;
  }
  // fn(i, up, dn) for this thread's levels in ascending order
  auto levels = [&](int n, auto&& fn) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (tid + k * T < n) fn(tid + k * T, e0[k], e1[k]);
    for (int i = tid + PER * T; i < n; i += T) fn(i, i < nb ? a.e[0][i] : 0.0, i < nb ? a.e[1][i] : 0.0);
  };
  levels(nb, [&](int, double u, double d) {
    lo = fmin(lo, fmin(u, d));
    hi = fmax(hi, fmax(u, d));
  });
  lo = -wave_max(-lo);
  hi = wave_max(hi);
  if (lane == 0) {
    smin[wave] = lo;
    smax[wave] = hi;
  }
  __syncthreads();
  for (int q = 0; q < NW; ++q) {
    lo = fmin(lo, smin[q]);
    hi = fmax(hi, smax[q]);
  }
  lo -= 40.0 * kT;
  hi += 40.0 * kT;

  // the root to the count's rounding, and how far from it a midpoint's side is certain
  double root = 0.5 * (lo + hi), margin = 1e300;
  {
    double l = lo, h = hi, step = hi - lo;
    for (int it = 0; it < 24; ++it) {
      double s[2] = {0.0, 0.0};
      levels(nb, [&](int, double u, double v) {
        const double fu = occ(u, root, beta), fv = occ(v, root, beta);
        s[0] += fu + fv;
        s[1] += fu * (1.0 - fu) + fv * (1.0 - fv);
      });
      block_sums<NW, 2, false>(s, sums, buf);
      const double resid = s[0] - n_e, slope = beta * s[1];
      const double near = SPECTRUM_NOISE * n_e / slope + 1e-14 * fabs(root);
      if (fabs(resid) <= 0.05 * SPECTRUM_NOISE * n_e) {
        if (near < 0.1 * kT) margin = near;
        break;
      }
      if (resid < 0.0) l = root; else h = root;
      double next = root - resid / slope;
      // the bracket halved where Newton leaves it or has not halved its last step
      if (!(next > l && next < h) || fabs(next - root) > 0.5 * step) next = 0.5 * (l + h);
      step = fabs(next - root);
      root = next;
    }
  }
  const auto ended = [&](double mid) __attribute__((always_inline)) { return hi - lo <= 1e-15 * fmax(1.0, fabs(mid)); };
  bool end = false;
  // the halvings of a certain outcome, up to the first that is to be counted, by one wave
  if (margin < 1e300) {
    if (wave == 0) {
      if (margin > 1e-15 * fmax(1.0, fmax(fabs(lo), fabs(hi)))) {
        // half the bracket stays above the margin, so the width at which the bisection ends is
        // not reached. Four halvings to a branch, by the halves of lo and hi (0.5 (lo + hi) to the bit).
        double hl = 0.5 * lo, hh = 0.5 * hi;
        bool on = true;
        for (int iter = 0; iter < 400 && on; iter += 4)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double mid = hl + hh, d = mid - root, half = 0.5 * mid;
            on = on && fabs(d) > margin;
            hl = on && d < 0.0 ? half : hl;
            hh = on && !(d < 0.0) ? half : hh;
          }
        lo = 2.0 * hl;
        hi = 2.0 * hh;
      } else {
        for (int iter = 0; iter < 400; ++iter) {
          const double mid = 0.5 * (lo + hi);
          if (!(fabs(mid - root) > margin)) break;
          if (mid < root) lo = mid; else hi = mid;
          if ((end = ended(mid))) break;
        }
      }
      if (lane == 0) {
        ends[0] = lo;
        ends[1] = hi;
        ends[2] = end;
      }
    }
    __syncthreads();
    lo = ends[0];
    hi = ends[1];
    end = ends[2] != 0.0;
  }
  for (int iter = 0; iter < 400 && !end; ++iter) {
    const double mid = 0.5 * (lo + hi);
    bool below = mid < root;
    if (!(fabs(mid - root) > margin)) {
      double c[1] = {0.0};
      levels(nb, [&](int, double u, double v) { c[0] += occ(u, mid, beta) + occ(v, mid, beta); });
      block_sums<NW, 1, true>(c, sums, buf);
      below = c[0] < n_e;
    }
    if (below) lo = mid; else hi = mid;
    end = ended(mid);
  }
  double mu = 0.5 * (lo + hi);
  for (int it = 0; it < 3; ++it) {
    double s[2] = {0.0, 0.0};
    levels(nb, [&](int, double u, double v) {
      const double fu = occ(u, mu, beta), fd = occ(v, mu, beta);
      s[0] += fu + fd;
      s[1] += fu * occ(-u, -mu, beta) + fd * occ(-v, -mu, beta);
    });
    block_sums<NW, 2, true>(s, sums, buf);
    const double d = s[1] * beta, resid = s[0] - n_e;
    if (d <= 0.0 || fabs(resid) <= 1e-13 * n_e) break;
    mu -= resid / d;
  }
  if (tid == 0) *a.mu = mu;
  double ws[1] = {0.0};
  levels(a.np, [&](int i, double u, double v) {  // whole waves: np and the strides are multiples of 64
    double w[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bool in = i < nb;
      const double e = s ? v : u, f = in ? occ(e, mu, beta) : 0.0, fc = in ? occ(-e, -mu, beta) : 0.0;
      w[s] = in ? beta * f * fc : 0.0;
      a.eps[s][i] = in ? e : 0.0;
      a.f[s][i] = f;
      a.fc[s][i] = fc;
      a.w[s][i] = w[s];
    }
    ws[0] += w[0] + w[1];
  });
  block_sums<NW, 1, true>(ws, sums, buf);
  if (tid == 0) *a.wsum = ws[0];
}

// The window tables of a spectrum, one block for each spin.
__global__ void __launch_bounds__(SPECTRUM_MAX_THREADS) window_tables(const SpectrumArgs a) {
  constexpr int T = SPECTRUM_MAX_THREADS, NW = T / WAVE;
  __shared__ double smin[NW], smax[NW], sref[NW];
  __shared__ double bmin[WIN_MAX_BLOCKS], bmax[WIN_MAX_BLOCKS];  // levels of each window block
  __shared__ double bf[WIN_MAX_BLOCKS], bfc[WIN_MAX_BLOCKS];     // its largest f and 1 - f
  __shared__ int blo[WIN_MAX_BLOCKS], bhi[WIN_MAX_BLOCKS], wcount[NW];
  static_assert(WIN == WAVE, "a wave's levels are a window block");
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE, nb = a.nb, s = blockIdx.x;
  const int nblk = a.np / WIN;
  const double beta = a.beta, mu = *a.mu;
  double e_min = 1e300, e_max = -1e300, ref = 0.0;  // of both spins
  for (int i = tid; i < a.np; i += T) {             // whole waves: np and the strides are multiples of 64
    const bool in = i < nb;
    const double e = a.eps[s][i], other = a.eps[1 - s][i];
    if (in) {
      e_min = fmin(e_min, fmin(e, other));
      e_max = fmax(e_max, fmax(e, other));
      ref = fmax(ref, fmax(a.f[s][i] * a.fc[s][i], a.f[1 - s][i] * a.fc[1 - s][i]));
    }
    // the block's lowest and highest level; a NaN makes them unbounded, an all-padding block keeps
    // them reversed
    const bool nan = __any(in && !(e == e && mu == mu));
    double bl = in ? e : INFINITY, bh = in ? e : -INFINITY;
    bl = -wave_max(-bl);
    bh = wave_max(bh);
    if (lane == 0) {
      bmin[i / WIN] = nan ? -INFINITY : bl;
      bmax[i / WIN] = nan ? INFINITY : bh;
    }
  }
  e_min = -wave_max(-e_min);
  e_max = wave_max(e_max);
  ref = wave_max(ref);
  if (lane == 0) {
    smin[wave] = e_min;
    smax[wave] = e_max;
    sref[wave] = ref;
  }
  __syncthreads();
  for (int q = 0; q < NW; ++q) {
    e_min = fmin(e_min, smin[q]);
    e_max = fmax(e_max, smax[q]);
    ref = fmax(ref, sref[q]);
  }
  const double wide = beta * (e_max - e_min);
  ref = fmax(ref, occ(e_min, mu, beta) * occ(-e_max, -mu, beta) * (wide > 0.0 ? -expm1(-wide) / wide : 1.0));
  const double cut = a.exact_cut ? a.cut : a.cut * ref;
  for (int b = tid; b < nblk; b += T) {  // f falls with the level, so the block's ends bound it
    const bool any = bmin[b] <= bmax[b];
    bf[b] = any ? (isinf(bmin[b]) ? 1.0 : occ(bmin[b], mu, beta)) : 0.0;
    bfc[b] = any ? (isinf(bmax[b]) ? 1.0 : occ(-bmax[b], -mu, beta)) : 0.0;
    blo[b] = INT_MAX;
    bhi[b] = 0;
  }
  __syncthreads();
  for (int p = tid; p < nblk * nblk; p += T) {
    const int I = p / nblk, J = p - I * nblk;
    const double imin = bmin[I], imax = bmax[I], jmin = bmin[J], jmax = bmax[J];
    double bound = 0.0;
    if (!(imin > jmax)) bound = bf[I] * bfc[J];
    if (!(jmin > imax)) bound = fmax(bound, bf[J] * bfc[I]);
    const double z = beta * fmax(jmin - imax, imin - jmax);
    if (z > 1.0) bound /= z;
    const bool on = imin <= imax && jmin <= jmax && !(bound < cut);
    if (on) {
      atomicMin(&blo[J], I);
      atomicMax(&bhi[J], I + 1);
    }
    a.act[s][p] = on || I == J;
  }
  __syncthreads();
  for (int b = tid; b < nblk; b += T) a.range[s][b] = bhi[b] > 0 ? make_int2(blo[b] * WIN, bhi[b] * WIN) : make_int2(0, 0);
  int on_before = 0, off_before = 0;
  for (int base = 0; base < a.ntiles; base += T) {
    const int t = base + tid;
    bool on = false;
    int2 tile = make_int2(0, 0);
    if (t < a.ntiles) {
      tile = a.tiles_in[t];
      for (int i = 0; i < a.bm; ++i)
        for (int j = 0; j < a.bn; ++j) on |= a.act[s][(size_t)(tile.x * a.bm + i) * nblk + tile.y * a.bn + j] != 0;
    }
    const unsigned long long ball = __ballot(on);
    if (lane == 0) wcount[wave] = __popcll(ball);
    __syncthreads();
    int before = 0, total = 0;
    for (int q = 0; q < NW; ++q) {
      if (q < wave) before += wcount[q];
      total += wcount[q];
    }
    before += __popcll(ball & ((1ull << lane) - 1));
    if (t < a.ntiles)
      a.tiles[s][on ? on_before + before : a.ntiles - 1 - (off_before + tid - before)] = tile;
    on_before += total;
    off_before += min(T, a.ntiles - base) - total;
    __syncthreads();
  }
  if (tid == 0) a.count[s] = on_before;
}

// out[s*natoms + I] = sum_{i in I} sum_k X_s[i][k] * Y_s[i][k] * wk_s[k], one block of
// ROW_DOTS_THREADS threads per atom (blockIdx.x) and spin (blockIdx.y). A thread takes the columns
// k = tid, tid + T, ... of one row after another; ROW_DOTS_BATCH of these are loaded before the
// first is used, so that the block keeps enough loads in flight (it is bound by HBM, and by
// latency in small systems: 16 atoms 9.8 -> 4.0 us, 128 atoms 40 -> 10 us, 1024 atoms 645 -> 501 us
// against one block per atom for both spins, a load at a time); the sum's order and roundings do not depend on the batch. ncols >= 1.
constexpr int ROW_DOTS_THREADS = 256, ROW_DOTS_BATCH = 9;
__global__ void __launch_bounds__(ROW_DOTS_THREADS)
    atom_row_dots(const double* __restrict__ x0, const double* __restrict__ x1, int ldx,
                  const double* __restrict__ y0, const double* __restrict__ y1, int ldy,
                  const double* __restrict__ wk0, const double* __restrict__ wk1, int ncols,
                  const int* __restrict__ offsets, int natoms, double* __restrict__ out) {
  __shared__ double sh[17];
  const int a = blockIdx.x, s = blockIdx.y;
  const int r0 = offsets[a], r1 = offsets[a + 1];
  const double *x = s ? x1 : x0, *y = s ? y1 : y0, *wk = s ? wk1 : wk0;
  double acc = 0.0;
  int i = r0, k = threadIdx.x;
  if (k >= ncols) i = r1;
  while (i < r1) {
    double xv[ROW_DOTS_BATCH], yv[ROW_DOTS_BATCH], wv[ROW_DOTS_BATCH];
#pragma unroll
    for (int q = 0; q < ROW_DOTS_BATCH; ++q) {
      const bool in = i < r1;
      xv[q] = in ? x[(size_t)i * ldx + k] : 0.0;
      yv[q] = in ? y[(size_t)i * ldy + k] : 0.0;
      wv[q] = in ? wk[k] : 0.0;
      k += ROW_DOTS_THREADS;
      if (k >= ncols) {
        k = threadIdx.x;
        ++i;
      }
    }
#pragma unroll
    for (int q = 0; q < ROW_DOTS_BATCH; ++q) {
#pragma clang fp contract(off)
      const double p = xv[q] * yv[q];
      acc += p * wv[q];
    }
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) out[s * natoms + a] = acc;
}

// Mulliken projection of caller density-matrix changes (Sec. III.A):
// dn^s_I = sum_{i in I} sum_j dD^s_ij S_ji, S symmetric so S_ji = S_ij.
// Output (dq, dm) = (dn_up + dn_dn, dn_up - dn_dn). One block per atom and item.
__global__ void mulliken_rows(const double* __restrict__ dup, const double* __restrict__ ddn, int nb,
                              const double* __restrict__ S, int lds, const int* __restrict__ offsets,
                              int natoms, double* __restrict__ dqm) {
  __shared__ double sh[17];
  const int a = blockIdx.x, b = blockIdx.y;
  const size_t mat = (size_t)nb * nb * b;
  const int r0 = offsets[a], r1 = offsets[a + 1];
  double su = 0.0, sd = 0.0;
  for (int i = r0; i < r1; ++i) {
    const double* pu = dup + mat + (size_t)i * nb;
    const double* pd = ddn + mat + (size_t)i * nb;
    const double* ps = S + (size_t)i * lds;
    for (int k = threadIdx.x; k < nb; k += blockDim.x) {
      const double s = ps[k];
      su += pu[k] * s;
      sd += pd[k] * s;
    }
  }
  su = block_sum(su, sh);
  sd = block_sum(sd, sh);
  if (threadIdx.x == 0) {
    dqm[(size_t)b * 2 * natoms + a] = su + sd;
    dqm[(size_t)b * 2 * natoms + natoms + a] = su - sd;
  }
}

// Per-orbital spin potentials for a batch of directions (Sec. III.A):
// u^s_I = sum_J gamma_IJ v_q[J] + sign_s W v_m[I], written to every orbital of
// atom I in u[(b*2 + s)*np + i]. One wave per (atom, direction). With gamma
// NULL the coupling is the identity, u^s_I = v_q[I] + sign_s W v_m[I] (the
// reverse pass uses it with W = 1 to apply the transposed response).
__device__ __forceinline__ void potentials_dev(const double* __restrict__ gamma, int natoms, double W,
                                               const double* __restrict__ v, int batch,
                                               const int* __restrict__ offsets, int np, double* __restrict__ u,
                                               const int* __restrict__ stop, int bx) {
  if (stop != nullptr && *stop != 0) return;
  const int wid = (bx * blockDim.x + threadIdx.x) / WAVE;
  const int lane = threadIdx.x & (WAVE - 1);
  if (wid >= natoms * batch) return;
  const int b = wid / natoms, a = wid - b * natoms;
  const double* vb = v + (size_t)b * 2 * natoms;
  double s = 0.0;
  if (gamma != nullptr) {
    const double* g = gamma + (size_t)a * natoms;
    for (int j = lane; j < natoms; j += WAVE) s += g[j] * vb[j];
    s = wave_sum(s);
  } else {
    s = vb[a];
  }
  const double up = s + W * vb[natoms + a];
  const double dn = s - W * vb[natoms + a];
  for (int i = offsets[a] + lane; i < offsets[a + 1]; i += WAVE) {
    u[((size_t)b * 2 + 0) * np + i] = up;
    u[((size_t)b * 2 + 1) * np + i] = dn;
  }
}

__global__ void potentials(const double* __restrict__ gamma, int natoms, double W,
                           const double* __restrict__ v, int batch, const int* __restrict__ offsets,
                           int np, double* __restrict__ u, const int* __restrict__ stop) {
  potentials_dev(gamma, natoms, W, v, batch, offsets, np, u, stop, blockIdx.x);
}

// Combine the two spins (Sec. II.C, III.A): dmu from the diagonal of X,
// Mulliken sums per atom, and q1 = (dn_up + dn_dn, dn_up - dn_dn).
//   xdiag[(b*2+s)*np + i], part[(b*2+s)][p][np], t[s*natoms + I] = sum_{i in I}
//   sum_k C_ik w_k G_ik (the response to a unit chemical-potential shift),
//   wsum = sum_s sum_i w_i.
// One wave per atom: its lanes split the partial rows, each adds the atom's
// orbitals of its rows, and the wave reduces. Grid: (ceil(natoms / waves per
// block), batch); every block also reduces dmu over all orbitals (cached reads).
__device__ __forceinline__ void combine_dev(const double* __restrict__ xdiag, const double* __restrict__ part,
                                            int nparts, int part_stride, const double* __restrict__ w_up,
                                            const double* __restrict__ w_dn, const double* __restrict__ wsum_p,
                                            const double* __restrict__ t, int nb, int np,
                                            const int* __restrict__ offsets, int natoms, double* __restrict__ q1,
                                            const int* __restrict__ stop, int bx, int by,
                                            const double* __restrict__ vsub = nullptr, double* __restrict__ ft = nullptr) {
  if (stop != nullptr && *stop != 0) return;
  __shared__ double sh[17];
  const int b = by;
  const double* xu = xdiag + ((size_t)b * 2 + 0) * np;
  const double* xd = xdiag + ((size_t)b * 2 + 1) * np;
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) s += w_up[i] * xu[i] + w_dn[i] * xd[i];
  s = block_sum(s, sh);
  const double wsum = *wsum_p;
  const double dmu = wsum > 0.0 ? s / wsum : 0.0;
  const int lane = threadIdx.x & (WAVE - 1);
  const int a = bx * (blockDim.x / WAVE) + (int)(threadIdx.x / WAVE);
  if (a >= natoms) return;
  const int i0 = offsets[a], i1 = offsets[a + 1];
  double dn[2];
  for (int sp = 0; sp < 2; ++sp) {
    const double* pp = part + ((size_t)b * 2 + sp) * part_stride * np;
    double acc = 0.0;
    for (int p = lane; p < nparts; p += WAVE)
      for (int i = i0; i < i1; ++i) acc += pp[(size_t)p * np + i];
    dn[sp] = wave_sum(acc) + dmu * t[sp * natoms + a];
  }
  if (lane == 0) {
    const double qa = dn[0] + dn[1], ma = dn[0] - dn[1];
    q1[(size_t)b * 2 * natoms + a] = qa;
    q1[(size_t)b * 2 * natoms + natoms + a] = ma;
    if (ft != nullptr) {  // the preconditioned directional derivative with K0 = -I: -(q1 - v)
      ft[a] = -(qa - vsub[a]);
      ft[natoms + a] = -(ma - vsub[natoms + a]);
    }
  }
}

// Blocks of the combine kernels: COMBINE_THREADS threads, one wave per atom.
constexpr int COMBINE_THREADS = 256;
constexpr int COMBINE_ATOMS = COMBINE_THREADS / WAVE;

__global__ void combine(const double* __restrict__ xdiag, const double* __restrict__ part, int nparts,
                        const double* __restrict__ w_up, const double* __restrict__ w_dn,
                        const double* __restrict__ wsum_p, const double* __restrict__ t, int nb, int np,
                        const int* __restrict__ offsets, int natoms, double* __restrict__ q1,
                        const int* __restrict__ stop, const double* __restrict__ vsub = nullptr,
                        double* __restrict__ ft = nullptr) {
  combine_dev(xdiag, part, nparts, nparts, w_up, w_dn, wsum_p, t, nb, np, offsets, natoms, q1, stop, blockIdx.x,
              blockIdx.y, vsub, ft);
}

// sum of both spins' w (one block).
__global__ void sum_two(const double* __restrict__ a, const double* __restrict__ b, int n,
                        double* __restrict__ out) {
  __shared__ double sh[17];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += a[i] + b[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) *out = s;
}

// ---------------------------------------------------------------------------
// Krylov loop (Sec. II.G)

struct KrylovState {
  int rank;       // accepted directions
  int stop;       // 1 after a breakdown, a zero starting vector or reaching the residual target
  int status;     // 0 ok, 1 breakdown, -5 singular Gram matrix
  int done;       // directions whose residual_test ended the expansion; 0: none did
  double min_pivot, max_pivot;
  double ls_residual;  // ||F~ c - f~|| / ||f~|| of the last solve
};

// What a solve tells a host that waits for it, in pinned host memory. word = 2 seq + stop is one
// store, so the host may act on it while the kernel still runs; st is whole once the stream
// has passed the kernel.
struct SolveReport {
  unsigned long long word;
  KrylovState st;
};

// y = K0 (x - sub) (sub may be null), or -(x - sub) when K0 is null.
// One wave per row. Skipped after a breakdown when stop is given. With reset given (the
// first launch of an update, stop null) thread 0 also clears that Krylov state.
__global__ void precondition(const double* __restrict__ K0, const double* __restrict__ x,
                             const double* __restrict__ sub, double* __restrict__ y, int n2,
                             const int* __restrict__ stop, KrylovState* reset = nullptr) {
  if (reset != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
    reset->rank = 0; reset->stop = 0; reset->status = 0; reset->done = 0;
    reset->min_pivot = 0.0; reset->max_pivot = 0.0; reset->ls_residual = 1.0;
  }
  if (stop != nullptr && *stop != 0) return;
  const int row = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int lane = threadIdx.x & (WAVE - 1);
  if (row >= n2) return;
  if (K0 == nullptr) {
    if (lane == 0) y[row] = -(x[row] - (sub ? sub[row] : 0.0));
    return;
  }
  const double* kr = K0 + (size_t)row * n2;
  double s = 0.0;
  for (int j = lane; j < n2; j += WAVE) s += kr[j] * (x[j] - (sub ? sub[j] : 0.0));
  s = wave_sum(s);
  if (lane == 0) y[row] = s;
}

// Orthogonalize src against the accepted directions V[0..rank) with modified
// Gram-Schmidt, two passes; accept it as V[rank] if its norm kept more than
// BREAKDOWN_TOL of its starting norm, else stop the expansion. One block of
// at least n2 / 8 threads.
__device__ __forceinline__ void orth_dev(const double* __restrict__ src, double* __restrict__ V, int n2,
                                         KrylovState* st) {
  __shared__ double sh[17];
  if (st->stop) return;
  const int rank = st->rank;
  constexpr int PER = 8;  // n2 <= 8 * 1024
  double w[PER];
  double nn = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int i = threadIdx.x + e * blockDim.x;
    w[e] = i < n2 ? src[i] : 0.0;
    nn += w[e] * w[e];
  }
  const double start = sqrt(block_sum(nn, sh));
  // Two passes of projections against v_0 .. v_{rank-1}, in order; the entries of
  // the next v_j are loaded before the current projection's reduction, so the
  // loop waits on reductions, not on loads. Entries past n2 are zero in w and v.
  auto load_row = [&](int j, double* dst) {
    const double* vj = V + (size_t)j * n2;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = threadIdx.x + e * blockDim.x;
      dst[e] = i < n2 ? vj[i] : 0.0;
    }
  };
  const int steps = 2 * rank;
  double cur[PER], nxt[PER] = {};
  if (steps > 0) load_row(0, cur);
  for (int t = 0; t < steps; ++t) {
    if (t + 1 < steps) load_row((t + 1) % rank, nxt);
    double d = 0.0;
#pragma unroll
    for (int e = 0; e < PER; ++e) d += cur[e] * w[e];
    d = block_sum(d, sh);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      w[e] -= d * cur[e];
      cur[e] = nxt[e];
    }
  }
  nn = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) nn += w[e] * w[e];
  const double nrm = sqrt(block_sum(nn, sh));
  if (!(nrm > BREAKDOWN_TOL * start) || rank >= MAX_RANK) {
    if (threadIdx.x == 0) {
      st->stop = 1;
      if (rank > 0) st->status = 1;
    }
    return;
  }
  double* vr = V + (size_t)rank * n2;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int i = threadIdx.x + e * blockDim.x;
    if (i < n2) vr[i] = w[e] / nrm;
  }
  __syncthreads();
  if (threadIdx.x == 0) st->rank = rank + 1;
}

__global__ void __launch_bounds__(1024) krylov_orthonormalize(const double* __restrict__ src,
                                                              double* __restrict__ V, int n2,
                                                              KrylovState* st) {
  orth_dev(src, V, n2, st);
}

// O = F~^T F~, rhs = F~^T f~ of the first r directions, Cholesky O = L L^T, c = O^-1 rhs, with x given
// x = V c (0 on a non-positive pivot), and the projected residual ||F~ c - f~|| / ||f~|| formed
// explicitly, returned to thread 0. One block of at most 16 waves; lds: solve_lds(r) doubles. Ends
// without a barrier. Every result has the same bits whatever the number of waves and whether x is
// given: an adaptive update ends at a rank that its inputs alone decide, wherever its tests ran.
struct Solution {
  double residual, min_pivot, max_pivot;
  bool ok;  // every pivot positive
};
constexpr int SOLVE_ROWS = 8 * 1024 / WAVE;  // n2 <= 8 * 1024
constexpr int solve_lds(int r) { return r * (r + 1) + r + 2 * SOLVE_ROWS + 3; }
__device__ __forceinline__ Solution least_squares(const double* __restrict__ V, const double* Ft,
                                                  const double* __restrict__ ftilde, int n2, int r,
                                                  double* __restrict__ x, double* lds) {
  const int ldo = r + 1;
  double *const O = lds, *const c = O + r * ldo, *const sr = c + r, *const fin = sr + 2 * SOLVE_ROWS;
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  // The r (r + 1) / 2 entries of O and the r of the right-hand side, one wave each (fixed
  // lane order and reduction tree, so the result is deterministic); 4 loads per lane in flight.
  {
    const int npairs = r * (r + 1) / 2;
    for (int p = wave; p < npairs + r; p += nw) {
      int a, b = -1;
      if (p < npairs) {
        a = 0;
        while ((a + 1) * (a + 2) / 2 <= p) ++a;
        b = p - a * (a + 1) / 2;
      } else {
        a = p - npairs;
      }
      const double* fa = Ft + (size_t)a * n2;
      const double* y = b >= 0 ? Ft + (size_t)b * n2 : ftilde;
      double d4[4] = {0.0, 0.0, 0.0, 0.0};
      for (int base = 0; base < n2; base += 4 * WAVE) {
        double xa[4], xb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int i = base + lane + k * WAVE;
          xa[k] = i < n2 ? fa[i] : 0.0;
          xb[k] = i < n2 ? y[i] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) d4[k] += xa[k] * xb[k];
      }
      const double d = wave_sum_dpp((d4[0] + d4[1]) + (d4[2] + d4[3]));
      if (lane == 0) {
        if (b >= 0) { O[a * ldo + b] = d; O[b * ldo + a] = d; }
        else c[a] = d;
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    // Cholesky O = L L^T in wave 0, lane i owning row i (r <= MAX_RANK = WAVE): column j's
    // entries l_ij = O_ij / l_jj, then the trailing update O_ik -= l_ij l_kj (k <= i), l_kj
    // taken from lane k. One wave's LDS accesses complete in order.
    int good = 1;
    double pmin = 0.0, pmax = 0.0;
    for (int j = 0; j < r; ++j) {
      const double dj = O[j * ldo + j];
      if (!(dj > 0.0)) {  // the same value in every lane
        good = 0;
        break;
      }
      pmin = (j == 0) ? dj : fmin(pmin, dj);
      pmax = (j == 0) ? dj : fmax(pmax, dj);
      const double ljj = sqrt(dj);
      const bool below = lane > j && lane < r;
      const double lij = below ? O[lane * ldo + j] / ljj : 0.0;
      if (lane == j) O[j * ldo + j] = ljj;
      if (below) O[lane * ldo + j] = lij;
      for (int k = j + 1; k < r; ++k) {
        const double lkj = lane_f64(lij, k);
        if (below && k <= lane) O[lane * ldo + k] -= lij * lkj;
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (good) {
      double ci = lane < r ? c[lane] : 0.0;
      for (int j = 0; j < r; ++j) {  // L y = rhs
        const double yj = lane_f64(ci / O[j * ldo + j], j);
        if (lane == j) ci = yj;
        else if (lane > j && lane < r) ci -= O[lane * ldo + j] * yj;
      }
      for (int j = r - 1; j >= 0; --j) {  // L^T c = y
        const double xj = lane_f64(ci / O[j * ldo + j], j);
        if (lane == j) ci = xj;
        else if (lane < j) ci -= O[j * ldo + lane] * xj;
      }
      if (lane < r) c[lane] = ci;
    }
    if (lane == 0) {
      fin[0] = good;
      fin[1] = pmin;
      fin[2] = pmax;
    }
  }
  __syncthreads();
  const bool okv = fin[0] != 0.0;
  // The residual's sums of a row of WAVE entries each, added up in the rows' order
  for (int base = wave * WAVE; base < n2; base += blockDim.x) {
    const int i = base + lane;
    double rr = 0.0, ff = 0.0;
    if (i < n2) {
      double s = 0.0, fi = 0.0;
      if (okv) {
        int k = 0;
        for (; k + 4 <= r; k += 4) {
          double vv[4], fv[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            vv[q] = x != nullptr ? V[(size_t)(k + q) * n2 + i] : 0.0;
            fv[q] = Ft[(size_t)(k + q) * n2 + i];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            s += c[k + q] * vv[q];
            fi += c[k + q] * fv[q];
          }
        }
        for (; k < r; ++k) {
          s += c[k] * (x != nullptr ? V[(size_t)k * n2 + i] : 0.0);
          fi += c[k] * Ft[(size_t)k * n2 + i];
        }
      }
      if (x != nullptr) x[i] = s;
      const double fti = ftilde[i], e = fi - fti;
      rr = e * e;
      ff = fti * fti;
    }
    rr = wave_sum_dpp(rr);
    ff = wave_sum_dpp(ff);
    if (lane == 0) {
      sr[base / WAVE] = rr;
      sr[SOLVE_ROWS + base / WAVE] = ff;
    }
  }
  __syncthreads();
  double rr = 0.0, ff = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < (n2 + WAVE - 1) / WAVE; ++q) {
      rr += sr[q];
      ff += sr[SOLVE_ROWS + q];
    }
  return {ff > 0.0 ? sqrt(rr / ff) : 0.0, fin[1], fin[2], okv};
}

// The solve on the accepted directions. On a non-positive pivot x = 0 and status = -5. With
// stop_tol > 0 a residual <= stop_tol ends the expansion (used by the adaptive-rank call after
// each direction). One block.
__device__ __forceinline__ void solve_dev(const double* __restrict__ V, const double* Ft,
                                          const double* __restrict__ ftilde, int n2, KrylovState* st,
                                          double* __restrict__ x, double stop_tol, SolveReport* report = nullptr,
                                          unsigned long long seq = 0) {
  __shared__ double lds[solve_lds(MAX_RANK)];
  const Solution sol = least_squares(V, Ft, ftilde, n2, st->rank, x, lds);
  if (threadIdx.x == 0) {
    if (!sol.ok) st->status = -5;
    st->min_pivot = sol.min_pivot;
    st->max_pivot = sol.max_pivot;
    st->ls_residual = sol.residual;
    int stop = st->stop;
    if (stop_tol > 0.0 && sol.ok && sol.residual <= stop_tol) st->stop = stop = 1;
    if (report != nullptr) {
      __hip_atomic_store(&report->word, 2 * seq + (stop != 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      report->st = *st;
    }
  }
}

// An adaptive update's test between two directions as one block of a launch of the second of them
// (rank > 0; tol > 0): whether the residual of the first `rank` directions is <= tol. The word goes
// into st->done, which nothing in that launch reads; the next orth_potentials or solve ends
// the expansion at that rank (settle). As a launch of its own, 9 us a direction at 16 and
// 10 us at 128 atoms, it stood in the chain between two directions.
struct ResidualTest {
  const double *Ft, *ftilde;
  KrylovState* st;
  double tol;
  int n2, rank;
};
constexpr int RESIDUAL_TEST_MAX_RANK = 16;
__device__ __forceinline__ void residual_test(const ResidualTest& t, double* lds) {
  if (t.st->rank < t.rank || t.st->done != 0) return;  // the expansion had ended before
  const Solution sol = least_squares(nullptr, t.Ft, t.ftilde, t.n2, t.rank, nullptr, lds);
  if (threadIdx.x == 0 && sol.ok && sol.residual <= t.tol) t.st->done = t.rank;
}
// The end of the expansion that a residual_test found, whatever the directions after it did. One thread.
__device__ __forceinline__ void settle(KrylovState* st, int done) {
  st->stop = 1;
  st->rank = done;
  st->status = 0;
}

// Host-side copies of the argument lists of precondition and krylov_solve (SolveArgs; declaration
// order), read from and written back to a kernel node of a captured graph so that a replay
// can take other input and output pointers.
template <class T>
inline T kernel_arg(void** kp, int i) {
  T v;
  __builtin_memcpy(&v, kp[i], sizeof v);
  return v;
}

struct PreconditionArgs {
  static constexpr int COUNT = 7;
  const double *K0, *x, *sub;
  double* y;
  int n2;
  const int* stop;
  KrylovState* reset;
  static PreconditionArgs from(void** kp) {
    return {kernel_arg<const double*>(kp, 0), kernel_arg<const double*>(kp, 1), kernel_arg<const double*>(kp, 2),
            kernel_arg<double*>(kp, 3),       kernel_arg<int>(kp, 4),           kernel_arg<const int*>(kp, 5),
            kernel_arg<KrylovState*>(kp, 6)};
  }
  void pointers(void** out) {
    out[0] = &K0; out[1] = &x; out[2] = &sub; out[3] = &y; out[4] = &n2; out[5] = &stop; out[6] = &reset;
  }
};

// (q, m) Mulliken vector of per-spin atom populations: out = (p_up + p_dn - ref, p_up - p_dn),
// ref = neutral-atom populations (may be null).
__global__ void mix_spins(const double* __restrict__ p, const double* __restrict__ ref, int natoms,
                          double* __restrict__ out) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= natoms) return;
  const double u = p[a], d = p[natoms + a];
  out[a] = u + d - (ref ? ref[a] : 0.0);
  out[natoms + a] = u - d;
}

// Extended-Lagrangian update of the electronic coordinates (Sec. II.F):
//   n(t+dt) = 2 n(t) - n(t-dt) - kappa K f + alpha sum_k c_k n(t - k dt),
// hist[k] = n(t - k dt) for k = 0..kmax (row-major (kmax+1) x n2), Kf the
// kernel applied to the residual f = q[n] - n, c on the device.
__global__ void xlbomd_update(const double* __restrict__ hist, int kmax, int n2, const double* __restrict__ Kf,
                              double kappa, double alpha, const double* __restrict__ c,
                              double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n2) return;
  const double n0 = hist[i];
  const double n1 = kmax >= 1 ? hist[(size_t)n2 + i] : n0;
  double diss = 0.0;
  for (int k = 0; k <= kmax; ++k) diss += c[k] * hist[(size_t)k * n2 + i];
  out[i] = 2.0 * n0 - n1 - kappa * Kf[i] + alpha * diss;
}

}  // namespace kk
