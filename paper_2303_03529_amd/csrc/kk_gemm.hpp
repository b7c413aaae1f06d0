// FP64 MFMA tile GEMM for gfx950 with three fused epilogues.
//
// Every dense contraction of the response runs through one kernel shape:
//   acc[m][n] = sum_k A[k][m] * B[k][n]
// with both operands stored k-major (row k contiguous along m or n), padded to
// a multiple of 128 so no access needs a bounds check. In that layout the
// forward eigenbasis transform X = C^T U~ G (+ its transpose) and the
// back-transform P = C Y (with C^T stored) read both panels along rows, which
// is the coalesced direction.
//
// Tile: BM x BN per workgroup of WAVES_M x WAVES_N waves; each wave owns a
// (BM/WAVES_M) x (BN/WAVES_N) block of v_mfma_f64_16x16x4 accumulators. K
// advances BK per stage through double-buffered LDS with the next stage's
// global loads in flight while the current stage is multiplied.
//
// Epilogues
//   EPI_STORE   out[m][n] = acc                                (setup products)
//   EPI_FERMI   Sec. II.C first-order Fermi response in the eigenbasis:
//               X = 1/2 acc (acc accumulates C^T U~ G + G^T U~ C over a K of
//               2 Nb), Y_mn = F_mn X_mn for m < n written to (m,n) and (n,m),
//               Y_mm = -w_m X_mm and X_mm saved for the chemical-potential
//               shift. Tiles entirely below the diagonal are not launched;
//               elements below it are skipped.
//   EPI_MULLIKEN  Sec. III.A Mulliken rows: part[p][m] = sum over the wave's
//               columns n of acc[m][n] * G[m][n]; the caller sums the parts.
//   EPI_ACCUM   out[m][n] += acc                                (adjoint sums)
//   EPI_XSTORE  out[m][n] = acc with the row scale applied like EPI_FERMI: the
//               product A = C^T U~ G over full tiles (one K half), which
//               fermi_symmetrize_f64 turns into Y in place
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace kk {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

// Cross-lane moves of doubles that stay in the VALU: DPP within rows of 16 lanes, permlane swaps
// between rows. The general shuffle goes through the LDS crossbar, two trips of about a hundred
// cycles for a double, and competes with a kernel's LDS reads; the reductions that end almost every
// kernel here are chains of them.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// v of lane ^ B in x or y: x holds the lower lanes' (rows', halves') values in both places, y the
// upper ones'.
template <int B>
__device__ __forceinline__ void swap_u32(unsigned v, unsigned& x, unsigned& y) {
  static_assert(B == 16 || B == 32, "rows or halves");
  if constexpr (B == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    x = r[0];
    y = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    x = r[0];
    y = r[1];
  }
}
template <int B>
__device__ __forceinline__ void swap_f64(double v, double& x, double& y) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  unsigned xl, yl, xh, yh;
  swap_u32<B>((unsigned)b, xl, yl);
  swap_u32<B>((unsigned)(b >> 32), xh, yh);
  x = __builtin_bit_cast(double, ((unsigned long long)xh << 32) | xl);
  y = __builtin_bit_cast(double, ((unsigned long long)yh << 32) | yl);
}
// v of lane ^ B
template <int B>
__device__ __forceinline__ double lane_xor(double v) {
  if constexpr (B == 1) {
    return dpp_f64<0xB1>(v);  // quad_perm [1, 0, 3, 2]
  } else if constexpr (B == 2) {
    return dpp_f64<0x4E>(v);  // quad_perm [2, 3, 0, 1]
  } else if constexpr (B == 4) {  // row_shl:4 for the lower quad of each eight, row_shr:4 for the upper
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    auto move = [](int w) {
      const int r = __builtin_amdgcn_update_dpp(0, w, 0x104, 0xf, 0x5, false);
      return (unsigned)__builtin_amdgcn_update_dpp(r, w, 0x114, 0xf, 0xa, false);
    };
    return __builtin_bit_cast(double, ((unsigned long long)move((int)(unsigned)(b >> 32)) << 32) | move((int)(unsigned)b));
  } else if constexpr (B == 8) {
    return dpp_f64<0x128>(v);  // row_ror:8
  } else {
    double x, y;
    swap_f64<B>(v, x, y);
    return (threadIdx.x & B) ? x : y;
  }
}
// v + (v of lane ^ B)
template <int B>
__device__ __forceinline__ double add_xor(double v) {
  if constexpr (B < 16) {
    return v + lane_xor<B>(v);
  } else {
    double x, y;
    swap_f64<B>(v, x, y);
    return x + y;
  }
}
// Sum over the row of 16 lanes by exchanges with lane ^ 1, 2, 4, 8 in turn (after the first two steps
// a quad holds one value, so a mirrored half row is the exchange with lane ^ 4).
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x128>(v);  // row_ror:8
  return v;
}

constexpr int PAD = 128;    // every padded dimension is a multiple of this
constexpr int MAX_GEMM_BATCH = 16;

enum { EPI_STORE = 0, EPI_FERMI = 1, EPI_MULLIKEN = 2, EPI_ACCUM = 4, EPI_XSTORE = 5 };

struct GemmItem {
  const double* a0;   // first K half: A operand, [K][n] row-major
  const double* b0;   // first K half: B operand
  const double* a1;   // second K half (EPI_FERMI) or unused
  const double* b1;
  const double* scale;  // per-k scale of A rows (EPI_FERMI: u~ per orbital), length n
  double* out;          // EPI_STORE: product; EPI_FERMI: Y
  const double* g;      // EPI_MULLIKEN: G, [n][n]
  const double* eps;    // EPI_FERMI: eigenvalues (padded with 0)
  const double* f;      // occupations f
  const double* fc;     // 1 - f
  const double* w;      // beta f (1 - f)
  double* xdiag;        // EPI_FERMI: diag X
  double* part;         // EPI_MULLIKEN: [parts][n]
  double* xout;         // symmetrizing pass of the reverse pass: X (a0 then holds A, out receives Y)
};

// Where the divided differences F of a prepared spectrum are negligible (built by window_tables
// from the levels alone; kk_kernels.hpp has the rule). Two levels that are both filled, or
// both empty, up to a few ten kT from mu do not respond, so blocks of Y = F o X between such
// levels are zero: the forward transform leaves their tiles out, the symmetrizing pass writes
// zeros there, and the back-transform contracts only over the rows that remain. In blocks of
// WIN x WIN levels, per spin. With ascending levels the active blocks are all but two squares
// on the diagonal; any other order is as correct, with less left out. On spectra 60 eV wide at
// kT = 0.25 eV, 1024 atoms, 84 % (forward, by tiles) and 83 % (back, by rows) of the products remain, in
// FP16 x 3, whose cut is higher, 77 and 74 %; from kT = 1 eV on all of them (FP64 then 1 % slower at 265-350 atoms than
// without the tables). m = 12 FP64 1024 atoms 1092 -> 920 ms, eight responses at 250 atoms 11.8 -> 10.2 ms;
// FP16 x 3 at 432 atoms m = 8 12.9 -> 11.7 ms (3.2 rounds of 256 x 128 tiles for 4).
constexpr int WIN = 64;
struct Window {
  const unsigned char* act[2];  // nblk x nblk: 1 where Y may be non-zero (symmetric; the diagonal always)
  const int2* range[2];         // per column block: rows [x, y) hold its active blocks
  const int2* tiles[2];         // forward tile list: the active tiles in launch order, then the others
  const int* count;             // active tiles of each spin
  int nblk;                     // n / WIN
};

// Hardware hands workgroup ids to the 8 XCDs round-robin; give each XCD a
// contiguous range of logical tiles so neighbouring tiles share its L2.
__device__ __forceinline__ int xcd_remap(int bid, int total) {
  const int x = bid & 7, slot = bid >> 3;
  const int q = total >> 3, r = total & 7;
  return (x < r) ? x * (q + 1) + slot : r * (q + 1) + (x - r) * q + slot;
}

// Forward launch: its active tiles, and the item and tile of the `logical` one of them. Items are
// (direction, spin).
__device__ __forceinline__ int window_total(const Window& w, int nitems) {
  return (w.count[0] + w.count[1]) * (nitems / 2);
}
__device__ __forceinline__ void window_tile(const Window& w, int logical, int& z, int2& tile) {
  const int n0 = w.count[0], per = n0 + w.count[1];
  const int set = logical / per, r = logical - set * per, s = r >= n0;
  z = 2 * set + s;
  tile = w.tiles[s][s ? r - n0 : r];
}
// The rest of the forward launch's blocks, one per inactive tile.
__device__ __forceinline__ void window_rest(const Window& w, int ntiles, int nitems, int& z, int2& tile) {
  const int n0 = w.count[0], n1 = w.count[1];
  const int idx = (int)blockIdx.x - (n0 + n1) * (nitems / 2), r0 = ntiles - n0, per = r0 + ntiles - n1;
  const int set = idx / per, r = idx - set * per, s = r >= r0;
  z = 2 * set + s;
  tile = w.tiles[s][s ? n1 + r - r0 : n0 + r];
}
// Back-transform: the rows [lo, hi) of a contraction over [0, k_len) that the columns of `blocks`
// blocks from block c need, lo rounded down to a multiple of `align`; the first `least` rows where
// none or fewer remain.
__host__ __device__ __forceinline__ int2 window_rows(const int2* range, int c, int blocks, int k_len, int align,
                                                     int least) {
  int lo = 1 << 30, hi = 0;
  for (int q = 0; q < blocks; ++q) {
    const int2 r = range[c + q];
    if (r.y > r.x) {
      lo = r.x < lo ? r.x : lo;
      hi = r.y > hi ? r.y : hi;
    }
  }
  lo = lo / align * align;
  hi = k_len < hi ? k_len : hi;
  return hi > lo && hi - lo >= least ? make_int2(lo, hi) : make_int2(0, least);
}
__device__ __forceinline__ bool window_active(const unsigned char* act, int nblk, int I, int J) {
  return act == nullptr || act[(size_t)I * nblk + J] != 0;
}

struct GemmArgs {
  int n;          // padded dimension; M = N = n, row stride n
  int k_half;     // rows per K half (= n)
  int two_halves; // 1: K runs over both halves (a0,b0) then (a1,b1)
  int ntiles;     // tiles per item
  int nitems;     // batch items
  int cus;        // CUs of the chip (windowed launches: Tail)
  const int2* tiles;  // tile coordinates (tm, tn), in launch order
  const int* stop;    // if non-null and *stop != 0 the launch does nothing
  double beta;        // 1 / kT (EPI_FERMI)
  Window win;         // all null: every tile, every row
  GemmItem item[MAX_GEMM_BATCH];
};

// (f_lo - f_hi)/(e_lo - e_hi) for the pair, lo = lower eigenvalue, written as
// -beta f_lo (1 - f_hi) phi(beta (e_lo - e_hi)), phi(z) = expm1(z)/z, phi(0) = 1.
__device__ __forceinline__ double fermi_divided_difference(double em, double fm, double fcm,
                                                           double en, double fn, double fcn,
                                                           double beta) {
  double flo, fchi, z;
  if (em <= en) {
    flo = fm; fchi = fcn; z = beta * (em - en);
  } else {
    flo = fn; fchi = fcm; z = beta * (en - em);
  }
  const double phi = (z == 0.0) ? 1.0 : expm1(z) / z;
  return -beta * flo * fchi * phi;
}

// ONE_ROW: the Mulliken sums of a tile's waves along n are added up into one partial row.
template <int BM_, int BN_, int BK_, int WAVES_M_, int WAVES_N_, int MINB_, bool ONE_ROW_ = false>
struct TileCfg {
  using Tile = TileCfg;  // the configuration itself (OneLds)
  static constexpr bool ONE_ROW = ONE_ROW_;
  static constexpr int PART_ROWS = ONE_ROW ? 1 : WAVES_N_;  // Mulliken partial rows of a tile
  static constexpr int BM = BM_, BN = BN_, BK = BK_;
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
  static constexpr int THREADS = 64 * WAVES_M * WAVES_N;
  static constexpr int WTM = BM / WAVES_M / 16;  // MFMA tiles per wave along m
  static constexpr int WTN = BN / WAVES_N / 16;  // along n
  static constexpr int MIN_BLOCKS = MINB_;
  // MIN_BLOCKS co-resident workgroups need this many waves per SIMD, which caps
  // the registers per lane the compiler may use (512 / WAVES_PER_EU).
  static constexpr int WAVES_PER_EU = (MIN_BLOCKS * THREADS / 64 + 3) / 4;
  // global -> LDS staging: each thread moves double2 pieces
  static constexpr int A_PIECES = BK * BM / 2 / THREADS;
  static constexpr int B_PIECES = BK * BN / 2 / THREADS;
  static_assert(BM % (16 * WAVES_M) == 0 && BN % (16 * WAVES_N) == 0, "wave tiling");
  static_assert(BK % 4 == 0, "BK");
  static_assert(A_PIECES >= 1 && B_PIECES >= 1, "staging");
  static_assert((BK * BM / 2) % THREADS == 0 && (BK * BN / 2) % THREADS == 0, "staging split");
  static_assert(PAD % BM == 0 && PAD % BN == 0, "tile must divide the padding");
  static constexpr int LDS_BYTES = 2 * BK * (BM + BN) * 8;
};

// Where a tile's contraction rows come from: rows(k0) sets A and B to row k0 of the contraction
// (k0 a multiple of the K stage), scale(k0) gives the row scales from there.

// The k_half rows from k_lo of the item's first operands, then (two_halves) of its second.
struct HalfRows {
  const GemmItem& it;
  int n, k_lo, k_half;
  bool two_halves;
  __device__ __forceinline__ int stages(int bk) const { return (two_halves ? 2 * k_half : k_half) / bk; }
  __device__ __forceinline__ void rows(int k0, const double*& A, const double*& B) const {
    A = it.a0;
    B = it.b0;
    if (two_halves && k0 >= k_half) {
      A = it.a1; B = it.b1; k0 -= k_half;
    }
    A += (size_t)(k_lo + k0) * n;
    B += (size_t)(k_lo + k0) * n;
  }
  __device__ __forceinline__ const double* scale(int k0) const {
    if (two_halves && k0 >= k_half) k0 -= k_half;
    return it.scale + k_lo + k0;
  }
};

// The reverse pass's sum over directions k of Y_b Xa + Y_a Xb as one contraction: 2 directions
// operand pairs of `per` K stages (bk rows) each from row k_lo, of which this tile takes the stages
// from first on. X and Y hold the items (a up, a dn, b up, b dn) of every direction, np2 apart.
struct PairRows {
  const double *X, *Y;  // of the tile's spin, direction 0
  size_t np2;
  int n, k_lo, per, bk, first, count;
  unsigned long long magic;  // ceil(2^32 / per): stage / per for stages below 2^32 / per
  __device__ __forceinline__ int stages(int) const { return count; }
  __device__ __forceinline__ void rows(int k0, const double*& A, const double*& B) const {
    const unsigned t = first + k0 / bk;
    const unsigned q = (unsigned)((t * magic) >> 32), r = t - q * per;
    const size_t dir = (size_t)(q >> 1) * 4 * np2, row = (size_t)(k_lo + r * bk) * n;
    A = Y + dir + ((q & 1) ? 0 : 2) * np2 + row;
    B = X + dir + ((q & 1) ? 2 : 0) * np2 + row;
  }
  __device__ __forceinline__ const double* scale(int) const { return nullptr; }
};

// LDS of f64_tile: two stages of each operand, those of LdsCfg, where a kernel runs tiles of two
// configurations. Two objects (one, whose accesses the compiler orders, is 1.2 % slower on 128 x 128
// tiles at 150 atoms), or one (OneLds) for the 64 x 64 tiles of single systems (171 atoms, a
// transform 303 -> 297 us). Functions rather than references to the arrays: with those the
// batches' tiles took a register more per lane and 1.2 % longer.
template <class Cfg>
struct OneLds : Cfg {
  using Tile = Cfg;
};
template <class Cfg, class LdsCfg>
__device__ __forceinline__ double (&tile_a())[2][Cfg::BK][Cfg::BM] {
  if constexpr (std::is_same<Cfg, LdsCfg>::value) {
    __shared__ double As[2][Cfg::BK][Cfg::BM];
    return As;
  } else if constexpr (std::is_same<OneLds<Cfg>, LdsCfg>::value) {
    __shared__ double As[2 * Cfg::BK * (Cfg::BM + Cfg::BN)];
    return *reinterpret_cast<double (*)[2][Cfg::BK][Cfg::BM]>(&As[0]);
  } else {
    static_assert(Cfg::BK * Cfg::BM <= LdsCfg::BK * LdsCfg::BM, "LDS");
    return *reinterpret_cast<double (*)[2][Cfg::BK][Cfg::BM]>(&tile_a<typename LdsCfg::Tile, LdsCfg>());
  }
}
template <class Cfg, class LdsCfg>
__device__ __forceinline__ double (&tile_b())[2][Cfg::BK][Cfg::BN] {
  if constexpr (std::is_same<Cfg, LdsCfg>::value) {
    __shared__ double Bs[2][Cfg::BK][Cfg::BN];
    return Bs;
  } else if constexpr (std::is_same<OneLds<Cfg>, LdsCfg>::value) {
    return *reinterpret_cast<double (*)[2][Cfg::BK][Cfg::BN]>(&tile_a<Cfg, LdsCfg>()[0][0][0] + 2 * Cfg::BK * Cfg::BM);
  } else {
    static_assert(Cfg::BK * Cfg::BN <= LdsCfg::BK * LdsCfg::BN, "LDS");
    return *reinterpret_cast<double (*)[2][Cfg::BK][Cfg::BN]>(&tile_b<typename LdsCfg::Tile, LdsCfg>());
  }
}

// One output tile: both operands n x n (row stride n), contracted over src's rows. Ends with a
// barrier, so a workgroup may run several tiles in sequence.
template <int EPI, class Cfg, class LdsCfg = Cfg, class Rows>
__device__ __forceinline__ void f64_tile(const GemmItem& it, const Rows& src, const int n, const int2 tile,
                                         const double beta_arg) {
  constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK;
  constexpr int WTM = Cfg::WTM, WTN = Cfg::WTN;
  constexpr int AP = Cfg::A_PIECES, BP = Cfg::B_PIECES;
  constexpr int APR = BM / 2;  // double2 pieces per A row
  constexpr int BPR = BN / 2;
  const int m0 = tile.x * BM, n0 = tile.y * BN;

  const int tid = threadIdx.x;
  const int nk = src.stages(BK);
  const int wave = tid >> 6, lane = tid & 63;
  const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;
  const int lr = lane >> 4, lc = lane & 15;

  d4 acc[WTM][WTN];
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int j = 0; j < WTN; ++j) acc[i][j] = (d4){0.0, 0.0, 0.0, 0.0};

  // Global -> register -> LDS staging, one stage ahead: the loads of stage kt + 1 are
  // issued at the start of step kt and written to LDS at its end, and nothing in
  // between waits for them; the loads are unconditional (the last step reloads the last
  // stage, written to the idle buffer and never read), because a conditional load makes
  // the compiler wait for every load in flight before the write.
  // The forward transform's row scales go through a 3-slot LDS ring: the BK scales of
  // stage s are loaded by the first BK threads at the start of step s - 2, put in slot
  // s % 3 at its end, and multiplied in when stage s is written to LDS (end of step s - 1).
  constexpr bool SCALED = EPI == EPI_FERMI || EPI == EPI_XSTORE;
  __shared__ double Ss[SCALED ? 3 : 1][BK];
  d2 ra[AP], rb[BP];
  double sreg = 0.0;
  // Byte offsets of this thread's staging pieces within a K stage (loop invariant; BK
  // rows of n <= 65536 doubles span at most 8 MB, so 32 bits hold them); the stage's
  // uniform part goes into the base pointers.
  unsigned aoff[AP], boff[BP];
#pragma unroll
  for (int p = 0; p < AP; ++p) {
    const int idx = tid + p * Cfg::THREADS;
    const int row = idx / APR, col = (idx % APR) * 2;
    aoff[p] = (unsigned)(row * n + col) * 8u;
  }
#pragma unroll
  for (int p = 0; p < BP; ++p) {
    const int idx = tid + p * Cfg::THREADS;
    const int row = idx / BPR, col = (idx % BPR) * 2;
    boff[p] = (unsigned)(row * n + col) * 8u;
  }
  auto gload = [&](const int kt) __attribute__((always_inline)) {
    const double *A, *B;
    src.rows(kt * BK, A, B);
    const char* Ab = reinterpret_cast<const char*>(A + m0);
    const char* Bb = reinterpret_cast<const char*>(B + n0);
#pragma unroll
    for (int p = 0; p < AP; ++p) ra[p] = *reinterpret_cast<const d2*>(Ab + aoff[p]);
#pragma unroll
    for (int p = 0; p < BP; ++p) rb[p] = *reinterpret_cast<const d2*>(Bb + boff[p]);
  };
  auto sload = [&](const int kt) __attribute__((always_inline)) {
    if constexpr (SCALED) {
      if (tid < BK) sreg = src.scale(kt * BK)[tid];
    }
  };
  auto sstore = [&](const int kt) __attribute__((always_inline)) {
    if constexpr (SCALED) {
      if (tid < BK) Ss[kt % 3][tid] = sreg;
    }
  };
  auto lstore = [&](const int buf, const int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < AP; ++p) {
      const int idx = tid + p * Cfg::THREADS;
      d2 v = ra[p];
      if constexpr (SCALED) v *= Ss[kt % 3][idx / APR];
      *reinterpret_cast<d2*>(&tile_a<Cfg, LdsCfg>()[buf][idx / APR][(idx % APR) * 2]) = v;
    }
#pragma unroll
    for (int p = 0; p < BP; ++p) {
      const int idx = tid + p * Cfg::THREADS;
      *reinterpret_cast<d2*>(&tile_b<Cfg, LdsCfg>()[buf][idx / BPR][(idx % BPR) * 2]) = rb[p];
    }
  };

  gload(0);
  sload(0);
  sstore(0);
  sload(min(1, nk - 1));
  sstore(1);
  __syncthreads();
  lstore(0, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    gload(min(kt + 1, nk - 1));
    sload(min(kt + 2, nk - 1));
#pragma unroll
    for (int kk = 0; kk < BK / 4; ++kk) {
      double a[WTM], b[WTN];
#pragma unroll
      for (int i = 0; i < WTM; ++i) a[i] = tile_a<Cfg, LdsCfg>()[buf][kk * 4 + lr][wm * (BM / Cfg::WAVES_M) + i * 16 + lc];
#pragma unroll
      for (int j = 0; j < WTN; ++j) b[j] = tile_b<Cfg, LdsCfg>()[buf][kk * 4 + lr][wn * (BN / Cfg::WAVES_N) + j * 16 + lc];
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    lstore(buf ^ 1, kt + 1);
    sstore(kt + 2);
    __syncthreads();
  }

  // Accumulator element (i, j, r) of this lane sits at
  //   m = m0 + wm*(BM/WAVES_M) + i*16 + lr + 4r,  n = n0 + wn*(BN/WAVES_N) + j*16 + lc.
  const int mw = m0 + wm * (BM / Cfg::WAVES_M) + lr;
  const int nw = n0 + wn * (BN / Cfg::WAVES_N) + lc;
  if constexpr (EPI == EPI_STORE || EPI == EPI_ACCUM || EPI == EPI_XSTORE) {
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double* o = it.out + (size_t)(mw + i * 16 + 4 * r) * n + nw + j * 16;
          if constexpr (EPI == EPI_ACCUM) *o += acc[i][j][r];
          else *o = acc[i][j][r];
        }
  } else if constexpr (EPI == EPI_FERMI) {
    const double beta = beta_arg;
    // Column spectra are re-read per row (cached) rather than held, which keeps the
    // epilogue inside the main loop's register budget.
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = mw + i * 16 + 4 * r;
        const double em = it.eps[m], fm = it.f[m], fcm = it.fc[m];
#pragma unroll
        for (int j = 0; j < WTN; ++j) {
          const int c = nw + j * 16;
          if (m > c) continue;
          const double en = it.eps[c], fn = it.f[c], fcn = it.fc[c];
          const double x = 0.5 * acc[i][j][r];
          if (m == c) {
            it.xdiag[m] = x;
            it.out[(size_t)m * n + m] = -it.w[m] * x;
          } else {
            const double y = fermi_divided_difference(em, fm, fcm, en, fn, fcn, beta) * x;
            it.out[(size_t)m * n + c] = y;
            it.out[(size_t)c * n + m] = y;
          }
        }
      }
  } else {  // EPI_MULLIKEN
    const int p = Cfg::ONE_ROW ? tile.y : tile.y * Cfg::WAVES_N + wn;
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = mw + i * 16 + 4 * r;
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < WTN; ++j) s += acc[i][j][r] * it.g[(size_t)m * n + nw + j * 16];
        s = row16_sum(s);
        if constexpr (Cfg::ONE_ROW) {
          if (lc == 0) tile_a<Cfg, LdsCfg>()[0][wn][m - m0] = s;  // (the last stage's reads ended with a barrier)
        } else {
          if (lc == 0) it.part[(size_t)p * n + m] = s;
        }
      }
    if constexpr (Cfg::ONE_ROW) {
      __syncthreads();
      if (tid < BM) {
        double s = tile_a<Cfg, LdsCfg>()[0][0][tid];
#pragma unroll
        for (int w = 1; w < Cfg::WAVES_N; ++w) s += tile_a<Cfg, LdsCfg>()[0][w][tid];
        it.part[(size_t)p * n + m0 + tid] = s;
      }
      __syncthreads();
    }
  }
}

// The last, partly empty round of a windowed launch. Its tiles past the last multiple of the chip's
// CUs are cut into PIECES tiles of a quarter or half the size, where that ends the round sooner:
// the active tiles are known on the device only, so the choice is made there. tail_begin: the
// first tile that is cut (total: none), where the pieces of the rest take less than a whole tile's
// time. Most of the CUs were left waiting for a few whole tiles. m = 4: FP64 (quarters)
// 250 atoms, 572 and 648 tiles on 256 CUs, 7.29 -> 5.68 ms, 265 atoms 7.63 -> 7.12, 350 atoms 15.7 -> 14.6,
// 300 atoms (no cut: 200 tiles past the last multiple of 256) level; FP16 x 3 (halves) 265 atoms
// 1.97 -> 1.87 ms, 171 atoms 0.795 -> 0.777, 432 atoms 5.60 -> 5.44; BF16 265 atoms 3.23 -> 3.02.
// The 64 x 64 FP64 tiles, three workgroups per CU, gain while their quarters fit beside the whole
// tiles: 160 atoms 1.90 -> 1.79 ms, 171 atoms 2.46 -> 2.30, 178 atoms 2.55 -> 2.45; after more rounds a
// quarter takes a slot that a whole tile would have filled (182 atoms, 72 tiles after five
// rounds, back-transform 315 us whole, 347 us cut).
template <class Cfg>
struct Tail {
  // REST: most tiles that are cut, in sixteenths of the CUs; REST_LONG: after more than four rounds
  static constexpr int PIECES = 1, REST = 0, REST_LONG = 0;
};
template <int EPI, class Cfg>
constexpr bool f64_tail() {
  return Tail<Cfg>::PIECES > 1 && (EPI == EPI_XSTORE || EPI == EPI_MULLIKEN);
}
template <class Cfg>
__host__ __device__ inline int tail_begin(int total, int cus) {
  const int rest = total % cus, most = total - rest <= 4 * cus ? Tail<Cfg>::REST : Tail<Cfg>::REST_LONG;
  return 16 * rest <= most * cus ? total - rest : total;
}

// Where workgroup b of a windowed launch works: `logical` tile of the launch's `total`, and with piece >= 0
// which piece of it. false: nowhere.
template <class Cfg>
__device__ __forceinline__ bool tail_place(int b, int total, int cus, int& logical, int& piece) {
  constexpr int S = Tail<Cfg>::PIECES;
  const int whole = S > 1 ? tail_begin<Cfg>(total, cus) : total;
  piece = -1;
  if (b < whole) {
    logical = xcd_remap(b, whole);
    return true;
  }
  const int pieces = (total - whole) * S, q = b - whole;  // whole is a multiple of 8 here, so q keeps b's XCD
  if (q >= pieces) return false;
  const int at = xcd_remap(q, pieces);
  logical = whole + at / S;
  piece = at % S;
  return true;
}

// WINDOWED: the launch goes by args.win. (A choice at run time cost the smallest systems, whose
// launches are all latency, 0.2 us a kernel.)
template <int EPI, class Cfg, bool WINDOWED = false>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::MIN_BLOCKS) void gemm_f64(const GemmArgs args) {
  static_assert(Cfg::BN % WIN == 0 && Cfg::BM % WIN == 0, "tiles are whole window blocks");
  if (args.stop != nullptr && *args.stop != 0) return;
  constexpr bool ACTIVE = WINDOWED && (EPI == EPI_FERMI || EPI == EPI_XSTORE);  // only the active tiles
  constexpr bool TAIL = WINDOWED && f64_tail<EPI, Cfg>();
  const int total = ACTIVE ? window_total(args.win, args.nitems) : args.ntiles * args.nitems;
  int z, logical, piece = -1;
  if constexpr (TAIL) {
    if (!tail_place<Cfg>(blockIdx.x, total, args.cus, logical, piece)) return;
  } else {
    if (ACTIVE && (int)blockIdx.x >= total) {
      if constexpr (EPI == EPI_FERMI) {  // no pass follows that would write the inactive tiles' zeros
        int2 tile;
        window_rest(args.win, args.ntiles, args.nitems, z, tile);
        static_assert(Cfg::BM == Cfg::BN, "a tile and its mirror");
        double* const out = args.item[z].out;
        for (int e = threadIdx.x; e < Cfg::BM * Cfg::BN; e += Cfg::THREADS) {
          const size_t r = e / Cfg::BN, c = e % Cfg::BN;
          out[(tile.x * Cfg::BM + r) * args.n + tile.y * Cfg::BN + c] = 0.0;
          out[(tile.y * Cfg::BM + r) * args.n + tile.x * Cfg::BN + c] = 0.0;
        }
      }
      return;
    }
    logical = xcd_remap(blockIdx.x, total);
  }
  int2 tile, rows = make_int2(0, args.k_half);
  if constexpr (ACTIVE) {
    window_tile(args.win, logical, z, tile);
  } else {
    z = logical / args.ntiles;
    tile = args.tiles[logical - z * args.ntiles];
  }
  using Lds = typename std::conditional<(Cfg::MIN_BLOCKS > 2), OneLds<Cfg>, Cfg>::type;
  if constexpr (TAIL) {
    if (piece >= 0) {
      using Sub = typename Tail<Cfg>::Cfg;
      constexpr int SM = Cfg::BM / Sub::BM, SN = Cfg::BN / Sub::BN;
      static_assert(SM * SN == Tail<Cfg>::PIECES && Sub::THREADS == Cfg::THREADS &&
                    SN * Sub::PART_ROWS == Cfg::PART_ROWS, "the pieces of a tile");
      const int2 part = make_int2(tile.x * SM + piece % SM, tile.y * SN + piece / SM);
      if constexpr (EPI == EPI_MULLIKEN)
        rows = window_rows(args.win.range[z & 1], part.y * Sub::BN / WIN, (Sub::BN + WIN - 1) / WIN, args.k_half,
                           Sub::BK, 0);
      const HalfRows src{args.item[z], args.n, rows.x, rows.y - rows.x, args.two_halves != 0};
      f64_tile<EPI, Sub, Lds>(args.item[z], src, args.n, part, args.beta);
      return;
    }
  }
  if constexpr (WINDOWED && EPI == EPI_MULLIKEN)
    rows = window_rows(args.win.range[z & 1], tile.y * (Cfg::BN / WIN), Cfg::BN / WIN, args.k_half, Cfg::BK, 0);
  const HalfRows src{args.item[z], args.n, rows.x, rows.y - rows.x, args.two_halves != 0};
  f64_tile<EPI, Cfg, Lds>(args.item[z], src, args.n, tile, args.beta);
}

// The commutator sums of the reverse pass: out + (2 c + s) np2 (+)= chunk c of spin s's
// contraction (PairRows), over all tiles. With `range` (Window) the rows where no Y of the tile's
// row block lies are left out. One launch for all directions in place of one each: 2 x 81 tiles of
// 128 atoms fill 256 CUs only when the contraction is cut, and the sums stay in registers between
// directions (128 atoms, 8 directions: 8 x 314 us -> 1514 us, 65 TFLOP/s).
struct PairArgs {
  const double *X, *Y;  // [directions][4][n][n]
  double* out;          // [chunks][2][n][n]
  const int2* tiles;
  const int2* range[2];
  int n, k, directions, ntiles, chunks;
};
template <class Cfg, bool ACCUMULATE>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::MIN_BLOCKS) void gemm_pairs(const PairArgs a) {
  const int logical = xcd_remap(blockIdx.x, a.ntiles * 2 * a.chunks);
  const int z = logical / a.ntiles, s = z & 1, c = z >> 1;
  const int2 tile = a.tiles[logical - z * a.ntiles];
  int2 rows = make_int2(0, a.k);
  if (a.range[0] != nullptr)
    rows = window_rows(a.range[s], tile.x * (Cfg::BM / WIN), Cfg::BM / WIN, a.k, Cfg::BK, Cfg::BK);
  const size_t np2 = (size_t)a.n * a.n;
  const int per = (rows.y - rows.x) / Cfg::BK;
  const long total = (long)2 * a.directions * per;
  const int first = (int)(total * c / a.chunks), last = (int)(total * (c + 1) / a.chunks);
  const PairRows src{a.X + s * np2, a.Y + s * np2, np2, a.n, rows.x, per, Cfg::BK, first, last - first,
                     ((1ull << 32) + per - 1) / per};
  GemmItem it{};
  it.out = a.out + (2 * (size_t)c + s) * np2;
  f64_tile<ACCUMULATE ? EPI_ACCUM : EPI_STORE, Cfg>(it, src, a.n, tile, 0.0);
}

// Second pass of the FP64 forward transform when it runs as a full-tile product
// (EPI_XSTORE): out holds A = C^T U~ G; for each B x B block pair (I <= J),
// X = (A + A^T) / 2, Y = F o X off the diagonal and Y_ii = -w_i X_ii (X_ii to
// xdiag), written in place over A: block (I, J) element by element by the
// thread that read it, block (J, I) through LDS after the whole of it was read.
// pair indexes the upper triangle row-major; T threads. Small handles: 32 x 32 blocks of
// 256 threads; large handles and FP64 batches: 64 x 64 blocks of 512 threads (512-byte rows).
constexpr int SYM64_B = 32;
constexpr int SYM64_B_LARGE = 64, SYM64_T_LARGE = 512;
static_assert(PAD % SYM64_B_LARGE == 0, "the symmetrizing blocks must divide the padding");
template <int B = SYM64_B, int T = 256>
__device__ __forceinline__ void fermi_symmetrize_f64_dev(const GemmItem& it, const int n, const double beta,
                                                         const int pair, const unsigned char* act, const int nblk64) {
  static_assert(T % B == 0 && B % (T / B) == 0, "thread mapping");
  const int nblk = n / B;
  int I = 0, rem = pair;
  while (rem >= nblk - I) {
    rem -= nblk - I;
    ++I;
  }
  const int J = I + rem;
  __shared__ double At[B][B + 1];  // block (J, I) of A, then the mirror of Y
  const int tx = threadIdx.x % B, ty = threadIdx.x / B;
  constexpr int RS = T / B;
  double* const Y = it.out;
  if (!window_active(act, nblk64, I * B / WIN, J * B / WIN)) {
    for (int r = ty; r < B; r += RS) {
      Y[(size_t)(I * B + r) * n + J * B + tx] = 0.0;
      Y[(size_t)(J * B + r) * n + I * B + tx] = 0.0;
    }
    return;
  }
  for (int r = ty; r < B; r += RS) At[r][tx] = Y[(size_t)(J * B + r) * n + I * B + tx];
  __syncthreads();
  const int c = J * B + tx;
  const double en = it.eps[c], fn = it.f[c], fcn = it.fc[c];
  double yv[B / RS];
#pragma unroll
  for (int q = 0; q < B / RS; ++q) {
    const int r = ty + q * RS, m = I * B + r;
    double* const o = Y + (size_t)m * n + c;
    const double x = 0.5 * (*o + At[tx][r]);
    double y;
    if (m == c) {
      it.xdiag[m] = x;
      y = -it.w[m] * x;
    } else {
      y = fermi_divided_difference(it.eps[m], it.f[m], it.fc[m], en, fn, fcn, beta) * x;
    }
    *o = y;
    yv[q] = y;
  }
  if (I == J) return;  // a diagonal block is symmetric by construction
  __syncthreads();     // every read of At is done
#pragma unroll
  for (int q = 0; q < B / RS; ++q) At[tx][ty + q * RS] = yv[q];
  __syncthreads();
  for (int r = ty; r < B; r += RS) Y[(size_t)(J * B + r) * n + I * B + tx] = At[r][tx];
}

// Single system: blockIdx.x = block pair, blockIdx.y = item.
template <int B, int T>
__global__ __launch_bounds__(T) void fermi_symmetrize_f64(const GemmArgs args) {
  if (args.stop != nullptr && *args.stop != 0) return;
  fermi_symmetrize_f64_dev<B, T>(args.item[blockIdx.y], args.n, args.beta, blockIdx.x, args.win.act[blockIdx.y & 1],
                                 args.win.nblk);
}

// Configurations. The default (128 x 128 tile, 8 waves of 32 x 64, two
// workgroups and 16 waves per CU) was the fastest of the shapes below for
// both transforms at Nb = 9216 and 3888 on MI355X; the others stay available
// for re-tuning (-DKK_FWD_CFG=..., -DKK_BACK_CFG=...).
using Cfg128x128 = TileCfg<128, 128, 16, 2, 2, 2>;
using Cfg128x64 = TileCfg<128, 64, 16, 2, 2, 2>;
using Cfg64x128 = TileCfg<64, 128, 16, 2, 2, 2>;
using Cfg128x128w8 = TileCfg<128, 128, 16, 4, 2, 2>;
using Cfg128x128k32 = TileCfg<128, 128, 32, 2, 2, 1>;
using Cfg128x128k8 = TileCfg<128, 128, 8, 2, 2, 2>;
using Cfg64x64 = TileCfg<64, 64, 16, 2, 2, 3>;

using Cfg128x128w16 = TileCfg<128, 128, 16, 4, 4, 1>;
using Cfg128x128w8n = TileCfg<128, 128, 16, 2, 4, 2>;

#ifndef KK_FWD_CFG
#define KK_FWD_CFG Cfg128x128w8
#endif
#ifndef KK_BACK_CFG
#define KK_BACK_CFG Cfg128x128w8
#endif
#ifndef KK_STORE_CFG
#define KK_STORE_CFG Cfg128x128w8
#endif
using FwdCfg = KK_FWD_CFG;
using BackCfg = KK_BACK_CFG;
using StoreCfg = KK_STORE_CFG;
template <>
struct Tail<Cfg64x64> {
  static constexpr int PIECES = 4, REST = 9, REST_LONG = 1;
  using Cfg = TileCfg<32, 32, 16, 2, 2, 3, true>;
};
template <>
struct Tail<Cfg128x128w8> {
  static constexpr int PIECES = 4, REST = 12, REST_LONG = 12;
  using Cfg = TileCfg<64, 64, 16, 4, 2, 2, true>;
};

}  // namespace kk
