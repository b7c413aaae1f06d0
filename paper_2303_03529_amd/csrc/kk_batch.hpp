// Batched rank-m Krylov kernel over many independent systems of uneven size.
//
// Every system keeps its own prepared state (a full single-system handle);
// the batch adds device descriptor tables so that each step of the Krylov
// loop is ONE launch for all systems: small kernels take the system from
// blockIdx.y, and the two dense transforms are persistent kernels that take
// tiles (system, spin, tile row, tile column) from queues, dearest first.
// The whole update is captured once into a hipGraph and replayed.
#pragma once

#include <hip/hip_runtime.h>

#include "kk_gemm.hpp"
#include "kk_gemm_mixed.hpp"
#include "kk_kernels.hpp"

namespace kk {

struct SysDesc {
  int natoms, nb, np, nparts;  // nparts: Mulliken partial rows written per spin by the tile class in use
  int part_stride, pad;        // rows reserved per spin in part
  double W, beta;
  const int* offsets;
  const double* gamma;
  double* u;        // 2 x np (spin potentials per orbital)
  double* xdiag;    // 2 x np
  double* part;     // 2 x nparts x np
  const double *w0, *w1, *wsum, *t;
  double *V, *Ft, *ftilde, *q1;
  KrylovState* kst;
  // split-precision path
  double* msc;             // 2 x 8
  const double* mconst;    // 8
  const double *CT0, *CT1;
  _Float16 *uct_h, *uct_l;  // 2 x np^2 each
};

struct BatchItemF64 {
  GemmItem g;
  int n, k;  // padded size; contraction length (rows past the system's nb are zero)
  const int* stop;
  double beta;
  const unsigned char* act;  // the item's spin of its system's Window
  const int2* range;
  int nblk;
};

struct BatchItemMixed {
  MixedItem g;
  int n, k;
  const int* stop;
  double beta;
  const unsigned char* act;  // the item's spin of its system's Window
  const int2* range;
  int nblk;
};

// Also clears the update's tile queue counters.
__global__ void b_reset(SysDesc* d, int* queue, int nqueue) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nqueue; i += gridDim.x * blockDim.x) queue[i] = 0;
  if (threadIdx.x == 0) {
    KrylovState* st = d[blockIdx.x].kst;
    st->rank = 0; st->stop = 0; st->status = 0; st->done = 0;
    st->min_pivot = 0.0; st->max_pivot = 0.0; st->ls_residual = 1.0;
  }
}

// f~ = K0 delta with K0 = -I; delta from the pointer table.
__global__ void b_init(const SysDesc* __restrict__ d, const double* const* __restrict__ delta) {
  const SysDesc& s = d[blockIdx.y];
  const int n2 = 2 * s.natoms;
  const double* x = delta[blockIdx.y];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += gridDim.x * blockDim.x) s.ftilde[i] = -x[i];
}

__global__ void __launch_bounds__(1024) b_orth(SysDesc* d, int k) {
  const SysDesc& s = d[blockIdx.x];
  const int n2 = 2 * s.natoms;
  const double* src = (k == 0) ? s.ftilde : s.Ft + (size_t)(k - 1) * n2;
  orth_dev(src, s.V, n2, s.kst);
}

__global__ void b_potentials(const SysDesc* __restrict__ d, int k) {
  const SysDesc& s = d[blockIdx.y];
  const int n2 = 2 * s.natoms;
  if ((int)(blockIdx.x * blockDim.x / WAVE) >= s.natoms) return;
  potentials_dev(s.gamma, s.natoms, s.W, s.V + (size_t)k * n2, 1, s.offsets, s.np, s.u, &s.kst->stop,
                 blockIdx.x);
}

__global__ void b_center(const SysDesc* __restrict__ d) {
  const SysDesc& s = d[blockIdx.x];
  center_potentials_dev(s.u, s.np, s.nb, s.w0, s.w1, &s.kst->stop, 0);
}

__global__ void b_mixed_scales(const SysDesc* __restrict__ d) {
  const SysDesc& s = d[blockIdx.y];
  mixed_scales_dev(s.u, s.np, s.mconst, s.beta, s.msc, &s.kst->stop, blockIdx.x);
}

// blockIdx.z = system, blockIdx.y = spin: the split forward operand (U~ C)^T
__global__ void b_split(const SysDesc* __restrict__ d) {
  const SysDesc& s = d[blockIdx.z];
  const int spin = blockIdx.y;
  const size_t np2 = (size_t)s.np * s.np;
  split_scaled_columns_dev(spin ? s.CT1 : s.CT0, s.np, s.u + (size_t)spin * s.np, s.msc + spin * 8 + 3,
                           s.uct_h + spin * np2, s.uct_l + spin * np2, &s.kst->stop, blockIdx.x, gridDim.x);
}

// The forward's symmetrizing pass over every item of the batch: blockIdx.x runs over
// the block pairs of all items, item z owning [pair_off[z], pair_off[z + 1]).
__device__ __forceinline__ int pair_item(const int* __restrict__ pair_off, int nitems, int g) {
  int lo = 0, hi = nitems;
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (pair_off[mid] <= g) lo = mid;
    else hi = mid;
  }
  return lo;
}
// Block side of the pair list: split batches pad every system to the large split tile and
// take its 64 x 64 block pairs (512 threads); FP64 batches (padded to 128) 64 x 64 as well.
constexpr int BATCH_SYM_B_MIXED = SYM_B_LARGE, BATCH_SYM_T_MIXED = SYM_T_LARGE;
constexpr int BATCH_SYM_B_F64 = SYM64_B_LARGE, BATCH_SYM_T_F64 = SYM64_T_LARGE;

// (Against the earlier pass with one element per thread and row: the same bits, and
// the 64-cluster split batch 19.59 -> 19.76 batch updates/s, one process.)
__global__ __launch_bounds__(BATCH_SYM_T_MIXED) void b_symmetrize(const BatchItemMixed* __restrict__ items,
                                                                  const int* __restrict__ pair_off, int nitems) {
  static_assert(BATCH_SYM_B_MIXED == 64 && BATCH_SYM_T_MIXED == 512, "64 x 64 pairs, 8 elements per thread");
  const int z = pair_item(pair_off, nitems, blockIdx.x);
  const BatchItemMixed& it = items[z];
  if (*it.stop) return;
  fermi_symmetrize_v8_dev<false, 2>(it.g, it.n, it.beta, blockIdx.x - pair_off[z], it.act, it.nblk);
}

__global__ __launch_bounds__(BATCH_SYM_T_F64) void b_symmetrize_f64(const BatchItemF64* __restrict__ items,
                                                        const int* __restrict__ pair_off, int nitems) {
  const int z = pair_item(pair_off, nitems, blockIdx.x);
  const BatchItemF64& it = items[z];
  if (*it.stop) return;
  fermi_symmetrize_f64_dev<BATCH_SYM_B_F64, BATCH_SYM_T_F64>(it.g, it.n, it.beta, blockIdx.x - pair_off[z], it.act,
                                                             it.nblk);
}

__global__ void b_combine(const SysDesc* __restrict__ d) {
  const SysDesc& s = d[blockIdx.y];
  if ((int)(blockIdx.x * (blockDim.x / WAVE)) >= s.natoms) return;
  combine_dev(s.xdiag, s.part, s.nparts, s.part_stride, s.w0, s.w1, s.wsum, s.t, s.nb, s.np, s.offsets, s.natoms, s.q1,
              &s.kst->stop, blockIdx.x, 0);
}

// f~_k = -(q1 - v_k) (K0 = -I)
__global__ void b_precond(const SysDesc* __restrict__ d, int k) {
  const SysDesc& s = d[blockIdx.y];
  if (s.kst->stop) return;
  const int n2 = 2 * s.natoms;
  const double* v = s.V + (size_t)k * n2;
  double* out = s.Ft + (size_t)k * n2;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += gridDim.x * blockDim.x)
    out[i] = -(s.q1[i] - v[i]);
}

__global__ void __launch_bounds__(1024) b_solve(SysDesc* d, double* const* out) {
  const SysDesc& s = d[blockIdx.x];
  solve_dev(s.V, s.Ft, s.ftilde, 2 * s.natoms, s.kst, out[blockIdx.x], 0.0);
}

__global__ void b_info(const SysDesc* __restrict__ d, int ns, KrylovState* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ns) out[i] = *d[i].kst;
}

// Whether a BM x BN forward tile holds a block in which Y may be non-zero.
template <class Cfg, class Item>
__device__ __forceinline__ bool window_tile_active(const Item& it, int tm, int tn) {
  bool any = false;
  for (int i = 0; i < Cfg::BM / WIN; ++i)
    for (int j = 0; j < Cfg::BN / WIN; ++j)
      any |= window_active(it.act, it.nblk, tm * (Cfg::BM / WIN) + i, tn * (Cfg::BN / WIN) + j);
  return any;
}

// Tile queues of a persistent transform: one per XCD, so that the workgroups of an XCD (blockIdx
// mod 8) work on the same systems' panels in its L2. tiles[off[x]..off[x + 1]) is queue x, filled
// by the host with whole row groups of systems, dearest first, to equal cost; next[x] counts
// what has been taken. A workgroup takes tiles from its own queue until that is empty, then from
// the others', so the launch ends level whatever the systems' stop flags and windows leave out,
// and a workgroup that starts late finds all queues empty and ends. Against a fixed stride over one
// list (tile t to workgroup t mod grid): 24 clusters of 16-250 atoms, FP64, m = 6, 54.9 -> 48.8 ms
// an update; 64 clusters FP16 x 3 49.8 -> 45.3 ms, FP64 5.33 -> 5.94 updates/s (the windows alone,
// whose gaps a stride cannot close, gave the 24 clusters 0.8 %).
constexpr int XCDS = 8;
struct TileQueues {
  const int4* tiles;
  const int* off;  // XCDS + 1
  int* next;       // XCDS counters, zero at the launch: tiles taken after the workgroups' first ones
};

// Takes the workgroup's next tile; false once there is none. A workgroup's first tile is its own
// place in its XCD's queue, without the counters, and one look at all counters finds a queue
// that is not empty: a counter's round trip is a microsecond and more, and walking the eight of
// them to the end of a launch cost the 64 x 64 class of 16 small clusters 46 us for 16.
struct QueueState {
  bool first = true;
};
__device__ __forceinline__ bool queue_take(const TileQueues& q, QueueState& st, int4& tile) {
  __shared__ int4 taken;
  if (threadIdx.x < WAVE) {
    const int lane = threadIdx.x, grid = gridDim.x, own = blockIdx.x % XCDS;
    const int x = lane % XCDS, off = q.off[x], len = q.off[x + 1] - off;
    const int ahead = (grid - x + XCDS - 1) / XCDS;  // first tiles of queue x's workgroups
    int4 got = make_int4(-1, 0, 0, 0);
    if (st.first && (int)(blockIdx.x / XCDS) < __shfl(len, own)) {
      got = q.tiles[__shfl(off, own) + blockIdx.x / XCDS];
    } else {
      for (;;) {
        const int used = __hip_atomic_load(&q.next[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned full = (unsigned)__ballot(ahead + used < len) & ((1u << XCDS) - 1);
        if (full == 0) break;  // every counter has reached its queue's end, and counters only grow
        // the own queue, or the next one after it that has tiles left
        const unsigned turned = ((full >> own) | (full << (XCDS - own))) & ((1u << XCDS) - 1);
        const int from = (own + __builtin_ctz(turned)) % XCDS;
        int at = 0;
        if (lane == 0) at = atomicAdd(&q.next[from], 1);
        at = __shfl(at, 0) + __shfl(ahead, from);
        if (at < __shfl(len, from)) {
          got = q.tiles[__shfl(off, from) + at];
          break;
        }
      }
    }
    if (lane == 0) taken = got;
  }
  st.first = false;
  __syncthreads();
  // uniform for the compiler too: the tile's pointers stay scalar
  tile = make_int4(__builtin_amdgcn_readfirstlane(taken.x), __builtin_amdgcn_readfirstlane(taken.y),
                   __builtin_amdgcn_readfirstlane(taken.z), 0);
  __syncthreads();  // taken is free for the next call
  return tile.x >= 0;
}

// Transforms over the tile queues (QUEUED), or one tile to each workgroup; a tile of a system whose
// Krylov expansion has stopped, or that its window leaves out, is skipped (uniformly for the workgroup).
// A launch whose tiles all run at once has neither queues nor windows, which could only add to its
// latency: 10 clusters of 30-70 atoms, FP16 x 3, 1.28 ms an update against 1.49 with the queues and 1.35
// with a stride loop; 16 of 20-60 atoms FP64, 2.10 against 2.15 and 2.14.
// Held to MIN_BLOCKS workgroups per CU: the two-half forward form with the Fermi
// epilogue, which this kernel ran before the full-tile forward, took ~164 registers per
// lane and one workgroup per CU when left to itself (13 % slower); the full-tile
// product and the back-transform fit without spilling.
template <int EPI, class Cfg, bool QUEUED>
__global__ __launch_bounds__(Cfg::THREADS) __attribute__((amdgpu_waves_per_eu(Cfg::WAVES_PER_EU)))
void b_gemm(const BatchItemF64* __restrict__ items, const TileQueues q) {
  if constexpr (!QUEUED) {
    const int4 tl = q.tiles[blockIdx.x];
    const BatchItemF64& it = items[tl.x];
    if (*it.stop) return;
    f64_tile<EPI, Cfg>(it.g, HalfRows{it.g, it.n, 0, it.k, false}, it.n, make_int2(tl.y, tl.z), it.beta);
  } else {
    QueueState take;
    int4 tl;
    while (queue_take(q, take, tl)) {
      const BatchItemF64& it = items[tl.x];
      if (*it.stop) continue;
      int2 rows = make_int2(0, it.k);
      if constexpr (EPI == EPI_MULLIKEN)
        rows = window_rows(it.range, tl.z * (Cfg::BN / WIN), Cfg::BN / WIN, it.k, Cfg::BK, 0);
      else if (!window_tile_active<Cfg>(it, tl.y, tl.z))
        continue;
      const HalfRows src{it.g, it.n, rows.x, rows.y - rows.x, false};
      f64_tile<EPI, Cfg>(it.g, src, it.n, make_int2(tl.y, tl.z), it.beta);
    }
  }
}

// Held to MIN_BLOCKS workgroups per CU as well (the two-half forward form with a staged
// mirror epilogue, which this kernel ran before the full-tile forward, took ~190 registers
// and one workgroup per CU when left to itself, 4 % slower).
template <int EPI, class Cfg, bool QUEUED>
__global__ __launch_bounds__(Cfg::THREADS) __attribute__((amdgpu_waves_per_eu((Cfg::MIN_BLOCKS * Cfg::THREADS / 64 + 3) / 4)))
void b_gemm(const BatchItemMixed* __restrict__ items, const TileQueues q) {
  if constexpr (!QUEUED) {
    const int4 tl = q.tiles[blockIdx.x];
    const BatchItemMixed& it = items[tl.x];
    if (*it.stop) return;
    mixed_tile<EPI, Cfg>(it.g, it.n, 0, it.k, make_int2(tl.y, tl.z));
  } else {
    QueueState take;
    int4 tl;
    while (queue_take(q, take, tl)) {
      const BatchItemMixed& it = items[tl.x];
      if (*it.stop) continue;
      int2 rows = make_int2(0, it.k);
      if constexpr (EPI == EPI_MULLIKEN)
        rows = window_rows(it.range, tl.z * (Cfg::BN / WIN), Cfg::BN / WIN, it.k, WIN_ROWS_MIXED<Cfg>, Cfg::BK);
      else if (!window_tile_active<Cfg>(it, tl.y, tl.z))
        continue;
      mixed_tile<EPI, Cfg>(it.g, it.n, rows.x, rows.y - rows.x, make_int2(tl.y, tl.z));
    }
  }
}

}  // namespace kk
