// Device-side problem description, workspace header and the importance load shared by all kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tsenor.h"

namespace tsenor_dev {

// Head of a matrix's workspace slice: what the kernels of a call pass to each other besides the potentials and masks of the blocks.
struct WsHeader {
  double tau_eff;         // multiplier of the importance, left by the iterations for the rounding (M >= 8, T > 0)
  // measurement aid: shader-clock cycles and constant-rate timer ticks that the first wave of the Dykstra kernel
  // spent in its iteration loop (their ratio is the clock the chip held under that load)
  unsigned long long loop_cycles, loop_ticks;
};
static_assert(sizeof(WsHeader) <= 256, "header must fit its slot");

// The importance maximum of a matrix (relative tau) travels as one partial maximum per workgroup of the
// pre-pass, in the workspace right after the header; the kernel that needs the maximum reduces them itself.
// No atomic, so nothing has to be cleared before a call.
constexpr int kMaxAbsmaxPartials = 1024;
// Once the iterations have read them, their place holds the partial sums of the objectives: a pair (mask found, previous
// mask) per workgroup of objective_kernel.
constexpr int kObjectiveGroups = 64;
static_assert(kObjectiveGroups * 2 * sizeof(double) <= kMaxAbsmaxPartials * sizeof(float), "the partial sums fit");

struct DevProblem {
  const void* W;
  const void* add;
  const float* col_scale;
  int64_t ld, cols, nblocks, bc;  // bc: blocks per block-row
  int dtype, N, T, transpose;
  int L;
  short strict, simple;  // simple: the ablation arm in place of Algorithm 2
  double tau;
  int tau_mode;
  float add_scale;
  int square;
  double tol;  // > 0: early exit of the iterations (see tsenor_problem.tol)
};

// One fused launch serves up to kMaxBatch matrices that share M and the kernel variant: every kernel gets the
// table by value, finds the matrix its workgroup belongs to from the prefix `first`, and reads that entry.
// A matrix owns whole workgroups, so the choice is uniform over a workgroup.
constexpr int kMaxBatch = 16;

struct BatchEntry {
  DevProblem p;
  int64_t rows;
  WsHeader* hdr;                // workspace slices of this matrix
  float* absmax_partial;        // partial maxima of the importance, absmax_count of them (relative tau only)
  int absmax_count;
  void* potentials;             // BlockPotentials of every block (M >= 8)
  void* rowmask;                // greedy's mask (M = 4) or the row normalisers (M >= 8), then the blocks' counters
  double* block_objective;      // NULL: no objective asked for
  uint8_t* mask;                // outputs of the caller (NULL where optional and not asked for)
  double* plan_out;
  double* tau_eff_out;
  int64_t* stats_out;
  uint8_t* packed_out;
  void* pruned_out;
  double* objective_out;
  const uint8_t* prev_mask;
  int* iters_done_out;
  // alignment of the caller's buffers
  uint8_t wide_store;           // mask rows can be written with 16-byte stores
  uint8_t wide_prev;            // the previous mask can be read with loads as wide as a block row (at most 16 bytes)
  uint8_t absmax_vec;           // rows of W (and of the additive term) can be read with 16-byte loads by the pre-pass
  uint8_t by_columns;           // the iterations take the blocks column by column, in the order of column_order_of()
  uint8_t emit_vec;             // everything the derived outputs read and write can be moved 8 weights at a time
};

struct Batch {
  int count;
  unsigned int first[kMaxBatch + 1];  // first workgroup of every matrix in the launch at hand
  BatchEntry e[kMaxBatch];
};
static_assert(sizeof(Batch) <= 4096, "the table travels as a kernel argument");

__device__ __forceinline__ int find_problem(const Batch& b, unsigned int workgroup) {
  int k = 0;
  while (k + 1 < b.count && workgroup >= b.first[k + 1]) ++k;
  return k;
}

// matrix position of a block.  A launch holds fewer than 2^31 blocks: a 32-bit division, a fraction of a 64-bit one
struct BlockAt {
  int64_t r0, c0;
};
__device__ __forceinline__ BlockAt block_at(const DevProblem& p, int64_t blk, int M) {
  const unsigned int b = (unsigned int)blk, bc = (unsigned int)p.bc, row = b / bc;
  return {(int64_t)row * M, (int64_t)(b - row * bc) * M};
}

constexpr size_t kAlign = 256;  // of the parts of a workspace slice
__host__ __device__ inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
// M words per block, 32-bit up to M = 32, 64-bit for M = 64: greedy's row bit masks (M = 4) or the row normalisers, then the
// block's counters
__host__ __device__ inline size_t rowmask_bytes_per_block(int M) { return (size_t)M * (M > 32 ? 8 : 4); }

// Block columns in the order the iterations take them (by_columns).  The list stands where something else is written after the
// iterations: the potentials, which the one kernel of the small tiles keeps to itself, or the blocks' objectives, behind the row masks.
enum { kOrderInPotentials = 1, kOrderInObjectives = 2 };
__device__ __forceinline__ uint16_t* column_order_of(const BatchEntry& e, int M) {
  char* at = static_cast<char*>(e.potentials);
  if (e.by_columns == kOrderInObjectives)
    at = static_cast<char*>(e.rowmask) + align_up((size_t)e.p.nblocks * rowmask_bytes_per_block(M));
  return reinterpret_cast<uint16_t*>(at);
}
// The block that the iterations take at place `k` of a matrix.  With a column scale the blocks of a column, which share it, converge
// in about the same number of iterations, and those under large scales in many times that of the others: so they go column by
// column, the largest scale first.  The blocks of a wave then stop together, and the long waves begin early instead of ending the
// launch alone (16:32 4096x14336 Wanda-style: the iterations a wave runs 113 -> 103 on average in fp32, and what the launch takes
// beyond an even load of its SIMDs 11-16 % -> 3-4 %).  orders_columns() in launch.hpp has the calls it pays for.
// (a branch of its own: with one division for both orders, launches without the list were 0.5-1 % slower.)
__device__ __forceinline__ BlockAt place_of(const BatchEntry& e, int64_t k, int M, int64_t& blk) {
  if (!e.by_columns) {
    blk = k;
    return block_at(e.p, k, M);
  }
  const unsigned at = (unsigned)k, block_rows = (unsigned)(e.rows / M), rank = at / block_rows, row = at - rank * block_rows,
                 column = column_order_of(e, M)[rank];
  blk = (int64_t)row * e.p.bc + column;
  return {(int64_t)row * M, (int64_t)column * M};
}

__device__ __forceinline__ float load_element(const void* base, int dtype, int64_t index) {
  if (dtype == TSENOR_BF16) {
    const unsigned int b = reinterpret_cast<const unsigned short*>(base)[index];
    return __uint_as_float(b << 16);
  }
  return reinterpret_cast<const float*>(base)[index];
}

// x = W + add_scale * add: the value a kept entry carries (Sec. 4; the ALPS D-update of Proposition 1).
// Explicitly rounded operations: no fused multiply-add, so that a host evaluation gives the same bits.
__device__ __forceinline__ float load_value(const DevProblem& p, int64_t r, int64_t c) {
  const float w = load_element(p.W, p.dtype, r * p.ld + c);
  if (!p.add) return w;
  return __fadd_rn(w, __fmul_rn(p.add_scale, load_element(p.add, p.dtype, r * p.ld + c)));
}

// importance of one weight: |x| (times col_scale[j]) (squared), every step one float operation
// (Sec. 4: Wanda-style scores; Proposition 1: (W + V/rho)^2)
__device__ __forceinline__ float load_importance(const DevProblem& p, int64_t r, int64_t c) {
  float a = fabsf(load_value(p, r, c));
  if (p.col_scale) a = __fmul_rn(a, p.col_scale[c]);
  if (p.square) a = __fmul_rn(a, a);
  return a;
}

// Tile loads.  A lane holds a TH x TW register tile of its block; the element offset of tile entry (a, b)
// is base + roff[a] + coff[b], and its column scale is csa[a] * csb[b] where one of the two factors is
// exactly 1 (which of them depends on whether the kernel works on the block or on its transpose), so the
// product with both is still the single rounded multiply of the definition above.  The point of this form:
// every choice (storage type, additive term, scale, transpose) is made once per tile, and the loads of a
// tile are one straight run of independent instructions instead of a chain of branches with a wait each.
template <int TH, int TW>
struct TileAddr {
  int64_t base;
  int64_t roff[TH], coff[TW];
  float csa[TH], csb[TW];
};

// ri[a], cj[b]: coordinates of the tile's rows and columns inside the (possibly transposed) block at
// matrix position (r0, c0)
template <int TH, int TW>
__device__ __forceinline__ TileAddr<TH, TW> tile_addr(const DevProblem& p, int64_t r0, int64_t c0, const int (&ri)[TH],
                                                      const int (&cj)[TW]) {
  TileAddr<TH, TW> t;
  t.base = r0 * p.ld + c0;
#pragma unroll
  for (int a = 0; a < TH; ++a) {
    t.roff[a] = p.transpose ? (int64_t)ri[a] : ri[a] * p.ld;
    t.csa[a] = 1.0f;
  }
#pragma unroll
  for (int b = 0; b < TW; ++b) {
    t.coff[b] = p.transpose ? cj[b] * p.ld : (int64_t)cj[b];
    t.csb[b] = 1.0f;
  }
  if (p.col_scale) {
    if (p.transpose) {
#pragma unroll
      for (int a = 0; a < TH; ++a) t.csa[a] = p.col_scale[c0 + ri[a]];
    } else {
#pragma unroll
      for (int b = 0; b < TW; ++b) t.csb[b] = p.col_scale[c0 + cj[b]];
    }
  }
  return t;
}

template <bool BF16, bool ADD, int A0, int NA, int TH, int TW>
__device__ __forceinline__ void tile_values(const DevProblem& p, const TileAddr<TH, TW>& t, float (&x)[NA][TW]) {
  float v[ADD ? NA : 1][ADD ? TW : 1];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < TW; ++b) {
      const int64_t off = t.base + t.roff[A0 + a] + t.coff[b];
      if constexpr (BF16) {
        x[a][b] = __uint_as_float((unsigned int)reinterpret_cast<const unsigned short*>(p.W)[off] << 16);
        if constexpr (ADD) v[a][b] = __uint_as_float((unsigned int)reinterpret_cast<const unsigned short*>(p.add)[off] << 16);
      } else {
        x[a][b] = reinterpret_cast<const float*>(p.W)[off];
        if constexpr (ADD) v[a][b] = reinterpret_cast<const float*>(p.add)[off];
      }
    }
  if constexpr (ADD) {
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < TW; ++b) x[a][b] = __fadd_rn(x[a][b], __fmul_rn(p.add_scale, v[a][b]));
  }
}

// importance of tile rows [A0, A0 + NA): the same operations, in the same order, as load_importance.  SHORT: branches around the
// multiplications by 1 and the square that is not asked for (three of four operations of an entry; small launches, which wait for
// every basic block, do without the branches: 0.6 us of a 512 x 512 call).  With exp_in_range() and the scalar row addresses of
// block_column_values(): 32:64 8192x8192 with the early exit 692 / 682 us, 32:64 6144x2048 Wanda-style, whose fp32 tiles are formed
// anew, 612 / 566, 4096x4096 583 / 575; 16- and 32-wide calls 0-2 % faster.
template <int A0, int NA, bool SHORT, int TH, int TW>
__device__ __forceinline__ void tile_importance(const DevProblem& p, const TileAddr<TH, TW>& t, float (&imp)[NA][TW]) {
  if (p.dtype == TSENOR_BF16) {
    if (p.add)
      tile_values<true, true, A0, NA>(p, t, imp);
    else
      tile_values<true, false, A0, NA>(p, t, imp);
  } else {
    if (p.add)
      tile_values<false, true, A0, NA>(p, t, imp);
    else
      tile_values<false, false, A0, NA>(p, t, imp);
  }
  if constexpr (SHORT) {
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < TW; ++b) imp[a][b] = fabsf(imp[a][b]);
    if (p.col_scale) {
      if (p.transpose) {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
          for (int b = 0; b < TW; ++b) imp[a][b] = __fmul_rn(imp[a][b], t.csa[A0 + a]);
      } else {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
          for (int b = 0; b < TW; ++b) imp[a][b] = __fmul_rn(imp[a][b], t.csb[b]);
      }
    }
    if (p.square) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b) imp[a][b] = __fmul_rn(imp[a][b], imp[a][b]);
    }
  } else {
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < TW; ++b) {
        float m = __fmul_rn(__fmul_rn(fabsf(imp[a][b]), t.csa[A0 + a]), t.csb[b]);
        if (p.square) m = __fmul_rn(m, m);
        imp[a][b] = m;
      }
  }
}

// a number of the wave's first active lane, in scalar registers
__device__ __forceinline__ int64_t of_first_lane(int64_t v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)v), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}
template <bool BF16>
__device__ __forceinline__ float element_at(const char* at) {
  if constexpr (BF16)
    return __uint_as_float((unsigned int)*reinterpret_cast<const unsigned short*>(at) << 16);
  else
    return *reinterpret_cast<const float*>(at);
}

// importance of the M entries (r0 .. r0+M-1, c) of one matrix column, loads issued together; the same
// operations, in the same order, as load_importance.
// ASCENDING: no lane's r0 is above that of a lane after it (blocks taken row by row: the kernels of their own that round).  The address of
// a row is then one scalar, of the first lane's blocks, and the lane's part a 32-bit offset from it that is not negative: the blocks of
// a wave lie in at most 64 rows and c is below ld, so the offset stays below 2^32 for ld < kFarLd.  (64-bit addresses of their own took
// the lanes two to four instructions per entry, twice, 7 % of the rounding of 64-wide blocks.)
constexpr int64_t kFarLd = (int64_t)1 << 21;
template <int M, bool BF16, bool ADD, bool ASCENDING>
__device__ __forceinline__ void block_column_values(const DevProblem& p, int64_t r0, int64_t c, float (&x)[M]) {
  constexpr int SIZE = BF16 ? 2 : 4;
  float v[ADD ? M : 1];
  const char *W = static_cast<const char*>(p.W), *V = static_cast<const char*>(p.add);
  const int64_t step = p.ld * SIZE;
  if (ASCENDING && p.ld < kFarLd) {
    const int64_t first = of_first_lane(r0);
    const unsigned off = ((unsigned)(r0 - first) * (unsigned)p.ld + (unsigned)c) * SIZE;
    W += first * step;
    if constexpr (ADD) V += first * step;
#pragma unroll
    for (int k = 0; k < M; ++k) {
      asm("" : "+s"(W), "+s"(V));  // (the row's address stays a scalar one, and `off` the lane's part of it)
      x[k] = element_at<BF16>(W + off);
      W += step;
      if constexpr (ADD) {
        v[k] = element_at<BF16>(V + off);
        V += step;
      }
    }
  } else {
    const int64_t off = (r0 * p.ld + c) * SIZE;
#pragma unroll
    for (int k = 0; k < M; ++k) {
      x[k] = element_at<BF16>(W + (off + k * step));
      if constexpr (ADD) v[k] = element_at<BF16>(V + (off + k * step));
      if (ASCENDING && k % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (their addresses would not fit the registers beside the rest)
    }
  }
  if constexpr (ADD) {
#pragma unroll
    for (int k = 0; k < M; ++k) x[k] = __fadd_rn(x[k], __fmul_rn(p.add_scale, v[k]));
  }
}
template <int M, bool ASCENDING>
__device__ __forceinline__ void block_column_importance(const DevProblem& p, int64_t r0, int64_t c, float (&imp)[M]) {
  if (p.dtype == TSENOR_BF16) {
    if (p.add)
      block_column_values<M, true, true, ASCENDING>(p, r0, c, imp);
    else
      block_column_values<M, true, false, ASCENDING>(p, r0, c, imp);
  } else {
    if (p.add)
      block_column_values<M, false, true, ASCENDING>(p, r0, c, imp);
    else
      block_column_values<M, false, false, ASCENDING>(p, r0, c, imp);
  }
  const float cs = p.col_scale ? p.col_scale[c] : 1.0f;
#pragma unroll
  for (int k = 0; k < M; ++k) imp[k] = __fmul_rn(fabsf(imp[k]), cs);  // times exactly 1 where there is no scale
  if (p.square) {
#pragma unroll
    for (int k = 0; k < M; ++k) imp[k] = __fmul_rn(imp[k], imp[k]);
  }
}

// multiplier of the importance in the log-kernel K (App. B.1 parameter choice for the relative mode).
// Called by whole waves: the partial maxima of the pre-pass are reduced across the lanes.
__device__ __forceinline__ double tau_eff_of(const BatchEntry& e) {
  const DevProblem& p = e.p;
  if (p.tau_mode == TSENOR_TAU_ABSOLUTE) return p.tau;
  float mx = 0.0f;
  for (int k = (int)(threadIdx.x & 63u); k < e.absmax_count; k += 64) mx = fmaxf(mx, e.absmax_partial[k]);
  for (int s = 1; s < 64; s <<= 1) mx = fmaxf(mx, __shfl_xor(mx, s, 64));
  return mx > 0.0f ? 1.0 / (p.tau * (double)mx) : 0.0;
}

}  // namespace tsenor_dev
