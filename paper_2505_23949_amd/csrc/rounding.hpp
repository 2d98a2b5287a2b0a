// Algorithm 2: greedy selection, local search and the mask write.
#pragma once
#include <limits>
#include <type_traits>

#include "lanes.hpp"
#include "problem.hpp"

namespace tsenor_dev {

// The rounding steps below belong to one wave each (whatever the size of its workgroup).  Its LDS accesses take effect in
// the order they are issued; what is needed between them is that the compiler keeps that order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Bit masks over the M columns (or rows) of a block.
template <int M>
using block_mask_t = typename std::conditional<(M > 32), unsigned long long, unsigned int>::type;

template <class mask_t>
__device__ __forceinline__ int mask_popc(mask_t v) {
  if constexpr (sizeof(mask_t) == 8)
    return __popcll((unsigned long long)v);
  else
    return __popc((unsigned int)v);
}

// LDS of the lane-parallel rounding steps for the G blocks a wave holds: the mask as row and column bit masks
// (rowm[r] bit c == colm[c] bit r == S[r][c]), column counters of the greedy selection, the importance block.
template <int M, int G>
struct RoundingLds {
  union {
    struct {
      block_mask_t<M> rowm[G][M], colm[G][M];
    };
    // until the sort keys are formed: minus the normaliser of every in-kernel row (BlockPotentials)
    double minus_largest[G][M];
  };
  unsigned int colcnt[G][M];
  // (rows padded by one float: lane r reads row r, and with a row length of M every lane would hit the same bank)
  static constexpr int kImpLd = M + 1;
  float imp[G][M * kImpLd];
};

// Transpose of an M x M bit matrix held as one M-bit row per lane (M consecutive lanes): afterwards the
// lane that held row r holds column r.  log2(M) block-swap steps.
template <int M, int S = M / 2, class mask_t>
__device__ __forceinline__ mask_t bit_transpose(mask_t x, int ql) {
  if constexpr (S >= 1) {
    // bits whose index has bit S clear: S ones, S zeros, repeated
    mask_t lowpat = 0;
    for (int k = 0; k < M; ++k)
      if (!(k & S)) lowpat |= (mask_t)1 << k;
    mask_t other;
    if constexpr (sizeof(mask_t) == 8)
      other = (mask_t)__double_as_longlong(lane_xor<S>(__longlong_as_double((long long)x)));
    else
      other = (mask_t)lane_xor_i32<S>((int)x);
    x = (ql & S) ? (mask_t)((x & ~lowpat) | ((other & ~lowpat) >> S)) : (mask_t)((x & lowpat) | ((other & lowpat) << S));
    return bit_transpose<M, S / 2>(x, ql);
  } else {
    return x;
  }
}

// The best of the swaps (i', j') of Eq. (5) that a lane i' may take part in: `cand` are its columns j', row_i and row_q the
// importance of row i and of its own.  Higher score wins, equal scores go to the lower column.  (A score that is not a
// number, as of importances that overflowed, counts as the lowest there is: any candidate is better than none.)
struct SwapBest {
  double score;
  int column;
};
__device__ __forceinline__ void scan_candidate(unsigned int& word, int first, const float* row_i, const float* row_q, double base,
                                               SwapBest& best) {
  const int j = first + __ffs((int)word) - 1;
  word &= word - 1;
  const double score = ((double)row_i[j] + base) - (double)row_q[j];
  if (score > best.score) {
    best.score = score;
    best.column = j;
  }
}
template <class mask_t>
__device__ __forceinline__ SwapBest best_candidate(mask_t cand, const float* row_i, const float* row_q, double base) {
  SwapBest best = {-std::numeric_limits<double>::infinity(), (sizeof(mask_t) == 8 ? __ffsll((long long)cand) : __ffs((int)cand)) - 1};
  unsigned int word = (unsigned int)cand;
  while (word != 0) scan_candidate(word, 0, row_i, row_q, base, best);
  if constexpr (sizeof(mask_t) == 8) {
    word = (unsigned int)(cand >> 32);
    while (word != 0) scan_candidate(word, 32, row_i, row_q, base, best);
  }
  return best;
}

// the mask of lane `lane`, which is to be the same number in every lane
__device__ __forceinline__ unsigned int mask_of_lane(unsigned int v, int lane) { return (unsigned)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ unsigned long long mask_of_lane(unsigned long long v, int lane) {
  return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)v, lane) |
         (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32;
}

template <int M, int STEP = 1>
__device__ __forceinline__ double group_sum(double v) {
  if constexpr (STEP < M) {
    v += lane_xor<STEP>(v);
    return group_sum<M, STEP * 2>(v);
  } else {
    return v;
  }
}

template <int M, int STEP = 1>
__device__ __forceinline__ int group_sum(int v) {
  if constexpr (STEP < M) {
    v += lane_xor_i32<STEP>(v);
    return group_sum<M, STEP * 2>(v);
  } else {
    return v;
  }
}

// Algorithm 2 lines 7-13 and the mask write for the blocks of one wave.  A block owns LPB >= M consecutive lanes,
// of which the first M take part: lane r owns row r and column r of the block as bit masks.  On entry lds.rowm
// holds the mask greedy selection left.  blk: the lane's block (a valid one also for idle lanes, which write
// nothing: `active`), at matrix position (r0, c0).  ASCENDING: of block_column_values.  To be called by whole waves.
template <int M, int LPB, bool ASCENDING>
__device__ __forceinline__ void local_search_and_write(const DevProblem& p, const BatchEntry& e, int64_t blk, bool active,
                                                       int64_t r0, int64_t c0, int lane, RoundingLds<M, kWave / LPB>& lds) {
  using mask_t = block_mask_t<M>;
  constexpr int LD = RoundingLds<M, kWave / LPB>::kImpLd;
  uint8_t* mask = e.mask;
  const int wide_store = e.wide_store;
  double* block_objective = e.block_objective;
  const uint8_t* prev_mask = e.prev_mask;
  const bool want_stats = e.stats_out != nullptr;
  constexpr bool kInLanes = LPB == kWave;  // a wave has one block (see the swaps below)
  const int g = kInLanes ? 0 : lane / LPB, ql = lane % LPB;
  const bool part = ql < M;
  const int qm = ql % M;  // (an index that stays inside the block's LDS rows also for the lanes that only tag along)
  const mask_t one = 1;

  // the transpose of the mask greedy selection left
  {
    const mask_t r = part ? lds.rowm[g][qm] : (mask_t)0;
    const mask_t c = bit_transpose<M>(r, qm);
    if (part) lds.colm[g][qm] = c;
  }
  wave_sync();
  const auto popc = [](mask_t v) { return mask_popc(v); };
  const int missing = want_stats ? group_sum<M>(part ? p.N - popc(lds.rowm[g][qm]) : 0) : 0;
  const unsigned long long gmask = (M == 64 ? ~0ull : ((1ull << M) - 1)) << (g * LPB);
  const bool any_short = __any(part && popc(lds.rowm[g][qm]) < p.N);
  if ((any_short || block_objective) && part) {
    // local search scores on the importance (Eq. 5), staged in LDS: this lane fetches column ql of its
    // block, all M loads in flight at once
    float col[M];
    block_column_importance<M, ASCENDING>(p, r0, c0 + qm, col);
#pragma unroll
    for (int k = 0; k < M; ++k) lds.imp[g][k * LD + qm] = col[k];
  }
  wave_sync();

  int rounds = 0, nonpos = 0;
  bool open = any_short;  // this block may still take swaps
  // A wave of one block keeps the masks in the registers of the rows' and columns' lanes and reads those of row i and column j
  // from there; several blocks to a wave have theirs in LDS.  Such a wave takes every decision from ballots, so that all its
  // lanes agree on i, j, the winner and whether to go on, those that only tag along too: readlane takes one lane number.
  mask_t Srow = part ? lds.rowm[g][qm] : (mask_t)0, Scol = part ? lds.colm[g][qm] : (mask_t)0;
  while (any_short) {
    if constexpr (!kInLanes) {
      Srow = part ? lds.rowm[g][qm] : (mask_t)0;
      Scol = part ? lds.colm[g][qm] : (mask_t)0;
    }
    const unsigned long long rb = __ballot(part && popc(Srow) < p.N) & gmask;
    const unsigned long long cb = __ballot(part && popc(Scol) < p.N) & gmask;
    if (rb == 0 || cb == 0 || (p.strict && rounds >= p.L)) open = false;
    if (!__any(open)) break;
    // line 10: the lowest-index row i and column j that are short
    const int i = kInLanes || open ? (__ffsll((long long)rb) - 1 - g * LPB) : 0;
    const int j = kInLanes || open ? (__ffsll((long long)cb) - 1 - g * LPB) : 0;
    // line 11 for i' = this lane: columns j' with S[i'][j'] = 1 and S[i][j'] = 0, provided S[i'][j] = 0
    mask_t row_i, col_j;
    if constexpr (kInLanes)
      row_i = mask_of_lane(Srow, i), col_j = mask_of_lane(Scol, j);
    else
      row_i = lds.rowm[g][i], col_j = lds.colm[g][j];
    mask_t cand = Srow & ~row_i;
    if (!open || !part || ((col_j >> qm) & 1)) cand = 0;
    const SwapBest best =
        best_candidate(cand, &lds.imp[g][i * LD], &lds.imp[g][qm * LD], (double)lds.imp[g][qm * LD + j]);
    // the best of the block: lanes are rows i', so among equal scores the first lane has the lowest flat index
    const double top = block_max<M>(best.score);
    const unsigned long long winners = __ballot(cand != 0 && best.score == top) & gmask;
    const int winner = winners ? __ffsll((long long)winners) - 1 : 0;
    const int ip = winner - g * LPB;
    const int jp = kInLanes ? __builtin_amdgcn_readlane(best.column, winner) : __shfl(best.column, winner, kWave);
    if (open) ++rounds;
    // (block_max() covers the block's M lanes: the maximum is the winner's)
    const bool gain = kInLanes ? (__ballot(top > 0.0) >> winner) & 1 : top > 0.0;
    const bool apply = winners != 0 && (!p.strict || gain);
    if (open && !apply) open = false;  // nothing changes any more for this block
    // line 13: remove (i', j'), insert (i', j) and (i, j')
    if constexpr (kInLanes) {
      if (apply) {
        if (ql == ip) Srow = (Srow & ~(one << jp)) | (one << j);
        if (ql == i) Srow |= one << jp;
        if (ql == jp) Scol = (Scol & ~(one << ip)) | (one << i);
        if (ql == j) Scol |= one << ip;
        if (!gain) ++nonpos;
      }
      continue;
    }
    wave_sync();
    if (apply && ql == 0) {
      lds.rowm[g][ip] = (lds.rowm[g][ip] & ~(one << jp)) | (one << j);
      lds.rowm[g][i] |= one << jp;
      lds.colm[g][jp] = (lds.colm[g][jp] & ~(one << ip)) | (one << i);
      lds.colm[g][j] |= one << ip;
      if (!gain) ++nonpos;
    }
    wave_sync();
  }
  if (kInLanes && any_short) {
    if (part) lds.rowm[g][qm] = Srow;
    wave_sync();
  }

  if (active && part) {
    const mask_t bits = lds.rowm[g][qm];
    uint8_t* dst = mask + (r0 + qm) * p.cols + c0;
    if (wide_store) {
      // 4 mask bytes per 32-bit word: bit k of a nibble goes to byte k
      unsigned int w[M / 4];
#pragma unroll
      for (int k = 0; k < M / 4; ++k) w[k] = (((unsigned int)(bits >> (4 * k)) & 0xFu) * 0x00204081u) & 0x01010101u;
      if constexpr (M == 4) {
        *reinterpret_cast<unsigned int*>(dst) = w[0];
      } else if constexpr (M == 8) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
      } else {
#pragma unroll
        for (int k = 0; k < M / 16; ++k)
          reinterpret_cast<uint4*>(dst)[k] = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
      }
    } else {
      for (int k = 0; k < M; ++k) dst[k] = (uint8_t)((bits >> k) & 1);
    }
  }
  if (block_objective) {
    // sum S * importance of this block for the mask found and for the caller's previous mask: every lane
    // sums its row left to right, the rows are then added in a fixed butterfly order
    double mine = 0.0, theirs = 0.0;
    if (part) {
      const mask_t bits = lds.rowm[g][qm];
      mask_t prev_bits = 0;
      if (prev_mask) {
        // the previous mask's row as bits: the byte loads are independent of each other
        const uint8_t* prev = prev_mask + (r0 + qm) * p.cols + c0;
        if (e.wide_prev) {
          unsigned int w[M / 4];
          if constexpr (M == 4) {
            w[0] = *reinterpret_cast<const unsigned int*>(prev);
          } else if constexpr (M == 8) {
            const uint2 v = *reinterpret_cast<const uint2*>(prev);
            w[0] = v.x, w[1] = v.y;
          } else {
#pragma unroll
            for (int k = 0; k < M / 16; ++k) {
              const uint4 v = reinterpret_cast<const uint4*>(prev)[k];
              w[4 * k] = v.x, w[4 * k + 1] = v.y, w[4 * k + 2] = v.z, w[4 * k + 3] = v.w;
            }
          }
#pragma unroll
          for (int k = 0; k < M; ++k) prev_bits |= (mask_t)((w[k / 4] & (0xFFu << (8 * (k % 4)))) != 0) << k;
        } else {
          uint8_t pm[M];
#pragma unroll
          for (int k = 0; k < M; ++k) pm[k] = prev[k];
#pragma unroll
          for (int k = 0; k < M; ++k) prev_bits |= (mask_t)(pm[k] != 0) << k;
        }
      }
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const double v = (double)lds.imp[g][qm * LD + k];
        mine += ((bits >> k) & 1) ? v : 0.0;
        theirs += ((prev_bits >> k) & 1) ? v : 0.0;
      }
    }
    mine = group_sum<M>(mine);
    theirs = group_sum<M>(theirs);
    if (active && ql == 0) {
      block_objective[2 * blk] = mine;
      block_objective[2 * blk + 1] = theirs;
    }
  }
  if (want_stats) {
    // a record per block where its mask from the greedy selection was (this wave has read it); stats_kernel adds them up.
    // (Atomic additions of every wave to the four counters took 0.24 ms for 24 000 waves.)
    const int left = group_sum<M>(part ? p.N - popc(lds.rowm[g][qm]) : 0);
    if (active && ql == 0)
      reinterpret_cast<uint4*>(static_cast<char*>(e.rowmask) + blk * (int64_t)(M * sizeof(mask_t)))[0] =
          make_uint4((unsigned)missing, (unsigned)nonpos, !p.strict && rounds > p.L ? 1u : 0u, (unsigned)left);
  }
}

// The stand-alone kernel (M = 4 on the large tiles): M lanes per block, 64/M blocks per wave, one wave per workgroup; the
// mask greedy selection left comes from the workspace.
template <int M>
__global__ __launch_bounds__(kWave) void finalize_kernel(Batch batch) {
  using mask_t = block_mask_t<M>;
  constexpr int G = kWave / M;
  __shared__ RoundingLds<M, G> lds;
  const int which = find_problem(batch, blockIdx.x);
  const DevProblem p = batch.e[which].p;
  const mask_t* rowmask = static_cast<const mask_t*>(batch.e[which].rowmask);
  const int lane = threadIdx.x, g = lane / M, ql = lane % M;
  int64_t blk = (int64_t)(blockIdx.x - batch.first[which]) * G + g;
  const bool active = blk < p.nblocks;
  if (!active) blk = p.nblocks - 1;  // idle groups shadow the last block and write nothing
  lds.rowm[g][ql] = rowmask[blk * M + ql];
  const BlockAt at = block_at(p, blk, M);
  local_search_and_write<M, M, true>(p, batch.e[which], blk, active, at.r0, at.c0, lane, lds);
}

// ------------------------------------------------------------------------------------------------------------------
// The whole of Algorithm 2 from the potentials the iterations leave (M >= 8, and M = 4 on the small tiles).
//
// The greedy selection needs no sort of the M*M entries.  It scans them in one common order (descending plan, ties by
// index) and keeps an entry while its row and its column have room; its result is the one stable assignment in which
// every row and every column prefers entries in that order and holds at most N of them (the first entry of the order is
// in every stable assignment, and what follows is the same problem with one place less; Gale and Shapley 1962, the
// common order makes the stable assignment unique).  So deferred acceptance finds it from the order INSIDE every row and
// every column alone: a row proposes to the columns of its first N entries; a column keeps the best N of its proposals
// and turns the others away; a row that was turned away proposes its next entries, until nobody proposes any more (about
// four rounds).  Two sorts of M keys in the registers of a lane (one lane per row, then one lane per column) replace a
// sort of M*M keys across the lanes of a block, and the M*M dependent steps of the scan are gone.
// ------------------------------------------------------------------------------------------------------------------

// What the iterations hand to the rounding, per block: log S = min((K - m) + (u + v), 0) with u per in-kernel row and v per
// in-kernel column (in-kernel rows are matrix columns under TSENOR_FLAG_COLS_FIRST), and m the normaliser of the in-kernel
// row, a float not below its largest K.  m and u stay apart: the largest K may be anything, and u - m in one number keeps
// of u what the size of m leaves (with K = 2^28 masks came out other than those of the same block shifted to K <= 640).
template <int M>
struct BlockPotentials {
  double u[M], v[M];
};
static_assert(sizeof(BlockPotentials<8>) <= 2 * 8 * 8, "fits the two bytes per weight the workspace has for it (M >= 8)");
// m is left where the block's counters go later, M floats of the slot that for M = 4 holds the greedy selection's mask
template <int M>
__device__ __forceinline__ float* normalisers_of(const BatchEntry& e, int64_t blk) {
  return reinterpret_cast<float*>(static_cast<char*>(e.rowmask) + blk * (int64_t)(M * sizeof(block_mask_t<M>)));
}

// Scan key of an entry: positive doubles whose order is descending plan, ties by ascending index.  `index` (below 2^12) is the
// entry's place in what is being sorted: a block, a row or a column.
constexpr int kIdxBits = 12;  // index bits: up to 64*64 entries
__device__ __forceinline__ double with_index(double key, unsigned int index) {
  return __hiloint2double(__double2hiint(key), (__double2loint(key) & ~((1 << kIdxBits) - 1)) | (int)index);
}
// log_plan: K + (u + v), to be capped at 0 (at -2^-1021: with the index bits in place the key is a normal double, and all
// capped entries tie)
__device__ __forceinline__ double scan_key(double log_plan, unsigned int index) {
  return with_index(fmax(-log_plan, 0x1p-1021), index);
}
// T = 0: the order is descending K itself.  Bit patterns of non-negative doubles order like the doubles:
// pattern(2^1023) - pattern(K) reverses the order for every finite K >= 0 and is again the pattern of a positive double
__device__ __forceinline__ double scan_key_of_k(double K, unsigned int index) {
  const unsigned long long bits = (unsigned long long)__double_as_longlong(K);
  return with_index(__longlong_as_double((long long)(0x7FE0000000000000ull - bits)), index);
}
// the index bytes of four keys whose index is below 2^8, next to each other
__device__ __forceinline__ unsigned int index_bytes(double a, double b, double c, double d) {
  const unsigned int ab = __builtin_amdgcn_perm((unsigned)__double2loint(b), (unsigned)__double2loint(a), 0x0c0c0400u);
  const unsigned int cd = __builtin_amdgcn_perm((unsigned)__double2loint(d), (unsigned)__double2loint(c), 0x0c0c0400u);
  return ab | cd << 16;
}

// (bare instructions: fmin() and fmax() first quiet possible signalling NaNs in keys that were put together from words)
__device__ __forceinline__ void compare_exchange_as_is(double& lo, double& hi) {
  double a;
  asm("v_min_f64 %0, %1, %2" : "=v"(a) : "v"(lo), "v"(hi));
  asm("v_max_f64 %0, %0, %1" : "+v"(hi) : "v"(lo));
  lo = a;
}

// Ascending sort of the E keys of a lane: Batcher's odd-even merge sort (191 comparators for 32 keys, 543 for 64; the
// bitonic network has 240 and 672), no data movement between lanes.
template <int E, int P = 1, int K = 1>
__device__ __forceinline__ void sort_in_lane(double (&c)[E]) {
  if constexpr (P < E) {
#pragma unroll
    for (int x = 0; x + K < E; ++x) {
      const int y = x - K % P;
      if (y >= 0 && y % (2 * K) < K && x / (2 * P) == (x + K) / (2 * P)) compare_exchange_as_is(c[x], c[x + K]);
    }
    if constexpr (E >= 32) __builtin_amdgcn_sched_barrier(0);  // stage by stage: stages that overlap need registers
    if constexpr (K > 1)
      sort_in_lane<E, P, K / 2>(c);
    else
      sort_in_lane<E, P * 2, P * 2>(c);
  }
}

// Algorithm 2 lines 1-6 for a 4 x 4 block in the registers of a lane, from its 16 keys in scan order (index = flat index):
// an entry is kept while its row and its column hold fewer than N.  Bit i*4+j of the result = S[i][j].
// `simple`: the ablation arm of App. B.2.1, row-wise then column-wise N:M rounding: an entry survives the row stage while its
// row has passed fewer than N entries, and a survivor is kept while its column holds fewer than N.
// ~250 instructions for 64 blocks behind the sort; as a kernel of its own the scan took 15 us of a 2:4 4096x4096 call, and its
// input two bytes per weight through memory.
__device__ __forceinline__ unsigned int select_in_lane(const double (&c)[16], int N, bool simple) {
  unsigned int kept = 0, passed = 0;  // the entries kept; the entries their row counts
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const unsigned int at = (unsigned int)__double2loint(c[k]) & 15u;
    const bool pass = __popc((passed >> (at & 12u)) & 15u) < N, keep = pass && __popc((kept >> (at & 3u)) & 0x1111u) < N;
    kept |= keep ? 1u << at : 0u;
    passed |= (simple ? pass : keep) ? 1u << at : 0u;
  }
  return kept;
}

// position of the N-th set bit (N >= 1) of a mask that has at least N
template <int M, class mask_t>
__device__ __forceinline__ int nth_set_bit(mask_t h, int N) {
  int pos = 0;
#pragma unroll
  for (int s = M / 2; s >= 1; s >>= 1) {
    const int below = mask_popc((mask_t)((h >> pos) & (((mask_t)1 << s) - 1)));
    if (below < N) {
      N -= below;
      pos += s;
    }
  }
  return pos;
}

// Algorithm 2 for the blocks of one wave.  A block owns LPB >= M consecutive lanes; lane r of the first M is its row r and
// its column r, further ones repeat what lane r % M does.  blk: the lane's block (a valid one also for idle lanes, which
// write nothing: `active`), at matrix position (r0, c0).  row_pot, col_pot (LDS, T > 0): the potentials of the matrix rows
// and columns of the wave's blocks; lds.minus_largest goes with them.  ASCENDING: of block_column_values.  To be called by whole
// waves.
template <int M, int LPB, bool ZERO_T, bool COLS_FIRST, bool ASCENDING = false>
__device__ __forceinline__ void round_blocks(const DevProblem& p, const BatchEntry& e, int64_t blk, bool active, int64_t r0,
                                             int64_t c0, int lane, double tau_eff, const double (*row_pot)[M],
                                             const double (*col_pot)[M], RoundingLds<M, kWave / LPB>& lds) {
  using mask_t = block_mask_t<M>;
  constexpr int LD = RoundingLds<M, kWave / LPB>::kImpLd;
  const int g = lane / LPB, ql = lane % M, N = p.N;
  // the importance of the block, a column per lane (coalesced), into LDS
  {
    float col[M];
    block_column_importance<M, ASCENDING>(p, r0, c0 + ql, col);
#pragma unroll
    for (int k = 0; k < M; ++k) lds.imp[g][k * LD + ql] = col[k];
  }
  wave_sync();

  // keys of the entries of this lane's row (ROWS) or column
  double c[M];
  auto keys = [&](auto rows_tag) {
    constexpr bool ROWS = decltype(rows_tag)::value;
    const auto importance = [&](int k) { return (double)lds.imp[g][ROWS ? ql * LD + k : k * LD + ql]; };
    if constexpr (ZERO_T) {
#pragma unroll
      for (int k = 0; k < M; ++k) {
        c[k] = scan_key_of_k(tau_eff * importance(k), k);
        if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      const double own = ROWS ? row_pot[g][ql] : col_pot[g][ql];
      // m belongs to the in-kernel row: this lane's line, or the line it crosses at k
      constexpr bool kMine = ROWS != COLS_FIRST;
      const double mine = lds.minus_largest[g][ql];
#pragma unroll
      for (int k = 0; k < M; ++k) {
        // (K - m) + (u + v), the same operations in both passes: an entry has one key
        const double other = ROWS ? col_pot[g][k] : row_pot[g][k];
        c[k] = scan_key(fma(tau_eff, importance(k), kMine ? mine : lds.minus_largest[g][k]) + (own + other), k);
        // a few entries at a time: with all their LDS reads in flight the keys no longer fit the registers
        if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  using yes = std::integral_constant<bool, true>;
  using no = std::integral_constant<bool, false>;

  // this lane's row in scan order: the column of every place, four to a register
  unsigned int row_list[M / 4];
  keys(yes{});
  sort_in_lane(c);
#pragma unroll
  for (int r = 0; r < M; r += 4) row_list[r / 4] = index_bytes(c[r], c[r + 1], c[r + 2], c[r + 3]);
  // this lane's column in scan order
  keys(no{});
  sort_in_lane(c);
  wave_sync();

  // From here the space of the importance holds three byte tables per block (rows padded by a word so that a lane per
  // row meets no other in a bank): rank of entry (i, j) within column j, the columns of row i in scan order, the rows
  // of column j in scan order.
  constexpr int LDB = M == 4 ? 4 : M + 4;
  static_assert(3 * M * LDB <= (int)sizeof(lds.imp[0]), "the tables fit where the importance was");
  unsigned char* rank = reinterpret_cast<unsigned char*>(&lds.imp[g][0]);
  unsigned char* columns_of = rank + M * LDB;
  unsigned char* rows_of = columns_of + M * LDB;
#pragma unroll
  for (int r = 0; r < M; ++r) {
    const unsigned int i = (unsigned int)__double2loint(c[r]) & (M - 1);
    rank[i * LDB + ql] = (unsigned char)r;
    if (r % 4 == 3) {
      *reinterpret_cast<unsigned int*>(rows_of + ql * LDB + r - 3) = index_bytes(c[r - 3], c[r - 2], c[r - 1], c[r]);
      *reinterpret_cast<unsigned int*>(columns_of + ql * LDB + r - 3) = row_list[r / 4];
    }
  }
  // lds.rowm[i]: the columns row i holds; lds.colm[j]: the ranks (within column j) of the entries column j holds;
  // lds.colcnt[j]: entries of a higher rank than this one it would turn away
  const mask_t one = 1;
  lds.colm[g][ql] = 0;
  wave_sync();
  mask_t held = 0;
  // (half of the row at a time: with N = M / 2 the other half is neither looked up nor proposed; 32:64 with the early exit 686 -> 680 us,
  // 226 -> 207 registers, and 16:32 no longer spills)
  constexpr int kAtOnce = M == 4 ? M : M / 2;
#pragma unroll
  for (int half = 0; half < M; half += kAtOnce) {
    if (half >= N) break;
    unsigned int cr[kAtOnce];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k)
      cr[k] = rank[ql * LDB + ((row_list[(half + k) / 4] >> (8 * (k % 4))) & 0xFFu)] & (unsigned)(M - 1);
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k)
      if (half + k < N) {
        const unsigned int j = (row_list[(half + k) / 4] >> (8 * (k % 4))) & 0xFFu;
        atomicOr(&lds.colm[g][j], one << cr[k]);
        held |= one << j;
      }
  }
  lds.rowm[g][ql] = held;
  int next = N;  // the first place of its order this row has not proposed
  for (;;) {
    wave_sync();
    const mask_t h = lds.colm[g][ql];
    mask_t surplus = 0;
    int limit = M;
    if (mask_popc(h) >= N) {
      limit = nth_set_bit<M>(h, N);
      surplus = h & ~(((one << limit) << 1) - 1);
      lds.colm[g][ql] = h ^ surplus;
    }
    lds.colcnt[g][ql] = (unsigned)limit;
    while (surplus != 0) {
      const int at = sizeof(mask_t) == 8 ? __ffsll((long long)surplus) - 1 : __ffs((int)surplus) - 1;
      surplus &= surplus - 1;
      atomicAnd(&lds.rowm[g][rows_of[ql * LDB + at]], ~(one << ql));
    }
    wave_sync();
    held = lds.rowm[g][ql];
    int lacks = p.simple ? 0 : N - mask_popc(held);
    bool proposed = false;
    while (lacks > 0 && next < M) {
      // four places of the row's order per LDS round trip (a row that stays short looks at all that is left of it)
      const int first = next & ~3;
      const unsigned int four = *reinterpret_cast<const unsigned int*>(columns_of + ql * LDB + first);
      unsigned int at[4], below[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned int j = (four >> (8 * k)) & 0xFFu;
        at[k] = rank[ql * LDB + j];
        below[k] = lds.colcnt[g][j];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (first + k >= next && lacks > 0) {
          next = first + k + 1;
          if (at[k] < below[k]) {
            const unsigned int j = (four >> (8 * k)) & 0xFFu;
            atomicOr(&lds.colm[g][j], one << at[k]);
            held |= one << j;
            --lacks;
            proposed = true;
          }
        }
    }
    lds.rowm[g][ql] = held;
    if (!__any(proposed)) break;
  }
  wave_sync();
  local_search_and_write<M, LPB, ASCENDING>(p, e, blk, active, r0, c0, lane, lds);
}

// The stand-alone kernel: 64/M blocks per wave, one wave per workgroup; the potentials come from the workspace.
// Bound by instruction issue: 3 650 vector instructions per wave (M = 32, the swaps of 16:32 4096x14336 included), of which the
// two sorts are 764 and the keys 384; 2 060 up to the first proposals.  57 344 blocks of 16:32: 0.198 ms, where the sort across
// lanes (0.20 ms of the iteration kernel), the scan kernel (0.077 ms) and the swap kernel (0.104 ms) took 0.38 ms; 57 344 of
// 32:64: 0.97-1.15 ms (7 100 vector instructions per wave, two waves per SIMD: 207 registers, 19 KB of LDS).  None spill.
template <int M, bool ZERO_T>
__global__ __launch_bounds__(kWave, M <= 32 ? 4 : 2) void round_kernel(Batch batch) {
  constexpr int G = kWave / M;
  __shared__ RoundingLds<M, G> lds;
  __shared__ double row_pot[ZERO_T ? 1 : G][M], col_pot[ZERO_T ? 1 : G][M];
  const int which = find_problem(batch, blockIdx.x);
  const BatchEntry& e = batch.e[which];
  const DevProblem p = e.p;
  const int lane = threadIdx.x, g = lane / M, ql = lane % M;
  const unsigned int group = blockIdx.x - batch.first[which];
  int64_t blk = (int64_t)group * G + g;
  const bool active = blk < p.nblocks;
  if (!active) blk = p.nblocks - 1;  // idle groups shadow the last block and write nothing
  const BlockAt at = block_at(p, blk, M);
  double tau_eff;
  if constexpr (ZERO_T) {
    tau_eff = tau_eff_of(e);
    if (e.tau_eff_out && group == 0 && lane == 0) *e.tau_eff_out = tau_eff;
    if (active && ql == 0 && e.iters_done_out) e.iters_done_out[blk] = 0;
  } else {
    tau_eff = e.hdr->tau_eff;
    const BlockPotentials<M>* src = static_cast<const BlockPotentials<M>*>(e.potentials) + blk;
    const double of_row = src->u[ql], of_col = src->v[ql];
    lds.minus_largest[g][ql] = -(double)normalisers_of<M>(e, blk)[ql];
    row_pot[g][ql] = p.transpose ? of_col : of_row;
    col_pot[g][ql] = p.transpose ? of_row : of_col;
  }
  if (!ZERO_T && p.transpose)
    round_blocks<M, M, ZERO_T, true, true>(p, e, blk, active, at.r0, at.c0, lane, tau_eff, row_pot, col_pot, lds);
  else
    round_blocks<M, M, ZERO_T, false, true>(p, e, blk, active, at.r0, at.c0, lane, tau_eff, row_pot, col_pot, lds);
}

}  // namespace tsenor_dev
