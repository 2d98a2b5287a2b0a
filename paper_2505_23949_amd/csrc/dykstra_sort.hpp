// Tile load and Algorithm 1 (Dykstra iterations), one kernel.  For M >= 8 on the large tiles it leaves the potentials of
// every block for round_kernel; for M = 4 there the greedy selection follows; on the small tiles the whole of Algorithm 2
// does.
//
// How Algorithm 1 is evaluated.  With A = log S + log Q, the cap step (lines 5-6) gives
// log S = min(A, 0) and log Q = max(A, 0) after every iteration, and one iteration adds a row term
// and a column term to A.  So A = K + f_i + g_j with K = tau_eff * importance: the whole Dykstra
// state of a block is K plus 2M potentials.  With kappa_ij = exp(K_ij - max_j K_ij) (the first row
// scaling makes a per-row factor of the start irrelevant) and the scalings U_i = exp(f_i), V_j = exp(g_j)
// one iteration is
//     e_ij = min(kappa_ij U_i V_j, 1);   R_i = N / sum_j e_ij;   C_j = N / sum_i e_ij R_i;
//     U_i *= R_i;   V_j *= C_j
// which is lines 3-6 of Algorithm 1 in exact arithmetic: the row scaling acts on the plan capped by
// the previous iteration, the column scaling on the row-scaled plan, and the cap with its dual is the
// min(., 1) at the top of the next pass (App. A.2 listing, same order of operations).  The kernel forms
// kappa_ij U_i once per entry and iteration, so an iteration costs four operations per entry - multiply-and-clamp,
// add, fused multiply-add, multiply - and no transcendental.
//
// Precision.  Default: everything in double (MI355X issues fp64 vector operations at 16 lanes/clk/SIMD),
// which reproduces a double-precision reference to ~1e-13.  FAST: the first kWarmIters iterations in
// double, then the loop in fp32 (a shorter instruction, and half the registers: three or four waves per SIMD
// instead of two) on kappa32 = fl32(kappa U V) with fp32 scalings relative to the double ones.  fp32 has 8
// exponent bits, so every kChunk iterations the relative scalings are checked and, when one has drifted past
// 2^+-kDriftBits, they are multiplied into the double ones and kappa32 is rebuilt as
// fl32(exp(K - row max + log U + log V)) from a fresh read of the importance (kappa itself is not kept: the kernel is
// budgeted the registers of the fp32 loop).  Rebuilt entries are clamped to about
// [2^-120, 2^80]; within the drift bound (2^+-80 for a product of a row and a column scaling) a clamped
// entry is still >= 1 (capped) or <= 2^-40 (nothing).
//
// Layout.  A block is spread over LPB = GX*GY lanes as a GY x GX grid of TH x TW register tiles
// (TH = M/GY rows, TW = M/GX columns); a wave holds 64/LPB blocks.  Row sums are reduced across the GX
// lanes of a lane-row by recursive halving (reduce-scatter): after log2(GX) exchange steps every lane
// owns TH/GX complete row sums, computes their reciprocals once, and the results are gathered back the
// same way.  To keep every exchange a fixed set of registers (no selects), register a of lane gx holds
// tile row a ^ (gx << log2(TH/GX)); columns likewise over the GY lanes of a lane-column.
#pragma once
#include <type_traits>

#include "lanes.hpp"
#include "launch.hpp"
#include "problem.hpp"
#include "rounding.hpp"

namespace tsenor_dev {

constexpr double kMinLogKernel = -700.0;  // exp(-700) is still a normal double
constexpr int kWarmIters = 4;             // FAST: iterations done in double before switching to fp32
constexpr int kRowChunks64 = 2;           // M = 64: the 8 x 8 tile is loaded in this many pieces (loads in flight cost registers)
constexpr int kChunk = 8;                 // FAST: iterations between looks for a repetition and range checks of the scalings
constexpr int kRepeatWindow = 24;         // iterations over which a repetition is looked for (RepeatCheck); in double also between looks
constexpr int kRaiseBits = 512;           // kKeep: what goes from a large row scaling into its row of the tile (raise_rows)
constexpr double kRaiseAbove = 0x1p+400;
constexpr double kSmallStep = 0x1p-30;    // increments: factors of an iteration within this of 1 ...
constexpr double kNearCap = 0x1p-20;      // ... no entry of the plan as near to the cap as this ...
constexpr float kIncrementSum = 0x1p-25f; // ... and the sum of the increments before the plan is formed anew
constexpr float kNothingLeft = 0x1p-54f;  // ... and what is left of the iterations when they are as good as done
constexpr int kDriftBits = 40;            // FAST: fold the fp32 scalings back beyond 2^+-kDriftBits
constexpr double kLogFloor32 = -83.0;     // FAST: rebuilt entries are kept within [e^-83, e^55] ~ [2^-120, 2^80]
constexpr double kLogCeil32 = 55.0;


constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// Per-M tiling.  XM[s] / YM[s]: lane masks of the exchange steps along a lane-row / lane-column.
// The top bit of XM[s] is lane bit NX-1-s (mirror masks keep the exchanges on DPP); YM[s] is a single
// lane bit, listed cheapest mechanism first because the first step moves the most registers, or 7: a DPP move that also turns
// round the lanes along the lane-row, in place of one through the LDS crossbar (column_lane; 8:16 4096x4096 844 us a call with
// the crossbar, 828 with it, and with fp32 iterations 531 and 517).
// Small tiles: a finer tiling (more lanes per block, fewer entries per lane) for launches that cannot fill the
// chip anyway: the dependent chain of an iteration is shorter.  Where a tile has fewer rows than the
// lane-row has lanes, the last exchange steps of a reduction have no registers left to split: they add the
// partner's value into the same register instead (both lanes end up owning the same sum).
// kFinestTiles: a 16 x 16 block on a whole wave, for launches that leave SIMDs without a wave even so.
// kFinestOrderTiles: the small tiles of 16 x 16 blocks with their additions in the order of the finest ones.
// SWAPS: exchanges 16 lanes apart by v_permlane swaps (swap_step).  KEEP: form of an iteration in double (dykstra_iteration).
template <int M, int TILES = kLargeTiles>
struct Tiling;
template <>
struct Tiling<4, kLargeTiles> {
  static constexpr int NX = 0, NY = 0;
  static constexpr int XM[1] = {1}, YM[1] = {1};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<8, kLargeTiles> {
  static constexpr int NX = 1, NY = 1;
  static constexpr int XM[1] = {1}, YM[1] = {2};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<16, kLargeTiles> {
  static constexpr int NX = 2, NY = 1;  // 8 lanes per block, 8 x 4 tiles
  static constexpr int XM[2] = {3, 1}, YM[1] = {7};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<32, kLargeTiles> {
  static constexpr int NX = 3, NY = 2;  // 32 lanes per block, 8 x 4 tiles
  static constexpr int XM[3] = {7, 3, 1}, YM[2] = {8, 16};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = false;
};
template <>
struct Tiling<64, kLargeTiles> {
  static constexpr int NX = 3, NY = 3;  // 64 lanes per block, 8 x 8 tiles; too large to hold e as doubles
  static constexpr int XM[3] = {7, 3, 1}, YM[3] = {8, 16, 32};
  static constexpr bool STORE_E = false;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = false;
};
template <>
struct Tiling<4, kSmallTiles> {
  static constexpr int NX = 1, NY = 1;  // 4 lanes per block, 2 x 2 tiles
  static constexpr int XM[1] = {1}, YM[1] = {2};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<8, kSmallTiles> {
  static constexpr int NX = 2, NY = 2;  // 16 lanes per block, 2 x 2 tiles
  static constexpr int XM[2] = {3, 1}, YM[2] = {8, 7};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<16, kSmallTiles> {
  static constexpr int NX = 2, NY = 2;  // 16 lanes per block, 4 x 4 tiles
  static constexpr int XM[2] = {3, 1}, YM[2] = {8, 7};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<16, kFinestTiles> {
  static constexpr int NX = 3, NY = 3;  // 64 lanes per block, 2 x 2 tiles
  static constexpr int XM[3] = {7, 3, 1}, YM[3] = {8, 32, 16};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = true;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<16, kFinestOrderTiles> {
  static constexpr int NX = 2, NY = 2;  // 16 lanes per block, 4 x 4 tiles
  static constexpr int XM[2] = {3, 1}, YM[2] = {8, 4};  // (steps of the finest tiles' lane-columns after their first: 32 and 16)
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};
template <>
struct Tiling<32, kSmallTiles> {
  static constexpr int NX = 3, NY = 3;  // 64 lanes per block, 4 x 4 tiles
  static constexpr int XM[3] = {7, 3, 1}, YM[3] = {8, 16, 32};
  static constexpr bool STORE_E = true;
  static constexpr bool SWAPS = false;
  static constexpr bool KEEP = true;
};

// The exchanges of a wave that has its SIMD to itself (swap_step).  The sums are the same bit for bit: what differs is which
// register a lane holds a column in, and a row sum adds the columns of a lane in pairs.
template <class T>
struct LoneTiling : T {
  static constexpr bool SWAPS = true;
};

// Two layouts of a block that add in the same order, so that a launch may take either.  A sum of two numbers does not depend on
// which of two lanes forms it, so the exchange steps of a reduction are a tree over the rows or columns whatever the layout;
// what has an order is the run of fused multiply-adds down a column inside a lane.  The finer layout (16 x 16: 2 x 2 tiles on
// a wave; 64 x 64: eight rows of one column per lane, team.hpp) starts that run of column c at row r(c) and goes on with rows
// r(c) ^ 1, r(c) ^ 2, ..., since its rows are offset by r.  The coarser layout has columns of different r in a lane.  With one
// offset o for rows and columns both - register a holds row a ^ o, register b column b ^ o, o over all values along a lane-row
// and along a lane-column - the k-th row of the run, k ^ r(c) = k ^ b ^ o, is in register k ^ b: the same in every lane.
// order_run: length of those runs (0: a tiling without such a partner, one run over all rows of the tile).
template <int M, int TILES>
constexpr int order_run() {
  return M == 64 && TILES == kLargeTiles ? 8 : M == 16 && TILES == kFinestOrderTiles ? 2 : 0;
}
// Sum of the capped entries of a tile row in the finer layout's order: over the lanes that differ by 7, 3, 1 (64 x 64), or the
// two columns of a lane and then the next lane (16 x 16).
template <int RUN, class real, int TW, int H = TW / 2>
__device__ __forceinline__ real row_tree(real (&s)[TW]) {
  if constexpr (H >= 1) {
#pragma unroll
    for (int b = 0; b < H; ++b) s[b] += s[b ^ (RUN == TW ? 2 * H - 1 : H)];
    return row_tree<RUN, real, TW, H / 2>(s);
  } else {
    return s[0];
  }
}
// in-kernel column of a block that tile column `b` (its register with the lane's offset taken off) of lane-column gx is
template <int M, int TILES>
__device__ __forceinline__ int column_in_block(int gx, int b) {  // (gx: of column_lane)
  if constexpr (M == 16 && TILES == kFinestOrderTiles) {
    // the column pairs of two finest lanes 7 apart (a step of their row reduction), the pair in bit 0
    return 2 * (b & 1 ? gx ^ 7 : gx) + (b >> 1);
  } else {
    return gx * (M >> Tiling<M, TILES>::NX) + b;
  }
}

// Lane-column of a lane for its columns.  A step that pairs lanes 7 apart along a lane-column also turns round the order of
// four lanes along the lane-row: so does the assignment of columns in every other lane-row, and the two lanes hold the same ones.
template <class T>
__device__ __forceinline__ int column_lane(int gx, int q) {
  bool turned = false;
#pragma unroll
  for (int s = 0; s < T::NY; ++s) turned |= T::YM[s] == 7;
  return turned && (q & 4) ? gx ^ 3 : gx;
}

// Whether the last iterations of a wave are done in increments (iterate_increments).  Where a launch may take two layouts of a block
// whose waves hold other numbers of blocks (order_run) the results would differ.  4 x 4 blocks have 64 or 16 to a wave, too many to
// converge together; on the 8-wide small tiles it gained nothing (the look 1 %).
template <int M, int TILES>
constexpr bool increments_at_the_end() {
  return (TILES == kLargeTiles && (M == 8 || M == 16 || M == 32)) || (TILES == kSmallTiles && M >= 16);
}

// whether any step along a lane-column swaps registers, so that a lane's first ones need not be of the columns it owns
template <class T, int S = 0>
constexpr bool kSwaps = S < T::NY && (T::YM[S < T::NY ? S : 0] == 32 || (T::SWAPS && T::YM[S < T::NY ? S : 0] == 16) ||
                                      (S + 1 < T::NY && kSwaps<T, (S + 1 < T::NY ? S + 1 : S)>));

// registers a lane owns after a reduce-scatter of `count` values over 2^steps lanes (at least one)
constexpr int owned(int count, int steps) { return (count >> steps) > 0 ? (count >> steps) : 1; }
// lane coordinate -> register offset of the row mapping: the top log2(TH) bits of gx if the tile has fewer
// rows than the lane-row has lanes, gx shifted up otherwise
constexpr int shift_lane(int x, int sh) { return sh >= 0 ? x << sh : x >> -sh; }

// 1/d from the hardware estimate x0.  A scaling factor is applied once and the sums of the next iteration see
// its error, so errors of the reciprocal do not accumulate over the iterations, while every refinement step sits
// in the dependent chain of each of them.  Double: x0 has ~24 bits; with e = 1 - d x0 one Newton step
// x0 (1 + e) leaves e^2 ~ 2^-48, two fused operations.  Float: the estimate itself (1 ulp).
__device__ __forceinline__ double fast_rcp(double d) {
  const double x = __builtin_amdgcn_rcp(d);
  return fma(fma(-d, x, 1.0), x, x);
}
// n/d the same way; the multiplication stands beside the refinement instead of behind it
__device__ __forceinline__ double fast_div(double n, double d) {
  const double x = __builtin_amdgcn_rcp(d), nx = n * x;
  return fma(fma(-d, x, 1.0), nx, nx);
}
__device__ __forceinline__ float fast_rcp(float d) { return __builtin_amdgcn_rcpf(d); }
// n/d to the last bit or two from a quotient q of the above
__device__ __forceinline__ double refined(double q, double n, double d) { return fma(fma(-d, q, n), __builtin_amdgcn_rcp(d), q); }
// exp(x) for |x| <= 708, below 1 ulp of error: e^x = 2^n e^r with |r| <= ln2 / 2 (n by the addition that leaves it in the low word),
// e^r = 1 + r + r^2 q(r), q the polynomial of degree 9 that minimises the largest relative error (3.6e-18, Remez exchange).  16
// instructions; the library's exp() spends four more on results that leave the range of a double, which no entry of a tile does.
__device__ __forceinline__ double exp_in_range(double x) {
  constexpr double kLog2e = 0x1.71547652b82fep+0, kLn2Hi = 0x1.62e42fefa39efp-1, kLn2Lo = 0x1.abc9e3b39803fp-56, kRound = 0x1.8p+52;
  const double shifted = fma(x, kLog2e, kRound), n = shifted - kRound;
  const double r = fma(n, -kLn2Lo, fma(n, -kLn2Hi, x));
  double q = 0x1.ad7f6b5dc2ef6p-26;
  q = fma(q, r, 0x1.28ad72bf7e407p-22);
  q = fma(q, r, 0x1.71df255430ed3p-19);
  q = fma(q, r, 0x1.a0199a0c78972p-16);
  q = fma(q, r, 0x1.a01a012a57064p-13);
  q = fma(q, r, 0x1.6c16c1842a09fp-10);
  q = fma(q, r, 0x1.1111111127be6p-7);
  q = fma(q, r, 0x1.555555555087dp-5);
  q = fma(q, r, 0x1.55555555554fap-3);
  q = fma(q, r, 0x1.000000000000ap-1);
  q = fma(q, r, 1.0);
  q = fma(q, r, 1.0);
  return __builtin_amdgcn_ldexp(q, __double2loint(shifted));
}
__device__ __forceinline__ double clamp01(double x) { return fmin(fmax(x, 0.0), 1.0); }
__device__ __forceinline__ float clamp01(float x) { return fminf(fmaxf(x, 0.0f), 1.0f); }
__device__ __forceinline__ double vmax(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float vmax(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double vfma(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float vfma(float a, float b, float c) { return fmaf(a, b, c); }

// Recursive halving over the lanes of a lane-row.  v[0..TH): partial sums, register a <-> tile row
// a ^ shift_lane(gx, SH).  Afterwards v[0 .. owned(TH, NX)) hold complete sums.
template <class T, class real, int TH, int S = 0>
__device__ __forceinline__ void reduce_scatter_x(real (&v)[TH]) {
  if constexpr (S < T::NX) {
    constexpr int SH = ilog2(TH) - T::NX;
    constexpr int h = TH >> (S + 1);
    if constexpr (h >= 1) {
      constexpr int am = shift_lane(T::XM[S], SH) & (2 * h - 1);  // register index of the partner's matching value
#pragma unroll
      for (int a = 0; a < h; ++a) v[a] += lane_xor<T::XM[S]>(v[a ^ am]);
    } else {
      v[0] += lane_xor<T::XM[S]>(v[0]);  // no registers left to split: both lanes keep the sum
    }
    reduce_scatter_x<T, real, TH, S + 1>(v);
  }
}
template <class T, class real, int TH, int S = T::NX - 1>
__device__ __forceinline__ void all_gather_x(real (&v)[TH]) {
  if constexpr (S >= 0) {
    constexpr int SH = ilog2(TH) - T::NX;
    constexpr int h = TH >> (S + 1);
    if constexpr (h >= 1) {
      constexpr int am = shift_lane(T::XM[S], SH) & (2 * h - 1);
#pragma unroll
      for (int a = 0; a < h; ++a) v[a ^ am] = lane_xor<T::XM[S]>(v[a]);
    }
    all_gather_x<T, real, TH, S - 1>(v);
  }
}
// The smallest float not below x >= 0.  The normaliser of a row is to be such a float for its largest K, and no larger one: where
// K itself is near 2^32 a step of floats is 512 of the 700 that a row may spread.  Taken once per lane and row, of the
// largest K it holds (5 instructions; rounding every K upwards took 14 per entry, a third of the 64-wide prologue).
__device__ __forceinline__ float round_up(double x) {
  const float f = (float)x;
  return (double)f < x ? __uint_as_float(__float_as_uint(f) + 1u) : f;
}
// Maximum over the lanes of a lane-row of a value per tile row (all TH registers, butterfly): afterwards
// every lane holds the maximum of each of its tile rows.
template <class T, int TH, int S = 0>
__device__ __forceinline__ void all_reduce_max_x(float (&v)[TH]) {
  if constexpr (S < T::NX) {
    constexpr int SH = ilog2(TH) - T::NX;
    constexpr int am = shift_lane(T::XM[S], SH) & (TH - 1);
    float o[TH];
#pragma unroll
    for (int a = 0; a < TH; ++a) o[a] = lane_xor<T::XM[S]>(v[a ^ am]);
#pragma unroll
    for (int a = 0; a < TH; ++a) v[a] = fmaxf(v[a], o[a]);
    all_reduce_max_x<T, TH, S + 1>(v);
  }
}

// Whether a step along a lane-column is a v_permlane swap of two registers instead of a move: both lanes of a pair then hold
// the same columns in the same registers, the halving step keeps one of them (or the sum of one, in both) in each lane, and no
// lane selects.
// 32 lanes apart always (64 x 64: 8 of 382 instructions per iteration fewer in double, 4 of 283 in fp32); 16 lanes
// apart only where a wave has its SIMD to itself and waits out the latency of the LDS crossbar (4096x32 16:32: 99.6 us a call
// through the crossbar, 94.4 with swaps; with two waves on a SIMD 148.3 and 151.2), and for the finest tiles, whose steps
// have no register to split (512x640 8:16, two waves on some SIMDs: 80.0 and 76.3).
template <class T, int S>
constexpr bool swap_step() {
  return T::YM[S] == 32 || (T::SWAPS && T::YM[S] == 16);
}
// The same over the lanes of a lane-column; step s pairs lanes that differ by YM[s].
template <class T, class real, int TW, int S = 0>
__device__ __forceinline__ void reduce_scatter_y(real (&v)[TW]) {
  if constexpr (S < T::NY) {
    constexpr int h = TW >> (S + 1);
    if constexpr (swap_step<T, S>()) {
      if constexpr (h >= 1) {
#pragma unroll
        for (int b = 0; b < h; ++b) v[b] = swap_sum<T::YM[S]>(v[b], v[b + h]);
      } else {
        v[0] = swap_sum<T::YM[S]>(v[0], v[0]);
      }
    } else if constexpr (h >= 1) {
#pragma unroll
      for (int b = 0; b < h; ++b) v[b] += lane_xor<T::YM[S]>(v[b + h]);
    } else {
      v[0] += lane_xor<T::YM[S]>(v[0]);
    }
    reduce_scatter_y<T, real, TW, S + 1>(v);
  }
}
// (steps S down to LAST; the default is the whole gather)
template <class T, class real, int TW, int S = T::NY - 1, int LAST = 0>
__device__ __forceinline__ void all_gather_y(real (&v)[TW]) {
  if constexpr (S >= LAST && S >= 0) {
    constexpr int h = TW >> (S + 1);
    if constexpr (h >= 1) {
#pragma unroll
      for (int b = 0; b < h; ++b) {
        if constexpr (swap_step<T, S>())
          swap_spread<T::YM[S]>(v[b], v[b + h]);
        else
          v[b + h] = lane_xor<T::YM[S]>(v[b]);
      }
    }
    all_gather_y<T, real, TW, S - 1, LAST>(v);
  }
}
// the lowest step of all_gather_y whose move goes through the LDS crossbar (0: none does, or it is the last one)
template <class T, int TW, int S = 0>
constexpr int gather_split_y() {
  if constexpr (S < T::NY) {
    constexpr int m = T::YM[S];
    constexpr bool crossbar = m < 32 && m != 1 && m != 2 && m != 3 && m != 7 && m != 15 && m != 8;
    if constexpr (crossbar && (TW >> (S + 1)) >= 1)
      return S;
    else
      return gather_split_y<T, TW, S + 1>();
  } else {
    return 0;
  }
}
// register offset of a lane along y: lane bit s of the lane-column set <-> register bit log2(TW >> (s+1)).  OWN: of the columns it
// owns after a reduction; else of the columns in its tile, for which the pairs of a swap step agree.
template <class T, int TW, bool OWN, int S = 0>
__device__ __forceinline__ int reg_xor_y(int q) {
  if constexpr (S < T::NY) {
    constexpr int bit = T::YM[S] == 7 ? 4 : T::YM[S];  // (xor 7: the lane-column's part of the mask)
    const int mine = !OWN && swap_step<T, S>() ? 0 : (q & bit) ? (TW >> (S + 1)) : 0;
    return mine | reg_xor_y<T, TW, OWN, S + 1>(q);
  } else {
    return 0;
  }
}

// How factors and scalings of the rows go round: moves between lanes; both through LDS; factors by moves, scalings through LDS
enum Gather { kLanesOnly, kRowsInLds, kScalingsInLds };

// An iteration alternates between two kinds of code: long runs of independent per-entry arithmetic, and the
// short dependent chains between them (exchange steps of a reduction, reciprocal, gather of the result) on
// which the next run waits.  A wave raises its priority for the chains, so that the SIMD issues their few
// instructions ahead of another wave's long run instead of behind it: with equal priorities the waves of a
// SIMD fell into step and stalled together (measured: 11-16 % of the fp32 loop, 1-2 % of the double one).
// A wave alone on its SIMD has nobody to be ahead of, and every instruction of its own counts (LONE: 512x512 2:4 31.0 us a call
// with the six instructions of an iteration, 28.1 without; with two waves on a SIMD 52.0 and 55.5).  That is so while its stream is
// the only one: where launches of several streams share the SIMDs, the priorities would gain (16:32, 812 blocks, T = 300: one
// stream 96 us without, 101 with; four streams 290 and 285; 506 blocks on four streams 200 and 191).  The iterations in fp32 keep
// them: alone they cost a lone wave 2-3 %, with two to four streams 4-14 % are lost without (64 x 64, 306 blocks, T = 300: one stream
// 250 us without, 254 with; four streams 368 and 317; 4 x 4, 65 024 blocks 82 and 85, four streams 220 and 210).  (A fixed
// priority for every wave, by its slot on the SIMD, is worse than none: the last ones wait for the others to end.)
template <bool LONE = false>
__device__ __forceinline__ void chain_phase(bool on) {
  if constexpr (LONE) return;
  if (on)
    __builtin_amdgcn_s_setprio(1);
  else
    __builtin_amdgcn_s_setprio(0);
}

// One iteration of Algorithm 1 (lines 3-6) in double on the register tile of this lane.  Every entry costs a multiply with its
// column scaling; where the row scalings are is the FORM:
//   kKeep: kap stays as it is.  x holds kappa_ij U_i when an iteration begins, the capped entries after the row pass, and is
//     formed anew from kap at the end.  So the state is the scalings alone, which RepeatCheck relies on, and no rounding
//     accumulates in the tile.  U: the scalings of all rows of the tile.
//   kFold: the row scalings are folded into kap as they are found, U holds the owned rows only; x takes the capped entries.
//     32-wide large tiles: gathering U besides the factors through LDS made their loop 3 % slower.
//   kRecompute: the same for tiles too large to be held twice (no x): the capped entries are recomputed in the column pass
//     from an opaque copy of V (without the copy the compiler keeps the row pass's values alive and spills them).
// No sum needs a floor.  The first row sum holds the row's largest entry, and with every entry at least e^kMinLogKernel and every
// row factor at least N/M the first column sum is at least N e^kMinLogKernel, whose reciprocal is finite; later ones see lines
// that were scaled to N and then changed by factors of at least 1/M on either side.  (A floor as an addend, 1e-300 in every entry,
// took the place of the smallest entries: with rows that spread over 690 the plan was off by 1e-3, by 1e-7 over 680.)
// ADAPT (early exit): `frozen` lanes apply factors of exactly 1 (their block has stopped; its state no longer
// changes), and the largest |factor - 1| among the rows and columns this lane owns is returned.
// RUN: order_run() of the tiling.  LONE: no other wave shares the SIMD (chain_phase).
// REFINED: factors without the 2^-48 of fast_div (iterate_increments).
struct NoTile {};
// a count that is the same in all lanes, where the compiler cannot tell (in a vector register it costs the loop an instruction or two)
__device__ __forceinline__ int of_wave(int n) { return __builtin_amdgcn_readfirstlane(n); }
enum Form { kRecompute, kFold, kKeep };
template <class T, Form FORM, Gather GATHER = kLanesOnly, bool ADAPT = false, int RUN = 0, bool LONE = false, bool REFINED = false,
          class Tile, int TH, int TW, int NU>
__device__ __forceinline__ double dykstra_iteration(double (&kap)[TH][TW], Tile& x, double (&U)[NU], double (&V)[TW],
                                                    double (&Vown)[owned(TW, T::NY)], double Nd, double* xr = nullptr, int rx = 0,
                                                    bool frozen = false) {
  constexpr bool KEEP = FORM == kKeep, STORE = FORM != kRecompute;
  double worst = 0;
  constexpr int OWN_R = owned(TH, T::NX), OWN_C = owned(TW, T::NY);
  static_assert(NU == (KEEP ? TH : OWN_R), "scalings of every row, or of the owned ones");
  // Where no lane multiplies a scaling of another's row, the factors that go round are 1 / row sum, without their N: the column
  // sums then come out divided by N, and their reciprocals are the column factors.  (Not on the small tiles: M = 4 on the
  // large ones is the only block without lanes to exchange with.)
  constexpr bool BARE = KEEP && (GATHER != kLanesOnly || OWN_R == TH);
  double R[TH], C[TW];
  // projection onto C1 (line 3) of the plan capped by the previous iteration
  if constexpr (KEEP && RUN == 0) {
    constexpr bool PAIRS = T::NY == 3;
    // (column by column: the scalings of the owned columns are there before the gathered ones)
#pragma unroll
    for (int b = 0; b < TW; ++b)
#pragma unroll
      for (int a = 0; a < TH; ++a) {
        x[a][b] = clamp01(x[a][b] * V[b]);
        if constexpr (!PAIRS) R[a] = b == 0 ? x[a][b] : R[a] + x[a][b];  // (0 + x is not a no-op for the compiler)
      }
    if constexpr (PAIRS) {
      // in pairs: a shorter chain, and the same sum whatever the lane's offset of the columns is (see LoneTiling)
#pragma unroll
      for (int a = 0; a < TH; ++a) {
        double s[TW];
#pragma unroll
        for (int b = 0; b < TW; ++b) s[b] = x[a][b];
#pragma unroll
        for (int h = 1; h < TW; h *= 2)
#pragma unroll
          for (int b = 0; b < TW; b += 2 * h) s[b] += s[b + h];
        R[a] = s[0];
      }
    }
  } else {
#pragma unroll
    for (int a = 0; a < TH; ++a) {
      double s = 0, leaf[RUN ? TW : 1];
#pragma unroll
      for (int b = 0; b < TW; ++b) {
        double ev;
        if constexpr (KEEP)
          ev = clamp01(x[a][b] * V[b]);
        else
          ev = clamp01(kap[a][b] * V[b]);
        if constexpr (STORE) x[a][b] = ev;
        if constexpr (RUN > 0)
          leaf[b] = ev;
        else
          s = b == 0 ? ev : s + ev;
      }
      if constexpr (RUN > 0) s = row_tree<RUN>(leaf);
      R[a] = s;
    }
  }
  chain_phase<LONE>(true);
  reduce_scatter_x<T, double, TH>(R);
#pragma unroll
  for (int a = 0; a < OWN_R; ++a) {
    double factor;
    const double sum = R[a];
    if constexpr (BARE) {
      R[a] = fast_rcp(sum);
      if constexpr (REFINED) R[a] = refined(R[a], 1.0, sum);
      factor = Nd * R[a];
    } else {
      factor = fast_div(Nd, sum);
      if constexpr (REFINED) factor = refined(factor, Nd, sum);
    }
    if constexpr (ADAPT) {
      worst = vmax(worst, fabs(factor - 1.0));
      factor = frozen ? 1.0 : factor;
    }
    U[a] *= factor;
    if constexpr (!BARE) R[a] = factor;
  }
  if constexpr (GATHER == kRowsInLds) {
    // the owner of a row leaves its factor in LDS and every lane of the lane-row picks up all TH of them:
    // LDS instructions instead of vector-ALU moves.  The lanes of a wave run in lock step, so the exchange
    // needs no barrier, only that the compiler keeps the accesses where they are.
    static_assert(!KEEP, "");
#pragma unroll
    for (int a = 0; a < OWN_R; ++a) xr[a ^ rx] = R[a];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int a = OWN_R; a < TH; ++a) R[a] = xr[a ^ rx];  // (the owned rows' factors are at hand)
    asm volatile("" ::: "memory");
  } else {
    all_gather_x<T, double, TH>(R);
    if constexpr (GATHER == kScalingsInLds) {
      // the factors on DPP moves, for the column pass waits for them; the scalings, which it does not need, through LDS
      static_assert(KEEP && OWN_R % 2 == 0, "pairs of rows");
#pragma unroll
      for (int a = 0; a < OWN_R; a += 2) *reinterpret_cast<double2*>(xr + (a ^ rx)) = make_double2(U[a], U[a + 1]);
      asm volatile("" ::: "memory");
    } else if constexpr (KEEP) {
#pragma unroll
      for (int a = OWN_R; a < TH; ++a) U[a] *= R[a];
    }
  }
  chain_phase<LONE>(false);
  // projection onto C2 (line 4)
  double Vc[TW];
#pragma unroll
  for (int b = 0; b < TW; ++b) {
    Vc[b] = V[b];
    if constexpr (!STORE) asm volatile("" : "+v"(Vc[b]));
  }
#pragma unroll
  for (int b = 0; b < TW; ++b) {
    const auto entry = [&](int a) {
      if constexpr (STORE)
        return x[a][b];
      else
        return clamp01(kap[a][b] * Vc[b]);
    };
    double s = 0;
    if constexpr (RUN == 0) {
#pragma unroll
      for (int a = 0; a < TH; ++a) s = a == 0 ? entry(a) * R[a] : fma(entry(a), R[a], s);
    } else {
      static_assert(TH <= 2 * RUN, "at most two runs");
#pragma unroll
      for (int a0 = 0; a0 < TH; a0 += RUN) {
        double run = 0;
#pragma unroll
        for (int k = 0; k < RUN; ++k) {
          const int a = a0 + (k ^ (b % RUN));
          run = k == 0 ? entry(a) * R[a] : fma(entry(a), R[a], run);
        }
        s = a0 == 0 ? run : s + run;
      }
    }
    C[b] = s;
  }
  if constexpr (GATHER == kScalingsInLds) {
#pragma unroll
    for (int a = OWN_R; a < TH; a += 2) {
      const double2 u = *reinterpret_cast<const double2*>(xr + (a ^ rx));
      U[a] = u.x;
      U[a + 1] = u.y;
    }
    asm volatile("" ::: "memory");
  }
  chain_phase<LONE>(true);
  reduce_scatter_y<T, double, TW>(C);
#pragma unroll
  for (int b = 0; b < OWN_C; ++b) {
    const double sum = C[b];
    C[b] = BARE ? fast_rcp(sum) : fast_div(Nd, sum);
    if constexpr (REFINED) C[b] = refined(C[b], BARE ? 1.0 : Nd, sum);
    if constexpr (ADAPT) {
      worst = vmax(worst, fabs(C[b] - 1.0));
      C[b] = frozen ? 1.0 : C[b];
    }
  }
  // the owner of a column applies its factor and the new scalings (not the factors) are gathered: every lane
  // would have formed the same products
#pragma unroll
  for (int b = 0; b < OWN_C; ++b) V[b] = Vown[b] *= C[b];
  // the steps of the gather down to the last one that goes through the LDS crossbar are issued before the
  // rescaling of the tile, the rest after it: the tile's multiplies cover the latency of those moves
  constexpr int SPLIT = gather_split_y<T, TW>();
  all_gather_y<T, double, TW, T::NY - 1, SPLIT>(V);
  chain_phase<LONE>(false);
  if constexpr (SPLIT > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < TH; ++a)
#pragma unroll
    for (int b = 0; b < TW; ++b) {
      if constexpr (KEEP)
        x[a][b] = kap[a][b] * U[a];
      else
        kap[a][b] *= R[a];
    }
  if constexpr (SPLIT > 0) {
    __builtin_amdgcn_sched_barrier(0);
    all_gather_y<T, double, TW, SPLIT - 1>(V);
  }
  // lines 5-6 (cap and dual update) are the clamp at the top of the next pass
  return worst;
}

// The end of the iterations in double, in increments.  Once every factor of an iteration is within kSmallStep of 1 and no entry of
// the plan is within kNearCap of the cap, an entry stays on its side of it for as long as the scalings move by less than that, and
// an iteration is a linear map of the relative changes rho_i, gamma_j that the last one made to U_i and V_j (p: the plan where it
// is below the cap, n_i and m_j the entries at the cap in row i and column j):
//     rho'_i  = (n_i rho_i - sum_p p_ij gamma_j) / N
//     gamma'_j = (m_j gamma_j - sum_p p_ij rho'_i - sum_cap (rho'_i - rho_i)) / N
// up to their squares, 2^-60.  The increments are iterated in fp32, a relative error of 2^-24 of changes below 2^-30; eight of them at a
// time are summed in fp32, the rest in double, and those sums go into the double scalings.  An error of the iteration they start from
// is in all of them: a factor of fast_div carries 2^-48, which 1 / (1 - lambda) iterations of a slow block take up where fresh errors of
// as many iterations in double would partly cancel.  So that one has factors of 2^-52 (`refined`).
// When the iterations that are left, were each to change the plan by as much as the last one did, add up to less than kNothingLeft, all
// are done.  That the changes do not grow: each third of an iteration minimises a convex function (the dual of the projection problem)
// over the row, the column or the cap's potentials, so that on a fixed side of the cap changes of the potentials go through the three
// orthogonal projections of Gauss-Seidel in the norm of its second derivative, which at the end of an iteration is that of the plan,
// E^2 = sum p_ij (rho_i + gamma_j)^2 over the entries below the cap.  E does not grow (random plans and changes: ratios up to 0.9998),
// and an entry changes by sqrt(p_ij) E at most.  E <= M times the largest sqrt(p_ij) |rho_i + gamma_j|, and sqrt(N M) times the largest
// |rho_i + gamma_j|: 2^-49 in the plan where M = 32 at the very most.  An entry above the cap does not count in E and may move on while
// the plan stands still (a block of two parts that entries near 2^-36 connect: 2^-39 per iteration): it must not get to the cap.
// 96 plain fp32 instructions per lane of a 32 x 32 block for the 120 of an iteration in double, and exchanges of one instruction
// instead of three: 115 at 2.5-4 cycles where an iteration in double has 162 at 4.  Calls before / with it (us): 16:32 4096x14336
// bf16 Wanda-style, T = 300, 2792 / 2515; 8:16 3280x12832 Wanda-style tau = 0.02 2199 / 1276; 4:8 4096x4096 student-t 537 / 326; 8:16
// 1072x2928 with its plan, small tiles, 198 / 178; 16:32 1600x1920 student-t, T = 500, small tiles, 176 / 117; normal weights, which never
// come so near, 842 / 841 (8:16), 2535 / 2548 (4:8) and 143 / 145 (16:32 1088x1472, small tiles).
// Error of the plan (2-norm) against 80-bit iterations, relative to that of iterations in double to the end (8, 16 and 32 wide on the
// tilings that do this, K up to 10, 40 and 100, T = 100 to 500, three distributions): 0.34 on average and at most 1.06, where no increment
// came or the rounding of the entries' logarithms is what there is, 5e-16; T = 30 000 on 8 x 8 normal blocks 0.16.  (With sums in fp32 and factors of fast_div before them 0.97 and, T = 30 000, 6.5.)
// The first condition: no scaling of a wave has moved by more than that from what it was, U_before and V_before.
template <int OWN_R, int OWN_C, int NU>
__device__ __forceinline__ bool hardly_moves(const double (&U)[NU], const double (&Vown)[OWN_C], const double (&U_before)[OWN_R],
                                             const double (&V_before)[OWN_C]) {
  bool moves = false;
#pragma unroll
  for (int a = 0; a < OWN_R; ++a) moves |= !(fabs(U[a] - U_before[a]) <= kSmallStep * U_before[a]);
#pragma unroll
  for (int b = 0; b < OWN_C; ++b) moves |= !(fabs(Vown[b] - V_before[b]) <= kSmallStep * V_before[b]);
  return !__any(moves);
}
// The second: no entry of the plan is beside the cap (from an opaque copy of V: the products of the look are not kept for the iteration
// that follows).
template <Form FORM, class Tile, int TH, int TW>
__device__ __forceinline__ bool away_from_cap(const double (&kap)[TH][TW], const Tile& x, const double (&V)[TW]) {
  bool near = false;
  double Vc[TW];
#pragma unroll
  for (int b = 0; b < TW; ++b) {
    Vc[b] = V[b];
    asm volatile("" : "+v"(Vc[b]));
  }
#pragma unroll
  for (int a = 0; a < TH; ++a) {
#pragma unroll
    for (int b = 0; b < TW; ++b) near |= !(fabs((FORM == kKeep ? x[a][b] : kap[a][b]) * Vc[b] - 1.0) > kNearCap);
    __builtin_amdgcn_sched_barrier(0);
  }
  return !__any(near);
}
// The iterations behind the t that are done, U_before and V_before the scalings before the last of them, for which both hold.
// Returns the number of iterations done; if that is less than `iters` the state is that after them.
template <class T, Form FORM, bool LDS, bool ADAPT, int LPB, bool LONE, class Tile, class Freeze, int TH, int TW, int NU>
__device__ __forceinline__ int iterate_increments(double (&kap)[TH][TW], Tile& x, double (&U)[NU], double (&V)[TW],
                                                  double (&Vown)[owned(TW, T::NY)], const double (&U_before)[owned(TH, T::NX)],
                                                  const double (&V_before)[owned(TW, T::NY)], int N, int t, int iters, double tol,
                                                  float2* xr, int rx, const bool& frozen, Freeze& freeze_if) {
  constexpr int OWN_R = owned(TH, T::NX), OWN_C = owned(TW, T::NY);
  static_assert(FORM != kRecompute, "the increments take the registers of the capped entries");
  // the plan and the entries at the cap, over N
  const float inv = 1.0f / (float)N;
  float p[TH][TW], c[TH][TW];
#pragma unroll
  for (int a = 0; a < TH; ++a) {
#pragma unroll
    for (int b = 0; b < TW; ++b) {
      const double entry = (FORM == kKeep ? x[a][b] : kap[a][b]) * V[b];
      const bool at_cap = entry > 1.0;
      p[a][b] = at_cap ? 0.0f : (float)entry * inv;
      c[a][b] = at_cap ? inv : 0.0f;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  float rho[TH], gamma[TW], rows_at_cap[TH], cols_at_cap[TW];
#pragma unroll
  for (int a = 0; a < TH; ++a) {
    rows_at_cap[a] = c[a][0];
#pragma unroll
    for (int b = 1; b < TW; ++b) rows_at_cap[a] += c[a][b];
  }
#pragma unroll
  for (int b = 0; b < TW; ++b) {
    cols_at_cap[b] = c[0][b];
#pragma unroll
    for (int a = 1; a < TH; ++a) cols_at_cap[b] += c[a][b];
  }
  reduce_scatter_x<T, float, TH>(rows_at_cap);
  reduce_scatter_y<T, float, TW>(cols_at_cap);
  float gamma_own[OWN_C];
  double moved_r[OWN_R] = {}, moved_c[OWN_C] = {};  // sums of the increments
#pragma unroll
  for (int a = 0; a < OWN_R; ++a) rho[a] = (float)((U[a] - U_before[a]) * __builtin_amdgcn_rcp(U_before[a]));
#pragma unroll
  for (int b = 0; b < OWN_C; ++b)
    gamma[b] = gamma_own[b] = (float)((Vown[b] - V_before[b]) * __builtin_amdgcn_rcp(V_before[b]));
  if constexpr (!LDS) all_gather_x<T, float, TH>(rho);
  all_gather_y<T, float, TW>(gamma);
  int looks = 0;
  for (bool go_on = true; go_on;) {
    // (up to a multiple of kChunk, so that a check for the tolerance comes just before what follows)
    const int stop = min(iters, (t | (kChunk - 1)) + 1);
    float largest = 0.0f, s[TH], sum_r[OWN_R] = {}, sum_c[OWN_C] = {};
    for (; t < stop; ++t) {
      float d[TH], q[TW];
      if constexpr (T::NY == 3) {
        // in pairs, as the row sums in double: the same whatever the lane's offset of the columns is (LoneTiling)
#pragma unroll
        for (int a = 0; a < TH; ++a) {
          float leaf[TW];
#pragma unroll
          for (int b = 0; b < TW; ++b) leaf[b] = p[a][b] * gamma[b];
#pragma unroll
          for (int h = 1; h < TW; h *= 2)
#pragma unroll
            for (int b = 0; b < TW; b += 2 * h) leaf[b] += leaf[b + h];
          s[a] = leaf[0];
        }
      } else {
#pragma unroll
        for (int b = 0; b < TW; ++b)
#pragma unroll
          for (int a = 0; a < TH; ++a) s[a] = b == 0 ? p[a][b] * gamma[b] : fmaf(p[a][b], gamma[b], s[a]);
      }
      chain_phase<LONE>(true);
      reduce_scatter_x<T, float, TH>(s);
      largest = 0.0f;
#pragma unroll
      for (int a = 0; a < OWN_R; ++a) {
        s[a] = fmaf(rows_at_cap[a], rho[a], -s[a]);
        if constexpr (ADAPT) s[a] = frozen ? 0.0f : s[a];
        d[a] = s[a] - rho[a];
        rho[a] = s[a];
        sum_r[a] += s[a];
        largest = fmaxf(largest, fabsf(s[a]));
      }
      if constexpr (LDS) {
#pragma unroll
        for (int a = 0; a < OWN_R; ++a) xr[a ^ rx] = make_float2(s[a], d[a]);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int a = OWN_R; a < TH; ++a) {
          const float2 rd = xr[a ^ rx];
          s[a] = rd.x;
          d[a] = rd.y;
        }
        asm volatile("" ::: "memory");
      } else {
        all_gather_x<T, float, TH>(s);
#pragma unroll
        for (int a = OWN_R; a < TH; ++a) {
          d[a] = s[a] - rho[a];
          rho[a] = s[a];
        }
      }
      chain_phase<LONE>(false);
#pragma unroll
      for (int b = 0; b < TW; ++b) {
#pragma unroll
        for (int a = 0; a < TH; ++a) {
          q[b] = a == 0 ? p[a][b] * s[a] : fmaf(p[a][b], s[a], q[b]);
          q[b] = fmaf(c[a][b], d[a], q[b]);
        }
      }
      chain_phase<LONE>(true);
      reduce_scatter_y<T, float, TW>(q);
#pragma unroll
      for (int b = 0; b < OWN_C; ++b) {
        gamma_own[b] = fmaf(cols_at_cap[b], gamma_own[b], -q[b]);
        if constexpr (ADAPT) gamma_own[b] = frozen ? 0.0f : gamma_own[b];
        sum_c[b] += gamma_own[b];
        gamma[b] = gamma_own[b];
        largest = fmaxf(largest, fabsf(gamma_own[b]));
      }
      all_gather_y<T, float, TW>(gamma);
      chain_phase<LONE>(false);
      if constexpr (ADAPT) {
        // (a tolerance that only factors of exactly 1 meet, 1 + an increment below 2^-54: the block has stopped but for what the sum
        // of all that are left makes of them)
        if ((t + 1) % TSENOR_ADAPTIVE_CHECK_EVERY == 0)
          freeze_if(block_max<LPB>((double)largest) <= fmax(tol, 0x1p-54), t + 1, tol >= 0x1p-53);
      }
    }
#pragma unroll
    for (int a = 0; a < OWN_R; ++a) moved_r[a] += (double)sum_r[a];
#pragma unroll
    for (int b = 0; b < OWN_C; ++b) moved_c[b] += (double)sum_c[b];
    // What the last one changed in the logarithm of an entry is rho_i + gamma_j (opposite constants in the two change nothing, and
    // the map keeps what rounding leaves of them).
    const float left = (float)(iters - t);
    float rho_hi = s[0], rho_lo = s[0], gamma_hi = gamma[0], gamma_lo = gamma[0], moved = 0.0f;
#pragma unroll
    for (int a = 1; a < TH; ++a) rho_hi = fmaxf(rho_hi, s[a]), rho_lo = fminf(rho_lo, s[a]);
#pragma unroll
    for (int b = 1; b < TW; ++b) gamma_hi = fmaxf(gamma_hi, gamma[b]), gamma_lo = fminf(gamma_lo, gamma[b]);
    const float step = fmaxf(fabsf(rho_hi + gamma_hi), fabsf(rho_lo + gamma_lo));
#pragma unroll
    for (int a = 0; a < OWN_R; ++a) moved = fmaxf(moved, fabsf((float)moved_r[a]));
#pragma unroll
    for (int b = 0; b < OWN_C; ++b) moved = fmaxf(moved, fabsf((float)moved_c[b]));
    bool done = !__any(!(step * left < kNothingLeft));
    // (Now and then by what it changed in the plan itself: where a block falls into parts that only entries near e^-100 connect, each
    // part has a constant of its own, and a sum over two parts stays.  That it must not take an entry to the cap is asked as well.)
    if (!done && ++looks % 3 == 0) {
      float change = 0.0f;
#pragma unroll
      for (int a = 0; a < TH; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b) {
          const float log_change = (s[a] + gamma[b]) * 0x1p+40f;  // (squares in the range of a float)
          change = fmaxf(change, p[a][b] * (log_change * log_change));
        }
      done = !__any(!(change * (float)N * (left * left) < (kNothingLeft * 0x1p+40f) * (kNothingLeft * 0x1p+40f) &&
                      step * left < 0.25f * (float)kNearCap));
    }
    if (done) t = iters;
    go_on = t < iters && !__any(!(moved < kIncrementSum && largest <= 2.0f * (float)kSmallStep));
  }
  // (a scaling has taken the product of the 1 + increments, e to their sum)
  double by[TH];
#pragma unroll
  for (int a = 0; a < OWN_R; ++a) {
    by[a] = fma(0.5 * moved_r[a], moved_r[a], moved_r[a]);
    U[a] = fma(U[a], by[a], U[a]);
  }
#pragma unroll
  for (int b = 0; b < OWN_C; ++b) V[b] = Vown[b] = fma(Vown[b], fma(0.5 * moved_c[b], moved_c[b], moved_c[b]), Vown[b]);
  all_gather_y<T, double, TW>(V);
  // (the tile also when all iterations are done: it need not be kept beside p and c then)
  all_gather_x<T, double, TH>(by);
#pragma unroll
  for (int a = 0; a < TH; ++a) {
    if constexpr (FORM == kKeep) {
      if (a >= OWN_R) U[a] = fma(U[a], by[a], U[a]);
    }
#pragma unroll
    for (int b = 0; b < TW; ++b) {
      if constexpr (FORM == kKeep)
        x[a][b] = kap[a][b] * U[a];
      else
        kap[a][b] = fma(kap[a][b], by[a], kap[a][b]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return t;
}

// x * y with the result clamped to [0, 1] by the output modifier: one instruction at the full fp32 rate
// (measured on MI355X: 1.2 ns per wave-instruction per SIMD, as a plain v_mul_f32; v_min_f32 / v_max_f32 /
// v_med3_f32 take 1.9 ns).  Written as the bare instruction so that it stays this one.
__device__ __forceinline__ float mul_clamp01(float x, float y) {
  float r;
  asm("v_mul_f32_e64 %0, %1, %2 clamp" : "=v"(r) : "v"(x), "v"(y));
  return r;
}

// max(a, b) as the bare instruction: fmaxf() first quiets a possible signalling NaN in an operand the compiler
// has not just computed (the loop-invariant floor below), one more instruction in every iteration
__device__ __forceinline__ float max_as_is(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// The same iteration in single precision.  kap stays as rebuilt (no rounding accumulates in it); the scalings
// U (every tile row) and V (every tile column) are kept as numbers, and the capped entry is
//     e_ij = clamp(kap_ij * (U_i V_j)):  a multiply, a multiply with the clamp modifier, the add of the row
// sum and the multiply-add of the column sum per entry, all at the full fp32 rate.  A scaling grows by at most
// 2^10 per iteration (keeps everything finite on degenerate input).
// ADAPT as in dykstra_iteration.
template <class T, bool LDS_GATHER = false, bool ADAPT = false, int TH, int TW>
__device__ __forceinline__ float dykstra_iteration_f32(const float (&kap)[TH][TW], float (&U)[TH], float (&V)[TW],
                                                       float (&Vown)[owned(TW, T::NY)], float Nf, float2* xr = nullptr, int rx = 0,
                                                       bool frozen = false) {
  constexpr int OWN_R = owned(TH, T::NX), OWN_C = owned(TW, T::NY);
  // (the factors of a lane's own rows without their N, as in dykstra_iteration: four of 92 instructions of 4 x 4 blocks)
  constexpr bool BARE = OWN_R == TH;
  [[maybe_unused]] const float cap = 1024.0f / Nf;
  float worst = 0;
  float e[TH][TW], R[TH], C[TW];
#pragma unroll
  for (int a = 0; a < TH; ++a) {
#pragma unroll
    for (int b = 0; b < TW; ++b) {
      e[a][b] = mul_clamp01(kap[a][b], U[a] * V[b]);
      R[a] = b == 0 ? e[a][b] : R[a] + e[a][b];
    }
  }
  chain_phase(true);
  reduce_scatter_x<T, float, TH>(R);
#pragma unroll
  for (int a = 0; a < OWN_R; ++a) {
    // factor of an owned row (a NaN from an empty row gives the cap)
    R[a] = BARE ? fminf(fast_rcp(R[a]), cap) : fminf(Nf * fast_rcp(R[a]), 1024.0f);
    if constexpr (ADAPT) {
      worst = fmaxf(worst, fabsf((BARE ? Nf * R[a] : R[a]) - 1.0f));
      if constexpr (!BARE) R[a] = frozen ? 1.0f : R[a];
    }
  }
  if constexpr (LDS_GATHER) {
    // the owner of a row updates its scaling and leaves factor and scaling in LDS; the other lanes of the
    // lane-row pick both up in one 8-byte read per row instead of multiplying each scaling themselves
#pragma unroll
    for (int a = 0; a < OWN_R; ++a) {
      U[a] *= R[a];
      xr[a ^ rx] = make_float2(R[a], U[a]);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int a = OWN_R; a < TH; ++a) {
      const float2 ru = xr[a ^ rx];
      R[a] = ru.x;
      U[a] = ru.y;
    }
    asm volatile("" ::: "memory");
  } else {
    all_gather_x<T, float, TH>(R);
#pragma unroll
    for (int a = 0; a < TH; ++a) U[a] *= !BARE ? R[a] : ADAPT && frozen ? 1.0f : Nf * R[a];
  }
  chain_phase(false);
#pragma unroll
  for (int b = 0; b < TW; ++b) {
#pragma unroll
    for (int a = 0; a < TH; ++a) C[b] = a == 0 ? e[a][b] * R[a] : fmaf(e[a][b], R[a], C[b]);
  }
  chain_phase(true);
  reduce_scatter_y<T, float, TW>(C);
#pragma unroll
  for (int b = 0; b < OWN_C; ++b) {
    C[b] = BARE ? fast_rcp(max_as_is(C[b], 0x1p-10f)) : Nf * fast_rcp(max_as_is(C[b], Nf * 0x1p-10f));
    if constexpr (ADAPT) {
      worst = fmaxf(worst, fabsf(C[b] - 1.0f));
      C[b] = frozen ? 1.0f : C[b];
    }
  }
#pragma unroll
  for (int b = 0; b < OWN_C; ++b) V[b] = Vown[b] *= C[b];
  all_gather_y<T, float, TW>(V);
  chain_phase(false);
  return worst;
}

// Whether the iterations of a wave have begun to repeat themselves.  An iteration is a function of the scalings alone (the
// tile it reads stays as it is), so once the scalings of all blocks of a wave are, bit for bit, what they were d iterations
// ago, all later states are known, and whole periods of d iterations are as good as done.
// Once a block has converged to the precision of its numbers its last bits run through a short cycle: of 512 blocks of 16:32
// with fp32 iterations 57 % end in one of period 2, 14 % of 1, 4, 6 or 8, hardly any in a period that does not divide 24.  So
// the fp32 loops compare the state every kChunk iterations with one 8, 16 or 24 iterations old, the double ones every kRepeatWindow
// iterations with the one before those.  The large tiles that fold (32 x 32 and 64 x 64 in double), the team and the kernels of the
// early exit do not look.  (In double the increments usually come first where there are any.)
// IN_LDS: that state is kept in LDS (`space`), for the kernels whose register budget is that of their loop; small launches, where a
// wave has its SIMD to itself and waits for every LDS access, keep it in registers.
template <class real, int OWN_R, int OWN_C, bool IN_LDS>
struct RepeatCheck {
  using Space = std::conditional_t<IN_LDS, real[OWN_R + OWN_C][kWave], char>;
  using Seen = std::conditional_t<IN_LDS, Space&, real[OWN_R + OWN_C]>;  // the scalings this lane owns, `noted` iterations done
  Seen seen;
  int lane, noted;
  static __device__ __forceinline__ RepeatCheck make(Space& space, int lane) {
    if constexpr (IN_LDS)
      return {space, lane, 0};
    else
      return {{}, lane, 0};
  }
  __device__ __forceinline__ real& at(int k) {
    if constexpr (IN_LDS)
      return seen[k][lane];
    else
      return seen[k];
  }
  static __device__ __forceinline__ bool differ(float x, float y) { return __float_as_uint(x) != __float_as_uint(y); }
  static __device__ __forceinline__ bool differ(double x, double y) { return __double_as_longlong(x) != __double_as_longlong(y); }
  template <int NU, int NV>
  __device__ __forceinline__ void note(const real (&U)[NU], const real (&V)[NV], int t) {
#pragma unroll
    for (int a = 0; a < OWN_R; ++a) at(a) = U[a];
#pragma unroll
    for (int b = 0; b < OWN_C; ++b) at(OWN_R + b) = V[b];
    noted = t;
  }
  // whether the state is the one noted
  template <int NU, int NV>
  __device__ __forceinline__ bool same(const real (&U)[NU], const real (&V)[NV], real first) {
    // (the whole state only if a first scaling of every lane is as it was)
    bool changed = __any(differ(U[0], first));
    if (!changed) {
#pragma unroll
      for (int a = 1; a < OWN_R; ++a) changed |= differ(U[a], at(a));
#pragma unroll
      for (int b = 0; b < OWN_C; ++b) changed |= differ(V[b], at(OWN_R + b));
      changed = __any(changed);
    }
    return !changed;
  }
  // t iterations are done: the number that are as good as done
  template <int NU, int NV>
  __device__ __forceinline__ int look(const real (&U)[NU], const real (&V)[NV], int t, int T, real first) {
    const int d = t - noted;
    if (same(U, V, first)) {
      while (T - t >= d) t += d;
      noted = t;
    } else if (d >= kRepeatWindow) {
      note(U, V, t);
    }
    return t;
  }
};

// calls f(integral_constant<A0>) for A0 = 0, NA, 2 NA, ... < TH: a tile is loaded NA rows at a time
template <int A0, int NA, int TH, class F>
__device__ __forceinline__ void row_chunks(F& f) {
  if constexpr (A0 < TH) {
    f(std::integral_constant<int, A0>{});
    row_chunks<A0 + NA, NA, TH>(f);
  }
}

template <int M, bool FAST, bool ADAPT = false, int TILES = kLargeTiles, bool LONE = false>
struct DykstraLaunch {
  // with the early exit the waves of a launch run for very different times; one-wave workgroups let the
  // dispatcher refill every wave slot as it frees (a four-wave workgroup holds its slots until its slowest wave).
  // The 64-wide fp32 waves, one block each, leave when their block repeats itself: two to a workgroup (8192x28672 student, T =
  // 500: 2.91 ms, one 2.94, four 3.25; 4096x4096 normal, which does not repeat, T = 300: 563 us, 610, 581).  In a launch of one
  // wave per SIMD four, which go to the four of a CU (2048x2048 normal, T = 300: 285 us, two 302).
  // The iterations in double of 8-, 16- and 32-wide blocks end at different times too (increments): one (16:32 4096x14336
  // Wanda-style 2515 us, two 2534, four 2578; normal weights the same within 0.3 %).
  // The small tiles carry the rounding behind the iterations, whose steps synchronise one wave at a time.
  static constexpr int kWavesPerGroup = (ADAPT || TILES != kLargeTiles) ? 1
                                        : M == 64 && FAST && !LONE      ? 2
                                        : FAST || M == 4 || M == 64     ? 4
                                                                        : 1;
  static constexpr int kThreads = kWavesPerGroup * kWave;
  // Waves per SIMD the register budget is set for.  Double: the loop holds twice the state of the fp32 one, two waves of up
  // to 256 registers; the 8-wide large tiles and the 16-wide small ones three of 168, no spills (with four of 128 the increments spill 14
  // and 19 outside the loops; four / three, us: 4:8 4096x4096 with all outputs 995 / 981, student-t 1536x2048 86.4 / 85.3, 8:16 2048x1024
  // T = 500 normal 200.4 / 196.5, student-t 111.2 / 108.9, 1792x1792 student-t 73.5 / 74.1).  With the early exit the 16-wide ones
  // four: launches of just under four waves per SIMD run at once (3936x1056 normal 245 / 270; 17 registers spill).
  // FAST: the more waves, the nearer the issue of plain fp32 instructions comes to its limit (1.13 ns
  // per instruction and SIMD with two waves, 1.05 with four).  M = 32: four waves of 128 registers, the loop fits and 38
  // registers of the double-precision code around it spill (whole calls with four / three waves, us: 4096x14336 Wanda-style 1364 /
  // 1464, normal 1745 / 1764; 4096 blocks, two waves to a SIMD anyway, 172 / 168).  M = 16: three (four the same to 0.4 % slower).
  // M = 8: four (eight spill outside the loop).  M = 4: four fit whatever is asked for (two spill outside the loop; five waves:
  // 1 % slower).  M = 64: three, 133 registers spill outside the loop.  With three / two waves, T = 300 normal and T = 500 student-t,
  // of which blocks run from 50 iterations to all: 57 344 blocks 7046 / 7128 and 3080 / 3200, 16 384 Wanda-style 1924 / 2066; 4096
  // blocks 572 / 532 and 549 / 531, 1024 blocks, a wave to a SIMD, 269 / 254 and 394 / 379: full launches decide.  With the early
  // exit, where a block may run a dozen iterations and the code around the loop is most of the work, two (8192x8192: 0.85 ms,
  // three 1.05).
  static constexpr int kWavesPerSimd =
      FAST && !(M == 64 && ADAPT)                  ? (M == 16 || M == 64 ? 3 : 4)
      : M == 8 && TILES == kLargeTiles             ? 3
      : !LONE && M == 16 && TILES == kSmallTiles ? (ADAPT ? 4 : 3)
                                                   : 2;
};

// ZERO_T: the instantiation for T = 0 (no iterations, keys are K itself).  It is a template parameter
// rather than a branch because keeping both paths in one kernel costs the iterating path ~40 registers.
// TILES: the finer tilings are for launches that cannot fill the chip.  There the whole path stays in this kernel: a block
// lives in one wave from its tile load to its mask, the potentials that Algorithm 2 starts from go to LDS instead of the
// workspace, and Algorithm 2 runs behind; no further kernel follows.  (4096 x 32, 16:32, T = 300: 120 us a call with a sort
// across the lanes and the scan of its result, 106 with round_blocks.)
// LONE: for a launch that gives a SIMD no second wave.
template <int M, bool FAST, bool ZERO_T = false, int TILES = kLargeTiles, bool ADAPT = false, bool LONE = false>
__global__ __launch_bounds__((DykstraLaunch<M, FAST, ADAPT, TILES, LONE>::kThreads),
                             (DykstraLaunch<M, FAST, ADAPT, TILES, LONE>::kWavesPerSimd)) void dykstra_sort_kernel(Batch batch) {
  using T = std::conditional_t<LONE && TILES != kLargeTiles, LoneTiling<Tiling<M, TILES>>, Tiling<M, TILES>>;
  constexpr bool SMALL = TILES != kLargeTiles;
  const int which = find_problem(batch, blockIdx.x);
  const DevProblem p = batch.e[which].p;
  double* plan_out = batch.e[which].plan_out;
  double* tau_eff_out = batch.e[which].tau_eff_out;
  const unsigned int group = blockIdx.x - batch.first[which];  // workgroup index within the matrix
  constexpr int GX = 1 << T::NX, GY = 1 << T::NY, TH = M / GY, TW = M / GX, LPB = GX * GY, BPW = kWave / LPB,
                E = TH * TW, SHX = ilog2(TH) - T::NX, WPG = DykstraLaunch<M, FAST, ADAPT, TILES, LONE>::kWavesPerGroup;
  const int lane = threadIdx.x & (kWave - 1), wave_in_group = threadIdx.x / kWave;
  const int64_t wave = (int64_t)group * WPG + wave_in_group;
  const int q = lane % LPB, gx = q % GX, gy = q / GX, gc = column_lane<T>(gx, q);
  int64_t blk = wave * BPW + lane / LPB;
  const bool active = blk < p.nblocks;
  if (!active) blk = p.nblocks - 1;  // idle lanes shadow the last block and write nothing
  const BlockAt at = place_of(batch.e[which], blk, M, blk);
  const int64_t r0 = at.r0, c0 = at.c0;
  const double tau_eff = tau_eff_of(batch.e[which]);
  if (tau_eff_out && group == 0 && threadIdx.x == 0) *tau_eff_out = tau_eff;

  // register (a, b) of this lane <-> in-kernel coordinates (ri, cj) of the block.  Each phase of the
  // kernel takes its own opaque copy of the lane offsets, so that element addresses are recomputed where
  // they are needed instead of being kept in registers across the iteration loop.
  constexpr int RUN = FAST ? 0 : order_run<M, TILES>();
  const int rx_own = shift_lane(gx, SHX), ry_tile = reg_xor_y<T, TW, false>(q);
  const int rx = RUN ? rx_own ^ ry_tile : rx_own, ry = RUN ? rx : ry_tile;
  const int ry_own = ry ^ ry_tile ^ reg_xor_y<T, TW, true>(q);  // offset of the columns this lane owns
  auto fresh = [](int v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  // with `transpose` the in-kernel rows are the matrix columns, which turns "rows first" into
  // "columns first" (TSENOR_FLAG_COLS_FIRST)
  auto mat_row = [&](int ri, int cj) { return p.transpose ? cj : ri; };
  auto mat_col = [&](int ri, int cj) { return p.transpose ? ri : cj; };

  // tile addressing of one phase, from that phase's copy of the lane offsets
  auto addr_of = [&](int rxp, int ryp) {
    int ri[TH], cj[TW];
#pragma unroll
    for (int a = 0; a < TH; ++a) ri[a] = gy * TH + (a ^ rxp);
#pragma unroll
    for (int b = 0; b < TW; ++b) cj[b] = column_in_block<M, TILES>(gc, b ^ ryp);
    return tile_addr<TH, TW>(p, r0, c0, ri, cj);
  };
  // rows of a tile loaded at a time: the fp32 variant lives in half the registers (two halves); the 8 x 8
  // tiles of M = 64 would keep 64 loads with their addresses in flight and spill
  constexpr int NA = M == 64 ? TH / kRowChunks64 : (FAST && TH >= 8) ? TH / 2 : TH;

  // Blocks are rounded from their potentials (in a kernel of their own for the large tiles); only for 4 x 4 blocks on the
  // large tiles, a lane each, the greedy selection is done here (round_kernel would give them four lanes)
  constexpr bool kPotentials = M >= 8 || SMALL;
  [[maybe_unused]] double c[kPotentials ? 1 : E];  // sort keys
  __shared__ double pot[2][kPotentials && SMALL ? BPW : 1][M];  // small tiles: potentials of the matrix rows and columns
  using RoundingSpace = std::conditional_t<SMALL, RoundingLds<M, BPW>, char>;
  [[maybe_unused]] __shared__ RoundingSpace lds;
  int iters_done = 0;
  double kap[ZERO_T ? 1 : TH][ZERO_T ? 1 : TW];
  // Normaliser of every in-kernel row: kappa = exp(K - mrow) <= ~1.  Any per-row constant gives the same
  // iterates, because the first step of Algorithm 1 rescales every row (with TSENOR_FLAG_COLS_FIRST: every
  // column, which is the in-kernel row); the single precision value next above the row's largest K is
  // enough.  Per row rather than per block, so that one huge entry does not push the other rows of its
  // block below the range of a double.
  float mrow[TH];
  {
    const int rx0 = fresh(rx), ry0 = fresh(ry);
    const auto addr = addr_of(rx0, ry0);
    // the plan (a diagnostic output) in a pass of its own, before the keys exist and with its own loads: an
    // exp() inside the key pass, or keys kept alive across it, costs registers (spills for M = 64)
    if constexpr (ZERO_T) {
      if (plan_out && active) {
        auto plan_rows = [&](auto first) {
          constexpr int A0 = decltype(first)::value;
          float imp[NA][TW];
          tile_importance<A0, NA, !SMALL>(p, addr, imp);
#pragma unroll
          for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b) {
              const int ri = gy * TH + ((A0 + a) ^ rx0), cj = column_in_block<M, TILES>(gc, b ^ ry0);
              plan_out[(r0 + mat_row(ri, cj)) * p.cols + c0 + mat_col(ri, cj)] = exp(tau_eff * (double)imp[a][b]);
              __builtin_amdgcn_sched_barrier(0);
            }
        };
        row_chunks<0, NA, TH>(plan_rows);
      }
      if constexpr (kPotentials) return;  // (launched for the plan alone: round_kernel forms the keys itself)
    }
    auto rows = [&](auto first) {
      constexpr int A0 = decltype(first)::value;
      float imp[NA][TW];
      tile_importance<A0, NA, !SMALL>(p, addr, imp);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b) {
          const double K = tau_eff * (double)imp[a][b];  // K of Algorithm 1 line 1
          if constexpr (ZERO_T) {
            // no iterations: the greedy order is descending K itself
            const int ri = gy * TH + ((A0 + a) ^ rx0), cj = column_in_block<M, TILES>(gc, b ^ ry0);
            if constexpr (!kPotentials) c[(A0 + a) * TW + b] = scan_key_of_k(K, mat_row(ri, cj) * M + mat_col(ri, cj));
          } else {
            kap[A0 + a][b] = K;
          }
        }
      if constexpr (!ZERO_T) {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          double largest = kap[A0 + a][0];
#pragma unroll
          for (int b = 1; b < TW; ++b) largest = vmax(largest, kap[A0 + a][b]);
          mrow[A0 + a] = round_up(largest);
        }
      }
    };
    row_chunks<0, NA, TH>(rows);
  }
  if constexpr (!ZERO_T) {
    all_reduce_max_x<T, TH>(mrow);
#pragma unroll
    for (int a = 0; a < TH; ++a)
#pragma unroll
      for (int b = 0; b < TW; ++b) {
        kap[a][b] = exp_in_range(fmax(kap[a][b] - (double)mrow[a], kMinLogKernel));
        __builtin_amdgcn_sched_barrier(0);  // one exp at a time: interleaving them only costs registers
      }

    const double Nd = (double)p.N;
    iters_done = p.T;
    const long long cycles0 = clock64(), ticks0 = wall_clock64();
    // scalings of the rows and columns this lane owns (the first registers after a reduce-scatter); the other lanes of the
    // lane-row / lane-column hold the same values for theirs.  FAST: in the form own * 2^exponent, so that the factors of
    // any number of chunks can be multiplied in; their logarithms (76 instructions each) are only taken where they are used (2:4
    // 4096x4096: 462 -> 450 us a call).
    constexpr int OWN_R = owned(TH, T::NX), OWN_C = owned(TW, T::NY);
    double u_own[OWN_R], v_own[OWN_C];
    // whether the tile is held twice (see dykstra_iteration)
    constexpr Form kForm = FAST || !T::STORE_E ? kRecompute : T::KEEP ? kKeep : kFold;
    constexpr bool kKept = kForm == kKeep;
    [[maybe_unused]] int u_exp[OWN_R] = {}, v_exp[OWN_C] = {};
    // early exit: a block whose factors have passed the tolerance is frozen at that iteration
    bool frozen = false;
    auto freeze_if = [&](bool passed, int t_done, bool stop = true) {
      if (!frozen && passed) {
        frozen = stop;
        iters_done = min(iters_done, t_done);
      }
    };
    // FAST: the tile of the fp32 phase, fl32(kap U V)
    float kap32[FAST ? TH : 1][FAST ? TW : 1];
    {
      double Uown[kKept ? TH : OWN_R], V[TW], Vown[OWN_C];
#pragma unroll
      for (double& u : Uown) u = 1.0;
#pragma unroll
      for (int b = 0; b < TW; ++b) V[b] = 1.0;
#pragma unroll
      for (double& v : Vown) v = 1.0;
      if constexpr (FAST) {
        // the entries are recomputed in the column pass: this phase must fit the registers of the fp32 loop
        const int t_double = p.T < kWarmIters ? p.T : kWarmIters;
        NoTile once;
        for (int t = 0; t < t_double; ++t) {
          double worst = dykstra_iteration<T, kRecompute, kLanesOnly, ADAPT>(kap, once, Uown, V, Vown, Nd, nullptr, 0, frozen);
          if constexpr (ADAPT) {
            if ((t + 1) % TSENOR_ADAPTIVE_CHECK_EVERY == 0) freeze_if(block_max<LPB>(worst) <= p.tol, t + 1);
          }
        }
      } else {
        // In the 32- and 64-wide kernels the row factors of an iteration are gathered through LDS (measured
        // ~1 % faster than DPP moves; doing the same for the column scalings as well exposed a second LDS round
        // trip and gained nothing), in the 8- and 16-wide ones the row scalings (two respectively eight multiplies fewer):
        // lane-row r of the wave keeps those of its rows at xrows[wave][r][0..TH)
        constexpr Gather kGather = SMALL || LPB == 1 ? kLanesOnly : kForm == kKeep ? kScalingsInLds : kRowsInLds;
        using Tile = std::conditional_t<kForm != kRecompute, double[TH][TW], NoTile>;
        constexpr bool kLds = kGather != kLanesOnly;
        __shared__ __align__(16) double xrows[kLds ? WPG : 1][kLds ? kWave >> T::NX : 1][TH];
        double* xr = kLds ? &xrows[wave_in_group][lane >> T::NX][0] : nullptr;
        Tile x;
        if constexpr (kKept) {
#pragma unroll
          for (int a = 0; a < TH; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b) x[a][b] = kap[a][b];
        }
        const auto iterate = [&]() {
          return dykstra_iteration<T, kForm, kGather, ADAPT, RUN, LONE>(kap, x, Uown, V, Vown, Nd, xr, rx, frozen);
        };
        // A row whose entries but one lie near e^-700 has its scaling grow to their reciprocal and, on the way to the others'
        // balance, beyond the range of a double (15:16, every entry 0 or 1, spread 680: e^717; as an infinity it would stay one).
        // So what is large of it goes into the row of the tile, by a power of two: the products are the same bit for bit.  Looked
        // for every kRepeatWindow iterations: a row sums to N / M^2 at least, so in these it grows by 2^288 at most.
        [[maybe_unused]] int raised = 0;  // bit a: tile row a
        [[maybe_unused]] const auto raise_rows = [&]() {
          bool large = false;
#pragma unroll
          for (int a = 0; a < OWN_R; ++a) large |= Uown[a] > kRaiseAbove;
          if (__builtin_expect(__any(large), 0)) {
#pragma unroll
            for (int a = 0; a < (kKept ? TH : 0); ++a) {
              const bool raise = Uown[a] > kRaiseAbove && !((raised >> a) & 1);
              Uown[a] = raise ? ldexp(Uown[a], -kRaiseBits) : Uown[a];
#pragma unroll
              for (int b = 0; b < TW; ++b) kap[a][b] = raise ? ldexp(kap[a][b], kRaiseBits) : kap[a][b];
              raised |= raise ? 1 << a : 0;
            }
          }
        };
        constexpr bool kEnd = increments_at_the_end<M, TILES>();
        // Behind a window of iterations over which a scaling of every lane has hardly changed (`first`: what it was before them): one
        // more iteration, with refined factors, and the rest in increments if that may be.  Whether any was done in increments.
        [[maybe_unused]] const auto try_the_end = [&]([[maybe_unused]] int& t, [[maybe_unused]] double first,
                                                      [[maybe_unused]] auto&& one_more) {
          if constexpr (kEnd) {
            if (t + 1 >= p.T || __any(!(fabs(Uown[0] - first) <= kRepeatWindow * kSmallStep * first))) return false;
            if (!away_from_cap<kForm>(kap, x, V)) return false;
            double U_before[OWN_R], V_before[OWN_C];
#pragma unroll
            for (int a = 0; a < OWN_R; ++a) U_before[a] = Uown[a];
#pragma unroll
            for (int b = 0; b < OWN_C; ++b) V_before[b] = Vown[b];
            one_more(dykstra_iteration<T, kForm, kGather, ADAPT, RUN, LONE, true>(kap, x, Uown, V, Vown, Nd, xr, rx, frozen));
            if (!hardly_moves(Uown, Vown, U_before, V_before)) return false;
            t = iterate_increments<T, kForm, kLds, ADAPT, LPB, LONE>(kap, x, Uown, V, Vown, U_before, V_before, p.N, t, p.T, p.tol,
                                                                     reinterpret_cast<float2*>(xr), rx, frozen, freeze_if);
            return true;
          } else {
            return false;
          }
        };
        // (the same numbers; said so, both have one register in the loop)
        [[maybe_unused]] const auto one_register = [&]() {
          if constexpr (!kSwaps<T>) {
#pragma unroll
            for (int b = 0; b < OWN_C; ++b) Vown[b] = V[b];
          }
        };
        if constexpr (ADAPT) {
          // iteration count as a bound: every TSENOR_ADAPTIVE_CHECK_EVERY-th iteration the largest |factor - 1|
          // of the block is compared with the tolerance; a block that passes is frozen, the wave leaves when
          // all its blocks are
          bool all_frozen = false;
          int t = 0;
          const auto count = [&](double worst) {
            ++t;
            if (t % TSENOR_ADAPTIVE_CHECK_EVERY == 0) {
              // (a block whose factors are exactly 1 is not where refined ones would leave it)
              freeze_if(block_max<LPB>(worst) <= p.tol, t, !kEnd || p.tol >= 0x1p-53);
              all_frozen = __all(frozen);
            }
          };
          for (int end = 0; t < p.T && !all_frozen;) {
            end = of_wave((kKept || kEnd) && p.T - end > kRepeatWindow ? end + kRepeatWindow : p.T);
            t = of_wave(t);
            [[maybe_unused]] const double first = Uown[0];
            while (t < end && !all_frozen) {
              // The three of four that no check follows need no factor's distance from 1, which the compiler leaves out here.
              // Whole calls at tol = 1e-5, distances in all / one of four (us): 16:32 1184x256 Wanda-style 118.8 / 110.2, 4000x5408
              // student-t 306.5 / 301.0; 32:64 2688x576 student-t 122.3 / 118.6; with fp32 iterations 16:32 672x960 student-t 61.4 / 58.5.
              one_register();
              for (const int last = of_wave(min(end, t | (TSENOR_ADAPTIVE_CHECK_EVERY - 1))); t < last; ++t) iterate();
              if (t < end) count(iterate());
            }
            if constexpr (kKept) raise_rows();
            if (!all_frozen && try_the_end(t, first, count)) end = t;
          }
        } else if constexpr (kKept) {
          using Repeat = RepeatCheck<double, OWN_R, OWN_C, !SMALL>;
          __shared__ typename Repeat::Space seen[WPG];
          Repeat repeat = Repeat::make(seen[wave_in_group], lane);
          repeat.note(Uown, Vown, 0);
          // (`end`: of the windows, which stay kRepeatWindow apart also where try_the_end() has run one iteration in vain: states are
          // compared over a whole number of their short periods)
          for (int t = 0, end = 0; t < p.T;) {
            end = of_wave(p.T - end > kRepeatWindow ? end + kRepeatWindow : p.T);
            t = of_wave(t);
            const double first = repeat.at(0);
            for (; t < end; ++t) iterate();
            raise_rows();
            // (noted one window ago, so that the period divides kRepeatWindow)
            const bool again = repeat.same(Uown, Vown, first);
            if (!again) repeat.note(Uown, Vown, t);
            const bool summed = try_the_end(t, first, [&](double) { ++t; });
            one_register();
            if (summed) {
              repeat.note(Uown, Vown, t);
              end = t;
            } else if (again) {
              while (p.T - t >= kRepeatWindow) t += kRepeatWindow;
              end = t;
            }
          }
        } else if constexpr (kEnd) {
          for (int t = 0, end = 0; t < p.T;) {
            end = of_wave(p.T - end > kRepeatWindow ? end + kRepeatWindow : p.T);
            t = of_wave(t);
            const double first = Uown[0];
            for (; t < end; ++t) iterate();
            if (try_the_end(t, first, [&](double) { ++t; })) end = t;
            one_register();
          }
        } else {
          for (int t = 0; t < p.T; ++t) iterate();
        }
        if constexpr (kKept) {
#pragma unroll
          for (int a = 0; a < OWN_R; ++a) u_exp[a] = (raised >> a) & 1 ? kRaiseBits : 0;
        }
      }
      if constexpr (FAST) {
        // The first tile of the fp32 phase comes from the double-precision tile while it is still at hand (it
        // holds kap U; a multiply with V and a conversion per entry, clamped like a rebuilt entry); only a later
        // rebuild has to read the importance again and go through exp().
        const double floor32 = 0x1.31c5957a47de2p-120, ceil32 = 0x1.45e3076d61699p+79;  // e^kLogFloor32, e^kLogCeil32
#pragma unroll
        for (int a = 0; a < TH; ++a)
#pragma unroll
          for (int b = 0; b < TW; ++b) kap32[a][b] = (float)fmin(fmax(kap[a][b] * V[b], floor32), ceil32);
      }
#pragma unroll
      for (int a = 0; a < OWN_R; ++a) u_own[a] = Uown[a];
#pragma unroll
      for (int b = 0; b < OWN_C; ++b) v_own[b] = Vown[b];
    }
    double lu_own[OWN_R], lv_own[OWN_C];  // (set by take_logs)
    auto take_logs = [&]() {
      constexpr double kLn2 = 0x1.62e42fefa39efp-1;
#pragma unroll
      for (int a = 0; a < OWN_R; ++a) {
        lu_own[a] = log(u_own[a]);
        if constexpr (FAST || kKept) lu_own[a] = fma((double)u_exp[a], kLn2, lu_own[a]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int b = 0; b < OWN_C; ++b) {
        lv_own[b] = log(v_own[b]);
        if constexpr (FAST) lv_own[b] = fma((double)v_exp[b], kLn2, lv_own[b]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    if constexpr (FAST) {
      if (p.T > kWarmIters && !(ADAPT && __all(frozen))) {
        // fp32 phase: kap32 = fl32(kap U V) for the double scalings U V reached so far, and fp32 scalings
        // U32, V32 relative to them.  kap is not kept: a rebuild reloads the importance.
        float U32[TH], V32[TW], V32own[OWN_C];
        const float Nf = (float)p.N;
        const float hi = __builtin_ldexpf(1.0f, kDriftBits), lo = __builtin_ldexpf(1.0f, -kDriftBits);
        auto rebuild = [&]() {
          const int rx1 = fresh(rx), ry1 = fresh(ry);
          double lu[TH], lv[TW];
#pragma unroll
          for (int a = 0; a < OWN_R; ++a) lu[a] = lu_own[a];
#pragma unroll
          for (int b = 0; b < OWN_C; ++b) lv[b] = lv_own[b];
          all_gather_x<T, double, TH>(lu);
          all_gather_y<T, double, TW>(lv);
          const auto addr = addr_of(rx1, ry1);
          auto rows = [&](auto first) {
            constexpr int A0 = decltype(first)::value;
            float imp[NA][TW];
            tile_importance<A0, NA, !SMALL>(p, addr, imp);
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
              for (int b = 0; b < TW; ++b) {
                const double K = tau_eff * (double)imp[a][b];
                const double full = (K - (double)mrow[A0 + a]) + (lu[A0 + a] + lv[b]);
                kap32[A0 + a][b] = (float)exp_in_range(fmin(fmax(full, kLogFloor32), kLogCeil32));
                __builtin_amdgcn_sched_barrier(0);
              }
          };
          row_chunks<0, NA, TH>(rows);
#pragma unroll
          for (int a = 0; a < TH; ++a) U32[a] = 1.0f;
#pragma unroll
          for (int b = 0; b < TW; ++b) V32[b] = 1.0f;
#pragma unroll
          for (float& v : V32own) v = 1.0f;
        };
        auto fold = [&]() {
#pragma unroll
          for (int a = 0; a < OWN_R; ++a) {
            const double u = u_own[a] * (double)U32[a];
            u_exp[a] += __builtin_amdgcn_frexp_exp(u);
            u_own[a] = __builtin_amdgcn_frexp_mant(u);
          }
#pragma unroll
          for (int b = 0; b < OWN_C; ++b) {
            const double v = v_own[b] * (double)V32own[b];
            v_exp[b] += __builtin_amdgcn_frexp_exp(v);
            v_own[b] = __builtin_amdgcn_frexp_mant(v);
          }
        };
#pragma unroll
        for (int a = 0; a < TH; ++a) U32[a] = 1.0f;
#pragma unroll
        for (int b = 0; b < TW; ++b) V32[b] = 1.0f;
#pragma unroll
        for (float& v : V32own) v = 1.0f;
        bool all_frozen = false;
        using Repeat = RepeatCheck<float, OWN_R, OWN_C, true>;
        __shared__ typename Repeat::Space seen[ADAPT ? 1 : WPG];
        Repeat repeat = Repeat::make(seen[ADAPT ? 0 : wave_in_group], lane);
        if constexpr (!ADAPT) repeat.note(U32, V32own, kWarmIters);
        for (int t = kWarmIters; t < p.T && !all_frozen;) {
          // (on its way from LDS while the iterations run; the 64-wide kernel has no register to spare for it: full launches lost 1 %)
          constexpr bool kEarly = M != 64;
          [[maybe_unused]] const float first = ADAPT || !kEarly ? 0.0f : repeat.at(0);
          const int stop = (p.T - t > kChunk) ? t + kChunk : p.T;
          // (in fp32 the exchange also carries the updated scalings, which pays wherever a block spans lanes:
          // -6 % for M = 8, -10 % for M = 16)
          constexpr bool kLdsGather32 = M >= 8;
          __shared__ float2 xrows32[kLdsGather32 ? WPG : 1][kLdsGather32 ? kWave >> T::NX : 1][TH];
          float2* xr = kLdsGather32 ? &xrows32[wave_in_group][lane >> T::NX][0] : nullptr;
          if constexpr (ADAPT) {
            while (t < stop && !all_frozen) {
              for (const int last = min(stop, t | (TSENOR_ADAPTIVE_CHECK_EVERY - 1)); t < last; ++t)
                dykstra_iteration_f32<T, kLdsGather32, true>(kap32, U32, V32, V32own, Nf, xr, rx, frozen);
              if (t >= stop) break;
              const float worst =
                  dykstra_iteration_f32<T, kLdsGather32, true>(kap32, U32, V32, V32own, Nf, xr, rx, frozen);
              ++t;
              if (t % TSENOR_ADAPTIVE_CHECK_EVERY == 0) {
                freeze_if(block_max<LPB>((double)worst) <= p.tol, t);
                all_frozen = __all(frozen);
              }
            }
          } else {
            for (; t < stop; ++t) dykstra_iteration_f32<T, kLdsGather32>(kap32, U32, V32, V32own, Nf, xr, rx);
          }
          if constexpr (!ADAPT) t = repeat.look(U32, V32own, t, p.T, kEarly ? first : repeat.at(0));
          // (the scalings of the rows and columns this lane owns: every row and column has its owner, and the
          // other copies of a scaling are the same number)
          float mxs = U32[0], mns = U32[0];
#pragma unroll
          for (int a = 1; a < OWN_R; ++a) mxs = fmaxf(mxs, U32[a]), mns = fminf(mns, U32[a]);
#pragma unroll
          for (int b = 0; b < OWN_C; ++b) mxs = fmaxf(mxs, V32own[b]), mns = fminf(mns, V32own[b]);
          // wave-uniform: fold the fp32 scalings into the double ones when any lane's have drifted
          if (t < p.T && __any(!(mxs < hi && mns > lo))) {
            fold();
            take_logs();
            rebuild();
            if constexpr (!ADAPT) repeat.note(U32, V32own, t);
          }
        }
        fold();
      }
    }

    if (group == 0 && threadIdx.x == 0) {
      WsHeader* h = batch.e[which].hdr;
      h->loop_cycles = (unsigned long long)(clock64() - cycles0);
      h->loop_ticks = (unsigned long long)(wall_clock64() - ticks0);
    }

    take_logs();
    const int rx2 = fresh(rx), ry2 = fresh(ry), ryo = fresh(ry_own);
    if constexpr (kPotentials) {
      // every row and column of the block has an owner among its lanes (on fine tiles several, with the same values)
      if constexpr (SMALL) {
#pragma unroll
        for (int a = 0; a < OWN_R; ++a) {
          const int ri = gy * TH + (a ^ rx2);
          pot[p.transpose ? 1 : 0][lane / LPB][ri] = lu_own[a];
          lds.minus_largest[lane / LPB][ri] = -(double)mrow[a];
        }
#pragma unroll
        for (int b = 0; b < OWN_C; ++b) pot[p.transpose ? 0 : 1][lane / LPB][column_in_block<M, TILES>(gc, b ^ ryo)] = lv_own[b];
      } else {
        if (group == 0 && threadIdx.x == 0) batch.e[which].hdr->tau_eff = tau_eff;
        if (active) {
          BlockPotentials<M>* out = static_cast<BlockPotentials<M>*>(batch.e[which].potentials) + blk;
          float* largest = normalisers_of<M>(batch.e[which], blk);
#pragma unroll
          for (int a = 0; a < OWN_R; ++a) {
            const int ri = gy * TH + (a ^ rx2);
            out->u[ri] = lu_own[a];
            largest[ri] = mrow[a];
          }
#pragma unroll
          for (int b = 0; b < OWN_C; ++b) out->v[column_in_block<M, TILES>(gc, b ^ ryo)] = lv_own[b];
        }
      }
      if (active && q == 0 && batch.e[which].iters_done_out) batch.e[which].iters_done_out[blk] = iters_done;
    }
    if (!kPotentials || plan_out) {
      double lu[TH], lv[TW];
#pragma unroll
      for (int a = 0; a < OWN_R; ++a) lu[a] = lu_own[a];
#pragma unroll
      for (int b = 0; b < OWN_C; ++b) lv[b] = lv_own[b];
      all_gather_x<T, double, TH>(lu);
      all_gather_y<T, double, TW>(lv);
      const auto addr = addr_of(rx2, ry2);
      // K + f_i + g_j, of which log S^(T) is the minimum with 0
      // (K is not floored here as it is for kappa: entries too small for the iterations to see keep
      // their own order in the scan)
      auto log_plan = [&](float importance, int a, int b) {
        const double K = tau_eff * (double)importance;
        return (K - (double)mrow[a]) + (lu[a] + lv[b]);
      };
      // the plan (a diagnostic output) in a pass of its own, with its own loads: an exp() inside the key pass
      // costs it registers (spills for M = 64)
      if (plan_out && active) {
        auto plan_rows = [&](auto first) {
          constexpr int A0 = decltype(first)::value;
          float imp[NA][TW];
          tile_importance<A0, NA, !SMALL>(p, addr, imp);
#pragma unroll
          for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b) {
              const int ri = gy * TH + ((A0 + a) ^ rx2), cj = column_in_block<M, TILES>(gc, b ^ ry2);
              plan_out[(r0 + mat_row(ri, cj)) * p.cols + c0 + mat_col(ri, cj)] = exp(fmin(log_plan(imp[a][b], A0 + a, b), 0.0));
              __builtin_amdgcn_sched_barrier(0);
            }
        };
        row_chunks<0, NA, TH>(plan_rows);
      }
      if constexpr (!kPotentials) {
        auto rows = [&](auto first) {
          constexpr int A0 = decltype(first)::value;
          float imp[NA][TW];
          tile_importance<A0, NA, !SMALL>(p, addr, imp);
#pragma unroll
          for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b) {
              const int ri = gy * TH + ((A0 + a) ^ rx2), cj = column_in_block<M, TILES>(gc, b ^ ry2);
              c[(A0 + a) * TW + b] = scan_key(log_plan(imp[a][b], A0 + a, b), mat_row(ri, cj) * M + mat_col(ri, cj));
            }
        };
        row_chunks<0, NA, TH>(rows);
      }
    }
  }
  if constexpr (kPotentials) {
    if constexpr (SMALL) {
      wave_sync();
      if (p.transpose)
        round_blocks<M, LPB, false, true>(p, batch.e[which], blk, active, r0, c0, lane, tau_eff, pot[0], pot[1], lds);
      else
        round_blocks<M, LPB, false, false>(p, batch.e[which], blk, active, r0, c0, lane, tau_eff, pot[0], pot[1], lds);
    }
  } else {
    // a lane has its whole block: the greedy selection follows in registers
    static_assert(LPB == 1 && M == 4, "a lane per block");
    sort_in_lane(c);
    if (active) {
      const unsigned int m = select_in_lane(c, p.N, p.simple != 0);
      reinterpret_cast<uint4*>(batch.e[which].rowmask)[blk] = make_uint4(m & 15u, (m >> 4) & 15u, (m >> 8) & 15u, m >> 12);
      if (batch.e[which].iters_done_out) batch.e[which].iters_done_out[blk] = iters_done;
    }
  }
}

}  // namespace tsenor_dev
