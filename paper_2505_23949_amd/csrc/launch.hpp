// Interface between the host code of the library and the kernels that depend on the block size M.  The
// kernels of every M are compiled in a translation unit of their own (launch_m4.hip ... launch_m64.hip, all of
// them instantiating launch_impl.hpp), so that the library builds in parallel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "problem.hpp"

namespace tsenor_dev {

// how the Dykstra kernel spreads a block over lanes (see Tiling in dykstra_sort.hpp and team.hpp)
enum { kLargeTiles, kSmallTiles, kFinestTiles, kFinestOrderTiles, kTeam };

// kernel variant of a problem: problems with the same variant can share one fused launch
struct Variant {
  int M;
  bool fast, zero_t;
  // The Dykstra kernel's tiling, decided per problem, so that fusing never changes results.  kFinestTiles and kTeam, which only
  // pay in a small launch, each have a second layout that adds in the same order: which of the two runs is decided per launch.
  int tiles;
  bool simple;      // TSENOR_FLAG_SIMPLE_ROUNDING
  bool adaptive;    // tol > 0: the early-exit instantiation of the Dykstra kernel
  bool operator==(const Variant& o) const {
    return M == o.M && fast == o.fast && zero_t == o.zero_t && tiles == o.tiles &&
           simple == o.simple && adaptive == o.adaptive;
  }
};

// Whether the whole path of a matrix runs in the one kernel with the small tiles (M <= 32, double iterations): with few
// waves a SIMD holds one or two, whose iteration time is the dependent chain, and the rounding needs no launch of its own.
// `fp32`: the caller asked for single-precision iterations, which only the large tiles have, so they win earlier.  Both
// sides take their time in steps of whole waves per SIMD (1024 of them), so the lines lie where a step is full.  Whole
// calls, T = 300 (us, small / large double / large fp32):
//   M = 32 (a block per wave): 1792 blocks 147 / 159 / 153, 2070 blocks 208 / 221 / 161, 2944 blocks 204 / 228 / 169,
//     3080 blocks 268 / 230 / 168;
//   M = 16 (4): 7680 blocks 130 / 152 / 142, 8280 blocks 182 / 222 / 151, 57 344 blocks 797 / 827 / 509, 65 536 blocks
//     863 / 856 / 529;
//   M = 8 (4): 8280 blocks 83 / 83 / 85, 9216 blocks 87 / 83 / 85, 10 240 blocks 90 / 84 / 85;
//   M = 4 (16; the large tiles hold 64): 46 000 blocks 78 / 93 / 85, 49 283 blocks 97 / 93 / 85, 65 536 blocks 100 / 92 / 83,
//     66 000 blocks 113 / 159 / 94, 106 000 blocks 154 / 166 / 104, 114 920 blocks 179 / 165 / 102.
// T = 100 puts the lines at the same places; at T = 20 the small tiles stay ahead a little beyond them, by less than 2 us (M = 4,
// 52 000 blocks 21.0 / 22.1, M = 8, 9000 blocks 21.4 / 23.1), but for M = 16 (65 536 blocks 146 / 152).
// With the early exit (`adaptive`) a wave runs until the slowest of its blocks stops, and the large tiles put up to four times
// as many blocks into it, so M <= 8 keeps the small tiles for longer.  T = 300, normal weights, tol 1e-2 and 1e-3 (small /
// large double / large fp32):
//   M = 4: 52 000 blocks 67 / 87 / 72 and 116 / 115 / 95, 60 000 blocks 69 / 87 and 116 / 116, 120 000 blocks 117 / 133 and
//     211 / 195; M = 8: 9500 blocks 74 / 100 / 91 and 109 / 111 / 104, 12 500 blocks 76 / 100 / 90 and 130 / 108 / 99;
//   M = 4 and 8, heavy-tailed weights, tol 1e-3: 60 000 blocks 43 / 70, 12 500 blocks 37 / 43;
//   M = 16, heavy-tailed: 8600 blocks 54 / - / 57.
constexpr bool small_tiles_win(int M, bool fp32, bool adaptive, int64_t nblocks) {
  if (M == 4 && adaptive) return nblocks <= (fp32 ? 55000 : 114688);
  if (M == 4) return nblocks <= 49152 || (!fp32 && nblocks > 65536 && nblocks <= 114688);
  if (M == 8) return nblocks < (adaptive ? (fp32 ? 12000 : 13000) : 8700);
  if (M == 16) return nblocks <= (fp32 ? (adaptive ? 9000 : 8192) : 62000);
  return M == 32 && nblocks <= (fp32 ? 2048 : 3072);
}

// Below this many blocks in a matrix a 16 x 16 block adds in the order of the finest tiles, and in a launch of up to two waves
// per SIMD it has a wave of its own: 51 instead of 103 vector instructions in the chain of an iteration, four times the waves.
// Whole calls, T = 300 (us, finest / small tiles): 256 blocks 45 / 70, 1024 blocks 53.6 / 75, 1280 blocks 76.3 / 74.7, 1792 blocks
// 77.9 / 75.3; where blocks repeat a state (RepeatCheck) a wave of its own stops with its block: 1376 blocks of 12:16, Wanda-style,
// T = 200 60.5 / 64.3.  From three waves on a SIMD on, issue decides (2304 blocks 104 / 90).  Fused matrices of 1024 blocks (us,
// finest tiles / small tiles in their order): 2 85 / 94, 3 107 / 89, 4 131 / 90, 16 436 / 243.
constexpr int64_t finest_tiles_below_blocks(int M) { return M == 16 ? 1800 : 0; }
constexpr int64_t kFinestTilesLaunch = 2048;

// SIMDs of the chip: a launch of no more waves gives each of them at most one
constexpr unsigned kSimds = 1024;

// Below this many blocks in a launch a 64 x 64 block has a workgroup of its own (team.hpp), which iterates in double: one
// workgroup per CU.  Whole calls, T = 300 (us, team / large tiles in double / with fp32 iterations): 64 blocks 173 / 286 /
// 254, 256 blocks 180 / 296 / 270, 300 blocks 354 / 300.  Fused: 4 matrices of 256 blocks 677 / 307, 16 2684 / 1009.
constexpr int64_t team_below_blocks(int M) { return M == 64 ? 257 : 0; }
// Below as many blocks in a matrix it iterates in the team's order, in double whatever the fp32 flag says.  A call of its own
// gains from that (256 blocks 180 us, 270 with fp32 iterations on the large tiles); a fused launch of many takes the large
// tiles in double where they could iterate in single precision (16 matrices of 64 blocks 304 / 268, of 128 blocks 510 / 332,
// of 256 blocks 1009 / 673), which a caller that wants them asks for with TSENOR_FLAG_TILES_LARGE.

// Enqueues the kernels of one fused launch that depend on M: tile load + Algorithm 1 (for M = 4 with the greedy selection, on
// small launches the whole path), then Algorithm 2 + mask write.  `b.count` non-degenerate problems of variant v.
// ev (optional): events recorded after the first, and after the second where that is the whole of Algorithm 2 (M >= 8).
// Returns false if a launch could not be described (more workgroups than a grid holds).
template <int M>
bool launch_block_kernels(Batch& b, const Variant& v, hipStream_t stream, hipEvent_t ev_sorted, hipEvent_t ev_greedy);

extern template bool launch_block_kernels<4>(Batch&, const Variant&, hipStream_t, hipEvent_t, hipEvent_t);
extern template bool launch_block_kernels<8>(Batch&, const Variant&, hipStream_t, hipEvent_t, hipEvent_t);
extern template bool launch_block_kernels<16>(Batch&, const Variant&, hipStream_t, hipEvent_t, hipEvent_t);
extern template bool launch_block_kernels<32>(Batch&, const Variant&, hipStream_t, hipEvent_t, hipEvent_t);
extern template bool launch_block_kernels<64>(Batch&, const Variant&, hipStream_t, hipEvent_t, hipEvent_t);

}  // namespace tsenor_dev
