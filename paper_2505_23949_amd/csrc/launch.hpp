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
//   M = 32 (a block per wave): 3040 blocks 212 / 230 / 172, 3104 blocks 264 / 229 / 169; for fp32 1792 blocks 147 / - / 153, 2070
//     blocks 208 / - / 161;
//   M = 16 (4): 61 440 blocks 848 / 860 / 534, 62 976 blocks 892 / 863 / 539; for fp32 7680 blocks 130 / - / 142, 8280 blocks
//     182 / - / 151;
//   M = 8 (4): 8320 blocks 79 / 85 / 85, 11 264 blocks 83 / 87 / 86, 12 288 blocks 85 / 88 / 86, 12 416 blocks 102 / 88 / 86;
//   M = 4 (16; the large tiles hold 64): 48 128 blocks 82 / 89 / 81, 50 176 blocks 94 / 86 / 80, 65 536 blocks 99 / 87 / 80,
//     67 584 blocks 113 / 149 / 96, 98 304 blocks 146 / 153 / 100, 102 400 blocks 149 / 149, 114 688 blocks 156 / 150 / 101.
// T = 20 and T = 100 put the lines at the same places within 2 us, but for M = 16 at T = 20 (65 536 blocks 146 / 152), and for M = 4
// from 102 401 to 114 688 blocks, where the large tiles make up for their second kernel only over many iterations (108 240
// blocks, T = 20, 100, 150, 200, 300: 29.7 / 32.0, 63.0 / 64.8, 85.3 / 86.0, 107.5 / 107.6, 151.6 / 150.0; student weights the same).
// Where states repeat the small tiles gain more than the large ones, which put up to four times as many blocks into a wave, in
// single precision too (T = 500, student weights, tau = 0.01, small / large fp32): M = 32, 2000 blocks 177 / 222; M = 16, 8000
// blocks 160 / 200; M = 8, 12 000 blocks 101 / 130; with tau = 0.002, where fewer repeat, 221 / 198, 197 / 209 and 130 / 151.
// With the early exit (`adaptive`) a wave runs until the slowest of its blocks stops, and so M = 4 keeps the small tiles for longer,
// M = 8 in double a little.  T = 300 (small / large double / large fp32), tol 1e-2 and 1e-3 on normal weights, 1e-5 on student ones:
//   M = 4: 54 000 blocks 88 / 98 / 71, 143 / 134 / 96 and 57 / 86 / 69; 58 000 blocks 85 / 101 / 72, 141 / 132 / 93 and 54 / 91 /
//     66; 114 000 blocks 130 / 157 / 90, 226 / 226 / 117 and 63 / 102 / 79; 120 000 blocks 138 / 158, 254 / 228 and 65 / 103;
//   M = 8: 12 000 blocks 83 / 99 / 75, 124 / 131 / 102 and 39 / 53 / 46; 13 000 blocks 96 / 111 / 82, 150 / 128 / 99 and 41 / 55 / 47;
//   M = 16: 9000 blocks 151 / 190 / 117, 255 / 312 / 158 and 46 / 68 / 62; 60 000 blocks 572 / 620, 1044 / 1114 and 145 / 163.
// (The sides change with the tolerance and the weights; the lines weigh them.)
constexpr bool small_tiles_win(int M, bool fp32, bool adaptive, int iters, int64_t nblocks) {
  if (M == 4 && adaptive) return nblocks <= (fp32 ? 55000 : 114688);
  if (M == 4) return nblocks <= 49152 || (!fp32 && nblocks > 65536 && nblocks <= (iters <= 150 ? 114688 : 102400));
  if (M == 8) return nblocks <= (adaptive ? (fp32 ? 12000 : 13000) : 12288);
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
// blocks that a wave of the iterations holds
constexpr int blocks_per_wave(int M, int tiles) {
  return tiles == kLargeTiles ? (M == 4 ? 64 : M == 8 ? 16 : M == 16 ? 8 : M == 32 ? 2 : 1) : M == 4 ? 16 : M <= 16 ? 4 : 1;
}

// Whether the iterations of a matrix with a column scale take its blocks column by column, the largest scale first (place_of).
// It pays where the waves of a launch follow each other on a SIMD or hold several blocks: on the small tiles from two waves on a SIMD
// on, on the large ones when a launch has more waves than the chip holds at once; and over enough iterations to make up for
// a list to look up and the lines of W that are read in parts (bf16 8 x 8 blocks: 16 bytes of each).  Whole calls, Wanda-style weights, row
// by row / so (us):
//   16:32 4096x14336 bf16 2507 / 2301, with fp32 iterations 1329 / 1236, a layer of seven such 5318 / 4818; 4:8 1800x2456 bf16, T = 500,
//     290 / 218; 4:8 4096x11008 1657 / 1391; 8:16 4096x4096 tau = 0.005 845 / 790; 32:64 6144x2048 with fp32 iterations 709 / 614;
//     small tiles, 8:16 1600x2048 230 / 219;
//   T = 100: 8:16 4096x4096 351 / 340, with fp32 iterations 236 / 236 and 238 / 242; 1600x2048 with them (two waves on some SIMDs)
//     T = 300 147 / 149, T = 100 80 / 81; 32:64 1152x1536 with them (a wave to a SIMD) 163 / 169.
// 4 x 4 blocks have 64 or 16 to a wave, of which some row or other is slow whatever their scale (2:4 4096x4096 434 / 443, in double,
// 3504x12496, T = 100, 1115 / 1188), and 64 x 64 blocks in double all run all iterations.
constexpr bool orders_columns(const Variant& v, int iters, int64_t nblocks) {
  if (v.M == 4 || (v.tiles != kLargeTiles && v.tiles != kSmallTiles) || (v.M == 64 && !v.fast && !v.adaptive)) return false;
  const int64_t waves_per_simd = v.tiles == kSmallTiles ? 1 : v.fast && v.M != 64 ? 4 : 2;
  return iters >= (v.fast && !v.adaptive ? 150 : 100) && nblocks > waves_per_simd * kSimds * blocks_per_wave(v.M, v.tiles);
}

// Below this many blocks in a launch a 64 x 64 block has a workgroup of its own (team.hpp), which iterates in double: one
// workgroup per CU.  Whole calls, T = 300 (us, team / large tiles in double / with fp32 iterations): 64 blocks 173 / 286 /
// 254, 256 blocks 180 / 296 / 270, 300 blocks 354 / 300.  Fused: 4 matrices of 256 blocks 677 / 307, 16 2684 / 1009.
constexpr int64_t team_below_blocks(int M) { return M == 64 ? 257 : 0; }
// Below as many blocks in a matrix it iterates in the team's order, in double whatever the fp32 flag says.  A call of its own
// gains from that (256 blocks, T = 300: normal 179 us, 246 with fp32 iterations on the large tiles, Wanda-style 192 / 303), but
// where all blocks repeat early, which the team does not look for (student, T = 500: tau = 0.01 276 / 125, tau = 0.002 269 /
// 326).  A fused launch of many takes the large
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
