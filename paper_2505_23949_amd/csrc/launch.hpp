// Interface between the host code of the library and the kernels that depend on the block size M.  The
// kernels of every M are compiled in a translation unit of their own (launch_m4.hip ... launch_m64.hip, all of
// them instantiating launch_impl.hpp), so that the library builds in parallel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "problem.hpp"

namespace tsenor_dev {

// how the Dykstra kernel spreads a block over lanes (see Tiling in dykstra_sort.hpp)
enum { kLargeTiles, kSmallTiles, kFinestTiles, kTeam };

// kernel variant of a problem: problems with the same variant can share one fused launch
struct Variant {
  int M;
  bool fast, zero_t;
  int tiles;        // the Dykstra kernel's tiling (decided per problem, so that fusing never changes results)
  bool simple;      // TSENOR_FLAG_SIMPLE_ROUNDING
  bool adaptive;    // tol > 0: the early-exit instantiation of the Dykstra kernel
  bool operator==(const Variant& o) const {
    return M == o.M && fast == o.fast && zero_t == o.zero_t && tiles == o.tiles &&
           simple == o.simple && adaptive == o.adaptive;
  }
};

// Below this many blocks in a matrix the whole path runs in the one kernel with the small tiles (M <= 32, double
// iterations): with few waves a SIMD holds one or two, whose iteration time is the dependent chain, and the
// rounding needs no launches of its own.  `fp32`: the caller asked for single-precision iterations, which only
// the large tiles have, so they win earlier.  Measured crossovers of a whole call, T = 300 (ms, small / large
// fp64 / large fp32): M = 32: 3072 blocks 0.259 / 0.280 / 0.216, 3328 blocks 0.314 / 0.286 / 0.222, 2048 blocks
// 0.189 / 0.198 / 0.188; M = 16: 8192 blocks 0.165 / 0.202 / 0.182, 9216 blocks 0.209 / 0.258 / 0.196, 32 768
// blocks 0.484 / 0.492 / 0.367, 65 536 blocks 0.916 / 0.886 / 0.567; M = 8: 12 288 blocks 0.102 / 0.104 / 0.101,
// 16 384 blocks 0.128 / 0.107 / 0.102; M = 4: 49 152 blocks 0.085 / 0.104 / 0.095, 57 344 blocks 0.107 / 0.106 /
// 0.097, 81 920 blocks 0.133 / 0.174 / 0.113, 131 072 blocks 0.199 / 0.186 / 0.126.
constexpr int64_t small_tiles_below_blocks(int M, bool fp32) {
  return M == 4 ? (fp32 ? 55000 : 100000) : M == 8 ? (fp32 ? 12000 : 13000) : M == 16 ? (fp32 ? 9000 : 40000)
       : M == 32 ? (fp32 ? 2100 : 3200) : 0;
}

// Below this many blocks a 16 x 16 block has a wave of its own: 51 instead of 98 vector instructions in the chain of an
// iteration, four times the waves.  Whole calls, T = 300 (us, finest / small tiles): 256 blocks 67 / 88, 1024 blocks
// 73 / 89, 1536 blocks 81 / 90, 2304 blocks 104 / 90 (from three waves on a SIMD on, issue decides).
constexpr int64_t finest_tiles_below_blocks(int M) { return M == 16 ? 1800 : 0; }

// Below this many blocks a 64 x 64 block has a workgroup of its own (team.hpp), which iterates in double: one workgroup per
// CU.  Whole calls, T = 300 (us, team / large tiles in double / with fp32 iterations): 64 blocks 185 / 292 / 369, 256 blocks
// 189 / 299 / 377, 300 blocks 354 / 300.
constexpr int64_t team_below_blocks(int M) { return M == 64 ? 257 : 0; }

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
