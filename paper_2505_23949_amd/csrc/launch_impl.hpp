// Body of launch_block_kernels<M>: picks the instantiation of every kernel that depends on M and enqueues it.
// Included by exactly one translation unit per M.
#pragma once
#include "dykstra_sort.hpp"
#include "launch.hpp"
#include "team.hpp"

namespace tsenor_dev {

// prefix of workgroup counts when every matrix gets ceil(blocks / per_group) workgroups; false on overflow
inline bool assign_groups(Batch& b, int64_t per_group) {
  int64_t total = 0;
  for (int k = 0; k < b.count; ++k) {
    b.first[k] = (unsigned)total;
    total += (b.e[k].p.nblocks + per_group - 1) / per_group;
    if (total > 0x7FFFFFFF) return false;
  }
  for (int k = b.count; k <= kMaxBatch; ++k) b.first[k] = (unsigned)total;
  return true;
}

// Whether the workgroups assigned give a SIMD no second wave.
inline bool lone_waves(const Batch& b, int waves_per_group) { return (uint64_t)b.first[b.count] * waves_per_group <= kSimds; }
// Block sizes that come to the large tiles with so few without a flag: 64 x 64 (257 to 1024 blocks) and 4 x 4.  The others have
// the small tiles for launches like that.
template <int M>
constexpr bool kLoneOnLargeTiles = M == 64 || M == 4;

template <int M>
bool launch_block_kernels(Batch& b, const Variant& v, hipStream_t stream, hipEvent_t ev_sorted, hipEvent_t ev_greedy) {
  constexpr int BPW = kWave >> (Tiling<M>::NX + Tiling<M>::NY);
  static_assert(BPW == blocks_per_wave(M, kLargeTiles), "");
  int64_t nblocks = 0;  // of the whole launch
  for (int k = 0; k < b.count; ++k) nblocks += b.e[k].p.nblocks;
  const bool team_fits = nblocks < team_below_blocks(M);
  if (v.tiles != kLargeTiles && !(v.tiles == kTeam && !team_fits)) {
    // the small tiles carry Algorithm 2 behind the iterations: this one kernel is the whole path
    const auto launch = [&](auto tiles) {
      constexpr int TILES = decltype(tiles)::value;
      constexpr int BPWS = kWave >> (Tiling<M, TILES>::NX + Tiling<M, TILES>::NY);
      static_assert(TILES != kSmallTiles || BPWS == blocks_per_wave(M, kSmallTiles), "");
      using L = DykstraLaunch<M, false, false, TILES>;
      static_assert(L::kWavesPerGroup == 1 && DykstraLaunch<M, false, true, TILES>::kWavesPerGroup == 1, "");
      if (!assign_groups(b, (int64_t)BPWS)) return false;
      const bool lone = lone_waves(b, L::kWavesPerGroup);
      if (v.adaptive && lone)
        dykstra_sort_kernel<M, false, false, TILES, true, true><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
      else if (v.adaptive)
        dykstra_sort_kernel<M, false, false, TILES, true><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
      else if (lone)
        dykstra_sort_kernel<M, false, false, TILES, false, true><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
      else
        dykstra_sort_kernel<M, false, false, TILES><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
      return true;
    };
    bool ok = false;
    if constexpr (M <= 32) {
      if (v.tiles == kSmallTiles) ok = launch(std::integral_constant<int, kSmallTiles>{});
    }
    if constexpr (finest_tiles_below_blocks(M) > 0) {
      if (v.tiles == kFinestTiles)
        ok = nblocks <= kFinestTilesLaunch ? launch(std::integral_constant<int, kFinestTiles>{})
                                                    : launch(std::integral_constant<int, kFinestOrderTiles>{});
    }
    if constexpr (M == Team::M) {
      if (v.tiles == kTeam) {
        if (!assign_groups(b, 1)) return false;
        if (v.adaptive)
          team_kernel<true><<<b.first[b.count], Team::W * kWave, 0, stream>>>(b);
        else
          team_kernel<false><<<b.first[b.count], Team::W * kWave, 0, stream>>>(b);
        ok = true;
      }
    }
    if (!ok) return false;
    if (ev_sorted) (void)hipEventRecord(ev_sorted, stream);
    if (ev_greedy) (void)hipEventRecord(ev_greedy, stream);
    return true;
  } else if (v.fast && v.adaptive) {
    using L = DykstraLaunch<M, true, true>;
    if (!assign_groups(b, (int64_t)BPW * L::kWavesPerGroup)) return false;
    dykstra_sort_kernel<M, true, false, false, true><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
  } else if (v.fast) {
    // (fp32 iterations keep their priorities: a launch of lone waves differs in its workgroups, DykstraLaunch)
    using L = DykstraLaunch<M, true>;
    using LL = DykstraLaunch<M, true, false, kLargeTiles, true>;
    constexpr bool kLone = LL::kWavesPerGroup != L::kWavesPerGroup;
    if (!assign_groups(b, (int64_t)BPW * LL::kWavesPerGroup)) return false;
    if (kLone && lone_waves(b, LL::kWavesPerGroup)) {
      dykstra_sort_kernel<M, true, false, kLargeTiles, false, kLone><<<b.first[b.count], LL::kThreads, 0, stream>>>(b);
    } else {
      if (kLone && !assign_groups(b, (int64_t)BPW * L::kWavesPerGroup)) return false;
      dykstra_sort_kernel<M, true><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
    }
  } else {
    using L = DykstraLaunch<M, false>;
    using LA = DykstraLaunch<M, false, true>;
    if (!assign_groups(b, (int64_t)BPW * (v.adaptive ? LA::kWavesPerGroup : L::kWavesPerGroup))) return false;
    if (v.zero_t) {
      // (M >= 8: the rounding kernel starts from the importance itself, this one only writes a plan that is asked for)
      bool any_plan = M < 8;
      for (int k = 0; k < b.count; ++k) any_plan |= b.e[k].plan_out != nullptr;
      if (any_plan) dykstra_sort_kernel<M, false, true><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
    } else if (v.adaptive)
      dykstra_sort_kernel<M, false, false, false, true><<<b.first[b.count], LA::kThreads, 0, stream>>>(b);
    else if (kLoneOnLargeTiles<M> && lone_waves(b, L::kWavesPerGroup))
      dykstra_sort_kernel<M, false, false, kLargeTiles, false, kLoneOnLargeTiles<M>><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
    else
      dykstra_sort_kernel<M, false><<<b.first[b.count], L::kThreads, 0, stream>>>(b);
  }
  if (ev_sorted) (void)hipEventRecord(ev_sorted, stream);
  if constexpr (M >= 8) {
    // the whole of Algorithm 2 in one kernel
    if (!assign_groups(b, kWave / M)) return false;
    if (v.zero_t)
      round_kernel<M, true><<<b.first[b.count], kWave, 0, stream>>>(b);
    else
      round_kernel<M, false><<<b.first[b.count], kWave, 0, stream>>>(b);
    if (ev_greedy) (void)hipEventRecord(ev_greedy, stream);
  } else {
    if (ev_greedy) (void)hipEventRecord(ev_greedy, stream);
    if (!assign_groups(b, kWave / M)) return false;
    finalize_kernel<M><<<b.first[b.count], kWave, 0, stream>>>(b);
  }
  return true;
}

}  // namespace tsenor_dev
