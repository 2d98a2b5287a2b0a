// The whole path for launches of a few 64 x 64 blocks: a workgroup per block.
//
// A call of a column-by-column pruning loop holds 64 or 128 such blocks, far fewer than the chip has SIMDs.  What it takes is
// the dependent chain of an iteration, and a lone wave issues a vector instruction every ~2.6 ns whatever its kind: with a
// block on one wave (the large tiles) 384 of them, 1 us per iteration.  So a block is spread over the 8 waves of a workgroup,
// two on each SIMD of a CU.  Lane = in-kernel column; a wave holds 8 rows of all 64 columns:
//   * row sums stay inside a wave: reduce-scatter over 16 lanes on DPP, then v_permlane16_swap / v_permlane32_swap, whose
//     two results added are the sum over a pair of rows of lanes, in every lane, without a select;
//   * column sums cross the workgroup: every wave leaves its partial sums in LDS, one barrier, and every lane adds up its own
//     column - no gather, the lane that needs a column scaling is the one that forms it.  Two buffers, so that one barrier
//     per iteration is enough: a buffer is written again two barriers after it was read.
// The rows are rescaled between the LDS write and the barrier.  Rounding follows in the first wave (round_blocks).
// 64 blocks of 32:64, T = 300: 286 us a call on the large tiles (254 with fp32 iterations), 171 here; of the 0.5 us per
// iteration the issue of two waves' 93 instructions is 0.36, the LDS round trip with the barrier the rest.  (32 x 32 blocks on
// four waves the same way: 285 ns per iteration; one wave takes 267, for 115 instructions.)  A launch that fills the
// chip takes the large tiles, which add in the same order with fewer instructions per block (374 against 744).
#pragma once
#include "dykstra_sort.hpp"

namespace tsenor_dev {

struct Team {
  static constexpr int M = 64, W = 8, TH = M / W;  // waves, rows per wave
  static constexpr int NX = 4;                     // the lane-row of 16 (reduce_scatter_x and all_gather_x)
  static constexpr int XM[4] = {15, 7, 3, 1};
};

template <bool ADAPT>
__global__ __launch_bounds__(Team::W * kWave, 2) void team_kernel(Batch batch) {
  using T = Team;
  constexpr int M = T::M, TH = T::TH, SHX = ilog2(TH) - T::NX;
  static_assert(owned(TH, T::NX) == 1, "one owned row per lane");
  __shared__ double part[2][T::W][M];   // partial column sums
  __shared__ double pot[2][1][M];        // potentials of the matrix rows and columns
  __shared__ double wave_worst[T::W];
  __shared__ RoundingLds<M, 1> lds;
  const int which = find_problem(batch, blockIdx.x);
  const BatchEntry& e = batch.e[which];
  const DevProblem p = e.p;
  const int64_t blk = blockIdx.x - batch.first[which];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int row0 = wave * TH, rx = shift_lane(lane & 15, SHX);
  // The column of a lane, so that the row sums are added in the order of the large tiles (order_run in dykstra_sort.hpp): the
  // steps over lanes 15, 7 and 3 apart change rx and keep the parity of bits 0 and 1, the later ones change one of the rest.
  const int gx = (((lane ^ (lane >> 1)) & 1) * 7) ^ (((lane >> 4) & 1) * 3) ^ ((lane >> 5) & 1), col = gx * TH + rx;
  const BlockAt at = block_at(p, blk, M);
  const double tau_eff = tau_eff_of(e);
  if (e.tau_eff_out && blk == 0 && threadIdx.x == 0) *e.tau_eff_out = tau_eff;

  // register a of this lane <-> in-kernel entry (row0 + (a ^ rx), col); in-kernel rows are matrix columns under `transpose`
  int ri[TH];
  const int cj[1] = {col};
#pragma unroll
  for (int a = 0; a < TH; ++a) ri[a] = row0 + (a ^ rx);
  const auto addr = tile_addr<TH, 1>(p, at.r0, at.c0, ri, cj);
  double kap[TH];
  float mrow[TH];  // not below the largest K of every row (see dykstra_sort_kernel)
  {
    float imp[TH][1];
    tile_importance<0, TH, false>(p, addr, imp);
#pragma unroll
    for (int a = 0; a < TH; ++a) {
      kap[a] = tau_eff * (double)imp[a][0];
      mrow[a] = round_up(kap[a]);
    }
  }
  all_reduce_max_x<T, TH>(mrow);
#pragma unroll
  for (int a = 0; a < TH; ++a) {
    mrow[a] = fmaxf(mrow[a], lane_xor<16>(mrow[a]));
    mrow[a] = fmaxf(mrow[a], lane_xor<32>(mrow[a]));
    kap[a] = exp_in_range(fmax(kap[a] - (double)mrow[a], kMinLogKernel));
  }

  const double Nd = (double)p.N;
  double U = 1.0, V = 1.0;  // scalings of the owned row (register 0) and of this lane's column
  int iters_done = p.T;
  const long long cycles0 = clock64(), ticks0 = wall_clock64();
  for (int t = 0; t < p.T; ++t) {
    // projection onto C1 (line 3) of the plan capped by the previous iteration
    double ev[TH], R[TH];
#pragma unroll
    for (int a = 0; a < TH; ++a) R[a] = ev[a] = clamp01(kap[a] * V);
    reduce_scatter_x<T, double, TH>(R);
    R[0] = swap_sum<16>(R[0], R[0]);
    R[0] = swap_sum<32>(R[0], R[0]);
    R[0] = fast_div(Nd, R[0]);
    double worst = ADAPT ? fabs(R[0] - 1.0) : 0.0;
    U *= R[0];
    all_gather_x<T, double, TH>(R);
    // projection onto C2 (line 4)
    double C = ev[0] * R[0];
#pragma unroll
    for (int a = 1; a < TH; ++a) C = fma(ev[a], R[a], C);
    part[t & 1][wave][lane] = C;
#pragma unroll
    for (int a = 0; a < TH; ++a) kap[a] *= R[a];
    __syncthreads();
    double s[T::W];
#pragma unroll
    for (int k = 0; k < T::W; ++k) s[k] = part[t & 1][k][lane];
#pragma unroll
    for (int h = 1; h < T::W; h *= 2)  // (neighbours first, as the large tiles' lane-columns do)
#pragma unroll
      for (int k = 0; k < T::W; k += 2 * h) s[k] += s[k + h];
    C = fast_div(Nd, s[0]);
    V *= C;
    // lines 5-6 (cap and dual update) are the clamp at the top of the next pass
    if constexpr (ADAPT) {
      if ((t + 1) % TSENOR_ADAPTIVE_CHECK_EVERY == 0) {
        worst = block_max<kWave>(vmax(worst, fabs(C - 1.0)));
        if (lane == 0) wave_worst[wave] = worst;
        __syncthreads();
        worst = wave_worst[0];
#pragma unroll
        for (int w = 1; w < T::W; ++w) worst = vmax(worst, wave_worst[w]);
        if (worst <= p.tol) {
          iters_done = t + 1;
          break;
        }
      }
    }
  }
  if (blk == 0 && threadIdx.x == 0) {
    e.hdr->loop_cycles = (unsigned long long)(clock64() - cycles0);
    e.hdr->loop_ticks = (unsigned long long)(wall_clock64() - ticks0);
  }

  double lu[TH];
  lu[0] = log(U);
  const double lv = log(V);
  pot[p.transpose ? 1 : 0][0][ri[0]] = lu[0];
  lds.minus_largest[0][ri[0]] = -(double)mrow[0];
  pot[p.transpose ? 0 : 1][0][col] = lv;
  if (threadIdx.x == 0 && e.iters_done_out) e.iters_done_out[blk] = iters_done;
  if (e.plan_out) {
    all_gather_x<T, double, TH>(lu);
    float imp[TH][1];
    tile_importance<0, TH, false>(p, addr, imp);
#pragma unroll
    for (int a = 0; a < TH; ++a) {
      const int64_t r = at.r0 + (p.transpose ? col : ri[a]), c = at.c0 + (p.transpose ? ri[a] : col);
      e.plan_out[r * p.cols + c] = exp(fmin((tau_eff * (double)imp[a][0] - (double)mrow[a]) + (lu[a] + lv), 0.0));
    }
  }
  __syncthreads();
  if (wave == 0) {
    if (p.transpose)
      round_blocks<M, kWave, false, true>(p, e, blk, true, at.r0, at.c0, lane, tau_eff, pot[0], pot[1], lds);
    else
      round_blocks<M, kWave, false, false>(p, e, blk, true, at.r0, at.c0, lane, tau_eff, pot[0], pot[1], lds);
  }
}

}  // namespace tsenor_dev
