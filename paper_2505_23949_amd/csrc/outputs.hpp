// Kernels behind the optional outputs of a call: the objective of Eq. (1) with the safeguard verdict, and the
// outputs derived from the final mask (bit-packed mask, pruned values).  They do not depend on the block size.
#pragma once
#include "problem.hpp"

namespace tsenor_dev {

// Sums of the per-block objectives, workgroup by workgroup (blockIdx.y: matrix).  Every order is fixed: bitwise
// reproducible.  One workgroup per matrix took 0.1 ms for 262 144 blocks (256 dependent loads per thread); up to
// kObjectiveAloneBlocks (four) the first workgroup does it alone and writes the result, so that a call that wants only the
// sums of small matrices has one launch of one workgroup each for them (2:4, two matrices of 741 blocks: 18.0 us a call with
// 64 and a second launch, 17.0 so).
constexpr int64_t kObjectiveAloneBlocks = 4 * 256;
__device__ __forceinline__ bool previous_mask_wins(const BatchEntry& e, double2 sums) { return e.prev_mask && sums.y > sums.x; }
__device__ __forceinline__ void write_objectives(const BatchEntry& e, double2 sums) {
  e.objective_out[0] = previous_mask_wins(e, sums) ? sums.y : sums.x;
  e.objective_out[1] = e.prev_mask ? sums.y : 0.0;
}
__global__ __launch_bounds__(256) void objective_kernel(Batch batch) {
  const BatchEntry& e = batch.e[blockIdx.y];
  const bool alone = e.p.nblocks <= kObjectiveAloneBlocks;
  if (!e.block_objective || (alone && blockIdx.x != 0)) return;
  const double2* objective = reinterpret_cast<const double2*>(e.block_objective);
  __shared__ double2 part[4];
  double a = 0.0, b = 0.0;
  const int64_t step = (alone ? 1 : kObjectiveGroups) * 256;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < e.p.nblocks; k += step) {
    const double2 v = objective[k];
    a += v.x;
    b += v.y;
  }
  for (int s = 1; s < 64; s <<= 1) {
    a += __shfl_xor(a, s, 64);
    b += __shfl_xor(b, s, 64);
  }
  if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = make_double2(a, b);
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      a += part[w].x;
      b += part[w].y;
    }
    reinterpret_cast<double2*>(e.absmax_partial)[blockIdx.x] = make_double2(a, b);
    if (alone && e.objective_out) write_objectives(e, make_double2(a, b));
  }
}

// The objectives of the mask found and of the previous mask, in every lane of the calling wave (a butterfly gives all
// lanes the same sum; what one workgroup has summed comes through it as it is).
__device__ __forceinline__ double2 objectives_of(const BatchEntry& e) {
  static_assert(kObjectiveGroups == 64, "one partial sum per lane");
  const int lane = threadIdx.x % 64;
  double2 v = make_double2(0.0, 0.0);
  if (lane == 0 || e.p.nblocks > kObjectiveAloneBlocks) v = reinterpret_cast<const double2*>(e.absmax_partial)[lane];
  for (int s = 1; s < 64; s <<= 1) {
    v.x += __shfl_xor(v.x, s, 64);
    v.y += __shfl_xor(v.y, s, 64);
  }
  return v;
}

// round to nearest even; x is finite
__device__ __forceinline__ unsigned int bf16_bits(float x) {
  const unsigned int u = __float_as_uint(x);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// the 8 values x (load_value) from column c of row r on, with 16-byte loads
template <bool BF16>
__device__ __forceinline__ void load_8(const void* base, int64_t index, float (&x)[8]) {
  if constexpr (BF16) {
    const uint4 raw = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned short*>(base) + index);
    const unsigned int w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[2 * k] = __uint_as_float(w[k] << 16);
      x[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
    }
  } else {
    const float4* src = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + index);
    const float4 lo = src[0], hi = src[1];
    x[0] = lo.x, x[1] = lo.y, x[2] = lo.z, x[3] = lo.w, x[4] = hi.x, x[5] = hi.y, x[6] = hi.z, x[7] = hi.w;
  }
}
template <bool BF16>
__device__ __forceinline__ void prune_8(const DevProblem& p, void* out, int64_t from, int64_t to, unsigned int bits) {
  float x[8];
  load_8<BF16>(p.W, from, x);
  if (p.add) {
    float v[8];
    load_8<BF16>(p.add, from, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = __fadd_rn(x[k], __fmul_rn(p.add_scale, v[k]));
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = ((bits >> k) & 1) ? x[k] : 0.0f;
  if constexpr (BF16) {
    *reinterpret_cast<uint4*>(reinterpret_cast<unsigned short*>(out) + to) =
        make_uint4(bf16_bits(x[0]) | bf16_bits(x[1]) << 16, bf16_bits(x[2]) | bf16_bits(x[3]) << 16,
                   bf16_bits(x[4]) | bf16_bits(x[5]) << 16, bf16_bits(x[6]) | bf16_bits(x[7]) << 16);
  } else {
    float4* dst = reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + to);
    dst[0] = make_float4(x[0], x[1], x[2], x[3]);
    dst[1] = make_float4(x[4], x[5], x[6], x[7]);
  }
}

// Outputs derived from the final mask, 8 consecutive weights of a row per thread: the safeguard verdict of App. A.1
// (Assumption 1: the previous mask is kept if it scores strictly higher), the previous mask copied over the new one if
// the verdict says so, the bit-packed mask, and the pruned values x * S.  Bound by memory where the buffers are aligned
// (one load or store of 8 weights each).  With objective_kernel and the pre-pass on the additive term read the same way,
// a whole 4:8 call on 4096 x 4096 fp32 with all these outputs went from 1368 to 1090 us.
__global__ __launch_bounds__(256) void emit_kernel(Batch batch) {
  // blockIdx.z: matrix of the batch; x and y stride over its 8-weight vectors and rows
  const BatchEntry& e = batch.e[blockIdx.z];
  const uint8_t* prev_mask = e.prev_mask;
  uint8_t* packed_out = e.packed_out;
  void* pruned_out = e.pruned_out;
  const DevProblem p = e.p;
  bool use_prev = false;
  if (e.block_objective) {
    const double2 sums = objectives_of(e);
    use_prev = previous_mask_wins(e, sums);
    if (e.objective_out && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) write_objectives(e, sums);
  }
  if (!use_prev && !packed_out && !pruned_out) return;
  const int64_t rows = e.rows;
  uint8_t* mask = e.mask;
  const int64_t per_row = p.cols / 8;
  // a workgroup handles a contiguous band of rows
  const int64_t band = (rows + gridDim.y - 1) / gridDim.y;
  const int64_t r_end = (blockIdx.y + 1) * band < rows ? (blockIdx.y + 1) * band : rows;
  for (int64_t r = blockIdx.y * band; r < r_end; ++r)
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < per_row; v += (int64_t)gridDim.x * blockDim.x) {
      const int64_t c = v * 8, at = r * p.cols + c;
      if (e.emit_vec) {
        uint2 s = *reinterpret_cast<const uint2*>((use_prev ? prev_mask : mask) + at);
        if (use_prev) *reinterpret_cast<uint2*>(mask + at) = s;
        // the lowest bits of four bytes next to each other: no two products of the multiplication meet in a bit
        const unsigned int bits =
            (((s.x & 0x01010101u) * 0x10204080u) >> 28) | ((((s.y & 0x01010101u) * 0x10204080u) >> 28) << 4);
        if (packed_out) packed_out[r * per_row + v] = (uint8_t)bits;
        if (pruned_out) {
          if (p.dtype == TSENOR_BF16)
            prune_8<true>(p, pruned_out, r * p.ld + c, at, bits);
          else
            prune_8<false>(p, pruned_out, r * p.ld + c, at, bits);
        }
        continue;
      }
      unsigned int bits = 0;
      for (int k = 0; k < 8; ++k) {
        uint8_t s = mask[at + k];
        if (use_prev) {
          s = prev_mask[at + k];
          mask[at + k] = s;
        }
        bits |= (unsigned int)(s & 1) << k;
      }
      if (packed_out) packed_out[r * per_row + v] = (uint8_t)bits;
      if (pruned_out) {
        for (int k = 0; k < 8; ++k) {
          const float x = ((bits >> k) & 1) ? load_value(p, r, c + k) : 0.0f;
          if (p.dtype == TSENOR_BF16)
            reinterpret_cast<unsigned short*>(pruned_out)[at + k] = (unsigned short)bf16_bits(x);
          else
            reinterpret_cast<float*>(pruned_out)[at + k] = x;
        }
      }
    }
}

}  // namespace tsenor_dev
