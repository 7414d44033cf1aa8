// Cross-lane FP64 reductions on the DPP network and the permlane swaps
// (CDNA4, wave64).  Every lane of a reduced group ends with the same value:
// each step adds the same two partial sums, in either order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace odmd {

// LDS written by some lanes of a wavefront is read by others of it next (the
// wavefront's LDS operations complete in order; the fence keeps the compiler
// from reordering them)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  // (every lane is written, an inactive source lane reads as zero)
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// sum over each 16-lane row: quad swaps, then the half-row and row mirrors
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_move<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return v;
}

// the same over each 8-lane half of a row
__device__ __forceinline__ double oct_sum(double v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  return v;
}

__device__ __forceinline__ int oct_sum(int v) {
  v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
  v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
  v += __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);
  return v;
}

__device__ __forceinline__ double oct_prod(double v) {
  v *= dpp_move<0xB1>(v);
  v *= dpp_move<0x4E>(v);
  v *= dpp_move<0x141>(v);
  return v;
}

// v + the value of the same lane position in the neighbouring 16-lane row
// (rows 0 <-> 1, 2 <-> 3): the swap leaves own and partner value in its two
// outputs
__device__ __forceinline__ double add_row_pair(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  return __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) +
         __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
}

// v + the value of the same lane position in the other 32-lane half
__device__ __forceinline__ double add_half_pair(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  return __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) +
         __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
}

// the largest value of the wavefront (no NaN expected: fmax drops it)
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_move<0xB1>(v));
  v = fmax(v, dpp_move<0x4E>(v));
  v = fmax(v, dpp_move<0x141>(v));
  v = fmax(v, dpp_move<0x140>(v));
  uint64_t u = __builtin_bit_cast(uint64_t, v);
  auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
  auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  v = fmax(__builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)),
           __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32)));
  u = __builtin_bit_cast(uint64_t, v);
  lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
  hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  return fmax(__builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)),
              __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32)));
}

// sum over each 32-lane half
__device__ __forceinline__ double halfwave_sum(double v) { return add_row_pair(row_sum(v)); }

}  // namespace odmd
