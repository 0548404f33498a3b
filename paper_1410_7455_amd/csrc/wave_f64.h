// fp64 pieces that the eigen-solvers share: sums within a wavefront, reciprocals, Householder reflections.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ngsgd {

// Sum over the 64 lanes without LDS: the 16 lanes of a row through the vector ALU's cross-lane path, the four rows
// through scalar registers.
template <int CTRL>
__device__ __forceinline__ double dpp_add_f64(const double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double read_lane_f64(const double v, const int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double row16_sum_f64(double v) {
  v = dpp_add_f64<0xB1>(v);    // quad_perm [1,0,3,2]
  v = dpp_add_f64<0x4E>(v);    // quad_perm [2,3,0,1]
  v = dpp_add_f64<0x141>(v);   // row_half_mirror
  return dpp_add_f64<0x140>(v);   // row_mirror
}
template <int CTRL>
__device__ __forceinline__ double dpp_max_f64(const double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return fmax(v, __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double row16_max_f64(double v) {
  v = dpp_max_f64<0xB1>(v);
  v = dpp_max_f64<0x4E>(v);
  v = dpp_max_f64<0x141>(v);
  return dpp_max_f64<0x140>(v);
}
// Product over the lanes below (UP) or above this one in its row of 16; 1 where there are none.
template <int CTRL>
__device__ __forceinline__ double dpp_or_one_f64(const double v) {   // lanes without a source take 1
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0x3ff00000, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <bool UP>
__device__ __forceinline__ double row16_scan_product(double v) {
  constexpr int SHIFT = UP ? 0x110 : 0x100;   // row_shr, row_shl by the low bits
  v = dpp_or_one_f64<SHIFT + 1>(v);
  v *= dpp_or_one_f64<SHIFT + 1>(v);
  v *= dpp_or_one_f64<SHIFT + 2>(v);
  v *= dpp_or_one_f64<SHIFT + 4>(v);
  return v * dpp_or_one_f64<SHIFT + 8>(v);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_min_u32(const uint32_t v) {
  return min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ uint32_t row16_min_u32(uint32_t v) {
  v = dpp_min_u32<0xB1>(v);
  v = dpp_min_u32<0x4E>(v);
  v = dpp_min_u32<0x141>(v);
  return dpp_min_u32<0x140>(v);
}
// Sum over the 16 lanes that share (lane / 4) % 4, to all of them, by two instructions of the fp64 matrix unit (54 cycles; through the
// vector ALU's cross-lane path 12 instructions): v_mfma_f64_4x4x4_4b_f64 takes A[lane % 4][lane / 16] and B[lane / 16][lane % 4] and
// leaves D[lane / 16][lane % 4], for the four blocks (lane / 4) % 4.  The whole wavefront takes part.
__device__ __forceinline__ int group16_index() { return ((threadIdx.x >> 2) & 3); }                           // of the group
__device__ __forceinline__ int group16_member() { return (threadIdx.x & 3) | ((threadIdx.x >> 2) & 12); }   // within it
__device__ __forceinline__ int group16_lane(const int member) { return (member & 3) | ((member & 12) << 2); }   // of group 0
__device__ __forceinline__ double group16_sum_f64(const double v) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, __builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0), 0.0, 0, 0, 0);
}
// Over the 64 lanes, to all of them: 8 instructions where wave_sum_uniform takes 23, in one chain that is longer.
__device__ __forceinline__ double wave_sum_f64(double v) {
  v = group16_sum_f64(v);
  v = dpp_add_f64<0x141>(v);      // row_half_mirror: groups 0 and 1, 2 and 3
  return dpp_add_f64<0x140>(v);   // row_mirror
}
__device__ __forceinline__ double wave_sum_uniform(double v) {
  v = row16_sum_f64(v);
  return (read_lane_f64(v, 0) + read_lane_f64(v, 16)) + (read_lane_f64(v, 32) + read_lane_f64(v, 48));
}
// all 256 threads; `red` holds 4 doubles, and another call with the same array is a barrier away
__device__ __forceinline__ double block256_sum_f64(double v, double* red) {
  v = wave_sum_uniform(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// What a wavefront's lanes wrote to LDS before is what its lanes read behind it.  The hardware performs a wavefront's LDS
// operations in order; the fences keep the compiler to that order too (the barrier alone does not order memory for it).
// Costs no instruction.
__device__ __forceinline__ void wave_lds_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double reciprocal_f64(const double x) {   // hardware estimate, two Newton steps
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
// Reflection that maps (x0, tail) to (beta, 0), sigma the sum of squares of the tail: I - tau v v^T with v = (1, scale tail).
struct Reflection {
  double beta, tau, scale;
};
__device__ __forceinline__ Reflection reflection(const double x0, const double sigma) {
  Reflection h;
  h.beta = x0;
  h.tau = h.scale = 0.0;
  const double nn = fma(x0, x0, sigma);
  if (sigma > 0.0 && nn > 1.0e-290) {   // (below: the column is zero)
    double r = __builtin_amdgcn_rsq(nn);   // hardware estimate, two Newton steps
    r = fma(0.5 * r, fma(-nn * r, r, 1.0), r);
    r = fma(0.5 * r, fma(-nn * r, r, 1.0), r);
    const double norm = nn * r, size = fabs(x0) + norm;
    h.beta = x0 > 0.0 ? -norm : norm;
    h.tau = fma(fabs(x0), r, 1.0);
    h.scale = reciprocal_f64(x0 > 0.0 ? size : -size);
  }
  return h;
}

}  // namespace ngsgd
