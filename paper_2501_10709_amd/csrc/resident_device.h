// Helpers shared by the rollout kernels that hold the ensemble's second-layer weights on chip.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "mlp_device.h"

namespace fm {

constexpr int kRK = 3, kRH = 256, kRKK = 8;  // actors, hidden units, k-steps of 32 per hidden layer
constexpr int kRX0 = 40;                     // state-row stride (bfloat16): cash, <= 31 holdings, zeros
constexpr int kRIn = 256;                    // market entries per day, (2 + I) * D <= 256
// An input buffer in LDS: close[t] | close[t+1] in floats 0 .. 2D-1, ind[t+1] from float kRInd
// (the fetch writes whole runs of 64 floats, so the two parts do not overlap).
constexpr int kRInd = 64;
constexpr int kRInBuf = kRInd + 256;

// An opaque zero: values derived from it are recomputed where they are used instead of being
// hoisted out of the step loop and held in registers.
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+s"(z));
  return z;
}

// Four activations as bfloat16 (round to nearest even), 8 bytes.
__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const bf16x2 lo = {static_cast<__bf16>(a), static_cast<__bf16>(b)};
  const bf16x2 hi = {static_cast<__bf16>(c), static_cast<__bf16>(d)};
  return uint2{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
}

// Trajectory stores go through buffer resources that cover the tile's rows of one step: a lane
// with nothing to store passes an offset beyond the range, which the hardware drops, so the
// stores need no branches; a trajectory that is not requested gets an empty range.
constexpr int kNoStore = 1 << 30;  // beyond every range; adding a row offset stays below 2^31
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void* base, size_t elem_offset, size_t elem_bytes,
                                                            int n_elems) {
  if (!base) return __builtin_amdgcn_make_buffer_rsrc(nullptr, 0, 0, 0x00020000);
  return __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(static_cast<const char*>(base)) + elem_offset * elem_bytes, 0,
      static_cast<int>(elem_bytes * n_elems), 0x00020000);
}
__device__ __forceinline__ void store_f32(__amdgpu_buffer_rsrc_t r, int byte_off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, byte_off, 0, 0);
}
// A load through such a resource returns 0 beyond its range.
__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t r, int byte_off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0));
}

// The market rows close[t] | close[t+1] | ind[t+1] of day t into an input buffer in LDS by one
// wavefront, 64 floats per load, lanes past a range writing zeros.
__device__ __forceinline__ void fetch_market(const EnvConst& C, int t, float* in, int lane) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rows_rsrc(C.close, static_cast<size_t>(t) * C.D, 4, 2 * C.D), in, 4, 4 * lane,
                                           0, 0, 0);
  const int n = C.I * C.D;
  const __amdgpu_buffer_rsrc_t ri = rows_rsrc(C.ind, static_cast<size_t>(t + 1) * n, 4, n);
  for (int q = 0; 64 * q < n; ++q)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ri, in + kRInd + 64 * q, 4, 4 * (lane + 64 * q), 0, 0, 0);
}

}  // namespace fm
