// Ensemble MLP building blocks on MFMA (gfx950).
//
// Each actor is S -> H -> H -> A with tanh after every layer.  A workgroup evaluates one layer
// for a tile of 16 or 32 states: the tile's activations sit in LDS (row-major, padded rows), the
// layer's weights are pre-packed so that every lane of a wavefront fetches the B-operand of an
// MFMA with one contiguous load, and the wavefronts of the workgroup split the layer's
// 16-column output tiles between them.
//
//   float32:  v_mfma_f32_16x16x4_f32, B packed [col tile][k/16][lane][4]
//             (element e of lane l is W[16 kq + 4 e + l/16][16 c + l%16])
//   bfloat16: v_mfma_f32_16x16x32_bf16, B packed [col tile][k/32][lane][8]
//             (element j of lane l is W[32 kk + 8 (l/16) + j][16 c + l%16])
//
// In both, lane l holds rows 4(l/16)..4(l/16)+3 of column l%16 of the 16x16 accumulator.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;

enum { kF32 = 0, kBF16 = 1 };

template <int DT>
struct MT;
template <>
struct MT<kF32> {
  using act_t = float;
  static constexpr int kKGroup = 16;  // k covered by one packed load per lane
  static constexpr int kElem = 4;     // bytes per weight
};
template <>
struct MT<kBF16> {
  using act_t = __bf16;
  static constexpr int kKGroup = 32;
  static constexpr int kElem = 2;
};

__host__ __device__ inline int round_up(int x, int m) { return (x + m - 1) / m * m; }

// Device view of a packed ensemble.
struct EnsDev {
  int K, S, H, A;
  int S_pad, A_pad;  // layer-1 input and layer-3 output, padded
  const unsigned char* base;
  size_t actor_stride;
  size_t off_w1, off_w2, off_w3, off_b1, off_b2, off_b3;
  const float* mix;  // [K]
  // Split first layer (bfloat16 ensembles whose input is a trading state [cash, closes(A),
  // holdings(A), indicators]): W1 = W1e (rows of the per-environment entries: cash, holdings)
  // + W1m (rows of the market entries shared by all environments of a day).  split_a = A when
  // present, else 0.  Regions hold all actors back to back, from base.
  int split_a;
  int ke_pad;           // per-environment rows padded to a multiple of 32
  size_t off_w1e;       // [K][H/16][ke_pad/32][64][8] bfloat16 MFMA fragments
  size_t off_w1m;       // [K][S-1-A][H] bfloat16, row-major
};

// tanh from one exponential and one reciprocal: tanh|x| = (1 - e^{-2|x|}) / (1 + e^{-2|x|}).
// Absolute error below 1e-6 over the whole range.
__device__ __forceinline__ float fast_tanh(float x) {
  const float t = __builtin_amdgcn_exp2f(-2.8853900817779268f * fabsf(x));  // e^{-2|x|}
  const float y = (1.0f - t) * __builtin_amdgcn_rcpf(1.0f + t);
  return copysignf(y, x);
}

__device__ __forceinline__ floatx4 mfma_f32(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma_bf16(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace fm
