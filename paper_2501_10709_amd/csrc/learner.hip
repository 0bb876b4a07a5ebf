// The learner that consumes the rollout's samples (include/learner.h): the policy gradient of
// eq. (4) with the agent-diversity term of eq. (5), by the chain rule through agent i's network.
//
// Pipeline, all on the caller's stream: the K actors' forward passes over the T*N sample rows
// (agent i last, so its layer activations stay in the workspace); the returns R_n; per row the
// derivative of the objective with respect to mu_i, times tanh' (the layer-3 delta); then back
// through layers 3, 2, 1: each weight and bias gradient [X | 1]^T G is a reduction over the rows,
// split over row chunks into float32 partial products and summed in float64 in chunk order; each
// delta of the layer below is (G W^T) * (1 - X^2), written over the activation it masks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>
#include <type_traits>

#include "../../include/learner.h"
#include "device_common.h"
#include "mlp_device.h"
#include "status.h"

namespace fm {
namespace lrn {

constexpr int kMaxK = 8;
constexpr int kBK = 32, kThreads = 512, kWaves = kThreads / 64;

enum Epilogue { kBiasTanh = 0, kMaskTanhGrad = 1, kStore = 2 };

// C(m, n) = sum_k A(m, k) B(k, n) over k in the block's range; C is [M][ldc].  A chunk of kc values
// of k (split reductions) offsets C by chunk * scz.  The epilogue fixes the operands' layouts:
//   kBiasTanh      A [M][lda], B [K][ldb]: C = tanh(acc + bias[n]) (from one exp2 and one
//                  reciprocal, absolute error below 1e-6);
//   kMaskTanhGrad  A [M][lda], B [N][ldb]: C = acc * (1 - X^2) with X at the same place as C (C may
//                  be X itself: each element is read and written by one thread);
//   kStore         A [K][lda], B [K][ldb]: C = acc.
struct Gemm {
  const float* A;
  const float* B;
  float* C;
  const float* bias;
  const float* X;
  int lda, ldb, ldc;
  long scz;
  int M, N, K, kc, chunks;
  // kStore (bias gradients): C has a row ones_row with the column sums of B.  With ONES, rows
  // m >= ones_row of A (inside M) read as 1; else the workgroups of row tile 0 sum B's columns over
  // their k range (float32), without a row tile for that row when ones_row fills whole tiles.
  int ones_row;
};

// Float32 products on the bfloat16 matrix cores.  A float32 x is the sum of three bfloat16 values,
// hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid (24 bits in three times 8), exact where lo is not
// below the smallest bfloat16 (|x| of 2^-110 and more), and x y is the sum of nine products, of which
// mid*lo, lo*mid and lo*lo are below 2^-25 |x y| and left out.  The other six take 6 x 16 cycles of a
// SIMD's matrix core for a 16 x 16 x 32 block, where v_mfma_f32_16x16x4 takes 8 x 32.  The matrix core
// rounds a sum that starts from zero to nearest, but adds a non-zero accumulator with its lower bits cut
// off, towards minus infinity: a bias that is the same in every row and adds up over a gradient
// (seven times the float32 form's error).  So 32 terms of hi*hi are summed from zero, those of the
// five small products in a chain of their own (where what is cut off is 2^-8 of that), and both
// are added to the running float32 sum by ordinary additions.
// Operands are split at 2^16 times their value, which has all bits of every float32 above the smallest
// bfloat16 (2^-133), and the sums are taken back by 2^-32; neither rounds.  It takes 1 to 1.5% of the
// gradient of a 2048 x 252 rollout (5.13 to 5.18 ms, 5.15 to 5.23 on another card); without it gradients
// of 1e-36 were 2e-4 off, of 1e-37 2e-3.
// An operand that is infinite, NaN or beyond 2^112, or a sum beyond 2^96, makes a sum infinite or NaN; a
// wavefront that finds one sums its elements again in float32.
constexpr float kUp = 0x1p16f, kDown = 0x1p-32f;
__device__ __forceinline__ void split2(float x0, float x1, unsigned (&p)[3]) {
  x0 = x0 * kUp;
  x1 = x1 * kUp;
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  const auto pk = [](float a, float b) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f2{a, b}, b2)); };
  const auto lo_of = [](unsigned v) { return __uint_as_float(v << 16); };
  const auto hi_of = [](unsigned v) { return __uint_as_float(v & 0xffff0000u); };
  p[2] = pk(x0, x1);
  const float r0 = x0 - lo_of(p[2]), r1 = x1 - hi_of(p[2]);
  p[1] = pk(r0, r1);
  p[0] = pk(r0 - lo_of(p[1]), r1 - hi_of(p[1]));
}

// An operand tile of R rows (m or n) by kBK k in LDS: three planes (lo, mid, hi) of MFMA fragments
// [R / 16][64 lanes][8], lane 16 kg + r of a fragment holding row r, k 8 kg .. 8 kg + 7, with r
// XORed by 4 kg so that neither the fragment reads nor the writes of either load order conflict.
// KF: the matrix has k as its unit-stride index ([rows][ld]), else the rows ([K][ld]).  The loads
// go through a buffer resource over the block's rows or k, moved along k, with 32-bit offsets that
// do not change; what lies beyond reads as zero.
template <int R, bool KF>
struct Operand {
  static constexpr int kItems = (R * 4 + kThreads - 1) / kThreads;  // (row, 8 k) units per thread
  static constexpr int kPlane = R * kBK;                            // elements per plane
  static constexpr unsigned kBeyond = 0x7ffffff0;
  float x[kItems][8];

  // Item e of this thread: row r and k group kg; walks the unit-stride index across threads.
  static __device__ __forceinline__ bool at(int e, int& r, int& kg) {
    const int q = threadIdx.x + kThreads * e;
    r = KF ? q >> 2 : q % R;
    kg = KF ? q & 3 : q / R;
    return q < 4 * R;
  }
  // Requests item e of the block of rows r0 .. and k0 .. (k < k_end).
  __device__ __forceinline__ void fetch(int e, const float* p, int ld, int r0, int rows, int k0, int k_end) {
    const int nr = min(R, rows - r0), nk = min(kBK, k_end - k0);
    const float* base = KF ? p + static_cast<long>(r0) * ld + k0 : p + static_cast<long>(k0) * ld + r0;
    const int bytes = 4 * (KF ? nr * ld - k0 : nk * ld - r0);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, bytes, 0x00020000);
    int r, kg;
    const bool mine = at(e, r, kg);
    if constexpr (KF) {
      const unsigned o = mine ? 4u * (r * ld + 8 * kg) : kBeyond;
      if (nk == kBK) {
        const auto u = __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0);
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x[e][j] = __uint_as_float(u[j]);
          x[e][4 + j] = __uint_as_float(v[j]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          x[e][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 8 * kg + j < nk ? o + 4 * j : kBeyond, 0, 0));
      }
    } else {
      const unsigned o = mine && r < nr ? 4u * (8 * kg * ld + r) : kBeyond;
      // One resource per k, so that the offset is the same register for all eight.
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const __amdgpu_buffer_rsrc_t rj = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(base) + static_cast<long>(j) * ld, 0, max(bytes - 4 * j * ld, 0), 0x00020000);
        x[e][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rj, o, 0, 0));
      }
    }
  }
  // Rows first .. rows - 1 of item e read as one (for k < k_end).
  __device__ __forceinline__ void ones(int e, int first, int rows, int r0, int k0, int k_end) {
    int r, kg;
    (void)at(e, r, kg);
    const bool one = r0 + r >= first && r0 + r < rows;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[e][j] = one && k0 + 8 * kg + j < k_end ? 1.0f : x[e][j];
  }
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  // Elements 2 j and 2 j + 1 of item e into the planes' registers.
  __device__ __forceinline__ void split(int e, int j, u4 (&pl)[3]) const {
    unsigned p[3];
    split2(x[e][2 * j], x[e][2 * j + 1], p);
#pragma unroll
    for (int q = 0; q < 3; ++q) pl[q][j] = p[q];
  }
  static __device__ __forceinline__ void store(int e, __bf16* lds, const u4 (&pl)[3]) {
    int r, kg;
    if (!at(e, r, kg)) return;
    const int o = (r / 16 * 64 + 16 * kg + ((r & 15) ^ (4 * kg))) * 8;
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<u4*>(lds + q * kPlane + o) = pl[q];
  }
  static __device__ __forceinline__ bf16x8 frag(const __bf16* lds, int plane, int block, int lane) {
    const int kg = lane >> 4;
    return *reinterpret_cast<const bf16x8*>(lds + plane * kPlane + (block * 64 + 16 * kg + ((lane & 15) ^ (4 * kg))) * 8);
  }
};

// The BI x BJ blocks of a wavefront (from blocks bm and bn of the tile) over k_begin .. k_end - 1 by the
// float32 matrix instruction, for operands that the split has no value for.  Straight from memory, 16 k
// a round: lane group q of the instruction's four has k 4 q .. 4 q + 3 of them, one per instruction, so
// that a lane's four are one 16-byte load where k is the unit-stride index, and the next round's
// operands are requested before this round's products.  Bound by the float32 matrix rate.  A NaN reward
// sends every wavefront of the weight gradients here: a 1000 x 20 rollout of 30 stocks (three actors, 256
// units) takes 1.49 ms then and 0.76 without one, a 2048 x 32 one 1.75 and 1.01 (one element at a time
// 87.6 and 93.2; products in float32 throughout 1.20 and 1.74).
template <int EPI, int TM, int TN, bool ONES, int BI, int BJ>
__device__ __forceinline__ void sum_f32(const Gemm& g, int m0, int n0, int bm, int bn, int k_begin, int k_end, int lane,
                                        floatx4 (&acc)[BI][BJ]) {
  constexpr unsigned kBeyond = 0x7ffffff0;
  const int q = lane >> 4, len = k_end - k_begin;
  // Elements k .. k + 3 (of the block's range) of row r of the tile of R rows from r0 on.
  const auto load = [&](auto kf, const float* p, int ld, int r0, int R, int rows, int r, int k) {
    const int nr = min(R, rows - r0);
    floatx4 x;
    if constexpr (kf) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(p) + static_cast<long>(r0) * ld, 0, 4 * nr * ld, 0x00020000);
      const auto u = __builtin_amdgcn_raw_buffer_load_b128(rs, 4u * (r * ld + k_begin + k), 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = k + e < len ? __uint_as_float(u[e]) : 0.0f;
    } else {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(p) + static_cast<long>(k_begin) * ld + r0, 0, 4 * (len * ld - r0), 0x00020000);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, r < nr ? 4u * ((k + e) * ld + r) : kBeyond, 0, 0));
    }
    return x;
  };
  floatx4 a[BI], b[BJ];
  const auto fetch = [&](int k) {
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const int r = 16 * (bm + i) + (lane & 15);
      a[i] = load(std::bool_constant<EPI != kStore>(), g.A, g.lda, m0, TM, min(g.M, g.ones_row), r, k + 4 * q);
      if (ONES && m0 + r >= g.ones_row && m0 + r < g.M)
#pragma unroll
        for (int e = 0; e < 4; ++e) a[i][e] = k + 4 * q + e < len ? 1.0f : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j)
      b[j] = load(std::bool_constant<EPI == kMaskTanhGrad>(), g.B, g.ldb, n0, TN, g.N, 16 * (bn + j) + (lane & 15), k + 4 * q);
  };
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  fetch(0);
#pragma unroll 1
  for (int k = 0; k < len; k += 16) {
    floatx4 ca[BI], cb[BJ];
#pragma unroll
    for (int i = 0; i < BI; ++i) ca[i] = a[i];
#pragma unroll
    for (int j = 0; j < BJ; ++j) cb[j] = b[j];
    if (k + 16 < len) fetch(k + 16);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j) acc[i][j] = mfma_f32(ca[i][e], cb[j][e], acc[i][j]);
  }
}

// A TM x TN tile of C per workgroup, eight wavefronts of BI x BJ blocks each.  Bound by instruction
// issue: a wavefront's 24 products per (block column, 32 k) leave room for about three vector
// instructions each, and the split (6.5 an element) and the sums (2 an element and 32 k) take most
// of it.  One workgroup per compute unit (two wavefronts per SIMD), the operand tiles
// double-buffered in LDS: while block k is multiplied, block k + 1 is split into the other buffer
// from registers and block k + 2 is requested.  Tiles are 256 wide where C is (every row of A is
// then read and split once), and as narrow as C's width otherwise.
template <int EPI, int TM, int TN, bool ONES>
__global__ __launch_bounds__(kThreads) void gemm_kernel(Gemm g) {
  constexpr int WN = TN >= 128 ? TN / 64 : 1, WM = kWaves / WN;  // wavefronts along n and m
  constexpr int BI = TM / WM / 16, BJ = TN / WN / 16;
  using OpA = Operand<TM, EPI != kStore>;
  using OpB = Operand<TN, EPI == kMaskTanhGrad>;
  using u4 = typename OpA::u4;
  constexpr bool kColsum = EPI == kStore && !ONES;
  extern __shared__ __align__(16) __bf16 lds[];
  constexpr int kBuf = 3 * (OpA::kPlane + OpB::kPlane);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bm = (wave / WN) * BI, bn = (wave % WN) * BJ;  // this wavefront's first blocks
  const int m0 = blockIdx.x * TM, n0 = blockIdx.y * TN;
  const int k_begin = blockIdx.z * g.kc, k_end = min(g.K, k_begin + g.kc);
  OpA a;
  OpB b;
  const auto fetch = [&](int k0) {
#pragma unroll
    for (int e = 0; e < OpA::kItems; ++e) a.fetch(e, g.A, g.lda, m0, min(g.M, g.ones_row), k0, k_end);
#pragma unroll
    for (int e = 0; e < OpB::kItems; ++e) b.fetch(e, g.B, g.ldb, n0, g.N, k0, k_end);
  };
  // Column sums of B: a thread's items are always the same columns.
  float csum[OpB::kItems];
#pragma unroll
  for (int e = 0; e < OpB::kItems; ++e) csum[e] = 0.0f;
  const auto commit = [&](int buf, int k0) {
    __bf16* l = lds + buf * kBuf;
#pragma unroll
    for (int e = 0; e < OpA::kItems; ++e) {
      if (ONES) a.ones(e, g.ones_row, g.M, m0, k0, k_end);
      u4 pl[3];
#pragma unroll
      for (int j = 0; j < 4; ++j) a.split(e, j, pl);
      OpA::store(e, l, pl);
    }
#pragma unroll
    for (int e = 0; e < OpB::kItems; ++e) {
      u4 pl[3];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        b.split(e, j, pl);
        if (kColsum) csum[e] = (csum[e] + b.x[e][2 * j]) + b.x[e][2 * j + 1];
      }
      OpB::store(e, l + 3 * OpA::kPlane, pl);
    }
  };
  constexpr floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  floatx4 acc[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = zero;
  if (k_begin < k_end) {
    fetch(k_begin);
    commit(0, k_begin);
    if (k_begin + kBK < k_end) fetch(k_begin + kBK);
  }
  __syncthreads();
  int buf = 0;
  for (int k0 = k_begin; k0 < k_end; k0 += kBK, buf ^= 1) {
    if (k0 + kBK < k_end) {
      commit(buf ^ 1, k0 + kBK);
      if (k0 + 2 * kBK < k_end) fetch(k0 + 2 * kBK);
    }
    const __bf16* la = lds + buf * kBuf;
    const __bf16* lb = la + 3 * OpA::kPlane;
    bf16x8 fa[BI][3];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p) fa[i][p] = OpA::frag(la, p, bm + i, lane);
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      bf16x8 fb[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) fb[p] = OpB::frag(lb, p, bn + j, lane);
      // Products (plane of A, plane of B): hi*hi, then the five small ones; BI independent sums
      // between dependent products.
      constexpr int PA[6] = {2, 0, 1, 2, 1, 2}, PB[6] = {2, 2, 1, 0, 2, 1};
      floatx4 big[BI], small[BI];
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < BI; ++i) {
          floatx4& t = q == 0 ? big[i] : small[i];
          t = mfma_bf16(fa[i][PA[q]], fb[PB[q]], q < 2 ? zero : t);
        }
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = acc[i][j][r] + (big[i][r] + small[i][r]);
    }
    __syncthreads();
  }
  float* Cz = g.C + blockIdx.z * g.scz;
  if (kColsum && m0 == 0) {
    // The partial column sums of the threads that share a column, in thread order.
    float* sums = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int e = 0; e < OpB::kItems; ++e)
      if (tid + kThreads * e < 4 * TN) sums[tid + kThreads * e] = csum[e];
    __syncthreads();
    if (tid < TN && n0 + tid < g.N)
      Cz[static_cast<long>(g.ones_row) * g.ldc + n0 + tid] =
          ((sums[tid] + sums[TN + tid]) + sums[2 * TN + tid]) + sums[3 * TN + tid];
  }
  // Lane l holds column l%16 and rows 4(l/16)..4(l/16)+3 of each 16 x 16 block.  Offsets in
  // bytes from the tile's first element, through a resource over the tile's rows; derived from
  // an opaque copy of the lane so that they are not kept in registers over the loop.
  int le = lane;
  asm volatile("" : "+v"(le));
  const int mb = 16 * bm + 4 * (le >> 4), nb = 16 * bn + (le & 15);
  const int mr = min(TM, g.M - m0), nr = g.N - n0;  // rows and columns of this tile
  const long first = static_cast<long>(m0) * g.ldc + n0;
  const int bytes = 4 * (mr * g.ldc - n0);
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(Cz + first, 0, bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(EPI == kMaskTanhGrad ? g.X + first : Cz + first), 0, bytes, 0x00020000);
  const auto mask = [&](unsigned o) {
    return EPI == kMaskTanhGrad ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, o, 0, 0)) : 0.0f;
  };
  const auto put = [&](unsigned o, float v, float bias, float x) {
    if (EPI == kBiasTanh) v = fast_tanh(v + bias);
    if (EPI == kMaskTanhGrad) v = v * (1.0f - x * x);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rc, o, 0, 0);
  };
  bool lost = false;
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) lost = lost || !(fabsf(acc[i][j][r]) <= 0x1.fffffep127f);
  float down = kDown;
  if (__builtin_amdgcn_ballot_w64(lost) != 0) {
    sum_f32<EPI, TM, TN, ONES>(g, m0, n0, bm, bn, k_begin, k_end, le, acc);
    down = 1.0f;
  }
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    const int n = nb + 16 * j;
    const bool on = n < nr;
    const float bias = EPI == kBiasTanh && on ? g.bias[n0 + n] : 0.0f;
    const unsigned o = on ? 4u * (mb * g.ldc + n) : OpA::kBeyond;
    // A column's masks are all requested before its first store (which they cannot pass).
    float x[BI][4];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[i][r] = mask(o + 4u * (16 * i + r) * g.ldc);
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) put(o + 4u * (16 * i + r) * g.ldc, acc[i][j][r] * down, bias, x[i][r]);
  }
}

// R_n = sum_t r[t][n] in ascending t.
__global__ void returns_kernel(const double* rew, int T, int N, double* R) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  double acc = 0.0;
  // Unrolled so that the loads issue ahead of the additions, which stay in ascending t.
#pragma unroll 8
  for (int t = 0; t < T; ++t) acc = acc + rew[static_cast<size_t>(t) * N + n];
  R[n] = acc;
}

struct Mix {
  float w[kMaxK];
};

// Layer-3 delta of agent i for row r = t*N + n and actions 4j..4j+3 (one noise block):
//   u = (R_n / N) (abar + sigma eps - mu_i) / sigma^2 + lambda/(N T) sum_{k != i} (mu_i - mu_k) / sigma^2
//   G3 = u (1 - mu_i^2).
__global__ void delta3_kernel(const float* mu, int K, int agent, Mix mix, int rows, int N, int T, int A,
                              const double* R, float sigma, uint64_t key, int64_t env_offset, int t0,
                              float lambda_kl, float* G3) {
  const int G = (A + 3) / 4;
  const long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<long>(rows) * G) return;
  const int r = static_cast<int>(i / G), j = static_cast<int>(i % G);
  const int t = r / N, n = r % N;
  float z[4];
  // Row t of the samples was drawn on day t0 + t: the noise is keyed by the absolute day.
  noise_block(key, static_cast<uint64_t>(env_offset + n), static_cast<uint64_t>(t0 + t), static_cast<uint64_t>(j), z);
  const float inv_s2 = 1.0f / (sigma * sigma);
  const float rn = static_cast<float>(R[n] / N);
  const float kl = lambda_kl / (static_cast<float>(N) * static_cast<float>(T));
  for (int q = 0; q < 4; ++q) {
    const int a = 4 * j + q;
    if (a >= A) break;
    const size_t off = static_cast<size_t>(r) * A + a;
    const size_t plane = static_cast<size_t>(rows) * A;
    const float mi = mu[agent * plane + off];
    float abar = 0.0f, div = 0.0f;
    for (int k = 0; k < K; ++k) {
      const float mk = mu[k * plane + off];
      abar = abar + mix.w[k] * mk;
      if (k != agent) div = div + (mi - mk);
    }
    const float u = rn * ((abar + sigma * z[q]) - mi) * inv_s2 + kl * div * inv_s2;
    G3[off] = u * (1.0f - mi * mi);
  }
}

// out[i] = sum over chunks c (ascending) of P[c][i], in float64, rounded once.
__global__ void reduce_kernel(const float* P, int len, int n_chunks, float* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= len) return;
  double acc = 0.0;
#pragma unroll 8
  for (int c = 0; c < n_chunks; ++c) acc = acc + static_cast<double>(P[static_cast<size_t>(c) * len + i]);
  out[i] = static_cast<float>(acc);
}

struct Layout {
  size_t mu, x1, x2, g3, R, P, total;
  int rows, chunk, n_chunks;
};

Layout layout(int K, int S, int H, int A, int N, int T) {
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  Layout L{};
  L.rows = N * T;
  L.chunk = std::max(2048, (L.rows + 255) / 256);
  L.n_chunks = (L.rows + L.chunk - 1) / L.chunk;
  const size_t rows = L.rows;
  size_t o = 0;
  L.mu = o;
  o = al(o + sizeof(float) * K * rows * A);
  L.x1 = o;
  o = al(o + sizeof(float) * rows * H);
  L.x2 = o;
  o = al(o + sizeof(float) * rows * H);
  L.g3 = o;
  o = al(o + sizeof(float) * rows * A);
  L.R = o;
  o = al(o + sizeof(double) * N);
  const size_t pmax = std::max({static_cast<size_t>(S + 1) * H, static_cast<size_t>(H + 1) * H,
                                static_cast<size_t>(H + 1) * A});
  L.P = o;
  o = al(o + sizeof(float) * L.n_chunks * pmax);
  L.total = o;
  return L;
}

// Rows of A that a workgroup takes for C's width (its tile width is the width rounded up to 32,
// 64, 128 or 256).
constexpr int tile_rows(int N) { return N <= 128 ? 256 : 128; }

template <int EPI, int TN, bool ONES>
hipError_t gemm_tiles(const Gemm& g, hipStream_t stream) {
  constexpr int TM = tile_rows(TN);
  constexpr size_t lds = 2 * 3 * sizeof(__bf16) * kBK * (TM + TN);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_kernel<EPI, TM, TN, ONES>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  const dim3 grid((g.M + TM - 1) / TM, (g.N + TN - 1) / TN, g.chunks);
  hipLaunchKernelGGL((gemm_kernel<EPI, TM, TN, ONES>), grid, dim3(kThreads), lds, stream, g);
  return hipGetLastError();
}

template <int EPI, bool ONES = false>
hipError_t gemm(const Gemm& g, hipStream_t stream) {
  if (g.N <= 32) return gemm_tiles<EPI, 32, ONES>(g, stream);
  if (g.N <= 64) return gemm_tiles<EPI, 64, ONES>(g, stream);
  if (g.N <= 128) return gemm_tiles<EPI, 128, ONES>(g, stream);
  return gemm_tiles<EPI, 256, ONES>(g, stream);
}

// Weight and bias gradients [X | 1]^T G: Xr [rows][kin] (row stride ldx), Gr [rows][kout]; the
// result [kin + 1][kout] (weights, then the bias as the row of ones) into out, which is the
// layout of W followed by b in the master weights.
hipError_t weight_grad(const Layout& L, const float* Xr, int kin, int ldx, const float* Gr, int kout, float* P,
                       float* out, hipStream_t stream) {
  Gemm g{};
  g.A = Xr;
  g.lda = ldx;
  g.B = Gr;
  g.ldb = kout;
  g.C = P;
  g.ldc = kout;
  g.scz = static_cast<long>(kin + 1) * kout;
  // With kin a multiple of the tile height the bias row (the column sums of G) would take a row
  // tile of its own; the first row tile's workgroups sum the columns instead.
  const bool own = kin % tile_rows(kout) == 0;
  g.M = own ? kin : kin + 1;
  g.N = kout;
  g.K = L.rows;
  g.kc = L.chunk;
  g.chunks = L.n_chunks;
  g.ones_row = kin;
  hipError_t e = own ? gemm<kStore>(g, stream) : gemm<kStore, true>(g, stream);
  if (e != hipSuccess) return e;
  const int len = (kin + 1) * kout;
  hipLaunchKernelGGL(reduce_kernel, dim3((len + 255) / 256), dim3(256), 0, stream, P, len, L.n_chunks, out);
  return hipGetLastError();
}

// Delta of the layer below: Gout [rows][kin] = (Gin [rows][kout] W^T) * (1 - X^2), W [kin][kout],
// written over X [rows][kin].
hipError_t back_delta(const Layout& L, const float* Gin, int kout, const float* W, int kin, float* X,
                      hipStream_t stream) {
  Gemm g{};
  g.A = Gin;
  g.lda = kout;
  g.B = W;
  g.ldb = kout;
  g.C = X;
  g.ldc = kin;
  g.X = X;
  g.M = L.rows;
  g.N = kin;
  g.K = kout;
  g.kc = kout;
  g.chunks = 1;
  g.ones_row = g.M;
  return gemm<kMaskTanhGrad>(g, stream);
}

// Y [rows][kout] = tanh(X [rows][kin] W + b).
hipError_t layer(const Layout& L, const float* X, int kin, const float* W, const float* b, int kout, float* Y,
                 hipStream_t stream) {
  Gemm g{};
  g.A = X;
  g.lda = kin;
  g.B = W;
  g.ldb = kout;
  g.C = Y;
  g.ldc = kout;
  g.bias = b;
  g.M = L.rows;
  g.N = kout;
  g.K = kin;
  g.kc = kin;
  g.chunks = 1;
  g.ones_row = g.M;
  return gemm<kBiasTanh>(g, stream);
}

bool dims_ok(int K, int S, int H, int A, int N, int T) {
  if (K < 1 || K > kMaxK || S < 1 || S > 1024 || H < 1 || H > 1024 || A < 1 || A > 128 || N < 1 || T < 1)
    return false;
  return static_cast<int64_t>(N) * T <= (int64_t(1) << 26);
}

}  // namespace lrn
}  // namespace fm

extern "C" {

size_t fm_pg_workspace_bytes(int32_t K, int32_t S, int32_t H, int32_t A, int32_t N, int32_t T) {
  if (!fm::lrn::dims_ok(K, S, H, A, N, T)) return 0;
  return fm::lrn::layout(K, S, H, A, N, T).total;
}

fm_status fm_policy_gradient(int32_t K, int32_t S, int32_t H, int32_t A, const float* d_w, const float* h_mix,
                             int32_t agent, const float* d_states, const double* d_rew, int32_t N, int32_t T,
                             float sigma, uint64_t noise_key, int64_t env_offset, int32_t t0, float lambda_kl,
                             float* d_grad, void* d_workspace, size_t workspace_bytes, hipStream_t stream) {
  using namespace fm::lrn;
  if (!dims_ok(K, S, H, A, N, T))
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: sizes out of range (K 1..8, S/H 1..1024, A 1..128, N*T <= 2^26)");
  if (agent < 0 || agent >= K) return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: agent out of range");
  if (!d_w || !d_states || !d_rew || !d_grad || !d_workspace)
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: NULL buffer");
  if (!(sigma > 0.0f) || !std::isfinite(sigma)) return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: sigma must be finite and > 0");
  if (!(lambda_kl >= 0.0f) || !std::isfinite(lambda_kl))
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: lambda_kl must be finite and >= 0");
  if (env_offset < 0) return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: env_offset must be >= 0");
  if (t0 < 0 || static_cast<int64_t>(t0) + T > (int64_t{1} << 31) - 1)
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: t0 must be >= 0 and t0 + T must fit int32");
  const Layout L = layout(K, S, H, A, N, T);
  if (workspace_bytes < L.total || reinterpret_cast<uintptr_t>(d_workspace) % 256)
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: workspace smaller than fm_pg_workspace_bytes or not 256-byte aligned");
  Mix mix{};
  for (int k = 0; k < K; ++k) {
    mix.w[k] = h_mix ? h_mix[k] : 1.0f / K;
    if (!std::isfinite(mix.w[k])) return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient: mix weights must be finite");
  }
  unsigned char* ws = static_cast<unsigned char*>(d_workspace);
  float* mu = reinterpret_cast<float*>(ws + L.mu);
  float* x1 = reinterpret_cast<float*>(ws + L.x1);
  float* x2 = reinterpret_cast<float*>(ws + L.x2);
  float* g3 = reinterpret_cast<float*>(ws + L.g3);
  double* R = reinterpret_cast<double*>(ws + L.R);
  float* P = reinterpret_cast<float*>(ws + L.P);
  const size_t per = static_cast<size_t>(S) * H + H + static_cast<size_t>(H) * H + H + static_cast<size_t>(H) * A + A;
  const size_t oW1 = 0, ob1 = static_cast<size_t>(S) * H, oW2 = ob1 + H, ob2 = oW2 + static_cast<size_t>(H) * H,
               oW3 = ob2 + H, ob3 = oW3 + static_cast<size_t>(H) * A;
  hipError_t e = hipSuccess;
  // Forward passes, agent i last so that x1, x2 hold its activations.
  for (int step = 0; step < K && e == hipSuccess; ++step) {
    const int k = step < K - 1 ? (step < agent ? step : step + 1) : agent;
    const float* w = d_w + per * k;
    e = layer(L, d_states, S, w + oW1, w + ob1, H, x1, stream);
    if (e == hipSuccess) e = layer(L, x1, H, w + oW2, w + ob2, H, x2, stream);
    if (e == hipSuccess) e = layer(L, x2, H, w + oW3, w + ob3, A, mu + static_cast<size_t>(k) * L.rows * A, stream);
  }
  if (e != hipSuccess) return fm::device_error(e, "fm_policy_gradient (forward)");
  hipLaunchKernelGGL(returns_kernel, dim3((N + 255) / 256), dim3(256), 0, stream, d_rew, T, N, R);
  const long nd = static_cast<long>(L.rows) * ((A + 3) / 4);
  hipLaunchKernelGGL(delta3_kernel, dim3(static_cast<unsigned>((nd + 255) / 256)), dim3(256), 0, stream, mu, K,
                     agent, mix, L.rows, N, T, A, R, sigma, noise_key, env_offset, t0, lambda_kl, g3);
  e = hipGetLastError();
  if (e != hipSuccess) return fm::device_error(e, "fm_policy_gradient (delta)");
  const float* wi = d_w + per * agent;
  // Layer 3, then the delta of layer 2 over x2, layer 2, the delta of layer 1 over x1, layer 1.
  e = weight_grad(L, x2, H, H, g3, A, P, d_grad + oW3, stream);
  if (e == hipSuccess) e = back_delta(L, g3, A, wi + oW3, H, x2, stream);
  if (e == hipSuccess) e = weight_grad(L, x1, H, H, x2, H, P, d_grad + oW2, stream);
  if (e == hipSuccess) e = back_delta(L, x2, H, wi + oW2, H, x1, stream);
  if (e == hipSuccess) e = weight_grad(L, d_states, S, S, x1, H, P, d_grad + oW1, stream);
  if (e != hipSuccess) return fm::device_error(e, "fm_policy_gradient (backward)");
  return FM_OK;
}

// ------------------------------------------------------------------------------------------
// The allocation-free variant: the same computation with its workspace in a file-scope device
// array instead of a caller buffer.  Each device the library runs on holds its own copy of the
// array; its address is looked up once per device (the array's name is a host-side stand-in, not
// a device address) and kept.  Every call on a device shares that device's array, so calls that
// overlap on one device race.  The workspace needs no clearing: every region is written before
// it is read within a call.
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[FM_PG_NOALLOC_MAX_BYTES];

fm_status fm_policy_gradient_noalloc(int32_t K, int32_t S, int32_t H, int32_t A, const float* d_w, const float* h_mix,
                                     int32_t agent, const float* d_states, const double* d_rew, int32_t N, int32_t T,
                                     float sigma, uint64_t noise_key, int64_t env_offset, int32_t t0, float lambda_kl,
                                     float* d_grad, hipStream_t stream) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  const size_t need = fm_pg_workspace_bytes(K, S, H, A, N, T);
  if (need == 0)
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient_noalloc: sizes out of range (K 1..8, S/H 1..1024, A 1..128, N*T <= 2^26)");
  if (need > FM_PG_NOALLOC_MAX_BYTES)
    return fm::set_error(FM_ERR_INVALID, "fm_policy_gradient_noalloc: the problem needs " + std::to_string(need) +
                                             " bytes of workspace, more than the " +
                                             std::to_string(FM_PG_NOALLOC_MAX_BYTES) + " the library holds");
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fm::device_error(e, "fm_policy_gradient_noalloc (hipGetDevice)");
  if (dev < 0 || dev >= kMaxDevices) return fm::set_error(FM_ERR_UNSUPPORTED, "fm_policy_gradient_noalloc: device index above 63");
  void* ws = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p) return fm::device_error(e != hipSuccess ? e : hipErrorInvalidSymbol,
                                                         "fm_policy_gradient_noalloc (hipGetSymbolAddress)");
      addr[dev] = p;
    }
    ws = addr[dev];
  }
  return fm_policy_gradient(K, S, H, A, d_w, h_mix, agent, d_states, d_rew, N, T, sigma, noise_key, env_offset, t0,
                            lambda_kl, d_grad, ws, FM_PG_NOALLOC_MAX_BYTES, stream);
}

}  // extern "C"
