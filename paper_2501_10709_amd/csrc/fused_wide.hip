// The wide resident schedule of the fused rollout: the resident schedule's shapes (K = 3, H = 256,
// D <= 31 stocks) for batches past eight environments per compute unit, up to 16 ET of them per
// workgroup (ET = 1 or 2 sixteen-environment columns of the matrix products).
//
// One workgroup of four wavefronts per compute unit.  W2 of all three actors lives in registers as
// in the resident schedule (wavefront w holds output tiles 4w .. 4w+3 of every actor), W3 and W1e in
// LDS (W1e refetched from L2 every step where it has no room of its own).  The layers run
// transposed (units x environments), so each accumulator holds 16 environments and all its lanes do
// work.  Per step, four workgroup barriers close the phases:
//   L1    all wavefronts, all actors;
//   L2    all wavefronts, W2 from registers; beside it the market entries of the step's state rows
//         go straight from LDS to the trajectory;
//   L3    wavefront w sums k-steps 2w and 2w+1 of both output tiles of every actor and leaves the
//         partial sums in LDS;
//   trade wavefront w trades environments 4 ET w .. +4 ET - 1, four at a time, one per 16-lane row
//         (row_chain.h), as in the resident schedule.
// The arithmetic is the streamed schedule's, operation by operation (accumulators from zero, then
// bias or table entry, fast_tanh; layer 3 in four k slices summed in order), so the two agree bit
// for bit.
//
// Bound by vector instruction issue: there is one wavefront per SIMD (the weights fill the register
// file), and a step of 32 environments is 192 tanh a lane at about 50 cycles each, beside 3.8 k
// cycles of matrix products, then the trade, a chain of dependent float64 steps.  In a build with clock
// stamps, which keep the phases apart, a step of 32 environments is 35.7 k cycles (16.1 us there): layer
// 1 5.8 k, layer 2 14.0 k, layer 3 1.5 k, the trade 11.9 k (half of it the buys), waits 2.6 k.  Without
// them, per step of D = 30 with states, actions and rewards stored: 13.1 us at N = 8192 (streamed schedule
// 20.7, resident 22.6), 7.6 us at N = 4096 (17.0, 11.6).
#include <utility>

#include "device_common.h"
#include "fused.h"
#include "mlp_device.h"
#include "resident_device.h"
#include "row_chain.h"

namespace fm {

namespace {

constexpr int kWT = 256;  // threads per workgroup

constexpr floatx4 kZero4 = {0.0f, 0.0f, 0.0f, 0.0f};

// LDS regions (byte offsets) for MR = 16 ET environments.
template <int ET>
struct WLds {
  static constexpr int MR = 16 * ET;
  // Hidden rows [K][MR][256] bfloat16, the 16-byte groups of a row XORed by the row (see xcol).
  static constexpr size_t xb = sizeof(__bf16) * kRK * MR * kRH;
  static constexpr size_t w3 = 0;                                            // [K][2][8][64] bf16x8
  static constexpr size_t x1 = w3 + sizeof(bf16x8) * kRK * 2 * kRKK * 64;    // layer-1 outputs
  static constexpr size_t part = x1;                                         // [K][4][MR][32] f32 (after L2)
  static constexpr size_t x2 = x1 + xb;                                      // layer-2 outputs
  static constexpr size_t x0 = x2 + xb;                                      // [MR][40] bf16
  static constexpr size_t b2 = x0 + sizeof(__bf16) * MR * kRX0;              // [K][256] f32
  static constexpr size_t b3 = b2 + sizeof(float) * kRK * kRH;               // [K][32] f32
  static constexpr size_t mix = b3 + sizeof(float) * kRK * 32;               // [4] f32
  static constexpr size_t mt = mix + 16;                                     // [K][256] f32
  static constexpr size_t in = mt + sizeof(float) * kRK * kRH;               // [2][320] f32
  static constexpr size_t state = in + sizeof(float) * 2 * kRInBuf;          // [MR] {cash, value, cumrew, 0} f64
  // W1e [K][16][64] bf16x8: with one column in a region of its own; with two in the layer-2 region,
  // which is free from layer 3 to the next layer 2, fetched again from L2 during every trade.
  static constexpr bool kRefetch = ET == 2;
  static constexpr size_t w1b = sizeof(bf16x8) * kRK * 16 * 64;
  static constexpr size_t w1e = kRefetch ? x2 : state + sizeof(double) * 4 * MR;
  static constexpr size_t total = state + sizeof(double) * 4 * MR + (kRefetch ? 0 : w1b);
  static_assert(!kRefetch || w1b <= xb, "W1e fits the layer-2 region");
  static_assert(sizeof(float) * kRK * 4 * MR * 32 <= xb, "the partial sums fit the layer-1 region");
  static_assert(total <= 160 * 1024, "LDS budget");
};

// Byte offset of 16-byte group g (8 units) of row r in a hidden plane: the group index XORed by the
// row's low four bits, so that 16 rows read at one g, or written at one, fall in distinct banks.
__device__ __forceinline__ int xgroup(int r, int g) { return r * (2 * kRH) + ((g ^ (r & 15)) << 4); }

// Four activations (units 16 c + 4 (l/16) .. +3 of environment row r) into a hidden plane.
__device__ __forceinline__ void put4(unsigned char* plane, int r, int c, int bgrp, const float (&t)[4]) {
  *reinterpret_cast<uint2*>(plane + xgroup(r, 2 * c + (bgrp >> 1)) + 8 * (bgrp & 1)) = pack_bf16x4(t[0], t[1], t[2], t[3]);
}

// fast_tanh of V values side by side: V independent instructions between dependent ones (a dependent
// vector instruction waits about twice as long as an independent one takes), fenced so that the
// compiler keeps them so.  tanh_step is one of its seven steps.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
// copysignf as one instruction in float32 (the compiler would convert to bfloat16 first and move
// the signs of the converted values one by one).
__device__ __forceinline__ float with_sign(float y, float x) {
  float r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(0x7fffffff), "v"(y), "v"(x));
  return r;
}
template <int V>
__device__ __forceinline__ void tanh_step(int step, const float (&x)[V], float (&t)[V], float (&r)[V]) {
#pragma unroll
  for (int q = 0; q < V; ++q) {
    if (step == 0) t[q] = -2.8853900817779268f * fabsf(x[q]);
    if (step == 1) t[q] = __builtin_amdgcn_exp2f(t[q]);
    if (step == 2) r[q] = 1.0f + t[q];
    if (step == 3) r[q] = __builtin_amdgcn_rcpf(r[q]);
    if (step == 4) t[q] = 1.0f - t[q];
    if (step == 5) t[q] = t[q] * r[q];
    if (step == 6) t[q] = with_sign(t[q], x[q]);
  }
  fence();
}

// Layer 1 in twelve (actor, tile) stages: stage i requests the operands of stage i + 2 (the weight
// fragment and the day's table entries), issues the products of stage i + 1 and computes the
// activations of stage i, fenced so that the vector work runs while the matrix cores work.
template <int ET>
__device__ __forceinline__ void wide_layer1(const bf16x8* __restrict__ w1e, const float* __restrict__ mt,
                                            const __bf16* __restrict__ x0, unsigned char* __restrict__ x1, int wave,
                                            int lane) {
  constexpr int N = 4 * kRK, MR = 16 * ET;
  const int env = lane & 15, bgrp = lane >> 4;
  bf16x8 X[ET], W[N];
  floatx4 T[N], acc[N][ET];
#pragma unroll
  for (int s = 0; s < ET; ++s) X[s] = *reinterpret_cast<const bf16x8*>(x0 + (16 * s + env) * kRX0 + 8 * bgrp);
  auto load = [&](int i) {
    const int c = 4 * wave + (i & 3);
    W[i] = w1e[((i >> 2) * 16 + c) * 64 + lane];
    T[i] = *reinterpret_cast<const floatx4*>(mt + (i >> 2) * kRH + 16 * c + 4 * bgrp);
  };
  load(0);
  load(1);
#pragma unroll
  for (int s = 0; s < ET; ++s) acc[0][s] = mfma_bf16(W[0], X[s], kZero4);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + 2 < N) load(i + 2);
#pragma unroll
    for (int s = 0; s < ET; ++s) {
      if (i + 1 < N) acc[i + 1][s] = mfma_bf16(W[i + 1], X[s], kZero4);
      float x[4], t[4], r[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = acc[i][s][q] + T[i][q];
      fence();
#pragma unroll
      for (int step = 0; step < 7; ++step) tanh_step(step, x, t, r);
      put4(x1 + (i >> 2) * MR * 2 * kRH, 16 * s + env, 4 * wave + (i & 3), bgrp, t);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Layer 2 in (actor, column, tile pair) stages of sixteen products (two tiles, eight k-steps), with
// the previous stage's eight activations spread between them: two products in a row would hold up
// the wavefront for as long as one takes, and one activation after another would wait for each
// exponential and reciprocal.  So two activations go through fast_tanh's operations together, a
// few instructions (about as long as two products take) after each product.  A column's
// inputs (eight fragments) are replaced by the next column's as its second pair consumes them.
// beside(st, kk) is called once per k-step.
template <int ET, class Beside>
__device__ __forceinline__ void wide_layer2(const bf16x8 (&w2)[kRK][kRKK][4], const float* __restrict__ b2,
                                            const unsigned char* __restrict__ x1, unsigned char* __restrict__ x2,
                                            int wave, int lane, Beside beside) {
  constexpr int KK = kRKK, MR = 16 * ET, NS = kRK * ET * 2;
  const int env = lane & 15, bgrp = lane >> 4;
  bf16x8 X[KK];
  auto load_x = [&](int col, int kk) {  // col = actor * ET + s
    X[kk] = *reinterpret_cast<const bf16x8*>(x1 + (col / ET) * MR * 2 * kRH + xgroup(16 * (col % ET) + env, 4 * kk + bgrp));
  };
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) load_x(0, kk);
  floatx4 acc[2][2], T[2];
  auto bias = [&](int st, int h) {
    T[h] = *reinterpret_cast<const floatx4*>(b2 + st / (2 * ET) * kRH + 16 * (4 * wave + 2 * (st & 1) + h) + 4 * bgrp);
  };
  float x[2], t[2], r[2], y[4];
  // Slice i (0..3) of values 2 v and 2 v + 1 (v 0..3) of stage st's pair.
  auto slice = [&](int st, int v, int i) {
    const int h = v >> 1, q0 = 2 * (v & 1);
    if (i == 0) {
#pragma unroll
      for (int q = 0; q < 2; ++q) x[q] = acc[st & 1][h][q0 + q] + T[h][q0 + q];
      fence();
      tanh_step(0, x, t, r);
    } else if (i == 1) {
      tanh_step(1, x, t, r);
    } else if (i == 2) {
      tanh_step(2, x, t, r);
      tanh_step(3, x, t, r);
    } else {
      tanh_step(4, x, t, r);
      tanh_step(5, x, t, r);
      tanh_step(6, x, t, r);
      y[q0] = t[0];
      y[q0 + 1] = t[1];
      if (q0 == 2)
        put4(x2 + st / (2 * ET) * MR * 2 * kRH, 16 * (st / 2 % ET) + env, 4 * wave + 2 * (st & 1) + h, bgrp, y);
    }
  };
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    const int a = st / (2 * ET), p = st & 1;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        acc[st & 1][h] = mfma_bf16(w2[a][kk][2 * p + h], X[kk], kk == 0 ? kZero4 : acc[st & 1][h]);
        if (h == 1 && p == 1 && st / 2 + 1 < kRK * ET) load_x(st / 2 + 1, kk);
        if (st > 0) slice(st - 1, kk / 2, 2 * (kk % 2) + h);
        // The next stage's bias entries, once this stage's activations have used theirs.
        if (h == 1 && (kk == 2 || kk == 6)) bias(st, kk / 4);
        if (h == 1) beside(st, kk);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int i = 0; i < 4; ++i) slice(NS - 1, v, i);
}

// Group g (4 stocks) of row r of the layer-3 partial sums [32] floats, XORed against conflicts.
__device__ __forceinline__ int part_at(int r, int d) { return r * 32 + (((d >> 2) ^ (r & 7)) << 2) + (d & 3); }

// Layer 3: this wavefront's two k-steps of both output tiles of every actor and column, the
// operands requested one (actor) ahead.
template <int ET>
__device__ __forceinline__ void wide_layer3(const bf16x8* __restrict__ w3, const unsigned char* __restrict__ x2,
                                            float* __restrict__ part, int wave, int lane) {
  constexpr int MR = 16 * ET;
  const int env = lane & 15, bgrp = lane >> 4;
  bf16x8 W[kRK][2][2], X[kRK][ET][2];
  auto load = [&](int a) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int h = 0; h < 2; ++h) W[a][h][q] = w3[((a * 2 + h) * kRKK + 2 * wave + q) * 64 + lane];
#pragma unroll
      for (int s = 0; s < ET; ++s)
        X[a][s][q] = *reinterpret_cast<const bf16x8*>(x2 + a * MR * 2 * kRH + xgroup(16 * s + env, 4 * (2 * wave + q) + bgrp));
    }
  };
  load(0);
#pragma unroll
  for (int a = 0; a < kRK; ++a) {
    if (a + 1 < kRK) load(a + 1);
    floatx4 acc[2][ET];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < ET; ++s) acc[h][s] = mfma_bf16(W[a][h][q], X[a][s][q], q == 0 ? kZero4 : acc[h][s]);
    float* p = part + (a * 4 + wave) * MR * 32;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < ET; ++s)
        *reinterpret_cast<floatx4*>(p + part_at(16 * s + env, 16 * h + 4 * bgrp)) = acc[h][s];
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int ET>
__global__ __launch_bounds__(kWT) __attribute__((amdgpu_waves_per_eu(1, 1)))
void fused_wide_kernel(EnvConst C, EnvState st, EnsDev E, FusedArgs F) {
  constexpr int K = kRK, H = kRH, KK = kRKK, MR = 16 * ET, PW = 4 * ET;  // PW: environments per wavefront
  using L = WLds<ET>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane0 = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = C.D, N = C.N, S = C.S;
  const int n0 = blockIdx.x * F.tile_envs;
  const int M = min(F.tile_envs, N - n0);
  const int n_mkt = (1 + C.I) * D;

  // ---------------------------------------------------------------- set-up
  // W2 fragments: actors 0 and 1 in the accumulation registers, actor 2 in the vector registers.
  bf16x8 w2[K][KK][4];
#pragma unroll
  for (int a = 0; a < K; ++a)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        w2[a][kk][i] = *reinterpret_cast<const bf16x8*>(E.base + a * E.actor_stride + E.off_w2 +
                                                        static_cast<size_t>((4 * wave + i) * KK + kk) * 1024 + lane0 * 16);
        if (a < 2) asm volatile("" : "+a"(w2[a][kk][i]));
      }
  {
    bf16x8* s_w3 = reinterpret_cast<bf16x8*>(smem + L::w3);
    float* s_b2 = reinterpret_cast<float*>(smem + L::b2);
    float* s_b3 = reinterpret_cast<float*>(smem + L::b3);
    float* s_mix = reinterpret_cast<float*>(smem + L::mix);
    __bf16* s_x0 = reinterpret_cast<__bf16*>(smem + L::x0);
    float* s_mt = reinterpret_cast<float*>(smem + L::mt);
    float* s_in = reinterpret_cast<float*>(smem + L::in);
    for (int f = wave; f < K * 2 * KK; f += 4) {
      const int a = f / (2 * KK), r = f - a * 2 * KK;
      s_w3[f * 64 + lane0] = *reinterpret_cast<const bf16x8*>(E.base + a * E.actor_stride + E.off_w3 +
                                                              static_cast<size_t>(r) * 1024 + lane0 * 16);
    }
    for (int i = tid; i < K * H; i += kWT) {
      const int a = i / H, c = i - a * H;
      s_b2[i] = reinterpret_cast<const float*>(E.base + a * E.actor_stride + E.off_b2)[c];
      s_mt[i] = F.mt[i];
    }
    if (tid < K * 32) {
      const int a = tid / 32, c = tid - a * 32;
      s_b3[tid] = reinterpret_cast<const float*>(E.base + a * E.actor_stride + E.off_b3)[c];
    }
    if (tid < K) s_mix[tid] = E.mix[tid];
    for (int i = tid; i < MR * kRX0; i += kWT) s_x0[i] = static_cast<__bf16>(0.0f);
    // Rows past M trade too: without cash, which covers their empty orders.
    if (tid < 4 * MR) reinterpret_cast<double*>(smem + L::state)[tid] = 0.0;
    for (int i = tid; i < kRInBuf; i += kWT) {  // the first step's market rows
      float v = 0.0f;
      if (i < 2 * D) v = C.close[static_cast<size_t>(F.t0) * D + i];
      else if (i >= kRInd && i - kRInd < C.I * D) v = C.ind[static_cast<size_t>(F.t0 + 1) * C.I * D + (i - kRInd)];
      s_in[i] = v;
    }
  }
  __syncthreads();

  // The trading state: pass q of wavefront w trades environments PW w + 4 q .. +3, 16-lane row r
  // working on PW w + 4 q + r, lane j of a row on stocks j and j + 16.  Holdings live in the lanes'
  // registers; cash, value and cumulative reward in LDS.
  int hold[ET][2];
#pragma unroll
  for (int q = 0; q < ET; ++q) {
    const int m = PW * wave + 4 * q + (lane0 >> 4), j = lane0 & 15;
    hold[q][0] = hold[q][1] = 0;
    if (m < M) {
      __bf16* s_x0 = reinterpret_cast<__bf16*>(smem + L::x0) + m * kRX0;
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (j + 16 * s < D) {
          hold[q][s] = st.hold[static_cast<size_t>(j + 16 * s) * N + n0 + m];
          s_x0[1 + j + 16 * s] = static_cast<__bf16>(static_cast<float>(hold[q][s]) * C.hold_scale);
        }
      if (j == 0) {
        const double cash = st.cash[n0 + m];
        s_x0[0] = static_cast<__bf16>(static_cast<float>(cash * static_cast<double>(C.cash_scale)));
        double* s_state = reinterpret_cast<double*>(smem + L::state) + 4 * m;
        s_state[0] = cash;
        s_state[1] = st.asset[n0 + m];
        s_state[2] = st.cumrew[n0 + m];
      }
    }
  }
  // W1e into LDS, 1 KB per load, a quarter by each wavefront.
  const auto fetch_w1e = [&](unsigned char* dst, int lane) {
    constexpr int kPer = K * 16 / 4;
    const __amdgpu_buffer_rsrc_t r = rows_rsrc(E.base, E.off_w1e, 1, static_cast<int>(L::w1b));
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int o = 1024 * (kPer * wave + i);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst + o, 16, 16 * lane + o, 0, 0, 0);
    }
  };
  fetch_w1e(smem + L::w1e, lane0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): no set-up load counts as pending in the loop

  for (int j = 0; j < F.n_steps; ++j) {
    const bool nxt = j + 1 < F.n_steps;
    // Addresses derived from the lane and the LDS base are recomputed every step rather than held
    // across the loop: the weights leave few registers for loop-invariant values.
    const int z = opaque_zero();
    const int lane = threadIdx.x % 64 + z;
    unsigned char* sm = smem + z;
    const bf16x8* s_w3 = reinterpret_cast<const bf16x8*>(sm + L::w3);
    unsigned char* s_x1 = sm + L::x1;
    float* s_part = reinterpret_cast<float*>(sm + L::part);
    unsigned char* s_x2 = sm + L::x2;
    __bf16* s_x0 = reinterpret_cast<__bf16*>(sm + L::x0);
    const float* s_b2 = reinterpret_cast<const float*>(sm + L::b2);
    const float* s_b3 = reinterpret_cast<const float*>(sm + L::b3);
    const float* s_mix = reinterpret_cast<const float*>(sm + L::mix);
    float* s_mt = reinterpret_cast<float*>(sm + L::mt);
    const float* in = reinterpret_cast<const float*>(sm + L::in) + (j & 1) * kRInBuf;
    float* in_next = reinterpret_cast<float*>(sm + L::in) + ((j + 1) & 1) * kRInBuf;
    double* s_state = reinterpret_cast<double*>(sm + L::state);
    const size_t row0 = static_cast<size_t>(j) * N + n0;  // the tile's first row of step j
    const __amdgpu_buffer_rsrc_t r_obs = rows_rsrc(F.obs_traj, row0 * S, 4, M * S);

    // ------------------------------------------------------------ L1
    wide_layer1<ET>(reinterpret_cast<const bf16x8*>(sm + L::w1e), s_mt, s_x0, s_x1, wave, lane);
    __syncthreads();  // 1: layer-1 outputs complete
    // ------------------------------------------------------------ L2
    // Beside the first stage's k-steps: this step's noise, and the next step's table row and market
    // rows straight into LDS.  Beside the next ones: the market entries of the step's state rows from
    // LDS straight to the trajectory, one store (64 entries of a row) per two k-steps (all compute
    // units are at the same place of the step: closer together, the stores come at the rate that the
    // memory takes them and hold up the wavefronts).
    float eps[ET][2];
    {
      constexpr int kFirst = 8, kRuns = K * H / 64 / 4;  // kRuns: 64-float runs of the table row per wavefront
      const __amdgpu_buffer_rsrc_t r_eps = rows_rsrc(F.sigma != 0.0f ? F.eps : nullptr, row0 * D, 4, M * D);
      const __amdgpu_buffer_rsrc_t r_mt = rows_rsrc(nxt ? F.mt : nullptr, static_cast<size_t>(j + 1) * K * H, 4, K * H);
      // Market entry u of a state row: close[t+1] (u < D), then ind[t+1].  Rows past M fall beyond
      // the range.
      int pos = kNoStore;
      float v = 0.0f;
      const auto entry = [&](int k) {
        const int u = lane + 64 * k;
        const bool cl = u < D;
        if (u < n_mkt) v = in[cl ? D + u : kRInd + u - D] * (cl ? C.price_scale : 1.0f);
        pos = u < n_mkt ? 4 * (PW * wave * S + 1 + u + (cl ? 0 : D)) : kNoStore;
      };
      wide_layer2<ET>(w2, s_b2, s_x1, s_x2, wave, lane, [&](int st, int kk) {
        const int i = 8 * st + kk;
        if (i < 2 * ET) {
          const int m = PW * wave + 4 * (i / 2) + (lane >> 4), d = (lane & 15) + 16 * (i & 1);
          eps[i / 2][i & 1] = load_f32(r_eps, m < M && d < D ? 4 * (m * D + d) : kNoStore);
        } else if (i < 2 * ET + kRuns) {
          const int o = 64 * (kRuns * wave + i - 2 * ET);
          if (nxt) __builtin_amdgcn_raw_ptr_buffer_load_lds(r_mt, s_mt + o, 4, 4 * (lane + o), 0, 0, 0);
        } else if (i == kFirst - 1) {
          if (nxt && wave == 3) fetch_market(C, F.t0 + j + 1, in_next, lane);
          entry(0);
        } else if (i >= kFirst && i < kFirst + 8 * PW && i % 2 == 0) {
          const int k = (i - kFirst) / 2 / PW, e = (i - kFirst) / 2 % PW;
          store_f32(r_obs, pos, v);
          pos += 4 * S;
          if (e == PW - 1 && k < 3) entry(k + 1);
        }
      });
    }
    __syncthreads();  // 2: layer-2 outputs complete
    // ------------------------------------------------------------ L3
    wide_layer3<ET>(s_w3, s_x2, s_part, wave, lane);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the next step's inputs are in LDS
    __syncthreads();                     // 3: the partial sums complete
    if (L::kRefetch && nxt) fetch_w1e(sm + L::w1e, lane);
    // ------------------------------------------------------------ the trading step
    {
#pragma clang fp contract(off)
      const int jl = lane & 15, m0 = PW * wave + (lane >> 4);  // pass q: environment m0 + 4 q
      double cash[ET], pro[2][ET];
      int sold[ET][2];
      float act[ET][2];
      BuySet B[ET][2];
#pragma unroll
      for (int q = 0; q < ET; ++q) {
        const int m = m0 + 4 * q;
        cash[q] = s_state[4 * m];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int d = jl + 16 * s;
          const bool on = m < M && d < D;
          // Action: a_bar = sum_k w_k tanh(z_k + b3_k), z_k the sum of the wavefronts' partial
          // sums, in actor order; noise, clip (Section 5.2.1).
          float mean = 0.0f;
#pragma unroll
          for (int a = 0; a < K; ++a) {
            const float* p = s_part + a * 4 * MR * 32 + part_at(m, d);
            const float zs = ((p[0] + p[MR * 32]) + p[2 * MR * 32]) + p[3 * MR * 32];
            const float v = s_mix[a] * fast_tanh(zs + s_b3[a * 32 + d]);
            mean = a == 0 ? v : mean + v;
          }
          const float noisy = F.sigma != 0.0f ? mean + F.sigma * eps[q][s] : mean;
          act[q][s] = on ? fminf(fmaxf(noisy, -1.0f), 1.0f) : 0.0f;
          // Order and sale of stock d; the whole-order and one-share debits.
          const float p = on ? in[d] : 0.0f;
          const int qo = on ? order_from_action(act[q][s], C.hmax_f) : 0;
          sold[q][s] = qo < 0 ? min(hold[q][s], -qo) : 0;
          hold[q][s] -= sold[q][s];
          const double pd = static_cast<double>(p);
          const int qd = qo > 0 ? qo : 0;
          pro[s][q] = (pd * static_cast<double>(sold[q][s])) * C.one_m;
          B[q][s].deb = (pd * static_cast<double>(qd)) * C.one_p;
          B[q][s].c1 = pd * C.one_p;
          B[q][s].pq = pack_pq(p, qd);
        }
      }
      // The cash recurrence: all sells in ascending stock order, then the buys (Section 3.1);
      // stocks beyond D carry zero terms, which leave the cash unchanged.
#pragma unroll
      for (int q = 0; q < ET; ++q) cash[q] = row_sum(row_sum(cash[q], pro[0][q]), pro[1][q]);
      int kown[ET][2];
#pragma unroll
      for (int q = 0; q < ET; ++q) kown[q][0] = kown[q][1] = 0;
      buy_all_seg4<ET>(cash, kown, lane, B, C.one_p);
      // The W1e fragments have landed (requested before the trade; the stores come after this wait, and
      // would queue behind the fragments if they came sooner).
      if (L::kRefetch) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      // Holdings, executed quantities, the new day's position values, value and reward.
      double val[2][ET], v_new[ET];
#pragma unroll
      for (int q = 0; q < ET; ++q)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int m = m0 + 4 * q, d = jl + 16 * s;
          const bool on = m < M && d < D;
          hold[q][s] += kown[q][s];
          const float pn = on ? in[D + d] : 0.0f;
          val[s][q] = static_cast<double>(pn) * static_cast<double>(hold[q][s]);
          const float he = static_cast<float>(hold[q][s]) * C.hold_scale;
          if (on) s_x0[m * kRX0 + 1 + d] = static_cast<__bf16>(he);
          const int o = on ? 4 * (m * D + d) : kNoStore;
          store_f32(rows_rsrc(F.act_traj, row0 * D, 4, M * D), o, act[q][s]);
          store_f32(rows_rsrc(F.qty_traj, row0 * D, 4, M * D), o, __int_as_float(kown[q][s] - sold[q][s]));
          store_f32(r_obs, on ? 4 * (m * S + 1 + D + d) : kNoStore, he);
        }
#pragma unroll
      for (int q = 0; q < ET; ++q) v_new[q] = cash[q];
      row_sums(v_new, val[0]);
      row_sums(v_new, val[1]);
#pragma unroll
      for (int q = 0; q < ET; ++q) {
        const int m = m0 + 4 * q;
        const bool own = m < M && jl == 0;
        const float ce = static_cast<float>(cash[q] * static_cast<double>(C.cash_scale));
        const double r = (v_new[q] - s_state[4 * m + 1]) * C.reward_scale;
        store_f32(r_obs, own ? 4 * m * S : kNoStore, ce);
        typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, r), rows_rsrc(F.rew_traj, row0, 8, M),
                                              own ? 8 * m : kNoStore, 0, 0);
        if (own) {
          s_state[4 * m] = cash[q];
          s_state[4 * m + 1] = v_new[q];
          s_state[4 * m + 2] = s_state[4 * m + 2] + r;
          s_x0[m * kRX0] = static_cast<__bf16>(ce);
        }
      }
    }
    __syncthreads();  // 4: the next state rows are in LDS
  }
  // The trading state back to HBM.
#pragma unroll
  for (int q = 0; q < ET; ++q) {
    const int m = PW * wave + 4 * q + (lane0 >> 4), j = lane0 & 15;
    if (m >= M) continue;
    if (j == 0) {
      const double* s_state = reinterpret_cast<const double*>(smem + L::state) + 4 * m;
      st.cash[n0 + m] = s_state[0];
      st.asset[n0 + m] = s_state[1];
      st.cumrew[n0 + m] = s_state[2];
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (j + 16 * s < D) st.hold[static_cast<size_t>(j + 16 * s) * N + n0 + m] = hold[q][s];
  }
}

template <int ET>
hipError_t go_wide(int grid, const EnvConst& C, const EnvState& st, const EnsDev& E, const FusedArgs& F,
                   hipStream_t stream) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fused_wide_kernel<ET>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(WLds<ET>::total));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fused_wide_kernel<ET>, dim3(grid), dim3(kWT), WLds<ET>::total, stream, C, st, E, F);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wide_chunk(const EnvConst& C, const EnvState& st, const EnsDev& E, const FusedArgs& F,
                             hipStream_t stream) {
  if (F.tile_envs < 1 || F.tile_envs > 32) return hipErrorInvalidValue;
  const int grid = (C.N + F.tile_envs - 1) / F.tile_envs;
  return F.tile_envs <= 16 ? go_wide<1>(grid, C, st, E, F, stream) : go_wide<2>(grid, C, st, E, F, stream);
}

}  // namespace fm
