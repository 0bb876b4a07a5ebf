// Ensemble kernels: weight packing, the per-actor MLP over 16- or 32-row tiles, and the combine step
// (weighted average of the actor means, Gaussian noise, clip) used by ensemble_act.
#include <algorithm>

#include "device_common.h"
#include "launch.h"
#include "mlp_device.h"

namespace fm {

namespace {

// Pack one float32 matrix W [kin][nout] (row-major) into the MFMA B-operand layout of DT.
template <int DT>
__global__ void pack_matrix_kernel(const float* __restrict__ w, int kin, int nout, int kin_pad,
                                   int nout_pad, void* __restrict__ out) {
  const size_t total = static_cast<size_t>(kin_pad) * nout_pad;
  const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= total) return;
  int k, col;
  if constexpr (DT == kF32) {
    // i = ((c * KQ + kq) * 64 + lane) * 4 + e
    const int e = static_cast<int>(i & 3);
    const int lane = static_cast<int>((i >> 2) & 63);
    const size_t rest = i >> 8;
    const int KQ = kin_pad / 16;
    const int kq = static_cast<int>(rest % KQ);
    const int c = static_cast<int>(rest / KQ);
    k = 16 * kq + 4 * e + (lane >> 4);
    col = 16 * c + (lane & 15);
    static_cast<float*>(out)[i] = (k < kin && col < nout) ? w[static_cast<size_t>(k) * nout + col] : 0.0f;
  } else {
    // i = ((c * KK + kk) * 64 + lane) * 8 + j
    const int j = static_cast<int>(i & 7);
    const int lane = static_cast<int>((i >> 3) & 63);
    const size_t rest = i >> 9;
    const int KK = kin_pad / 32;
    const int kk = static_cast<int>(rest % KK);
    const int c = static_cast<int>(rest / KK);
    k = 32 * kk + 8 * (lane >> 4) + j;
    col = 16 * c + (lane & 15);
    const float v = (k < kin && col < nout) ? w[static_cast<size_t>(k) * nout + col] : 0.0f;
    static_cast<__bf16*>(out)[i] = static_cast<__bf16>(v);  // round to nearest even
  }
}

// Rows 0 and A+1..2A of W1 [S][H] (cash, holdings) as bfloat16 MFMA fragments over ke_pad rows.
__global__ void pack_env_rows_kernel(const float* __restrict__ w1, int A, int H, int ke_pad,
                                     __bf16* __restrict__ out) {
  const size_t total = static_cast<size_t>(ke_pad) * H;
  const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= total) return;
  // i = ((c * KK + kk) * 64 + lane) * 8 + j
  const int j = static_cast<int>(i & 7);
  const int lane = static_cast<int>((i >> 3) & 63);
  const size_t rest = i >> 9;
  const int KK = ke_pad / 32;
  const int kk = static_cast<int>(rest % KK);
  const int c = static_cast<int>(rest / KK);
  const int k = 32 * kk + 8 * (lane >> 4) + j;
  const int col = 16 * c + (lane & 15);
  const int row = k == 0 ? 0 : (k <= A ? A + k : -1);
  const float v = (row >= 0 && col < H) ? w1[static_cast<size_t>(row) * H + col] : 0.0f;
  out[i] = static_cast<__bf16>(v);
}

// Rows 1..A and 2A+1..S-1 of W1 [S][H] (closes, indicators) as bfloat16 [S-1-A][H].
__global__ void gather_market_rows_kernel(const float* __restrict__ w1, int S, int H, int A,
                                          __bf16* __restrict__ out) {
  const size_t total = static_cast<size_t>(S - 1 - A) * H;
  const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int f = static_cast<int>(i / H), col = static_cast<int>(i - static_cast<size_t>(f) * H);
  const int row = f < A ? 1 + f : A + 1 + f;
  out[i] = static_cast<__bf16>(w1[static_cast<size_t>(row) * H + col]);
}

__global__ void copy_pad_kernel(const float* __restrict__ src, int n, int n_pad,
                                float* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_pad) dst[i] = i < n ? src[i] : 0.0f;
}

// Wavefronts of an MLP workgroup; a wavefront owns output tiles wave and wave + 16 of every layer.
constexpr int kMlpWaves = 16;

// LDS position of activation column c: in float32 the k-th group of 16 columns is stored by
// (c mod 4, c / 4), so that a lane's operands of the four products of a group are one 16-byte read.
template <int DT>
__device__ __forceinline__ int act_pos(int c) {
  return DT == kF32 ? (c & ~15) | ((c & 3) << 2) | ((c >> 2) & 3) : c;
}
// Row stride (elements) of the activation tiles: 16-byte rows, free of bank conflicts.
template <int DT>
__host__ __device__ inline int mlp_stride(int kin_pad) {
  return DT == kF32 ? round_up(kin_pad, 32) + 4 : kin_pad + 8;
}

// One layer's products for RT row tiles and up to TMAX column tiles c0, c0 + 16 of a wavefront over
// k groups kbeg .. kend - 1 (of KG; 16 k for float32, 32 for bfloat16).  start() requests the
// first RING groups' fragments, before the activations that they meet are there; run() walks the
// groups in straight line, so that it waits for the fragments that it needs and not for the
// ones requested after them (with a guard per group the compiler waits for all).
template <int DT, int RT, int TMAX>
struct LayerProducts {
  static constexpr int RING = 4;
  const unsigned char* w;
  int KG, kbeg, kend, tj;
  floatx4 b[RING][TMAX];

  // Requests without a branch around them (what is beyond the range or the tiles reads its last
  // fragment again): the compiler counts outstanding loads over all paths.
  template <int TJ>
  __device__ __forceinline__ void fetch(int s, int kg, int lane) {
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      b[s][j] = *reinterpret_cast<const floatx4*>(w + (static_cast<size_t>((j < tj ? kMlpWaves * j * KG : 0) + kg) << 10) + 16u * lane);
  }
  __device__ __forceinline__ void start(const unsigned char* wp, int c0, int ntiles, int kg_all, int k0, int k1, int lane) {
    tj = c0 >= ntiles ? 0 : (ntiles - c0 + kMlpWaves - 1) / kMlpWaves;
    KG = kg_all;
    kbeg = k0;
    kend = k1;
    w = wp + (static_cast<size_t>(min(c0, ntiles - 1) * KG) << 10);
#pragma unroll
    for (int s = 0; s < RING; ++s) fetch<TMAX>(s, min(kbeg + s, kend - 1), lane);
  }
  template <int TJ>
  __device__ __forceinline__ void run_tiles(const typename MT<DT>::act_t* in, int ist, int lane, floatx4 (&acc)[RT][TMAX]) {
    using act_t = typename MT<DT>::act_t;
    const act_t* row = in + (lane & 15) * ist + (16 / sizeof(act_t)) * (lane >> 4);
    // Activation fragments of the next group are read before the products of this one.
    floatx4 a[2][RT];
    const auto read = [&](int p, int kg) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
        a[p][r] = *reinterpret_cast<const floatx4*>(row + 16 * r * ist + MT<DT>::kKGroup * min(kg, kend - 1));
    };
    read(0, kbeg);
    const auto products = [&](int s, int kg) {
      read((s + 1) & 1, kg + 1);
      __builtin_amdgcn_sched_barrier(0x6);
      const floatx4(&aa)[RT] = a[s & 1];
      if constexpr (DT == kF32) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r][j] = mfma_f32(aa[r][e], b[s][j][e], acc[r][j]);
      } else {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int r = 0; r < RT; ++r)
            acc[r][j] = mfma_bf16(__builtin_bit_cast(bf16x8, aa[r]), __builtin_bit_cast(bf16x8, b[s][j]), acc[r][j]);
      }
    };
    // Keeps a request where it stands (only scalar or vector arithmetic may move past):
    // otherwise a round's requests all sink to its end, and the next round waits for them.
    const auto keep = [] { __builtin_amdgcn_sched_barrier(0x6); };
    int g = kbeg;
    for (; g + 2 * RING <= kend; g += RING) {
#pragma unroll
      for (int s = 0; s < RING; ++s) {
        products(s, g + s);
        fetch<TJ>(s, g + RING + s, lane);
        keep();
      }
    }
    // One full round or a short one is left, or a full and a short one.
    if (g + RING < kend) {
#pragma unroll
      for (int s = 0; s < RING; ++s) {
        products(s, g + s);
        fetch<TJ>(s, min(g + RING + s, kend - 1), lane);
        keep();
      }
      g += RING;
    }
#pragma unroll
    for (int s = 0; s < RING; ++s)
      if (g + s < kend) products(s, g + s);
  }
  __device__ __forceinline__ void run(const typename MT<DT>::act_t* in, int ist, int lane, floatx4 (&acc)[RT][TMAX]) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int j = 0; j < TMAX; ++j) acc[r][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if (tj == 1) run_tiles<1>(in, ist, lane, acc);
    if constexpr (TMAX == 2)
      if (tj == 2) run_tiles<2>(in, ist, lane, acc);
  }
};

// The MLP of actor blockIdx.y on rows [16 RT blockIdx.x, +16 RT) of obs [n][S]; writes tanh
// outputs to mu [K][n][A].  Bound by the float32 matrix instructions at large batches (32 cycles
// each, and the activations' vector instructions add to them: on this unit the two do not overlap),
// by its chain of latencies at small ones, so the first weights of a layer are requested before the
// activations of the layer before it.  2048 float32 rows, 256 units, three actors: 23.5 us a call
// against 29 with a guard around each group's loads and products.
// slices: layer 3's k range is cut in so many, part of the result's rounding.
template <int DT, int RT, int TMAX>
__global__ __launch_bounds__(64 * kMlpWaves) void mlp_kernel(EnsDev E, const float* __restrict__ obs, int n, int slices,
                                                             float* __restrict__ mu) {
  using act_t = typename MT<DT>::act_t;
  constexpr int R = 16 * RT, NW = kMlpWaves;
  extern __shared__ __align__(16) unsigned char smem[];
  const int k = blockIdx.y;
  const int row0 = blockIdx.x * R;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int st0 = mlp_stride<DT>(E.S_pad), sth = mlp_stride<DT>(E.H);
  // Two LDS regions: the state tile, then layer 2's outputs, in the first; layer 1's in the second.
  act_t* x0 = reinterpret_cast<act_t*>(smem);
  act_t* x1 = x0 + R * max(st0, sth);
  act_t* x2 = x0;

  const unsigned char* P = E.base + static_cast<size_t>(k) * E.actor_stride;
  const float* b1 = reinterpret_cast<const float*>(P + E.off_b1);
  const float* b2 = reinterpret_cast<const float*>(P + E.off_b2);
  const float* b3 = reinterpret_cast<const float*>(P + E.off_b3);
  const int row_q = 4 * (lane >> 4), col_l = lane & 15;
  const int ht = E.H / 16, nt3 = E.A_pad / 16;
  const int kg1 = E.S_pad / MT<DT>::kKGroup, kgh = E.H / MT<DT>::kKGroup;
  const int c3 = slices > 1 ? wave % nt3 : wave, sl = slices > 1 ? wave / nt3 : 0;

  // Biases of the wavefront's tiles (tiles that it does not have read another's).
  float bv[TMAX];
  const auto bias = [&](const float* b, int c0, int nout) {
#pragma unroll
    for (int j = 0; j < TMAX; ++j) bv[j] = b[min(16 * (c0 + NW * j) + col_l, nout - 1)];
  };
  LayerProducts<DT, RT, TMAX> L;
  floatx4 acc[RT][TMAX];
  // tanh(acc + bias) into the rows `out` (of tiles known as L.tj: read before the next start).
  const auto hidden = [&](act_t* out, int tj) {
#pragma unroll
    for (int j = 0; j < TMAX; ++j)
      if (j < tj)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          act_t* o = out + (16 * r + row_q) * sth + 16 * (wave + NW * j) + act_pos<DT>(col_l);
#pragma unroll
          for (int q = 0; q < 4; ++q) o[q * sth] = static_cast<act_t>(fast_tanh(acc[r][j][q] + bv[j]));
        }
  };

  bias(b1, wave, E.H);
  L.start(P + E.off_w1, wave, ht, kg1, 0, kg1, lane);
  // Stage the state tile, zero-padded to S_pad columns and R rows: a wavefront a row, four loads a
  // row in flight.
  for (int c0 = 0; c0 < E.S_pad; c0 += 256) {
    float v[RT][4];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[r][i] = obs[static_cast<size_t>(min(row0 + wave + NW * r, n - 1)) * E.S + min(c0 + 64 * i + lane, E.S - 1)];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = c0 + 64 * i + lane, row = wave + NW * r;
        if (c < E.S_pad)
          x0[row * st0 + act_pos<DT>(c)] = static_cast<act_t>(c < E.S && row0 + row < n ? v[r][i] : 0.0f);
      }
  }
  __syncthreads();
  L.run(x0, st0, lane, acc);
  const int tjh = L.tj;
  L.start(P + E.off_w2, wave, ht, kgh, 0, kgh, lane);
  hidden(x1, tjh);
  bias(b2, wave, E.H);
  __syncthreads();
  L.run(x1, sth, lane, acc);
  // Layer 3 has few output tiles (A_pad / 16): its k range is split over the otherwise idle
  // wavefronts, whose partial tiles meet in LDS (over layer 1's outputs, no longer needed) and
  // are summed in slice order.
  const int s3 = min(sl, slices - 1);
  L.start(P + E.off_w3, c3, nt3, kgh, s3 * kgh / slices, (s3 + 1) * kgh / slices, lane);
  if (sl >= slices) L.tj = 0;
  hidden(x2, tjh);
  bias(b3, c3, E.A);
  __syncthreads();
  L.run(x2, sth, lane, acc);
  float* mu_k = mu + static_cast<size_t>(k) * n * E.A;
  const auto out_epi = [&](int r, int c, int j, const floatx4& v) {
    const int col = 16 * c + col_l;
    if (col >= E.A) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = row0 + 16 * r + row_q + q;
      if (row < n) mu_k[static_cast<size_t>(row) * E.A + col] = fast_tanh(v[q] + bv[j]);
    }
  };
  if (slices == 1) {
#pragma unroll
    for (int j = 0; j < TMAX; ++j)
      if (j < L.tj)
#pragma unroll
        for (int r = 0; r < RT; ++r) out_epi(r, wave + NW * j, j, acc[r][j]);
    return;
  }
  floatx4* part = reinterpret_cast<floatx4*>(x1);  // [slices][nt3][RT][64]
  if (sl < slices)
#pragma unroll
    for (int r = 0; r < RT; ++r) part[((sl * nt3 + c3) * RT + r) * 64 + lane] = acc[r][0];
  __syncthreads();
  // Wavefront c3 + nt3 * (row tile) completes tile c3.
  if (sl < RT) {
    floatx4 v = part[(c3 * RT + sl) * 64 + lane];
    for (int q = 1; q < slices; ++q) {
      const floatx4 p = part[((q * nt3 + c3) * RT + sl) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] + p[e];
    }
    out_epi(sl, c3, 0, v);
  }
}

// a_bar = sum_k w_k mu_k; a = clip(a_bar + sigma * eps, -1, 1).  One thread per (row, group of
// four outputs) so each Philox block is drawn once.
__global__ void combine_kernel(int K, int n, int A, const float* __restrict__ mu,
                               const float* __restrict__ mix, float sigma, uint64_t key, int t,
                               int64_t env_offset, float* __restrict__ mean,
                               float* __restrict__ act) {
  const int G = (A + 3) >> 2;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * G) return;
  const int row = i / G, g = i - row * G;
  float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (sigma != 0.0f)
    noise_block(key, static_cast<uint64_t>(env_offset + row), static_cast<uint64_t>(t),
                static_cast<uint64_t>(g), z);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int d = 4 * g + r;
    if (d >= A) break;
    const size_t o = static_cast<size_t>(row) * A + d;
    float acc = 0.0f;
    for (int k = 0; k < K; ++k) acc = acc + mix[k] * mu[static_cast<size_t>(k) * n * A + o];
    if (mean) mean[o] = acc;
    float a = acc;
    if (sigma != 0.0f) a = acc + sigma * z[r];
    act[o] = fminf(fmaxf(a, -1.0f), 1.0f);
  }
}

template <int DT>
hipError_t launch_mlp_dt(const EnsDev& E, int units, const float* obs, int n, float* mu, hipStream_t stream) {
  // Sixteen wavefronts on tiles of 32 rows (each weight fragment serves two row tiles), or of 16
  // where those leave compute units idle.  Batches of at most 16 rows cut layer 3 into the
  // slices of a four-wavefront workgroup, larger ones into those of sixteen, whatever the tile.
  const int st0 = mlp_stride<DT>(E.S_pad), sth = mlp_stride<DT>(E.H);
  const auto lds_of = [&](int rt) { return static_cast<size_t>(16 * rt) * (std::max(st0, sth) + sth) * MT<DT>::kElem; };
  const bool fits = lds_of(2) <= 160 * 1024;
  const int tiles = (n + 15) / 16;
  const int rt = fits && tiles * E.K > units ? 2 : 1;
  // The library's limit on float32 networks past 16 rows: state width (rounded up to 32) and hidden width
  // together below 1280, where 32 rows of both with two floats of padding each fill 160 KB.  (Tiles of 16
  // rows would go further; what a call accepts does not depend on the tile that it takes.)
  if (DT == kF32 && n > 16 && round_up(E.S_pad, 32) + E.H >= 1280) return hipErrorInvalidValue;
  const int nt3 = E.A_pad / 16, nk3 = E.H / MT<DT>::kKGroup;
  const int cap = 16 * sth * MT<DT>::kElem / (nt3 * 1024);
  const int slices = std::max(1, std::min(std::min((n > 16 ? kMlpWaves : 4) / nt3, nk3), cap));
  const dim3 grid((n + 16 * rt - 1) / (16 * rt), E.K);
  const auto go = [&](auto kern) -> hipError_t {
    if (lds_of(rt) > 64 * 1024) {  // past the default limit
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_of(rt)));
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * kMlpWaves), lds_of(rt), stream, E, obs, n, slices, mu);
    return hipGetLastError();
  };
  if (E.H <= 16 * kMlpWaves) return rt == 2 ? go(mlp_kernel<DT, 2, 1>) : go(mlp_kernel<DT, 1, 1>);
  return rt == 2 ? go(mlp_kernel<DT, 2, 2>) : go(mlp_kernel<DT, 1, 2>);
}

}  // namespace

hipError_t launch_pack_matrix(int dtype, const float* w, int kin, int nout, int kin_pad,
                              int nout_pad, void* out, hipStream_t stream) {
  const size_t total = static_cast<size_t>(kin_pad) * nout_pad;
  const dim3 grid(static_cast<unsigned>((total + 255) / 256));
  if (dtype == kF32)
    hipLaunchKernelGGL(pack_matrix_kernel<kF32>, grid, dim3(256), 0, stream, w, kin, nout, kin_pad,
                       nout_pad, out);
  else
    hipLaunchKernelGGL(pack_matrix_kernel<kBF16>, grid, dim3(256), 0, stream, w, kin, nout, kin_pad,
                       nout_pad, out);
  return hipGetLastError();
}

hipError_t launch_pack_env_rows(const float* w1, int A, int H, int ke_pad, void* out, hipStream_t stream) {
  const size_t total = static_cast<size_t>(ke_pad) * H;
  hipLaunchKernelGGL(pack_env_rows_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, stream,
                     w1, A, H, ke_pad, static_cast<__bf16*>(out));
  return hipGetLastError();
}

hipError_t launch_gather_market_rows(const float* w1, int S, int H, int A, __bf16* out, hipStream_t stream) {
  const size_t total = static_cast<size_t>(S - 1 - A) * H;
  hipLaunchKernelGGL(gather_market_rows_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0,
                     stream, w1, S, H, A, out);
  return hipGetLastError();
}

hipError_t launch_copy_pad(const float* src, int n, int n_pad, float* dst, hipStream_t stream) {
  hipLaunchKernelGGL(copy_pad_kernel, dim3((n_pad + 255) / 256), dim3(256), 0, stream, src, n, n_pad,
                     dst);
  return hipGetLastError();
}

hipError_t launch_mlp(int dtype, const EnsDev& E, int units, const float* obs, int n, float* mu,
                      hipStream_t stream) {
  return dtype == kF32 ? launch_mlp_dt<kF32>(E, units, obs, n, mu, stream)
                       : launch_mlp_dt<kBF16>(E, units, obs, n, mu, stream);
}

hipError_t launch_combine(int K, int n, int A, const float* mu, const float* mix, float sigma,
                          uint64_t key, int t, int64_t env_offset, float* mean, float* act,
                          hipStream_t stream) {
  const int total = n * ((A + 3) >> 2);
  hipLaunchKernelGGL(combine_kernel, dim3((total + 255) / 256), dim3(256), 0, stream, K, n, A, mu, mix,
                     sigma, key, t, env_offset, mean, act);
  return hipGetLastError();
}

}  // namespace fm
