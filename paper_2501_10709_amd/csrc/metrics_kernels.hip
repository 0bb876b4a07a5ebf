// Backtest metrics of a reward trajectory (the financial metrics the paper evaluates agents with)
// over the equity curve v_{t+1} = v_t + r_t / scale of each environment.  Two kernels with the
// same arithmetic, every sum in day order:
//   metrics_kernel       a workgroup per kEnvs environments;
//   metrics_walk_kernel  a thread per environment.
// launch_metrics states the choice.
#include "launch.h"

namespace fm {

namespace {

constexpr int kEnvs = 8;     // environments per workgroup: 64-byte runs of a day's rewards
constexpr int kDays = 256;   // days per pass (a trading year in one)
constexpr int kThreads = 256;
constexpr int kPer = kDays * kEnvs / kThreads;  // days per thread of a pass

// The ten metrics from an environment's sums.
__device__ __forceinline__ void write_metrics(double* o, int T, double v0, double v, double mean, double ss, double up,
                                              double dn, double down2, double mdd, int wins, int losses, double P,
                                              double rfp) {
#pragma clang fp contract(off)
  const double sd = T > 1 ? sqrt(ss / (T - 1)) : __builtin_nan("");
  const double sqp = sqrt(P);
  const double cum = v / v0 - 1.0;
  const double ann = pow(v / v0, P / T) - 1.0;
  const double ex_mean = mean - rfp;
  const double down = sqrt(down2 / T);
  o[0] = cum;
  o[1] = ann;
  o[2] = sd * sqp;
  o[3] = ex_mean / sd * sqp;
  o[4] = mdd;
  o[5] = cum / fabs(mdd);
  o[6] = ex_mean / down * sqp;
  o[7] = ann / fabs(mdd);
  o[8] = up / dn;
  o[9] = static_cast<double>(wins) / static_cast<double>(losses);
}

// One thread walks an environment's curve twice, first for the sums, extrema and counts, then for
// the sample deviation around the mean return.  Loads of rew[t][n] are coalesced.
__global__ void metrics_walk_kernel(const double* __restrict__ rew, int T, int N, double v0_all,
                               const double* __restrict__ v0s, double scale, double P, double rf,
                               double* __restrict__ out) {
#pragma clang fp contract(off)
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const double v0 = v0s ? v0s[n] : v0_all;
  const double rfp = rf / P;
  double v = v0, peak = v0, mdd = 0.0, sum = 0.0, up = 0.0, dn = 0.0, down2 = 0.0;
  int wins = 0, losses = 0;
  for (int t = 0; t < T; ++t) {
    const double v_next = v + rew[static_cast<size_t>(t) * N + n] / scale;
    const double rho = v_next / v - 1.0;
    sum += rho;
    if (rho > 0.0) {
      up += rho;
      ++wins;
    } else if (rho < 0.0) {
      dn -= rho;
      ++losses;
    }
    const double ex = rho - rfp;
    if (ex < 0.0) down2 += ex * ex;
    v = v_next;
    peak = fmax(peak, v);
    mdd = fmin(mdd, v / peak - 1.0);
  }
  const double mean = sum / T;
  double ss = 0.0;
  double w = v0;
  for (int t = 0; t < T; ++t) {
    const double w_next = w + rew[static_cast<size_t>(t) * N + n] / scale;
    const double dev = (w_next / w - 1.0) - mean;
    ss += dev * dev;
    w = w_next;
  }
  write_metrics(out + static_cast<size_t>(n) * 10, T, v0, v, mean, ss, up, dn, down2, mdd, wins, losses, P, rfp);
}

// use(i, load(i)) for i = 0 .. len - 1 in order, the loads a whole batch ahead of their uses.
template <class Load, class Use>
__device__ __forceinline__ void serial_days(int len, Load load, Use use) {
  constexpr int kB = 16;
  double x[kB];
  for (int i = 0; i < len; i += kB) {
#pragma unroll
    for (int k = 0; k < kB; ++k) x[k] = load(i + k);  // past len: leftovers inside the plane
#pragma unroll
    for (int k = 0; k < kB; ++k)
      if (i + k < len) use(i + k, x[k]);
  }
}

// Latency bound: an environment is a few serial chains of T float64 additions, and a thread that
// walks them alone pays for each day's three divisions between two links.  Here all threads of a
// workgroup divide, one (day, environment) each, and only the additions run serially: the curve on
// one lane per environment of the first wavefront, then the four sums on one wavefront each, over
// terms in LDS, sixteen read ahead.  (The running peak is a maximum, so it is exact in any order.)
__global__ __launch_bounds__(kThreads) void metrics_kernel(const double* __restrict__ rew, int T, int N, double v0_all,
                                                           const double* __restrict__ v0s, double scale, double P,
                                                           double rf, double* __restrict__ out) {
#pragma clang fp contract(off)
  // [day][environment]: the curve before each day and after the last; the returns; a term.
  __shared__ double vs[(kDays + 1) * kEnvs], rhos[kDays * kEnvs], term[kDays * kEnvs];
  __shared__ double s_red[kThreads], s_sum[4][kEnvs];
  __shared__ int s_wins[kThreads], s_losses[kThreads];
  const int tid = threadIdx.x, e = tid % kEnvs, d0 = tid / kEnvs, wave = tid / 64;
  constexpr int kStep = kThreads / kEnvs;
  const bool serial = tid % 64 < kEnvs;  // the lanes of a wavefront that run a chain
  const int n0 = blockIdx.x * kEnvs, n = n0 + e;
  const bool on = n < N;
  const double rfp = rf / P;
  const double v0 = on ? (v0s ? v0s[n] : v0_all) : 1.0;

  // The curve over days t0 .. t0 + len - 1 from v (carried by the first wavefront's lanes), and
  // each day's return.  Entries past len hold leftovers that nothing uses.
  auto pass = [&](int t0, int len, double& v) {
    double r[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = d0 + k * kStep;
      r[k] = on && i < len ? rew[static_cast<size_t>(t0 + i) * N + n] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) term[(d0 + k * kStep) * kEnvs + e] = r[k] / scale;
    __syncthreads();
    if (wave == 0 && serial) {
      vs[e] = v;
      serial_days(len, [&](int i) { return term[i * kEnvs + e]; }, [&](int i, double d) {
        v = v + d;
        vs[(i + 1) * kEnvs + e] = v;
      });
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = d0 + k * kStep;
      const double rho = vs[(i + 1) * kEnvs + e] / vs[i * kEnvs + e] - 1.0;
      rhos[i * kEnvs + e] = rho;
      const double ex = rho - rfp;
      term[i * kEnvs + e] = ex < 0.0 ? ex * ex : 0.0;
    }
  };

  // First the sums, extrema and counts.  A day that has no part in a sum adds zero, which leaves
  // it as it is.
  double v = v0, peak = v0, mdd = 0.0, acc = 0.0;
  int wins = 0, losses = 0;
  for (int t0 = 0; t0 < T; t0 += kDays) {
    const int len = min(kDays, T - t0);
    pass(t0, len, v);
    // Thread d0 takes kPer consecutive days for the drawdowns: their peak, then the peaks before.
    const int i0 = d0 * kPer;
    double x[kPer], top = peak;
#pragma unroll
    for (int k = 0; k < kPer; ++k) x[k] = vs[(i0 + k + 1) * kEnvs + e];
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (i0 + k < len) top = fmax(top, x[k]);
    s_red[tid] = top;
    __syncthreads();
    top = peak;
    for (int j = 0; j < kStep; ++j) {
      const double other = s_red[j * kEnvs + e];
      if (j < d0) top = fmax(top, other);
      peak = fmax(peak, other);
    }
    double fall[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      top = fmax(top, x[k]);
      fall[k] = x[k] / top - 1.0;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (i0 + k < len) mdd = fmin(mdd, fall[k]);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = d0 + k * kStep;
      const double rho = rhos[i * kEnvs + e];
      wins += i < len && rho > 0.0;
      losses += i < len && rho < 0.0;
    }
    if (serial) {
      const auto rho_at = [&](int i) { return rhos[i * kEnvs + e]; };
      if (wave == 0) serial_days(len, rho_at, [&](int, double r) { acc = acc + r; });
      if (wave == 1) serial_days(len, rho_at, [&](int, double r) { acc = acc + fmax(r, 0.0); });
      if (wave == 2) serial_days(len, rho_at, [&](int, double r) { acc = acc + fmax(-r, 0.0); });
      if (wave == 3) serial_days(len, [&](int i) { return term[i * kEnvs + e]; }, [&](int, double d) { acc = acc + d; });
    }
    __syncthreads();  // the planes are free for the next pass
  }
  s_red[tid] = mdd;
  s_wins[tid] = wins;
  s_losses[tid] = losses;
  if (serial) s_sum[wave][e] = acc;
  __syncthreads();

  // Then the deviation around the mean return; a single pass's returns are still in LDS.
  const double mean = s_sum[0][e] / T;
  double ss = 0.0, w = v0;
  for (int t0 = 0; t0 < T; t0 += kDays) {
    const int len = min(kDays, T - t0);
    if (T > kDays) pass(t0, len, w);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = d0 + k * kStep;
      const double dev = rhos[i * kEnvs + e] - mean;
      term[i * kEnvs + e] = dev * dev;
    }
    __syncthreads();
    if (wave == 0 && serial)
      serial_days(len, [&](int i) { return term[i * kEnvs + e]; }, [&](int, double d) { ss = ss + d; });
    __syncthreads();
  }
  if (tid >= kEnvs || !on) return;
  for (int i = 1; i < kStep; ++i) {
    mdd = fmin(mdd, s_red[i * kEnvs + e]);
    wins += s_wins[i * kEnvs + e];
    losses += s_losses[i * kEnvs + e];
  }
  write_metrics(out + static_cast<size_t>(n) * 10, T, v0, v, mean, ss, s_sum[1][e], s_sum[2][e], s_sum[3][e], mdd, wins,
                losses, P, rfp);
}

}  // namespace

hipError_t launch_metrics(const double* rew, int T, int N, double v0, const double* v0s,
                          double reward_scale, double periods_per_year, double risk_free,
                          double* out, hipStream_t stream) {
  // Two workgroups of the first kind fit a compute unit, so past about 8192 environments they run
  // in several rounds while the second kind still has at most a wavefront per SIMD: 252 days of
  // 2048 environments take 26 us against 174, of 8192 61 against 190, of 16384 117 against 196 (but
  // 61 days of them 48 against 32).  Over a few days its fixed work (all of a pass's divisions)
  // does not pay: one day of 8192 environments takes 18 us against 8.7, launch included.  Whole calls: 32
  // days of 2048 take 27 us against 35, of 6144 35 against 36; 40 days of 8192 40 against 39, 48 of them
  // 40 against 43.
  if (N <= 8192 && T >= (N <= 6144 ? 32 : 48))
    hipLaunchKernelGGL(metrics_kernel, dim3((N + kEnvs - 1) / kEnvs), dim3(kThreads), 0, stream, rew, T, N, v0, v0s,
                       reward_scale, periods_per_year, risk_free, out);
  else
    hipLaunchKernelGGL(metrics_walk_kernel, dim3((N + 255) / 256), dim3(256), 0, stream, rew, T, N, v0, v0s,
                       reward_scale, periods_per_year, risk_free, out);
  return hipGetLastError();
}

}  // namespace fm
