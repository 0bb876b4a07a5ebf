// The trading chain of Section 3.1 run by a 16-lane row of a wavefront: lane j of the row owns
// stocks j and j + 16 (at most 32 stocks); the serial cash recurrences (the sells' proceeds, the
// buys, the value) run on terms broadcast along the row by DPP row broadcasts, in stock order, so
// every lane of the row holds the same cash.  Used by the row variant of the environment step and by the
// fused rollouts' resident, wide and (up to 32 stocks) generic schedules.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "device_common.h"

namespace fm {

// Lane L of each 16-lane row, broadcast to the whole row (64-bit DPP row broadcast).
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_update_dpp(__builtin_nondeterministic_value(v), v, 0x150 + L, 0xf, 0xf, true);
}
template <int L>
__device__ __forceinline__ long row_bcast(long v) {
  return __builtin_amdgcn_update_dpp(__builtin_nondeterministic_value(v), v, 0x150 + L, 0xf, 0xf, true);
}

// acc + v(lane 0) + v(lane 1) + ... + v(lane 15) of the row, in lane order.
template <int... L>
__device__ __forceinline__ double row_sum_impl(double acc, double v, std::integer_sequence<int, L...>) {
#pragma clang fp contract(off)
  ((acc = acc + row_bcast<L>(v)), ...);
  return acc;
}
__device__ __forceinline__ double row_sum(double acc, double v) {
  return row_sum_impl(acc, v, std::make_integer_sequence<int, 16>());
}

// One stock's buy terms, owned by one lane of the row: the whole order's debit (p q)(1+c), the
// one-share debit (p 1)(1+c), and the price and order packed as {float bits, int}.
struct BuySet {
  double deb, c1;
  long pq;
};
__device__ __forceinline__ long pack_pq(float p, int q) {
  return static_cast<long>((static_cast<unsigned long>(static_cast<unsigned>(q)) << 32) | __float_as_uint(p));
}
__device__ __forceinline__ float pq_price(long pq) { return __uint_as_float(static_cast<unsigned>(pq)); }
__device__ __forceinline__ int pq_order(long pq) { return static_cast<int>(static_cast<unsigned long>(pq) >> 32); }

// The buy of one stock whose whole order of q shares does not fit the cash while one share does
// (Section 3.1, reading 7): the largest k in [0, q-1] with debit(k) = (p k)(1+c) <= cash.  The
// estimate kd = floor(cash / c1), from the refined reciprocal of the one-share debit c1 and
// clamped to [0, q-1], is at most one share off; the debits of kd-1 .. kd+2 are formed side by
// side and the answer is the largest of kd-1, kd, kd+1 that fits.  If the answer were not in
// that range (kd-1 does not fit, or kd+2 does), ok is false and the caller takes unit steps.
__device__ __forceinline__ int partial_fill_sel(double cash, double p, double c1, int q, double one_p, double& debit,
                                               bool& ok) {
#pragma clang fp contract(off)
  double rc1 = __builtin_amdgcn_rcp(c1);
  rc1 = fma(fma(-c1, rc1, 1.0), rc1, rc1);
  const double kd = fmax(fmin(floor(cash * rc1), static_cast<double>(q - 1)), 0.0);
  const double dm = (p * (kd - 1.0)) * one_p, d0 = (p * kd) * one_p;
  const double dp = (p * (kd + 1.0)) * one_p, dpp = (p * (kd + 2.0)) * one_p;
  const bool fm = kd <= 1.0 || dm <= cash, f0 = kd <= 0.0 || d0 <= cash, fp = dp <= cash, fpp = dpp <= cash;
  ok = fm && !fpp;
  const int k = static_cast<int>(kd);
  debit = fp ? dp : (f0 ? d0 : (k >= 2 ? dm : 0.0));
  return fp ? k + 1 : (f0 ? k : (k >= 1 ? k - 1 : 0));
}

// acc - v(lane 0) - v(lane 1) - ... - v(lane 15) of the row, in lane order.
template <int... L>
__device__ __forceinline__ double row_sub_impl(double acc, double v, std::integer_sequence<int, L...>) {
#pragma clang fp contract(off)
  ((acc = acc - row_bcast<L>(v)), ...);
  return acc;
}

// The row's cash before each lane's stock under the serial recurrence P(j + 1) = P(j) - x(j),
// P(0) = start, x(j) held by lane j: carried along the row one lane per round by DPP row shifts
// (lane 0 has no source and keeps start), so lane j's value is the exact serial result of j
// subtractions in lane order.  total receives P(16).
__device__ __forceinline__ double row_shr1(double keep, double v) {
  return __builtin_amdgcn_update_dpp(keep, v, 0x111, 0xf, 0xf, false);
}
// row_sum of NQ independent sets step by step, so that their dependent chains fill each other's
// latencies, and the row prefixes above (t; totals P(16)) likewise.
template <int NQ, int L = 0>
__device__ __forceinline__ void row_sums(double (&acc)[NQ], const double (&v)[NQ]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int n = 0; n < NQ; ++n) acc[n] = acc[n] + row_bcast<L>(v[n]);
  if constexpr (L < 15) row_sums<NQ, L + 1>(acc, v);
}
template <int NQ>
__device__ __forceinline__ void row_prefixes(const double (&start)[NQ], const double (&x)[NQ], double (&t)[NQ],
                                             double (&total)[NQ]) {
#pragma clang fp contract(off)
  double d[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) t[n] = start[n];
#pragma unroll
  for (int r = 0; r < 15; ++r) {
#pragma unroll
    for (int n = 0; n < NQ; ++n) d[n] = t[n] - x[n];
#pragma unroll
    for (int n = 0; n < NQ; ++n) t[n] = row_shr1(t[n], d[n]);
  }
#pragma unroll
  for (int n = 0; n < NQ; ++n) total[n] = row_bcast<15>(t[n] - x[n]);
}

// The buys (Section 3.1, readings 5-7) of NQ sets of four environments, one per 16-lane row, the sets
// side by side (the steps below are chains of dependent instructions that leave most issue slots
// empty).  Rows may repeat one another.
// If every row's cash covers the sum of its whole orders with a margin far above the rounding of
// 32 subtractions, every whole order fits in sequence: the debits are subtracted in stock order
// and every order fills.  Otherwise one segment: with cash C, the candidates are the stocks with a
// buy order whose one-share debit fits C (the others cannot buy: the cash only falls during the
// buys).  Every candidate is assumed to fill its whole order; the row prefix of their debits gives
// the cash each one meets, exactly as the serial recurrence would, up to the first candidate e whose
// whole order does not fit that cash.  The candidates before e fill whole; e buys what its cash
// allows (a partial fill, or nothing when one share does not fit).  That usually leaves less cash
// than one share of e, and few later stocks are cheaper, so the buys go on as events: each row's
// next stock with a buy order whose one-share debit fits the cash buys its whole order or what the
// cash allows.  Both forms are exact; an event costs about a third of a segment.
// LEAVE: wavefronts without a candidate leave before the segment (agents that only buy are soon there:
// 100 given days of 30 stocks and 2048 environments take 188 us against 221, of 32 stocks and 8192 375
// against 418), in the row kernel and the resident schedule.  The others go without: the branch costs the
// batched form up to 4% and the wide schedule 0.5%.
template <int NQ, bool LEAVE = false>
__device__ __forceinline__ void buy_all_seg4(double (&cash)[NQ], int (&kown)[NQ][2], int lane, const BuySet (&B)[NQ][2],
                                             double one_p) {
#pragma clang fp contract(off)
  const int jl = lane & 15, rsh = lane & 48;  // rsh: this lane's row's bits in a ballot
  bool covered = true;
  double total[NQ], both[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    total[n] = 0.0;
    both[n] = B[n][0].deb + B[n][1].deb;  // any order: only a bound
  }
  row_sums(total, both);
#pragma unroll
  for (int n = 0; n < NQ; ++n) covered = covered && cash[n] >= total[n] * (1.0 + 0x1p-40);
  if (__builtin_amdgcn_ballot_w64(!covered) == 0) {
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      cash[n] = row_sub_impl(cash[n], B[n][0].deb, std::make_integer_sequence<int, 16>());
      cash[n] = row_sub_impl(cash[n], B[n][1].deb, std::make_integer_sequence<int, 16>());
      kown[n][0] = pq_order(B[n][0].pq);
      kown[n][1] = pq_order(B[n][1].pq);
    }
    return;
  }
  if constexpr (LEAVE) {
    bool some = false;
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int s = 0; s < 2; ++s) some = some || (pq_order(B[n][s].pq) > 0 && B[n][s].c1 <= cash[n]);
    if (__builtin_amdgcn_ballot_w64(some) == 0) return;
  }
  // One segment: every candidate's cash if those before it fill whole.
  double at[2][NQ], mid[NQ], end[NQ];  // the cash that the lane's stocks meet; after 16; after them all
  bool cand[2][NQ];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    double x[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      cand[s][n] = pq_order(B[n][s].pq) > 0 && B[n][s].c1 <= cash[n];
      x[n] = cand[s][n] ? B[n][s].deb : 0.0;
    }
    if (s == 0) row_prefixes(cash, x, at[0], mid);
    else row_prefixes(mid, x, at[1], end);
  }
  int dn[NQ];  // the rows' next stocks to consider
  bool more = false;
  // Stock e of each row (32: none), whose lane holds its cash pe, buys whole or what pe allows; the
  // row's cash becomes what is left, or `rest` where there is no such stock.
  const auto fill = [&](const int (&e)[NQ], const double (&pe)[NQ], const double (&rest)[NQ]) {
    bool slow = false, part[NQ], owner[NQ];
    int k[NQ];
    double nc[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const bool hi = e[n] >= 16;
      const double deb = hi ? B[n][1].deb : B[n][0].deb;
      const long pq = hi ? B[n][1].pq : B[n][0].pq;
      const double c1e = hi ? B[n][1].c1 : B[n][0].c1;
      owner[n] = e[n] < 32 && (e[n] & 15) == jl;
      const bool whole = deb <= pe[n];
      bool ok;
      double debit;
      k[n] = partial_fill_sel(pe[n], static_cast<double>(pq_price(pq)), c1e, pq_order(pq), one_p, debit, ok);
      part[n] = owner[n] && !whole && c1e <= pe[n] && !ok;
      slow = slow || part[n];
      k[n] = whole ? pq_order(pq) : c1e <= pe[n] ? k[n] : 0;
      debit = whole ? deb : c1e <= pe[n] ? debit : 0.0;
      nc[n] = owner[n] ? pe[n] - debit : rest[n];
    }
    if (__builtin_amdgcn_ballot_w64(slow) != 0) {
#pragma unroll
      for (int n = 0; n < NQ; ++n)
        if (part[n]) {
          const bool hi = e[n] >= 16;
          const long pq = hi ? B[n][1].pq : B[n][0].pq;
          const double c1e = hi ? B[n][1].c1 : B[n][0].c1;
          double rc1 = __builtin_amdgcn_rcp(c1e), debit;
          rc1 = fma(fma(-c1e, rc1, 1.0), rc1, rc1);
          k[n] = partial_fill(pe[n], static_cast<double>(pq_price(pq)), rc1, pq_order(pq), one_p, debit);
          nc[n] = pe[n] - debit;
        }
    }
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      if (owner[n] && e[n] < 16) kown[n][0] = k[n];
      if (owner[n] && e[n] >= 16) kown[n][1] = k[n];
      const int src = e[n] < 32 ? rsh + (e[n] & 15) : lane;
      const long nbits = __builtin_bit_cast(long, nc[n]);
      const int lo = __builtin_amdgcn_ds_bpermute(4 * src, static_cast<int>(nbits));
      const int hb = __builtin_amdgcn_ds_bpermute(4 * src, static_cast<int>(nbits >> 32));
      cash[n] = __builtin_bit_cast(
          double, static_cast<long>((static_cast<unsigned long>(static_cast<unsigned>(hb)) << 32) | static_cast<unsigned>(lo)));
      dn[n] = e[n] < 32 ? e[n] + 1 : 32;
    }
  };
  // The first stock of the row among two ballots (stocks 0-15, 16-31), or 32.
  const auto first_of = [&](unsigned long long b0, unsigned long long b1) {
    const unsigned mine = static_cast<unsigned>((b0 >> rsh) & 0xffffu) | (static_cast<unsigned>((b1 >> rsh) & 0xffffu) << 16);
    return mine != 0 ? __builtin_ctz(mine) : 32;
  };
  int e[NQ];
  double pe[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    e[n] = first_of(__builtin_amdgcn_ballot_w64(cand[0][n] && !(B[n][0].deb <= at[0][n])),
                    __builtin_amdgcn_ballot_w64(cand[1][n] && !(B[n][1].deb <= at[1][n])));
    if (cand[0][n] && jl < e[n]) kown[n][0] = pq_order(B[n][0].pq);
    if (cand[1][n] && jl + 16 < e[n]) kown[n][1] = pq_order(B[n][1].pq);
    pe[n] = e[n] >= 16 ? at[1][n] : at[0][n];
    more = more || e[n] < 32;
  }
  if (__builtin_amdgcn_ballot_w64(more) == 0) {  // every row filled all its candidates whole
#pragma unroll
    for (int n = 0; n < NQ; ++n) cash[n] = end[n];
    return;
  }
  fill(e, pe, end);
  for (int it = 0; it < 32; ++it) {
    more = false;
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      e[n] = first_of(
          __builtin_amdgcn_ballot_w64(pq_order(B[n][0].pq) > 0 && B[n][0].c1 <= cash[n] && jl >= dn[n]),
          __builtin_amdgcn_ballot_w64(pq_order(B[n][1].pq) > 0 && B[n][1].c1 <= cash[n] && jl + 16 >= dn[n]));
      more = more || e[n] < 32;
    }
    if (__builtin_amdgcn_ballot_w64(more) == 0) break;
    fill(e, cash, cash);
  }
}

// One set.
__device__ __forceinline__ void buy_all_rows(double& cash, int (&kown)[2], int lane, const BuySet (&B)[2], double one_p) {
  double c[1] = {cash};
  int k[1][2] = {{kown[0], kown[1]}};
  const BuySet S[1][2] = {{B[0], B[1]}};
  buy_all_seg4<1, true>(c, k, lane, S, one_p);
  cash = c[0];
  kown[0] = k[0][0];
  kown[1] = k[0][1];
}

}  // namespace fm
