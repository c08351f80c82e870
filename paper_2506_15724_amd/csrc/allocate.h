// Eq. 10-11 and Eq. 8 for one batch item by one wavefront: used by madakv_allocate and, with the segment layout in the
// same launch, by madakv_evict.
#pragma once
#include "common.h"
#include "mpa_split.h"

namespace madakv {

struct AllocArgs {
  const void* stats; const int32_t* n_mod; int32_t* budgets; long long* pool;
  int n, B, H, NL, layer0, nc, beta, rho, mpa_mode, hcc_mode, keep_all, M;
};

AllocArgs alloc_args(const Dims& dm, const madakv_config& c, int layer0, const void* stats, const int32_t* n_mod, int32_t* budgets, long long* pool_state);

// num / den and the remainder, for a quotient below 2^40: a double estimate is off by at most one either way.  (The
// compiler's 64-bit division takes some 150 instructions; there are four per layer, one layer after the other: 44 us for
// 28 layers, 31 with this, the next layer's counts on their way and the split taken out of the chain.)
__device__ __forceinline__ long long div_rem(long long num, long long den, long long& rem) {
  long long q = (long long)((double)num * (1.0 / (double)den));
  long long r = num - q * den;
  if (r < 0) { --q; r += den; }
  else if (r >= den) { ++q; r -= den; }
  if (r < 0) { --q; r += den; }
  else if (r >= den) { ++q; r -= den; }
  rem = r;
  return q;
}
__device__ __forceinline__ long long lane_sum(long long x) {               // of non-negative values, the same in every lane
  const unsigned long long s = wave_incl_scan_u64((unsigned long long)x);
  return (long long)(((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(s >> 32), 63) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)s, 63));
}

// +1 for the `extra` lanes with the largest remainder (ties: lower lane first).
__device__ __forceinline__ long long largest_remainder(long long base, long long rem, long long extra, int lane, int H) {
  int rank = 0;
  for (int o = 0; o < H; ++o) {
    const long long ro = ((long long)__builtin_amdgcn_readlane((int)(rem >> 32), o) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)rem, o);
    if (lane < H && (ro > rem || (ro == rem && o < lane))) ++rank;
  }
  return base + ((long long)rank < extra ? 1 : 0);
}

// Eq. 8 of one head with the total ah
__device__ __forceinline__ void split_one(const AllocArgs& a, int b, long long idx, long long ah) {
#pragma clang fp contract(off)
  constexpr int MAXM = 4;
  const int M = a.M;
  long long nm[MAXM], bm[MAXM];
  float wm[MAXM];
  const float* rec = reinterpret_cast<const float*>(a.stats) + idx * 2 * M;
#pragma unroll
  for (int m = 0; m < MAXM; ++m) { nm[m] = m < M ? a.n_mod[b * M + m] : 0; wm[m] = m < M ? rec[m] : 0.f; }
  if (a.keep_all) {
#pragma unroll
    for (int m = 0; m < MAXM; ++m) bm[m] = nm[m];
  } else {
    mpa_split_device(ah, wm, nm, M, a.mpa_mode, bm);
  }
  for (int m = 0; m < M; ++m) a.budgets[idx * M + m] = (int32_t)bm[m];
}

// Eq. 10-11, one wave: the heads' totals, left in the first slot of their budgets.  The layers are a serial chain; the
// Eq. 8 split of the totals is not part of it (split_totals).
__device__ __forceinline__ void allocate_wave(const AllocArgs& a, int b, int lane) {
  const bool act = lane < a.H;
  constexpr int MAXM = 4;
  const int M = a.M;
  if (a.keep_all) return;
  const long long H = a.H, nc = a.nc, rho = a.rho, beta = a.beta;
  long long R = (a.layer0 == 0) ? (long long)a.NL * H * beta : a.pool[b];
  long long bf = beta / (rho * rho);
  if (bf < 1) bf = 1;

  int32_t kn[MAXM];                               // the next layer's counts (a record: M float masses, M int32 counts)
  auto fetch = [&](int li) {
    const float* rec = reinterpret_cast<const float*>(a.stats) + (((long long)li * a.B + b) * a.H + lane) * 2 * M;
#pragma unroll
    for (int m = 0; m < MAXM; ++m) kn[m] = (act && m < M) ? reinterpret_cast<const int32_t*>(rec)[M + m] : 0;
  };
  fetch(0);
  for (int li = 0; li < a.n; ++li) {
    const int l = a.layer0 + li;
    const long long idx = ((long long)li * a.B + b) * a.H + lane;
    // the head's record: M float masses (Eq. 6) then M int32 counts (Eq. 9)
    long long km = 0;
#pragma unroll
    for (int m = 0; m < MAXM; ++m) km += kn[m];
    if (li + 1 < a.n) fetch(li + 1);
    long long ah;
    if (!a.hcc_mode) {
      ah = beta;
    } else {
      const long long rem = a.NL - l;
      long long r0;
      long long lo = div_rem(R + rho * H * rem - 1, rho * H * rem, r0);
      if (lo < 1) lo = 1;
      long long hi = div_rem(rho * R, H * rem, r0);
      if (hi > nc) hi = nc;
      long long dem = km;
      dem = dem < lo ? lo : (dem > hi ? hi : dem);
      if (!act) dem = 0;
      const long long D = lane_sum(dem);
      long long A;
      if (rem == 1) {
        A = R;
      } else {
        const long long amin = R - (rem - 1) * H * nc, amax = R - (rem - 1) * H * bf;
        A = D < amin ? amin : (D > amax ? amax : D);
      }
      if (a.hcc_mode == 2) {
        // Eq. 8 as printed: one budget per layer; the A mod H spare tokens go to the lowest heads
        ah = A / H + (lane < A % H ? 1 : 0);
      } else if (A == D) {
        ah = dem;
      } else if (A < D) {
        const long long num = A * dem;
        long long r;
        const long long base = div_rem(num, D, r);
        const long long extra = A - lane_sum(act ? base : 0);
        ah = largest_remainder(base, act ? r : -1, extra, lane, a.H);
      } else {
        const long long room = act ? nc - dem : 0;
        const long long S = A - D, Rm = lane_sum(room);
        const long long num = S * room;
        long long r;
        const long long base = div_rem(num, Rm, r);
        const long long extra = S - lane_sum(act ? base : 0);
        ah = dem + largest_remainder(base, act ? r : -1, extra, lane, a.H);
      }
      R -= A;
    }
    if (a.n == 1) { if (act) split_one(a, b, idx, ah); }      // (a call of one layer: no trip through memory, 2 us)
    else if (act) a.budgets[idx * M] = (int32_t)ah;
  }
  if (lane == 0) a.pool[b] = R;
}

// Eq. 8 of every (layer, head) of the batch item, by the whole workgroup, behind a barrier
__device__ __forceinline__ void split_totals(const AllocArgs& a, int b, int tid, int threads) {
  if (a.n == 1 && !a.keep_all) return;                        // (done by the wave)
  for (int f = tid; f < a.n * a.H; f += threads) {
    const long long idx = ((long long)(f / a.H) * a.B + b) * a.H + f % a.H;
    split_one(a, b, idx, a.keep_all ? 0 : a.budgets[idx * a.M]);
  }
}

}  // namespace madakv

