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

// num / den and the remainder, for a quotient below 2^40: a double estimate is off by at most one either way.
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

// floor(num / den) of whole numbers below 2^53 held in doubles; inv = 1 / den rounded: the estimate is off by at most one
// either way, the remainder is exact
__device__ __forceinline__ double div_floor(double num, double den, double inv) {
  const double q = floor(num * inv), r = fma(-q, den, num);
  return q + (r < 0. ? -1. : r >= den ? 1. : 0.);
}
__device__ __forceinline__ double lane_value(double x, int src) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return __longlong_as_double((long long)(((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(u >> 32), src) << 32) |
                                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, src)));
}

// Eq. 10-11, one wave: the heads' totals, left in the first slot of their budgets.  The layers are a serial chain; the
// Eq. 8 split of the totals is not part of it (split_totals).  The chain is what a call over many layers waits for, so it
// holds little: pool, bounds and demands are whole numbers in doubles (the pool is below 2^36, rho times it below 2^46; no conversion of
// 64-bit integers), the reciprocals of 32 layers come from 32 lanes at once, and so do their counts, through LDS.
// 28 layers of 4 heads: with the layout 39 -> 28 us, alone 30 -> 22 (0.5 us per layer).
constexpr int ALLOC_BATCH = 32;
__device__ __forceinline__ void allocate_wave(const AllocArgs& a, int b, int lane) {
  __shared__ int s_count[ALLOC_BATCH][64];
  const bool act = lane < a.H;
  constexpr int MAXM = 4;
  const int M = a.M;
  if (a.keep_all) return;
  const long long H = a.H, nc = a.nc, rho = a.rho, beta = a.beta;
  const double Hd = (double)H, rhod = (double)rho, ncd = (double)nc;
  double R = (double)((a.layer0 == 0) ? (long long)a.NL * H * beta : a.pool[b]);
  long long bf = beta / (rho * rho);
  if (bf < 1) bf = 1;

  for (int l0 = 0; l0 < a.n; l0 += ALLOC_BATCH) {
    const int nb = min(ALLOC_BATCH, a.n - l0);
    // a head's demand is the sum of its counts (a record: M float masses of Eq. 6, M int32 counts of Eq. 9)
#pragma unroll 4
    for (int f = lane; f < nb * a.H; f += 64) {
      const int j = f / a.H, h = f - j * a.H;
      const int32_t* rec = reinterpret_cast<const int32_t*>(a.stats) + (((long long)(l0 + j) * a.B + b) * a.H + h) * 2 * M + M;
      int km = 0;
#pragma unroll
      for (int m = 0; m < MAXM; ++m) km += m < M ? rec[m] : 0;
      s_count[j][h] = km;
    }
    const double rem_l = (double)max(1, a.NL - (a.layer0 + l0 + lane));       // layers left, lane j: at layer l0 + j
    const double inv_lo = 1. / (rhod * Hd * rem_l), inv_hi = 1. / (Hd * rem_l);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int km = s_count[0][lane];
    for (int j = 0; j < nb; ++j) {
      const int li = l0 + j;
      const long long idx = ((long long)li * a.B + b) * a.H + lane;
      const double count = (double)km;
      km = s_count[min(j + 1, nb - 1)][lane];
      long long ah;
      if (!a.hcc_mode) {
        ah = beta;
      } else {
        const int rem = a.NL - (a.layer0 + li);
        const double remd = (double)rem, den_hi = Hd * remd, den_lo = rhod * den_hi;
        const double lo = fmax(div_floor(R + den_lo - 1., den_lo, lane_value(inv_lo, j)), 1.);
        const double hi = fmin(div_floor(rhod * R, den_hi, lane_value(inv_hi, j)), ncd);
        const double dem = !act ? 0. : count < lo ? lo : fmin(count, hi);
        double D;
        if (__any(dem >= 33554432.)) D = (double)lane_sum((long long)dem);       // (no prompt has so many candidates)
        else D = (double)(uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan_u32((uint32_t)dem), 63);
        double A = R;
        if (rem != 1) {
          const double amin = R - (remd - 1.) * Hd * ncd, amax = R - (remd - 1.) * Hd * (double)bf;
          A = D < amin ? amin : (D > amax ? amax : D);
        }
        if (a.hcc_mode == 2) {
          // Eq. 8 as printed: one budget per layer; the A mod H spare tokens go to the lowest heads
          const long long Al = (long long)A;
          ah = Al / H + (lane < Al % H ? 1 : 0);
        } else if (A == D) {
          ah = (long long)(int)dem;
        } else {
          // shares of the layer's total: scaled by demand when it has to shrink, by room when it has to grow
          const long long Al = (long long)A, Dl = (long long)D, deml = (long long)dem;
          const bool shrink = Al < Dl;
          const long long total = shrink ? Al : Al - Dl, part = shrink ? deml : (act ? nc - deml : 0), whole = shrink ? Dl : lane_sum(part);
          long long r;
          const long long base = div_rem(total * part, whole, r);
          const long long extra = total - lane_sum(act ? base : 0);
          ah = (shrink ? 0 : deml) + largest_remainder(base, act ? r : -1, extra, lane, a.H);
        }
        R -= A;
      }
      if (a.n == 1) { if (act) split_one(a, b, idx, ah); }  // (a call of one layer: no trip through memory, 2 us)
      else if (act) a.budgets[idx * M] = (int32_t)ah;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (lane == 0) a.pool[b] = (long long)R;
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

