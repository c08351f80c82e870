// Per-head modality statistics over the candidates [0, L-W) (paper Sec. 3.3):
//   Eq. 6  w_t, w_v   attention mass on text / image candidates
//   Eq. 9  k_t, k_v   fewest top-scored tokens of a modality that cover theta of its mass
// plus the max-pooled scores used for ranking, and the candidate counts per modality.
//
// One workgroup per (layer, batch, KV head).  Masses are summed in 64-bit fixed point
// (2^-44 units; a head's scores sum to G*W <= 256, so the total stays below 2^52): integer
// adds commute, so LDS atomics give the same bits on every run
// and the counts k_m, which are integers decided by a mass threshold, are reproducible.
// k_m is found without sorting by a radix descent (descent.h) on the float bit pattern over mass
// histograms to the bin where the running mass crosses theta * w_m; the last level pins the threshold value tau exactly, and
//   k_m = #{psi > tau} + ceil((theta w_m - mass{psi > tau}) / tau).
// Counts are only taken at the last level (the keys above its range, and a count histogram of its bins).
//
// Bound by latency and instruction issue: with one head per compute unit a launch is a chain of a pass over the scores,
// a walk, two more passes and walks, and the instructions are cold at every launch.  Eight unrolled variants of the pooling
// and 32 elements per thread had made 72 KB of code, more than the instruction cache; this is 13 KB, the scores are read
// again at every level.  One launch over 128 heads: 25.7 -> 14.0 us for 1K candidates, 27.1 -> 17.6 for 8K, 28.3 -> 21.7 for
// 16K.  512 threads: 12.7, 18.5, 25.0; values kept in registers or addresses kept over the levels: spills, 26 to 90 us.
#include "descent.h"

namespace madakv {

constexpr int STATS_THREADS = 1024;
constexpr int STATS_CHUNK = 16384;               // candidates per workgroup where a head's chunks have workgroups of their own
constexpr float FX_SCALE = 17592186044416.0f;    // 2^44
constexpr float PSI_MAX = 256.0f;                // G * W <= 256 bounds any column sum
constexpr int SPLIT_MAX_HEADS = 128;             // most heads of a launch whose chunks get workgroups of their own
constexpr uint32_t STATS_SH1 = 20;               // plain first digit: the sign bit is clear

// what the walk of one level hands to the next, per head and modality (phases 1 and 2)
struct StatsCarry {
  DescentRange range;
  unsigned long long sum_gt, w, target, wwin;
  uint32_t n, alive, pad[2];
};

struct StatsArgs {
  const float* psi; const uint8_t* mask; float* psi_pool; void* stats; int32_t* n_mod;
  int B, H, L, W, nc, pool_r, pool_mode, share_mode, M;
  double theta;
  // Long heads on few heads (see launch_stats): the chunks of a head go to workgroups of their own.
  // phase 0 = the whole head in one workgroup, all levels; 1 = histogram of one chunk at `level`, added
  // to the head's histogram in memory; 2 = the walk over that histogram (one workgroup per head).
  int phase, level, heads;
  unsigned long long* gsum;                      // [3 levels][heads][M][BINS]
  uint32_t* gcnt;                                // the same shape; level 0: [0] = candidates; level 2: [bin] = count, [GCNT_ABOVE] = keys above the range
  StatsCarry* carry;                             // [heads][4]
};
constexpr int GCNT_ABOVE = LAST_BINS;

// Fixed point, rounded to nearest even: adding 2^52 leaves the integer in the low bits of a double (v * 2^44 <= 2^52).
__device__ __forceinline__ unsigned long long to_fx(float v) {
  v = __builtin_amdgcn_fmed3f(v, 0.f, PSI_MAX);    // (NaN: 0)
  const double d = fma((double)v, (double)FX_SCALE, 4503599627370496.0);
  return (unsigned long long)__double_as_longlong(d) - 0x4330000000000000ULL;
}
__device__ __forceinline__ uint32_t nonneg_bits(float v) {
  v = __builtin_amdgcn_fmed3f(v, 0.f, PSI_MAX);
  return __float_as_uint(v);                      // non-negative floats order like their bit patterns
}

// Thread t takes the groups of four consecutive candidates number t, t + STATS_THREADS, ..., so that a wave's loads
// and stores cover whole cache lines.  The scores are read again (from L2) at every level, one group ahead: kept in
// registers, their unrolled code is what filled the instruction cache.  What lies past the end is 0: it adds no mass, and
// no key is above it.
struct Group { f32x4_any_t x; uint32_t mw; };
__device__ __forceinline__ Group load_group(const float* psi, const uint8_t* mask, int i, int nc) {
  Group g;
  g.x = f32x4_any_t{0.f, 0.f, 0.f, 0.f};
  g.mw = 0u;
  if (i + 4 <= nc) {
    g.x = *reinterpret_cast<const f32x4_any_t*>(psi + i);
    g.mw = load_mask4(mask + i);
  } else {
#pragma unroll
    for (int q = 0; q < 3; ++q) if (i + q < nc) { g.x[q] = psi[i + q]; g.mw |= (uint32_t)mask[i + q] << (8 * q); }
  }
  return g;
}

// f(group, its first candidate) for this thread's groups, the next one on its way (two ahead gains nothing: 23.3 against
// 23.0 us for a head of 16K candidates, the instructions bound it)
template <typename F>
__device__ __forceinline__ void for_groups(const float* psi, const uint8_t* mask, int i_first, int i_end, F f) {
  Group next = load_group(psi, mask, i_first, i_end);
#pragma unroll 1
  for (int i = i_first; i < i_end; i += 4 * STATS_THREADS) {
    const Group g = next;
    next = load_group(psi, mask, i + 4 * STATS_THREADS, i_end);
    f(g, i);
  }
}

// Pooling of half-width R <= POOL_R_REG over the candidates [0, nc): positions outside do not take part.  A group's
// neighbours are in the vectors before and after it (in the caches: the lanes next to this one load them anyway).
constexpr int POOL_R_REG = 3;
__device__ __forceinline__ void pool_group(const float* psi, float* pool, int i, int nc, int R, bool avg, const f32x4_any_t& x) {
  if (R == POOL_R_REG && !avg && __all(i > 0 && i + 8 <= nc)) {          // the usual window, away from the ends
    const f32x4_any_t y = *reinterpret_cast<const f32x4_any_t*>(psi + i - 4), z = *reinterpret_cast<const f32x4_any_t*>(psi + i + 4);
    const float c = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));            // in all four windows
    const float l3 = y[3], l23 = fmaxf(y[2], l3), r0 = z[0], r01 = fmaxf(r0, z[1]);
    *reinterpret_cast<f32x4_any_t*>(pool + i) = f32x4_any_t{fmaxf(fmaxf(y[1], l23), c), fmaxf(fmaxf(l23, r0), c), fmaxf(fmaxf(l3, r01), c), fmaxf(fmaxf(r01, z[2]), c)};
    return;
  }
  const float none = avg ? 0.f : -__builtin_inff();          // what a position outside [0, nc), or past R, contributes
  float ext[12];
#pragma unroll
  for (int q = 0; q < 4; ++q) { ext[q] = none; ext[8 + q] = none; ext[4 + q] = i + q < nc ? x[q] : none; }
  if (R > 0) {
    if (i > 0) {
      const f32x4_any_t y = *reinterpret_cast<const f32x4_any_t*>(psi + i - 4);
#pragma unroll
      for (int q = 1; q < 4; ++q) ext[q] = y[q];
    }
    if (i + 8 <= nc) {
      const f32x4_any_t y = *reinterpret_cast<const f32x4_any_t*>(psi + i + 4);
#pragma unroll
      for (int q = 0; q < 3; ++q) ext[8 + q] = y[q];
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) if (i + 4 + q < nc) ext[8 + q] = psi[i + 4 + q];
    }
  }
  float o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = ext[4 + q];
  if (avg) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float sm = 0.f;                                          // left to right over the clipped neighbourhood
#pragma unroll
      for (int r = -POOL_R_REG; r <= POOL_R_REG; ++r) sm += abs(r) <= R ? ext[4 + q + r] : 0.f;
      o[q] = sm / (float)(min(i + q + R, nc - 1) - max(i + q - R, 0) + 1);
    }
  } else {
#pragma unroll
    for (int r = 1; r <= POOL_R_REG; ++r)
      if (r <= R) {
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = fmaxf(o[q], fmaxf(ext[4 + q - r], ext[4 + q + r]));
      }
  }
  if (i + 4 <= nc) {
    *reinterpret_cast<f32x4_any_t*>(pool + i) = f32x4_any_t{o[0], o[1], o[2], o[3]};
  } else {
#pragma unroll
    for (int q = 0; q < 3; ++q) if (i + q < nc) pool[i + q] = o[q];
  }
}
__device__ __forceinline__ void pool_group_wide(const float* psi, float* pool, int i0, int nc, int R, bool avg) {
#pragma unroll 1
  for (int i = i0; i < min(i0 + 4, nc); ++i) {
    const int lo = max(i - R, 0), hi = min(i + R, nc - 1);
    float acc = avg ? 0.f : psi[i];
#pragma unroll 1
    for (int j = lo; j <= hi; ++j) acc = avg ? acc + psi[j] : fmaxf(acc, psi[j]);
    pool[i] = avg ? acc / (float)(hi - lo + 1) : acc;
  }
}

template <int MM>   // modalities the kernel is built for (2 or 4)
__global__ __launch_bounds__(STATS_THREADS) __attribute__((amdgpu_waves_per_eu(MM == 2 ? 8 : 4))) void stats_kernel(StatsArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char stats_smem[];
  unsigned long long* sum = reinterpret_cast<unsigned long long*>(stats_smem);      // [M][BINS] masses
  uint32_t* cnt = reinterpret_cast<uint32_t*>(sum + (size_t)a.M * BINS);             // [M][LAST_BINS] counts (last level)
  __shared__ DescentRange s_range[MM];
  __shared__ uint32_t s_cnt_gt[MM], s_n[MM], s_alive[MM], s_bincnt[MM], s_above[MM], s_tau[MM];
  __shared__ uint32_t s_bin[MM];
  __shared__ unsigned long long s_sum_gt[MM], s_w[MM], s_target[MM], s_wwin[MM], s_next_sum[MM], s_next_target[MM], s_part[MM][8];
  const int M = a.M;

  const int tid0 = threadIdx.x;
  const int phase = a.phase;
  const int head = phase == 1 ? blockIdx.y : blockIdx.x;      // phase 1: grid (chunks, heads)
  const int b = (head / a.H) % a.B;
  const float* psi = a.psi + (long long)head * a.L;
  const uint8_t* mask = a.mask + (long long)b * a.L;
  float* pool = a.psi_pool + (long long)head * a.nc;

  const int i_end = phase == 2 ? 0 : (phase == 1 ? min(a.nc, ((int)blockIdx.x + 1) * STATS_CHUNK) : a.nc);
  const size_t hist_words = (size_t)M * BINS;
  unsigned long long* gsum = phase ? a.gsum + ((size_t)a.level * a.heads + head) * hist_words : nullptr;
  uint32_t* gcnt = phase ? a.gcnt + ((size_t)a.level * a.heads + head) * hist_words : nullptr;
  StatsCarry* carry = phase ? a.carry + (size_t)head * 4 : nullptr;
  const bool want_n = a.n_mod && head < a.B * a.H && (head % a.H) == 0;

  if (tid0 < M) {
    if (phase != 0 && a.level > 0) {             // what the walk of the level above left
      const StatsCarry cy = carry[tid0];
      s_range[tid0] = cy.range; s_n[tid0] = cy.n; s_alive[tid0] = cy.alive;
      s_sum_gt[tid0] = cy.sum_gt; s_w[tid0] = cy.w; s_target[tid0] = cy.target; s_wwin[tid0] = cy.wwin;
    } else {
      s_range[tid0] = phase ? descent_plain<STATS_SH1>() : descent_first(0u);
      s_n[tid0] = 0u; s_alive[tid0] = 1u; s_sum_gt[tid0] = 0ULL; s_w[tid0] = 0ULL; s_target[tid0] = 0ULL; s_wwin[tid0] = 0ULL;
    }
    s_cnt_gt[tid0] = 0u; s_bincnt[tid0] = 0u; s_tau[tid0] = 0u;
  }

  for (int level = phase ? a.level : 0;; ++level) {
    // (addresses that depend on the thread are computed level by level: kept over the loop they would spill, and a
    // trip to scratch memory costs more than the whole walk)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i_first = (phase == 1 ? (int)blockIdx.x * STATS_CHUNK : 0) + 4 * tid;
    {
      uint4* z = reinterpret_cast<uint4*>(stats_smem);                       // masses and counts lie next to each other
      const int nz = M * (BINS * 8 + LAST_BINS * 4) / 16;
      for (int e = tid; e < nz; e += STATS_THREADS) z[e] = make_uint4(0u, 0u, 0u, 0u);
      if (tid < M) s_above[tid] = 0u;
    }
    __syncthreads();
    if (level == 0 && a.share_mode && tid < a.W && phase != 1) {
      // the other reading of Eq. 6: the proxy columns count towards the masses as well
      const int i = a.nc + tid;
      atomicAdd(&s_wwin[min((int)mask[i], M - 1)], to_fx(psi[i]));
    }
    DescentRange rg[MM];
    uint32_t thr[MM];                              // last level: keys above its range are counted (else none is)
    bool last = false;
#pragma unroll
    for (int m = 0; m < MM; ++m) {
      rg[m] = descent_uniform(s_range[min(m, M - 1)]);
      const bool lm = rg[m].sh == 0 && __builtin_amdgcn_readfirstlane((int)s_alive[min(m, M - 1)]) == 1;
      thr[m] = lm ? rg[m].hi : 0xffffffffu;
      last = last || lm;
    }
    if (phase == 2) {                              // the head's histogram of this level, gathered by the chunks' workgroups
      for (int e = tid; e < M * BINS; e += STATS_THREADS) sum[e] = gsum[e];
      if (last) {
        for (int e = tid; e < M * LAST_BINS; e += STATS_THREADS) cnt[e] = gcnt[(e / LAST_BINS) * BINS + e % LAST_BINS];
        if (tid < M) s_above[tid] = gcnt[tid * BINS + GCNT_ABOVE];
      }
      if (level == 0 && tid < M) s_n[tid] = gcnt[tid * BINS];
    }
    uint32_t found[MM];                            // level 0: candidates; last level: keys above the range
#pragma unroll
    for (int m = 0; m < MM; ++m) found[m] = 0u;
    if (level == 0) {
      // every key is in range
      const uint32_t sh0 = rg[0].sh, sub0 = rg[0].sub;
      for_groups(psi, mask, i_first, i_end, [&](const Group& g, int i) {
        if (a.pool_r <= POOL_R_REG) pool_group(psi, pool, i, a.nc, a.pool_r, a.pool_mode != 0, g.x);   // pooled scores for ranking (raw values)
        else pool_group_wide(psi, pool, i, a.nc, a.pool_r, a.pool_mode != 0);
        const uint32_t ids = mask4_ids<MM>(g.mw, (uint32_t)(M - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = (int)id_of<MM>(ids, q);
          atomicAdd(&sum[m * BINS + descent_bin({0u, 0u, sh0, sub0}, nonneg_bits(g.x[q]))], to_fx(g.x[q]));
        }
        if (want_n) {
#pragma unroll
          for (int m = 0; m < MM; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) found[m] += (int)id_of<MM>(ids, q) == m && i + q < i_end ? 1u : 0u;
        }
      });
    } else {
      const uint32_t span0 = rg[0].hi - rg[0].lo, span1 = rg[1].hi - rg[1].lo;
      for_groups(psi, mask, i_first, i_end, [&](const Group& g, int) {
        const uint32_t ids = mask4_ids<MM>(g.mw, (uint32_t)(M - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = (int)id_of<MM>(ids, q);
          const uint32_t key = nonneg_bits(g.x[q]);
          // (the per-modality state is picked with selects where there are two: indexing a register array by m would spill it)
          const uint32_t lo = MM == 2 ? (m ? rg[1].lo : rg[0].lo) : s_range[m].lo, sp = MM == 2 ? (m ? span1 : span0) : s_range[m].hi - lo;
          if (key - lo <= sp) {
            const uint32_t s1 = MM == 2 ? (m ? rg[1].sh : rg[0].sh) : s_range[m].sh;
            const uint32_t bin = (key >> s1) - (MM == 2 ? (m ? rg[1].sub : rg[0].sub) : s_range[m].sub);
            atomicAdd(&sum[m * BINS + bin], to_fx(g.x[q]));
            if (s1 == 0u) atomicAdd(&cnt[m * LAST_BINS + bin], 1u);
          }
        }
        if (last) {
#pragma unroll
          for (int m = 0; m < MM; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) found[m] += (int)id_of<MM>(ids, q) == m && nonneg_bits(g.x[q]) > thr[m] ? 1u : 0u;
        }
      });
    }
    if (last || (level == 0 && want_n)) {
#pragma unroll
      for (int m = 0; m < MM; ++m) {
        const uint32_t x = wave_incl_scan_u32(found[m]);
        if (lane == 63 && m < M && x) atomicAdd(last ? &s_above[m] : &s_n[m], x);
      }
    }
    __syncthreads();
    if (phase == 1) {                              // add the chunk's bins to the head's and leave
      for (int e = tid; e < M * BINS; e += STATS_THREADS)
        if (sum[e]) atomicAdd(&gsum[e], sum[e]);
      if (last) {
        for (int e = tid; e < M * LAST_BINS; e += STATS_THREADS)
          if (cnt[e]) atomicAdd(&gcnt[(e / LAST_BINS) * BINS + e % LAST_BINS], cnt[e]);
        if (tid < M && s_above[tid]) atomicAdd(&gcnt[tid * BINS + GCNT_ABOVE], s_above[tid]);
      }
      if (level == 0 && tid < M && s_n[tid]) atomicAdd(&gcnt[tid * BINS], s_n[tid]);
      return;
    }
    // the walk from the top bin down, WPM waves per modality: lane 0 of the first of them has the top bins
    constexpr int WPM = STATS_THREADS / 64 / MM, PER = BINS / (WPM * 64);
    const int m = wave / WPM, part = wave % WPM;
    const bool walks = m < M && s_alive[min(m, M - 1)] == 1u;
    unsigned long long share = 0ULL, incl = 0ULL;
    const int top = BINS - 1 - (part * 64 + lane) * PER;      // bins top, top - 1, ..., top - PER + 1
    if (walks) {
#pragma unroll
      for (int j = 0; j < PER; ++j) share += sum[m * BINS + top - j];
      incl = wave_incl_scan_u64(share);
      if (lane == 63) s_part[m][part] = incl;
    }
    __syncthreads();
    if (walks) {
      const DescentRange r = s_range[m];
      unsigned long long wtot = 0ULL, base = s_sum_gt[m];
#pragma unroll
      for (int w = 0; w < WPM; ++w) { const unsigned long long x = s_part[m][w]; wtot += x; base += w < part ? x : 0ULL; }
      unsigned long long target = s_target[m];
      if (level == 0) {
        // smallest integer >= theta * w: the running mass c reaches theta*w iff c >= it
        const unsigned long long tg = (unsigned long long)ceil(a.theta * (double)wtot);
        target = tg < wtot ? tg : wtot;
        if (part == 0 && lane == 0) {
          s_w[m] = wtot; s_next_target[m] = target;
          if (wtot == 0ULL) s_alive[m] = 3u;       // no mass at all: k = 0
        }
      }
      unsigned long long before = base + incl - share;
      if (before < target && before + share >= target) {      // one lane of one wave: the bin is among its own
        uint32_t bin = (uint32_t)top;
#pragma unroll 1
        for (;;) {
          const unsigned long long x = sum[m * BINS + bin];
          if (before + x >= target) break;
          before += x; --bin;
        }
        s_next_sum[m] = before; s_bin[m] = bin;
        if (r.sh == 0) {
          s_tau[m] = r.sub + bin; s_bincnt[m] = cnt[m * LAST_BINS + bin];
        }
      }
    }
    __syncthreads();
    if (walks && part == 0) {                      // the next level's state (everybody has read this one's)
      const DescentRange r = s_range[m];
      const uint32_t bin = s_bin[m];
      uint32_t c = 0u;
      if (r.sh == 0) {                             // keys above the threshold's bin: those above the range and those in the bins above it
        for (int x = (int)bin + 1 + lane; x < LAST_BINS; x += 64) c += cnt[m * LAST_BINS + x];
        c = wave_incl_scan_u32(c);
      }
      if (lane == 63) {
        if (level == 0) s_target[m] = s_next_target[m];
        if (s_alive[m] == 3u) { s_alive[m] = 0u; s_range[m] = descent_none(); }
        else {
          s_sum_gt[m] = s_next_sum[m];
          if (r.sh == 0) { s_cnt_gt[m] = s_above[m] + c; s_alive[m] = 2u; s_range[m] = descent_none(); }
          else s_range[m] = descent_next<STATS_SH1>(r, bin);
        }
      }
    }
    __syncthreads();
    if (phase == 2) break;
    bool open = false;
    for (int m = 0; m < M; ++m) open = open || s_alive[m] == 1u;
    if (!open) break;
  }
  if (phase == 2 && a.level < 2) {               // hand over to the next level
    if (tid0 < M) {
      StatsCarry cy;
      cy.range = s_range[tid0]; cy.n = s_n[tid0]; cy.alive = s_alive[tid0];
      cy.sum_gt = s_sum_gt[tid0]; cy.w = s_w[tid0]; cy.target = s_target[tid0]; cy.wwin = s_wwin[tid0];
      cy.pad[0] = cy.pad[1] = 0u;
      carry[tid0] = cy;
    }
    return;
  }
  if (tid0 < M) {
    const int m = tid0;
    int32_t k = 0;
    if (s_alive[m] == 2u) {
      // s_tau is the full bit pattern of tau; every element in the last bin equals tau
      const unsigned long long q = to_fx(__uint_as_float(s_tau[m]));
      const unsigned long long need = s_target[m] - s_sum_gt[m];
      unsigned long long t = q ? (need + q - 1ULL) / q : 1ULL;
      if (t < 1ULL) t = 1ULL;
      if (t > (unsigned long long)s_bincnt[m]) t = s_bincnt[m];
      k = (int32_t)(s_cnt_gt[m] + (uint32_t)t);
    }
    const float w = (float)((double)(s_w[m] + s_wwin[m]) * (1.0 / (double)FX_SCALE));
    // a head's record: M float masses, then M int32 counts (two modalities: madakv_head_stats)
    float* rec = reinterpret_cast<float*>(a.stats) + (long long)head * 2 * M;
    rec[m] = w;
    reinterpret_cast<int32_t*>(rec)[M + m] = k;
    if (want_n) a.n_mod[b * M + m] = (int32_t)s_n[m];
  }
}

__global__ __launch_bounds__(256) void split_zero_kernel(uint32_t* p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

void launch_split_zero(uint32_t* p, long long words, hipStream_t st) {
  hipLaunchKernelGGL(split_zero_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, p, words);
}

// Chunks per head that go to workgroups of their own, or 0: heads of at least four 16384-candidate chunks
// (with two, the 16 small launches cost what the parallelism gains: measured on 28 heads of 32K candidates),
// so few of them that one workgroup per head would leave most of the chip idle.
int split_chunks(const Dims& dm) {
  const int nchunks = (dm.nc + STATS_CHUNK - 1) / STATS_CHUNK;
  return (nchunks >= 4 && dm.heads <= SPLIT_MAX_HEADS) ? nchunks : 0;
}
size_t split_buffer_bytes(int heads, int M, int nchunks) {
  const size_t hist = (size_t)3 * heads * M * BINS;
  return hist * (sizeof(unsigned long long) + sizeof(uint32_t)) + (size_t)heads * 4 * sizeof(StatsCarry) + (size_t)heads * nchunks * 16 + 256;
}

hipError_t launch_stats(const Dims& dm, const madakv_config& c, const float* psi, const uint8_t* mask,
                        float* psi_pool, void* stats, int32_t* n_mod, int layer0, hipStream_t st,
                        void* split_buf, size_t split_bytes) {
  StatsArgs a;
  a.psi = psi; a.mask = mask; a.psi_pool = psi_pool; a.stats = stats; a.n_mod = n_mod;
  a.B = dm.B; a.H = dm.H; a.L = dm.L; a.W = dm.W; a.nc = dm.nc; a.pool_r = (c.pool_k - 1) / 2;
  (void)layer0;
  a.pool_mode = c.pool_mode; a.share_mode = c.share_mode; a.theta = (double)c.theta;
  a.M = c.n_modalities;
  a.phase = 0; a.level = 0; a.heads = dm.heads; a.gsum = nullptr; a.gcnt = nullptr; a.carry = nullptr;
  const size_t lds = (size_t)a.M * (BINS * sizeof(unsigned long long) + LAST_BINS * sizeof(uint32_t));
  if (a.M == 2) {
    if (lds > 48 * 1024)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&stats_kernel<2>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  } else {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&stats_kernel<4>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  }
  const int nchunks = split_chunks(dm);
  if (nchunks && split_buf && split_bytes >= split_buffer_bytes(dm.heads, a.M, nchunks)) {
    // per level: the chunks' workgroups add their histograms into the head's (in memory), then one workgroup per
    // head walks it; the kernel boundary is the synchronisation
    const size_t hist = (size_t)3 * dm.heads * a.M * BINS;
    a.gsum = reinterpret_cast<unsigned long long*>(split_buf);
    a.gcnt = reinterpret_cast<uint32_t*>(a.gsum + hist);
    a.carry = reinterpret_cast<StatsCarry*>(a.gcnt + hist);
    const long long zw = (long long)(hist * 3);                // 32-bit words of the two histogram arrays
    launch_split_zero(reinterpret_cast<uint32_t*>(split_buf), zw, st);
    for (int level = 0; level < 3; ++level) {
      a.level = level;
      for (int phase = 1; phase <= 2; ++phase) {
        a.phase = phase;
        const dim3 grid = phase == 1 ? dim3(nchunks, dm.heads) : dim3(dm.heads);
        if (a.M == 2) hipLaunchKernelGGL((stats_kernel<2>), grid, dim3(STATS_THREADS), lds, st, a);
        else hipLaunchKernelGGL((stats_kernel<4>), grid, dim3(STATS_THREADS), lds, st, a);
      }
    }
    return hipGetLastError();
  }
  if (a.M == 2) hipLaunchKernelGGL((stats_kernel<2>), dim3(dm.heads), dim3(STATS_THREADS), lds, st, a);
  else hipLaunchKernelGGL((stats_kernel<4>), dim3(dm.heads), dim3(STATS_THREADS), lds, st, a);
  return hipGetLastError();
}

}  // namespace madakv
