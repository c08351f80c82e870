// Per-head modality statistics over the candidates [0, L-W) (paper Sec. 3.3):
//   Eq. 6  w_t, w_v   attention mass on text / image candidates
//   Eq. 9  k_t, k_v   fewest top-scored tokens of a modality that cover theta of its mass
// plus the max-pooled scores used for ranking, and the candidate counts per modality.
//
// One workgroup per (layer, batch, KV head).  Masses are summed in 64-bit fixed point
// (2^-44 units; a head's scores sum to G*W <= 256, so the total stays below 2^52): integer
// adds commute, so LDS atomics give the same bits on every run
// and the counts k_m, which are integers decided by a mass threshold, are reproducible.
// k_m is found without sorting by a radix descent (descent.h) on the float bit pattern: mass histograms down to the bin where the
// running mass crosses theta * w_m, over all scores at the first level, then over a list of the keys of that bin, until few are
// left that can be ranked one against the other.  With the threshold value tau
//   k_m = #{psi > tau} + ceil((theta w_m - mass{psi > tau}) / tau).
//
// Bound by latency and instruction issue: with one head per compute unit a launch is a chain of a pass over the scores, a
// walk over the bins, a second pass and the ranking.  Per head of 16K candidates, in us: clearing 0.7, masses and pooling 6.2,
// walk 2.1, list 4.0, for lists of more than RANK_MAX keys another walk 2 and list 1.1, ranking 1, record 0.6.  One launch over
// 128 heads of 16K: 23 -> 17.7 us against three levels over all scores, 32 heads of 8K 25 -> 12 (one head's scores were below
// the range of the first level), 112 of 32K 52 -> 28, 8 of 1K 13 -> 7.4.  A 64-register limit (two workgroups per compute unit)
// and nothing in scratch memory: the level-0 pass stands in front of the loop, the phases are kernels of their own.
#include "descent.h"

namespace madakv {

constexpr int STATS_THREADS = 1024;
constexpr int STATS_CHUNK = 16384;               // candidates per workgroup where a head's chunks have workgroups of their own
constexpr float FX_SCALE = 17592186044416.0f;    // 2^44
constexpr float PSI_MAX = 256.0f;                // G * W <= 256 bounds any column sum
constexpr int SPLIT_MAX_HEADS = 128;             // most heads of a launch whose chunks get workgroups of their own
constexpr uint32_t STATS_SH1 = 20;               // plain first digit: the sign bit is clear

// keys of the crossing bins: how many of a head's chunk (on average) fit the head's list in memory, and up to how many are
// ranked one against the other
constexpr int GLIST_PER_CHUNK = 1024, RANK_MAX = 128;

// Long heads on few heads (see launch_stats): what a head's chunks share, and what the first launch leaves to the second.
// All zero between calls but for the last line.
struct StatsMeet {
  uint32_t arrived[2], n[4], listed[4], above[4], pad[2];
  DescentRange range[4];
  unsigned long long sum_gt[4], w[4], target[4], wwin[4];
  uint32_t total[4], alive[4];
};

struct StatsArgs {
  const float* psi; const uint8_t* mask; float* psi_pool; void* stats; int32_t* n_mod;
  int B, H, L, W, nc, pool_r, pool_mode, share_mode, M;
  double theta;
  unsigned long long* xchg; long long xchg_per_head;   // the exchange words of the scoring kernels, to be emptied (Exchange)
  // Phase 0 = the whole head in one workgroup.  Long heads on few heads: a workgroup per chunk; 1 = its masses, added to the
  // head's in memory, which the last one to arrive walks; 2 = its keys of the crossing bins, added to the head's list, which
  // the last one to arrive ranks.
  char* split;                                   // a record of split_stride bytes per head (StatsSplit)
  long long split_stride;
};

// a head's record: [M][BINS] masses, StatsMeet, [M][gcap] list
struct StatsSplit { unsigned long long* sum; StatsMeet* meet; uint32_t* list; };
__host__ __device__ inline StatsSplit stats_split(char* p, int M) {
  StatsSplit x;
  x.sum = reinterpret_cast<unsigned long long*>(p);
  x.meet = reinterpret_cast<StatsMeet*>(x.sum + M * BINS);
  x.list = reinterpret_cast<uint32_t*>(x.meet + 1);
  return x;
}

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
// and stores cover whole cache lines.  The scores are read again (from L2) for the list, one group ahead.  What lies past the end is 0: it adds no mass, and
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
// 23.0 us for a head of 16K candidates, the instructions bound it).  WHOLE: all lanes of a wave make the same trips, some with
// groups past the end.
template <bool WHOLE = false, typename F>
__device__ __forceinline__ void for_groups(const float* psi, const uint8_t* mask, int i_first, int i_end, F f) {
  Group next = load_group(psi, mask, i_first, i_end);
#pragma unroll 1
  for (int i = i_first; (WHOLE ? __builtin_amdgcn_readfirstlane(i) : i) < i_end; i += 4 * STATS_THREADS) {
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
  float none = avg ? 0.f : -__builtin_inff();                // what a position outside [0, nc), or past R, contributes
  asm volatile("" : "+v"(none));                             // (made here: kept over the loop, twelve copies of it would spill)
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

// modalities the kernel is built for (2, or 4 for three and four), phase (StatsArgs), one that has to fit beside a gather
template <int MM, int PHASE, bool SMALL>
__global__ __launch_bounds__(STATS_THREADS) __attribute__((amdgpu_waves_per_eu(MM == 2 ? 8 : 4))) void stats_kernel(StatsArgs a) {
  constexpr int phase = PHASE, CAP = LIST_MAX<MM, SMALL>;
  const int M = MM == 2 ? 2 : a.M;
  extern __shared__ __attribute__((aligned(16))) unsigned char stats_smem[];
  unsigned long long* sum = reinterpret_cast<unsigned long long*>(stats_smem);      // [M][BINS] masses, [M][64] of the lowest bin
  unsigned long long* low = sum + (size_t)M * BINS;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(low + M * 64);                       // [M][LAST_BINS] counts (last level)
  uint32_t* list = cnt + M * LAST_BINS;                                            // [M][CAP] keys
  // a modality's few keys that are ranked: in the place of its masses
  unsigned long long* rank_gt = sum;                                                 // [M][RANK_MAX] mass of the larger ones
  uint32_t* rank_cnt = reinterpret_cast<uint32_t*>(rank_gt + (size_t)M * RANK_MAX);// [M][RANK_MAX] larger ones, equal ones << 16
  __shared__ DescentRange s_range[MM];
  __shared__ uint32_t s_cnt_gt[MM], s_n[MM], s_alive[MM], s_bincnt[MM], s_above[MM], s_tau[MM], s_listed[MM], s_glisted[MM], s_gabove[MM], s_flag;
  __shared__ uint32_t s_bin[MM];
  __shared__ unsigned long long s_sum_gt[MM], s_w[MM], s_target[MM], s_wwin[MM], s_next_sum[MM], s_next_target[MM], s_part[MM][8];

  const int tid0 = threadIdx.x;
  const int head = phase ? blockIdx.y : blockIdx.x;            // chunks: grid (chunks, heads)
  const int b = (head / a.H) % a.B;
  const float* psi = a.psi + (long long)head * a.L;
  const uint8_t* mask = a.mask + (long long)b * a.L;
  float* pool = a.psi_pool + (long long)head * a.nc;

  int i_begin = phase ? (int)blockIdx.x * STATS_CHUNK : 0;
  int i_end = phase ? min(a.nc, i_begin + STATS_CHUNK) : a.nc;
  const StatsSplit split = phase ? stats_split(a.split + head * a.split_stride, M) : StatsSplit{};
  StatsMeet* meet = split.meet;
  const bool want_n = a.n_mod && head < a.B * a.H && (head % a.H) == 0;

  if (tid0 < M) {
    if (phase == 2) {                             // what the walk over the masses left
      s_range[tid0] = meet->range[tid0]; s_n[tid0] = meet->total[tid0]; s_alive[tid0] = meet->alive[tid0];
      s_sum_gt[tid0] = meet->sum_gt[tid0]; s_w[tid0] = meet->w[tid0]; s_target[tid0] = meet->target[tid0]; s_wwin[tid0] = meet->wwin[tid0];
    } else {
      s_range[tid0] = descent_first(0u);
      s_n[tid0] = 0u; s_alive[tid0] = 1u; s_sum_gt[tid0] = 0ULL; s_w[tid0] = 0ULL; s_target[tid0] = 0ULL; s_wwin[tid0] = 0ULL;
    }
    s_cnt_gt[tid0] = 0u; s_bincnt[tid0] = 0u; s_tau[tid0] = 0u;
  }

  constexpr int WPM = STATS_THREADS / 64 / MM;                 // waves per modality
  const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6), m_of = wave / WPM, part = wave % WPM;
  const auto clear = [&](int tid) {
    uint4* z = reinterpret_cast<uint4*>(stats_smem);           // masses and counts lie next to each other
    for (int e = tid; e < M * (BINS * 8 + 64 * 8 + LAST_BINS * 4) / 16; e += STATS_THREADS) z[e] = make_uint4(0u, 0u, 0u, 0u);
  };

  if (phase != 2) {                                // level 0: the masses of all keys
    for (long long i = tid0 + (phase ? (int)blockIdx.x * STATS_THREADS : 0); i < a.xchg_per_head; i += (phase ? (int)gridDim.x : 1) * STATS_THREADS)
      a.xchg[head * a.xchg_per_head + i] = ~0ULL;
    const int tid = tid0, lane = tid & 63, i_first = i_begin + 4 * tid;
    clear(tid);
    __syncthreads();
    if (a.share_mode && tid < a.W && (phase == 0 || blockIdx.x == 0)) {
      // the other reading of Eq. 6: the proxy columns count towards the masses as well
      const int i = a.nc + tid;
      atomicAdd(&s_wwin[min((int)mask[i], M - 1)], to_fx(psi[i]));
    }
    {
      // every key is in range.  Those of the lowest bin, often most of a head's, have an address per lane (an atomic serialises
      // over the lanes that hit the same one)
      uint32_t found[MM];                          // candidates
#pragma unroll
      for (int m = 0; m < MM; ++m) found[m] = 0u;
      for_groups(psi, mask, i_first, i_end, [&](const Group& g, int i) {
        if (a.pool_r <= POOL_R_REG) pool_group(psi, pool, i, a.nc, a.pool_r, a.pool_mode != 0, g.x);   // pooled scores for ranking (raw values)
        else pool_group_wide(psi, pool, i, a.nc, a.pool_r, a.pool_mode != 0);
        const uint32_t ids = mask4_ids<MM>(g.mw, (uint32_t)(M - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = (int)id_of<MM>(ids, q);
          const int bin = descent_first_bin(nonneg_bits(g.x[q]), 0u);
          atomicAdd(&sum[bin > 0 ? m * BINS + bin : M * BINS + m * 64 + lane], to_fx(g.x[q]));
        }
        if (want_n) {
#pragma unroll
          for (int m = 0; m < MM; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) found[m] += (int)id_of<MM>(ids, q) == m && i + q < i_end ? 1u : 0u;
        }
      });
      if (want_n) {
#pragma unroll
        for (int m = 0; m < MM; ++m) {
          const uint32_t x = wave_incl_scan_u32(found[m]);
          if (lane == 63 && m < M && x) atomicAdd(&s_n[m], x);
        }
      }
    }
    __syncthreads();
    if (m_of < M && part == WPM - 1) {            // the lowest bin: its last lane will look at it
      const unsigned long long x = wave_incl_scan_u64(low[m_of * 64 + lane]);
      if (lane == 63) sum[m_of * BINS] = x;
    }
    if (phase == 1) {                              // add the chunk's bins to the head's; the last workgroup takes them all
      __syncthreads();
      unsigned long long* gsum = split.sum;
      for (int e = tid; e < M * BINS; e += STATS_THREADS)
        if (sum[e]) (void)__hip_atomic_fetch_add(&gsum[e], sum[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (tid < M && s_n[tid]) (void)__hip_atomic_fetch_add(&meet->n[tid], s_n[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (tid < M && blockIdx.x == 0) agent_store(&meet->wwin[tid], s_wwin[tid]);
      if (!arrive_last(&meet->arrived[0], gridDim.x, &s_flag)) return;
      for (int e = tid; e < M * BINS; e += STATS_THREADS) { sum[e] = agent_load(&gsum[e]); agent_store(&gsum[e], 0ULL); }
      if (tid < M) { s_n[tid] = agent_load(&meet->n[tid]); s_wwin[tid] = agent_load(&meet->wwin[tid]); agent_store(&meet->n[tid], 0u); }
      if (tid == 0) agent_store(&meet->arrived[0], 0u);
      __syncthreads();
    }
  }
  // the keys of the ranges: 0 = among the scores, 1 = in the list, 2 = in the head's list in memory
  int have = 0;
  const int gcap = (int)gridDim.x * GLIST_PER_CHUNK;
  uint32_t* glist = split.list;
  // (what is listed of a modality whose descent is over is nobody's business)
  const auto listed = [&](int m) { return s_alive[m] == 1u ? (int)s_listed[m] : 0; };
  const auto glisted = [&](int m) { return s_alive[m] == 1u ? (int)s_glisted[m] : 0; };
#pragma unroll 1
  for (int level = 0;; ++level) {
    // (addresses that depend on the thread are computed level by level: kept over the loop they would spill, and a
    // trip to scratch memory costs more than the whole walk)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    if (phase != 2 || level > 0) {
      // the walk from the top bin down, WPM waves per modality: lane 0 of the first of them has the top bins
      constexpr int PER = BINS / (WPM * 64);
      const int m = m_of;
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
      if (phase == 1) break;
      bool open = false;
      for (int m = 0; m < M; ++m) open = open || s_alive[m] == 1u;
      if (!open) break;
    }

    // ---- the next level
    int i_first = i_begin + 4 * tid;
    // The keys of the crossing bins, about a hundredth of all, go into a list: the descent goes on over that, or ends where they
    // are few enough to rank each of them against the others.  (One more pass over the scores instead of two.)
    if (have != 1) {
      if (tid < M) { s_listed[tid] = 0u; s_above[tid] = 0u; }
      __syncthreads();
    }
    DescentRange rg[MM];
    uint32_t found[MM];                          // keys above the range
#pragma unroll
    for (int m = 0; m < MM; ++m) { rg[m] = descent_uniform(s_range[min(m, M - 1)]); found[m] = 0u; }
    auto push = [&](int m, uint32_t key) {
      const uint32_t at = atomicAdd(&s_listed[m], 1u);
      if (at < (uint32_t)CAP) list[m * CAP + at] = key;
    };
    if (have == 0) {                             // from the scores (what lies past the end has the key 0)
      // (in the place of the masses, which have been walked)
      WaveBuf<unsigned long long> wb{reinterpret_cast<unsigned long long*>(stats_smem) + wave * WAVE_BUF, 0u};
      const auto take = [&](unsigned long long x) { push((int)(x >> 32), (uint32_t)x); };
      for_groups<true>(psi, mask, i_first, i_end, [&](const Group& g, int) {
        const uint32_t ids = mask4_ids<MM>(g.mw, (uint32_t)(M - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = (int)id_of<MM>(ids, q);
          const uint32_t key = nonneg_bits(g.x[q]);
          const uint32_t lo = MM == 2 ? (m ? rg[1].lo : rg[0].lo) : s_range[m].lo, hi = MM == 2 ? (m ? rg[1].hi : rg[0].hi) : s_range[m].hi;
          if (MM == 2) { const uint32_t gt = key > hi ? 1u : 0u; found[0] += gt; found[1] += m ? gt : 0u; }      // (all; of modality 1)
          else {
#pragma unroll
            for (int mm = 0; mm < MM; ++mm) found[mm] += m == mm && key > hi ? 1u : 0u;
          }
          wb.put(key - lo <= hi - lo, ((unsigned long long)m << 32) | key);
        }
        if (wb.n > 64u) wb.flush(lane, take);
      });
      wb.flush(lane, take);
      if (MM == 2) found[0] -= found[1];
    } else if (have == 2) {                      // from the head's list in memory
      for (int m = 0; m < M; ++m)
        for (int e = tid; e < glisted(m); e += STATS_THREADS) {
          const uint32_t key = agent_load(glist + m * gcap + e);
          if (key - s_range[m].lo <= s_range[m].hi - s_range[m].lo) push(m, key);
          else if (key > s_range[m].hi) atomicAdd(&s_above[m], 1u);
        }
      if (tid < M) atomicAdd(&s_above[tid], s_gabove[tid]);
    } else {                                     // from the list itself
      constexpr int PT = MM * CAP / STATS_THREADS;
      uint32_t key[PT];
      bool in[PT];
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const int e = tid + j * STATS_THREADS, m = e / CAP;
        in[j] = m < M && e % CAP < listed(min(m, M - 1));
        key[j] = in[j] ? list[e] : 0u;
      }
      __syncthreads();
      if (tid < M) s_listed[tid] = 0u;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const int m = min((tid + j * STATS_THREADS) / CAP, M - 1);
        if (in[j] && key[j] - s_range[m].lo <= s_range[m].hi - s_range[m].lo) push(m, key[j]);
        else if (in[j] && key[j] > s_range[m].hi) atomicAdd(&s_above[m], 1u);
      }
    }
    if (have == 0) {
#pragma unroll
      for (int m = 0; m < MM; ++m) {
        const uint32_t x = wave_incl_scan_u32(found[m]);
        if (lane == 63 && m < M && x) atomicAdd(&s_above[m], x);
      }
    }
    __syncthreads();
    if (phase == 2 && level == 0) {              // add the chunk's keys to the head's; the last workgroup goes on with them all
      __shared__ uint32_t s_base[MM];
      if (tid < M) {
        const uint32_t n = s_listed[tid];
        // (too many for the list: a number that says so, whatever the others add)
        s_base[tid] = n ? __hip_atomic_fetch_add(&meet->listed[tid], n <= (uint32_t)CAP ? n : 1u << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        if (s_above[tid]) (void)__hip_atomic_fetch_add(&meet->above[tid], s_above[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      for (int m = 0; m < M; ++m)
        for (int e = tid; e < min((int)s_listed[m], CAP); e += STATS_THREADS)
          if (s_base[m] + e < (uint32_t)gcap) agent_store(glist + m * gcap + s_base[m] + e, list[m * CAP + e]);
      if (!arrive_last(&meet->arrived[1], gridDim.x, &s_flag)) return;
      if (tid < M) {
        s_glisted[tid] = s_listed[tid] = agent_load(&meet->listed[tid]);
        s_gabove[tid] = s_above[tid] = agent_load(&meet->above[tid]);
        agent_store(&meet->listed[tid], 0u); agent_store(&meet->above[tid], 0u);
      }
      if (tid == 0) agent_store(&meet->arrived[1], 0u);
      __syncthreads();
      bool here = true, there = true;
      for (int m = 0; m < M; ++m) {
        here = here && (s_alive[m] != 1u || s_glisted[m] <= (uint32_t)CAP);
        there = there && (s_alive[m] != 1u || s_glisted[m] <= (uint32_t)gcap);
      }
      if (here)
        for (int m = 0; m < M; ++m)
          for (int e = tid; e < min((int)s_glisted[m], CAP); e += STATS_THREADS) list[m * CAP + e] = agent_load(glist + m * gcap + e);
      have = here ? 1 : there ? 2 : 0;
      __syncthreads();
      i_begin = 0; i_end = a.nc;                 // from here on the whole head is this workgroup's
      i_first = 4 * tid;
    } else if (have != 1) {
      bool here = true;
      for (int m = 0; m < M; ++m) here = here && (s_alive[m] != 1u || s_listed[m] <= (uint32_t)CAP);
      have = here ? 1 : have;
    }
    bool few = have == 1;
    for (int m = 0; m < M; ++m) few = few && (s_alive[m] != 1u || s_listed[m] <= (uint32_t)RANK_MAX);
    if (few) {
      for (int e = tid; e < M * RANK_MAX; e += STATS_THREADS) { rank_gt[e] = 0ULL; rank_cnt[e] = 0u; }
      __syncthreads();
      const bool mine = m_of < M && s_alive[min(m_of, M - 1)] == 1u;
      const int n = mine ? (int)s_listed[m_of] : 0;
      for (int i0 = 0; i0 < n; i0 += 64) {
        const uint32_t ki = list[m_of * CAP + min(i0 + lane, n - 1)];
        unsigned long long gt = 0ULL;
        uint32_t c = 0u;
        for (int j = part; j < n; j += WPM) {
          const uint32_t kj = list[m_of * CAP + j];
          gt += kj > ki ? to_fx(__uint_as_float(kj)) : 0ULL;
          c += kj > ki ? 1u : (kj == ki ? 65536u : 0u);
        }
        if (i0 + lane < n) { atomicAdd(&rank_gt[m_of * RANK_MAX + i0 + lane], gt); atomicAdd(&rank_cnt[m_of * RANK_MAX + i0 + lane], c); }
      }
      __syncthreads();
      if (mine && part * 64 + lane < n) {        // (RANK_MAX <= 64 * WPM)
        const int i = part * 64 + lane;
        const uint32_t key = list[m_of * CAP + i], c = rank_cnt[m_of * RANK_MAX + i];
        const unsigned long long before = s_sum_gt[m_of] + rank_gt[m_of * RANK_MAX + i], target = s_target[m_of];
        if (before < target && before + to_fx(__uint_as_float(key)) * (c >> 16) >= target) {      // (all that hold this key: the same values)
          s_tau[m_of] = key; s_bincnt[m_of] = c >> 16; s_cnt_gt[m_of] = s_above[m_of] + (c & 0xffffu);
          s_next_sum[m_of] = before;
        }
      }
      __syncthreads();
      if (tid < M && s_alive[tid] == 1u) { s_sum_gt[tid] = s_next_sum[tid]; s_alive[tid] = 2u; }
      __syncthreads();
      break;
    }

    clear(tid);
    __syncthreads();
    auto add = [&](int m, uint32_t key) {
      const DescentRange r = s_range[m];
      if (key - r.lo <= r.hi - r.lo) {
        const uint32_t bin = (key >> r.sh) - r.sub;
        atomicAdd(&sum[m * BINS + bin], to_fx(__uint_as_float(key)));
        if (r.sh == 0u) atomicAdd(&cnt[m * LAST_BINS + bin], 1u);
      }
    };
    if (have == 0) {
      for_groups(psi, mask, i_first, i_end, [&](const Group& g, int) {
        const uint32_t ids = mask4_ids<MM>(g.mw, (uint32_t)(M - 1));
        for (int q = 0; q < 4; ++q) add((int)id_of<MM>(ids, q), nonneg_bits(q & 2 ? (q & 1 ? g.x[3] : g.x[2]) : (q & 1 ? g.x[1] : g.x[0])));
      });
    } else {
      for (int m = 0; m < M; ++m)
        for (int e = tid; e < (have == 1 ? listed(m) : glisted(m)); e += STATS_THREADS) add(m, have == 1 ? list[m * CAP + e] : agent_load(glist + m * gcap + e));
    }
    __syncthreads();
  }
  if (phase == 1) {                               // hand over to the second launch
    if (tid0 < M) {
      meet->range[tid0] = s_range[tid0]; meet->total[tid0] = s_n[tid0]; meet->alive[tid0] = s_alive[tid0];
      meet->sum_gt[tid0] = s_sum_gt[tid0]; meet->w[tid0] = s_w[tid0]; meet->target[tid0] = s_target[tid0]; meet->wwin[tid0] = s_wwin[tid0];
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

// Chunks per head that go to workgroups of their own, or 0: heads of at least four 16384-candidate chunks, so few of them that
// one workgroup per head would leave most of the chip idle.  (Two launches for the statistics and three for the selection, the
// chunks of a head meeting at its record; 32 heads of 128K: 27 and 36 us, where a launch per pass and per walk, seven and nine
// of them, took 56 and 65.)
int split_chunks(const Dims& dm) {
  const int nchunks = (dm.nc + STATS_CHUNK - 1) / STATS_CHUNK;
  return (nchunks >= 4 && dm.heads <= SPLIT_MAX_HEADS) ? nchunks : 0;
}
// What the chunks of a head share, statistics and selection: a record per head at a place of its own, whichever layers a call is
// over.  Zero when it is handed over for the first time, and again after every launch (the lists and what a launch leaves to
// the next apart).
size_t stats_split_bytes(int M, int nchunks) {
  return (reinterpret_cast<size_t>(stats_split(nullptr, M).list + (size_t)M * nchunks * GLIST_PER_CHUNK) + 255) / 256 * 256;
}
size_t split_head_bytes(int M, int nchunks) { return (stats_split_bytes(M, nchunks) + select_split_bytes(M, nchunks) + 255) / 256 * 256; }

template <int MM, int PHASE, bool SMALL = false>
static hipError_t launch_stats_t(const StatsArgs& a, dim3 grid, hipStream_t st) {
  const size_t lds = (size_t)a.M * ((BINS + 64) * sizeof(unsigned long long) + LAST_BINS * sizeof(uint32_t) + LIST_MAX<MM, SMALL> * sizeof(uint32_t));
  if (lds > 48 * 1024) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&stats_kernel<MM, PHASE, SMALL>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((stats_kernel<MM, PHASE, SMALL>), grid, dim3(STATS_THREADS), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_stats(const Dims& dm, const madakv_config& c, const float* psi, const uint8_t* mask,
                        float* psi_pool, void* stats, int32_t* n_mod, const Exchange& x, hipStream_t st,
                        void* split_buf, size_t split_bytes, bool beside_gather) {
  StatsArgs a;
  a.psi = psi; a.mask = mask; a.psi_pool = psi_pool; a.stats = stats; a.n_mod = n_mod;
  a.B = dm.B; a.H = dm.H; a.L = dm.L; a.W = dm.W; a.nc = dm.nc; a.pool_r = (c.pool_k - 1) / 2;
  a.xchg = x.words; a.xchg_per_head = x.per_head;
  a.pool_mode = c.pool_mode; a.share_mode = c.share_mode; a.theta = (double)c.theta;
  a.M = c.n_modalities;
  a.split = nullptr; a.split_stride = 0;
  static_assert(STATS_THREADS / 64 * WAVE_BUF <= 2 * (BINS + 64 + LAST_BINS / 2), "the waves' buffers must fit the masses and counts");
  const int nchunks = split_chunks(dm);
  const dim3 whole(dm.heads), chunks(nchunks, dm.heads);
  if (nchunks && split_buf && split_bytes >= dm.heads * split_head_bytes(a.M, nchunks)) {
    a.split = static_cast<char*>(split_buf);
    a.split_stride = (long long)split_head_bytes(a.M, nchunks);
    hipError_t e = a.M == 2 ? launch_stats_t<2, 1>(a, chunks, st) : launch_stats_t<4, 1>(a, chunks, st);
    if (e == hipSuccess) e = a.M == 2 ? launch_stats_t<2, 2>(a, chunks, st) : launch_stats_t<4, 2>(a, chunks, st);
    return e;
  }
  if (beside_gather && a.nc <= SMALL_HEADS && a.M == 2) return launch_stats_t<2, 0, true>(a, whole, st);
  return a.M == 2 ? launch_stats_t<2, 0>(a, whole, st) : launch_stats_t<4, 0>(a, whole, st);
}

}  // namespace madakv
