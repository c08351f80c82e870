// Eviction (paper Sec. 3.3, modality-specific eviction per attention head): for each head
// keep, per modality, the b_m candidates with the largest pooled score; equal scores go to
// the lower position.  Output: kept positions in ascending order, then the W window
// positions, written into the head's segment of the ragged index array.
//
// offsets_kernel   lays the segments out: batch item b owns a fixed region of the reduced
//                  cache, inside it layers and heads follow each other; a segment has
//                  kv_len = b_t + b_v + W rows plus max_new_tokens free rows.  It also fills
//                  a table "first head that overlaps each 64-row block" for the gather.
// select_kernel    one workgroup per head.  A radix descent (descent.h) over count histograms of the order-preserving keys, over
//                  all candidates at the first level, then over a list of those of the crossing bin, until few are left that are
//                  ranked by key and position: the last one that is kept gives, per modality, the threshold key tau_m and the
//                  position up to which candidates of that key are kept.  The last pass writes what is above, 16384 candidates
//                  at a time; prefix sums over the workgroup give the output slots, so the result is ascending by
//                  construction.  (Where more candidates share a bin than a list holds, and do so to the last bit, the number
//                  of them that is still needed is handed out by rank, 4096 candidates at a time.)
//                  Bound like the statistics (stats.hip) by latency and instruction issue.  Per head of 16K candidates, in us:
//                  clearing 0.7, counts 3.5, walk 1.8, list 3.6, ranking 1, last pass 4.2.  One launch, against three levels
//                  over all candidates and a last pass 4096 at a time: 128 heads of 16K 21.8 -> 15.0 us, 112 of 32K 37 (the
//                  slowest 67) -> 25 (30), 32 of 8K 14.1 -> 11.2, 8 of 1K 10.1 -> 8.3.
#include "allocate.h"
#include "descent.h"

namespace madakv {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_CHUNK = 16384;                 // candidates per workgroup where a head's chunks have workgroups of their own
constexpr uint32_t SEL_SH1 = 21;                 // plain first digit of a 32-bit key

// candidates of the crossing bins: how many of a head's chunk (on average) fit the head's list in memory, and up to how many
// are ranked one against the other
constexpr int SEL_GLIST_PER_CHUNK = 1024, SEL_RANK_MAX = 256;
constexpr int SEL_MAX_CHUNKS = 64;               // 2^20 candidates

// Long heads on few heads (see launch_select): what a head's chunks share, and what a launch leaves to the next.  All zero
// between calls but for the last line.
struct SelMeet {
  uint32_t arrived[2], listed[4], pad[2];
  DescentRange range[4];
  uint32_t need[4], alive[4], tau[4], pos[4], done, pad2[3];
};

struct OffsetsArgs {
  const int32_t* budgets; int64_t* kv_off; int32_t* kv_len; int32_t* len1; long long* cursor; int32_t* blk2head; long long* call_range; int32_t* layer_maxlen;
  int n, B, H, L, W, layer0, max_new, keep_all, blocks_per_batch, M;
  long long region_tokens;       // rows of one batch item's region
  long long init_limit;          // rows of it the segments laid out here may fill
  int page_rows, tbl_entries;    // paged cache: segments are whole pages, no free rows reserved per head
  int32_t* page_tbl; unsigned long long* pool_top;
};

// One workgroup per batch item; thread f of a trip owns head f of the call's (layer, head)
// sequence.  Offsets are a prefix sum over that sequence (wave shuffles + one LDS hop).
// The workgroup is kept small (one wave per SIMD, few registers): it has to find room on a compute
// unit while the score sweeps or a gather of another layer group fill the chip, and a 1024-thread
// workgroup would wait there until that kernel's grid has drained.
constexpr int OFF_THREADS = 256;
constexpr int OFF_MAX_LAYERS = 1024;

// ALLOC: the first wave does the batch item's budget allocation first (madakv_evict: one launch less).
template <bool ALLOC>
__global__ __launch_bounds__(OFF_THREADS) void offsets_kernel(OffsetsArgs a, AllocArgs al) {
  __shared__ long long s_wtot[OFF_THREADS / 64];
  __shared__ long long s_used;
  __shared__ int s_first_bad;
  __shared__ int s_lmax[OFF_MAX_LAYERS];
  __shared__ int2 s_blk[OFF_THREADS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  const int nh = a.n * a.H;
  const long long start = (a.layer0 == 0) ? 0 : a.cursor[b];
  const long long region = (long long)b * a.region_tokens;
  const long long blk_base = start / GATHER_ROWS;            // the block table is relative to the call's first block
  for (int li = tid; li < a.n; li += OFF_THREADS) s_lmax[li] = 0;
  if (ALLOC) {                                                // (totals and budgets go through memory to the threads that read them)
    if (wave == 0) allocate_wave(al, b, lane);
    __syncthreads();
    split_totals(al, b, tid, OFF_THREADS);
  }
  if (tid == 0) { s_first_bad = 0x7fffffff; s_used = 0; }
  if (tid == 0 && a.page_rows && a.layer0 == 0) a.pool_top[b] = 0ULL;   // a new pass: every page taken for appended rows is free again
  __syncthreads();
  long long carry = 0;                                        // rows laid out by earlier trips
  bool overflowed = false;                                    // a head did not fit: every later head is empty
  for (int f0 = 0; f0 < nh; f0 += OFF_THREADS) {
    const int f = f0 + tid;
    const bool act = f < nh;
    const int li = act ? f / a.H : 0, h = act ? f % a.H : 0;
    const long long idx = ((long long)li * a.B + b) * a.H + h;
    long long len = 0;
    if (act) {
      len = a.keep_all ? a.L : a.W;
      if (!a.keep_all) for (int m = 0; m < a.M; ++m) len += a.budgets[idx * a.M + m];
    }
    long long seg = act ? len + a.max_new : 0;
    if (a.page_rows) seg = act ? (len + a.page_rows - 1) / a.page_rows * a.page_rows : 0;
    long long incl = seg;
    for (int o = 1; o < 64; o <<= 1) {
      long long t = shfl_i64(incl, max(lane - o, 0));
      if (lane >= o) incl += t;
    }
    if (lane == 63) s_wtot[wave] = incl;
    __syncthreads();
    long long before = 0, tot = 0;
    for (int w = 0; w < OFF_THREADS / 64; ++w) { const long long t = s_wtot[w]; if (w < wave) before += t; tot += t; }
    const long long abs_incl = carry + before + incl;         // rows up to and including this head's segment
    // Budgets that do not add up to the configured total could run past the batch item's
    // region: the first head that does not fit, and every head after it, gets an empty
    // segment (kv_len 0) at the end of what was laid out, so nothing is written outside.
    const bool bad = act && (overflowed || start + abs_incl > a.init_limit);
    if (bad && !overflowed) atomicMin(&s_first_bad, f);
    __syncthreads();
    const int first_bad = s_first_bad;
    if (!overflowed && first_bad == f) s_used = abs_incl - seg;
    __syncthreads();
    const bool now_over = first_bad != 0x7fffffff;
    const long long used = s_used;
    long long off;
    if (bad) { len = 0; seg = 0; off = start + used; }
    else off = start + abs_incl - seg;                        // relative to the region start
    if (act) {
      atomicMax(&s_lmax[li], (int)len);                       // longest segment of the layer, for the decode grid
      a.kv_off[idx] = region + off;
      a.kv_len[idx] = (int32_t)len;
      a.len1[idx] = (int32_t)len + 1;
      if (a.page_rows) a.page_tbl[(((long long)(a.layer0 + li) * a.B + b) * a.H + h) * a.tbl_entries] = (int32_t)(seg / a.page_rows);
      // blocks whose first row lies inside this segment, relative to the table
      const long long b0 = (off + GATHER_ROWS - 1) / GATHER_ROWS, b1 = seg > 0 ? (off + seg - 1) / GATHER_ROWS : b0 - 1;
      s_blk[tid] = make_int2((int)max(0LL, b0 - blk_base), (int)min((long long)a.blocks_per_batch - 1, b1 - blk_base));
      if (f == 0 && (start % GATHER_ROWS) != 0 && 0 < a.blocks_per_batch)
        a.blk2head[(long long)b * a.blocks_per_batch] = 0;    // the call starts inside a block: its first head is head 0
    }
    carry = now_over ? used : carry + tot;
    overflowed = now_over;
    __syncthreads();
    // the table, a wave per head (a thread per head took 6 us where 32 heads of 4K rows had 64 to 128 blocks each)
    for (int g = wave; g < min(OFF_THREADS, nh - f0); g += OFF_THREADS / 64)
      for (int t = s_blk[g].x + lane; t <= s_blk[g].y; t += 64) a.blk2head[(long long)b * a.blocks_per_batch + t] = f0 + g;
    __syncthreads();
  }
  for (int li = tid; li < a.n; li += OFF_THREADS) a.layer_maxlen[(long long)li * a.B + b] = s_lmax[li];
  if (tid == 0) {
    a.cursor[b] = start + carry;
    a.call_range[b * 2] = start;
    a.call_range[b * 2 + 1] = start + carry;
  }
}

struct SelectArgs {
  const float* psi_pool; const uint8_t* mask; const int32_t* budgets; const int64_t* kv_off; const int32_t* kv_len; int32_t* kept_idx;
  int B, H, L, W, nc, mpa_mode, keep_all, select_mode, sink_tokens, M;
  const int32_t* seg_len; const uint8_t* rowmod;   // ragged candidates (re-eviction), else null
  // Phase 0 = the whole head in one workgroup.  Long heads on few heads: a workgroup per chunk; 1 = its counts, added to the
  // head's in memory, which the last one to arrive walks; 2 = its candidates of the crossing bins, added to the head's list,
  // which the last one to arrive ranks; 3 = its kept positions written behind those of the chunks before it.
  char* split;                    // a record of split_stride bytes per head (SelSplit)
  long long split_stride;
};

// a head's record: [M][BINS] counts, SelMeet, [nchunks] kept for sure and then kept by the chunks before, [M][gcap] list
struct SelSplit { uint32_t* cnt; SelMeet* meet; uint32_t* chunk_kept; unsigned long long* list; };
__host__ __device__ inline SelSplit select_split(char* p, int M, int nchunks) {
  SelSplit x;
  x.cnt = reinterpret_cast<uint32_t*>(p);
  x.meet = reinterpret_cast<SelMeet*>(x.cnt + M * BINS);
  x.chunk_kept = reinterpret_cast<uint32_t*>(x.meet + 1);
  x.list = reinterpret_cast<unsigned long long*>(x.chunk_kept + (nchunks + 1) / 2 * 2);
  return x;
}

// the next group of four candidates of a thread: keys, and the bytes of their modality ids (0 where the mask is not used)
struct KeyGroup { f32x4_any_t x; uint32_t mw; };
__device__ __forceinline__ KeyGroup load_keys(const float* sc, const uint8_t* mask, int i, int nc, int use_mask) {
  KeyGroup g;
  g.x = f32x4_any_t{0.f, 0.f, 0.f, 0.f};
  g.mw = 0u;
  if (i + 4 <= nc) {
    g.x = *reinterpret_cast<const f32x4_any_t*>(sc + i);
    if (use_mask) g.mw = load_mask4(mask + i);
  } else {
#pragma unroll
    for (int q = 0; q < 3; ++q) if (i + q < nc) { g.x[q] = sc[i + q]; if (use_mask) g.mw |= (uint32_t)mask[i + q] << (8 * q); }
  }
  return g;
}

// Writes the kept positions of [i_begin, i_end): key > tau, or key == tau up to position last (-1: none), in ascending order from
// out[run] on; returns the end.  16384 candidates and one barrier per trip: a thread has four groups of four, 4096 apart, whose
// counts it scans together (16 bits hold the count of a group column: 4096).
template <int MM>
__device__ __forceinline__ uint32_t write_kept(const float* sc, const uint8_t* mask, int use_mask, int32_t* out, int i_begin, int i_end, uint32_t top,
                                               const uint32_t* s_tau, const uint32_t* s_pos, uint32_t run, uint32_t (*s_tot)[3][SEL_THREADS / 64]) {
  constexpr int NWAVES = SEL_THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t tau0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tau[0]), tau1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tau[1]);
  const int pos0 = __builtin_amdgcn_readfirstlane((int)s_pos[0]), pos1 = __builtin_amdgcn_readfirstlane((int)s_pos[1]);
  int buf = 0;
#pragma unroll 1
  for (int base = i_begin; base < i_end; base += 16 * SEL_THREADS, buf ^= 1) {
    KeyGroup g[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) g[j] = load_keys(sc, mask, base + 4 * (tid + j * SEL_THREADS), i_end, use_mask);
    uint32_t bits = 0u, pk[2] = {0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t ids = mask4_ids<MM>(g[j].mw, top);
      uint32_t kb = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = (int)id_of<MM>(ids, q), i = base + 4 * (tid + j * SEL_THREADS) + q;
        const uint32_t key = float_key(g[j].x[q]), t = MM == 2 ? (m ? tau1 : tau0) : s_tau[m];
        const int p = MM == 2 ? (m ? pos1 : pos0) : (int)s_pos[m];
        // (what lies past the end is not kept, whatever tau is)
        kb |= i < i_end && (key > t || (key == t && i <= p)) ? 1u << q : 0u;
      }
      bits |= kb << (4 * j);
      pk[j >> 1] += (uint32_t)__popc(kb) << (16 * (j & 1));
    }
    uint32_t ex[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      ex[f] = wave_incl_scan_u32(pk[f]);
      if (lane == 63) s_tot[buf][f][wave] = ex[f];
      ex[f] -= pk[f];
    }
    __syncthreads();                               // (two buffers: a wave that is a trip ahead writes the other one)
    uint32_t tot[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const uint32_t w = wave_incl_scan_u32(lane < NWAVES ? s_tot[buf][f][lane] : 0u);
      tot[f] = (uint32_t)__builtin_amdgcn_readlane((int)w, NWAVES - 1);
      ex[f] += wave ? (uint32_t)__builtin_amdgcn_readlane((int)w, wave - 1) : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t pos = run + ((ex[j >> 1] >> (16 * (j & 1))) & 0xffffu);
      const int i = base + 4 * (tid + j * SEL_THREADS);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if ((bits >> (4 * j + q)) & 1u) out[pos++] = i + q;
      run += (tot[j >> 1] >> (16 * (j & 1))) & 0xffffu;
    }
  }
  return run;
}

// LDS in front of the list: the counts, in whose place the waves' buffers and the ranks are when they have been walked
__host__ __device__ constexpr int select_front(int M, bool small) {
  const int counts = 4 * M * (BINS + 64), bufs = SEL_THREADS / 64 * (small ? WAVE_BUF_SMALL : WAVE_BUF) * 8;
  return counts > bufs ? counts : bufs;
}

// f(candidate's group, its first candidate) for this thread's groups of [i_first, i_end), the next one on its way.  WHOLE: all
// lanes of a wave make the same trips, some with groups past the end.
template <bool WHOLE = false, typename F>
__device__ __forceinline__ void for_key_groups(const float* sc, const uint8_t* mask, int i_first, int i_end, int use_mask, F f) {
  KeyGroup next = load_keys(sc, mask, i_first, i_end, use_mask);
#pragma unroll 1
  for (int i = i_first; (WHOLE ? __builtin_amdgcn_readfirstlane(i) : i) < i_end; i += 4 * SEL_THREADS) {
    const KeyGroup g = next;
    next = load_keys(sc, mask, i + 4 * SEL_THREADS, i_end, use_mask);
    f(g, i);
  }
}

// modalities the kernel is built for (2, or 4 for three and four), phase (SelectArgs), one that has to fit beside a gather
template <int MM, int PHASE, bool SMALL>
__global__ __launch_bounds__(SEL_THREADS) __attribute__((amdgpu_waves_per_eu(MM == 2 ? 8 : 4))) void select_kernel(SelectArgs a) {
  constexpr int NWAVES = SEL_THREADS / 64, WPM = NWAVES / MM;   // waves per modality
  constexpr int phase = PHASE, CAP = LIST_MAX<MM, SMALL>;
  extern __shared__ __attribute__((aligned(16))) unsigned char select_smem[];
  const int M = MM == 2 ? 2 : a.M;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(select_smem);                          // [M][BINS] counts, [M][64] of the lowest bin
  uint32_t* low = cnt + M * BINS;
  unsigned long long* list = reinterpret_cast<unsigned long long*>(select_smem + select_front(M, SMALL));   // [M][CAP] key, ~position
  uint32_t* rank = cnt;                                                              // [M][SEL_RANK_MAX] larger ones (in the place of the counts)
  __shared__ DescentRange s_range[MM];
  __shared__ uint32_t s_need[MM], s_alive[MM], s_tau[MM], s_pos[MM], s_before[MM], s_bin[MM], s_part[MM][NWAVES], s_listed[MM], s_glisted[MM], s_sure, s_flag;
  __shared__ uint32_t s_tot[2][3][NWAVES], s_chunk[SEL_MAX_CHUNKS];
  const int tid0 = threadIdx.x;
  const int head = phase ? blockIdx.y : blockIdx.x;            // chunks: grid (chunks, heads)
  const int b = (head / a.H) % a.B;
  // candidates of this head: the L - W prompt positions before the window with the batch item's modality
  // mask, or (ragged: the rows of a reduced cache, re-eviction) the rows before the head's last W with a
  // modality byte per row; scores and output are indexed the same way
  const bool ragged = a.seg_len != nullptr;
  const int nc = ragged ? a.seg_len[head] - a.W : a.nc;
  const float* sc = ragged ? a.psi_pool + a.kv_off[head] : a.psi_pool + (long long)head * a.nc;
  const uint8_t* mask = ragged ? a.rowmod + a.kv_off[head] : a.mask + (long long)b * a.L;
  int32_t* out = a.kept_idx + a.kv_off[head];

  if (a.kv_len[head] == 0) return;               // the segment did not fit the region: nothing to write
  if (phase == 0 && a.keep_all) {
    for (int i = tid0; i < a.L; i += SEL_THREADS) out[i] = i;
    return;
  }
  if (phase == 0 && a.select_mode == 1) {
    // score-free baseline: the first `sink` candidates and the most recent ones, then the window
    uint32_t btot = 0;
    for (int m = 0; m < M; ++m) btot += (uint32_t)a.budgets[(long long)head * M + m];
    const int total = min((int)btot, nc);
    const int sink = min(a.sink_tokens, total);
    for (int j = tid0; j < total + a.W; j += SEL_THREADS)
      out[j] = j < sink ? j : (j < total ? nc - (total - j) : nc + (j - total));
    return;
  }
  int i_begin = phase ? (int)blockIdx.x * SEL_CHUNK : 0;
  int i_end = phase ? min(nc, i_begin + SEL_CHUNK) : nc;
  const uint32_t top = (uint32_t)(M - 1);
  const SelSplit split = phase ? select_split(a.split + head * a.split_stride, M, gridDim.x) : SelSplit{};
  SelMeet* meet = split.meet;
  uint32_t* chunk_kept = split.chunk_kept;
  if (phase == 3 && meet->done) return;           // (written by the second launch)
  if (tid0 < MM) {
    if (phase >= 2 && tid0 < M) {                  // what the launches before left
      s_range[tid0] = meet->range[tid0]; s_need[tid0] = meet->need[tid0]; s_alive[tid0] = meet->alive[tid0]; s_tau[tid0] = meet->tau[tid0];
      s_pos[tid0] = meet->pos[tid0];
    } else {
      s_range[tid0] = descent_first(1u);
      s_need[tid0] = tid0 < M ? (uint32_t)a.budgets[(long long)head * M + tid0] : 0u;
      s_alive[tid0] = tid0 < M ? 1u : 0u; s_tau[tid0] = 0xffffffffu; s_pos[tid0] = 0xffffffffu;
    }
  }
  if constexpr (PHASE == 3) {
    __syncthreads();
    const uint32_t end = write_kept<MM>(sc, mask, a.mpa_mode, out, i_begin, i_end, top, s_tau, s_pos, chunk_kept[blockIdx.x], &s_tot[0]);
    if (i_end != nc) return;                       // the window positions follow the last chunk's
    for (int r = tid0; r < a.W; r += SEL_THREADS) out[end + r] = nc + r;
  } else {
  const int wave0 = __builtin_amdgcn_readfirstlane(tid0 >> 6), m_of = wave0 / WPM, part = wave0 % WPM;
  const auto clear = [&](int tid) {
    for (int e = tid; e < M * (BINS + 64) / 4; e += SEL_THREADS) reinterpret_cast<uint4*>(cnt)[e] = make_uint4(0u, 0u, 0u, 0u);
  };
  if (phase != 2) {                                // level 0: the counts of all keys; those of the lowest bin have an address per lane
    const int tid = tid0, lane = tid & 63;
    clear(tid);
    __syncthreads();
    for_key_groups(sc, mask, i_begin + 4 * tid, i_end, a.mpa_mode, [&](const KeyGroup& g, int i) {
      const uint32_t ids = mask4_ids<MM>(g.mw, top);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = (int)id_of<MM>(ids, q), bin = descent_first_bin(float_key(g.x[q]), 1u);
        if (i + q < i_end) atomicAdd(&cnt[bin > 0 ? m * BINS + bin : M * BINS + m * 64 + lane], 1u);
      }
    });
    __syncthreads();
    if (m_of < M && part == WPM - 1) {             // (the lane that gets the lowest bin looks at it)
      const uint32_t x = wave_incl_scan_u32(low[m_of * 64 + lane]);
      if (lane == 63) cnt[m_of * BINS] = x;
    }
    if (phase == 1) {                              // add the chunk's bins to the head's; the last workgroup takes them all
      __syncthreads();
      uint32_t* gcnt = split.cnt;
      for (int e = tid; e < M * BINS; e += SEL_THREADS) {
        const uint32_t x = cnt[e];
        if (x) (void)__hip_atomic_fetch_add(&gcnt[e], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (!arrive_last(&meet->arrived[0], gridDim.x, &s_flag)) return;
      for (int e = tid; e < M * BINS; e += SEL_THREADS) { cnt[e] = agent_load(&gcnt[e]); agent_store(&gcnt[e], 0u); }
      if (tid == 0) agent_store(&meet->arrived[0], 0u);
      __syncthreads();
    }
  }

  bool alone = phase == 0;                         // this workgroup writes all of the head's positions
  bool ranked = false;                             // tau and the last position that is kept with it are known from a list
  int have = 0;                                    // the keys of the ranges: 0 = among the scores, 1 = in the list, 2 = in the head's list in memory
  const int gcap = (int)gridDim.x * SEL_GLIST_PER_CHUNK;
  unsigned long long* glist = split.list;
  // (what is listed of a modality whose descent is over is nobody's business)
  const auto listed = [&](int m) { return s_alive[m] == 1u ? (int)s_listed[m] : 0; };
  const auto glisted = [&](int m) { return s_alive[m] == 1u ? (int)s_glisted[m] : 0; };
#pragma unroll 1
  for (int level = 0;; ++level) {
    // (addresses that depend on the thread are computed level by level: kept over the loop they would spill)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    if (phase != 2 || level > 0) {
      // the walk from the top bin down, WPM waves per modality: lane 0 of the first of them has the top bins
      constexpr int PER = BINS / (WPM * 64);
      const int m = m_of;
      const bool walks = m < M && s_alive[min(m, M - 1)] == 1u;
      const int tb = BINS - 1 - (part * 64 + lane) * PER;     // bins tb, tb - 1, ..., tb - PER + 1
      uint32_t share = 0u, incl = 0u;
      if (walks) {
#pragma unroll
        for (int j = 0; j < PER; ++j) share += cnt[m * BINS + tb - j];
        incl = wave_incl_scan_u32(share);
        if (lane == 63) s_part[m][part] = incl;
      }
      __syncthreads();
      uint32_t need = 0u;
      if (walks) {
        uint32_t total = 0u, before = incl - share;
#pragma unroll
        for (int w = 0; w < WPM; ++w) { const uint32_t x = s_part[m][w]; total += x; before += w < part ? x : 0u; }
        need = min(s_need[m], total);              // (first level: a budget above the candidate count keeps them all)
        if (before < need && before + share >= need) {        // one lane of one wave: the bin is among its own
          uint32_t bin = (uint32_t)tb;
#pragma unroll 1
          for (;;) {
            const uint32_t x = cnt[m * BINS + bin];
            if (before + x >= need) break;
            before += x; --bin;
          }
          s_before[m] = before; s_bin[m] = bin;
        }
      }
      __syncthreads();
      if (walks && part == 0 && lane == 0) {       // the next level's state (everybody has read this one's)
        if (need == 0u) { s_alive[m] = 0u; s_need[m] = 0u; s_range[m] = descent_none(); }     // nothing to keep: tau stays above every key
        else {
          const DescentRange r = s_range[m];
          s_need[m] = need - s_before[m];          // still needed from inside this bin
          if (r.sh == 0) { s_tau[m] = r.sub + s_bin[m]; s_alive[m] = 2u; s_range[m] = descent_none(); }
          else s_range[m] = descent_next<SEL_SH1>(r, s_bin[m]);
        }
      }
      __syncthreads();
      if (phase == 1) break;
      bool open = false, walked = false;
      for (int mm = 0; mm < M; ++mm) { open = open || s_alive[mm] == 1u; walked = walked || s_alive[mm] == 2u; }
      if (!open) { ranked = !walked; break; }      // (nothing to keep of any modality: as good as ranked)
    }

    // ---- the next level: the candidates of the crossing bins, about a hundredth of all, go into a list; the descent goes on over
    // that, or ends where they are few enough to rank each of them against the others
    if (have != 1) {
      if (tid < MM) s_listed[tid] = 0u;
      if (tid == 0) s_sure = 0u;
      __syncthreads();
    }
    auto push = [&](int m, unsigned long long x) {
      const uint32_t at = atomicAdd(&s_listed[m], 1u);
      if (at < (uint32_t)CAP) list[m * CAP + at] = x;
    };
    auto within = [&](int m, uint32_t key) { return key - s_range[m].lo <= s_range[m].hi - s_range[m].lo; };
    if (have == 0) {                               // from the scores
      // (in the place of the counts, which have been walked)
      WaveBuf<unsigned long long> wb{reinterpret_cast<unsigned long long*>(select_smem) + wave0 * (SMALL ? WAVE_BUF_SMALL : WAVE_BUF), 0u};
      const auto take = [&](unsigned long long x) {
        const uint32_t m = ((uint32_t)x >> 30) ^ 3u;
        push((int)m, x ^ (m << 30));
      };
      DescentRange rg[MM];
      uint32_t hi[MM], sure = 0u;                  // keys above hi are kept for sure (chunks)
#pragma unroll
      for (int m = 0; m < MM; ++m) {
        rg[m] = descent_uniform(s_range[min(m, M - 1)]);
        hi[m] = __builtin_amdgcn_readfirstlane((int)s_alive[min(m, M - 1)]) == 1 ? rg[m].hi : 0xffffffffu;
      }
      for_key_groups<true>(sc, mask, i_begin + 4 * tid, i_end, a.mpa_mode, [&](const KeyGroup& g, int i) {
        const uint32_t ids = mask4_ids<MM>(g.mw, top);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = (int)id_of<MM>(ids, q);
          const uint32_t key = float_key(g.x[q]);
          const uint32_t lo = MM == 2 ? (m ? rg[1].lo : rg[0].lo) : s_range[m].lo, sp = (MM == 2 ? (m ? rg[1].hi : rg[0].hi) : s_range[m].hi) - lo;
          // (a position takes 20 bits: two of the others say the modality)
          wb.put(i + q < i_end && key - lo <= sp, ((unsigned long long)key << 32) | (~(uint32_t)(i + q) ^ ((uint32_t)m << 30)));
          if (phase == 2) sure += i + q < i_end && key > pick(hi, m) ? 1u : 0u;
          if (SMALL && wb.n > 64u) wb.flush(lane, take);
        }
        if (!SMALL && wb.n > 64u) wb.flush(lane, take);
      });
      wb.flush(lane, take);
      if (phase == 2) {
        const uint32_t x = wave_incl_scan_u32(sure);
        if (lane == 63 && x) atomicAdd(&s_sure, x);
      }
    } else if (have == 2) {                        // from the head's list in memory
      for (int m = 0; m < M; ++m)
        for (int e = tid; e < glisted(m); e += SEL_THREADS) {
          const unsigned long long x = agent_load(glist + m * gcap + e);
          if (within(m, (uint32_t)(x >> 32))) push(m, x);
        }
    } else {                                       // from the list itself
      constexpr int PT = MM * CAP / SEL_THREADS;
      unsigned long long x[PT];
      bool in[PT];
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const int e = tid + j * SEL_THREADS, m = e / CAP;
        in[j] = m < M && e % CAP < listed(min(m, M - 1));
        x[j] = in[j] ? list[e] : 0ULL;
      }
      __syncthreads();
      if (tid < M) s_listed[tid] = 0u;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const int m = min((tid + j * SEL_THREADS) / CAP, M - 1);
        if (in[j] && within(m, (uint32_t)(x[j] >> 32))) push(m, x[j]);
      }
    }
    __syncthreads();
    if (phase == 2 && level == 0) {                // add the chunk's candidates to the head's; the last workgroup goes on with them all
      __shared__ uint32_t s_base[MM];
      if (tid < M) {
        const uint32_t n = s_listed[tid];
        // (too many for the list: a number that says so, whatever the others add)
        s_base[tid] = n ? __hip_atomic_fetch_add(&meet->listed[tid], n <= (uint32_t)CAP ? n : 1u << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      }
      if (tid == 0) agent_store(&chunk_kept[blockIdx.x], s_sure);
      __syncthreads();
      for (int m = 0; m < M; ++m)
        for (int e = tid; e < min((int)s_listed[m], CAP); e += SEL_THREADS)
          if (s_base[m] + e < (uint32_t)gcap) agent_store(glist + m * gcap + s_base[m] + e, list[m * CAP + e]);
      if (!arrive_last(&meet->arrived[1], gridDim.x, &s_flag)) return;
      if (tid < M) { s_glisted[tid] = s_listed[tid] = agent_load(&meet->listed[tid]); agent_store(&meet->listed[tid], 0u); }
      if (tid == 0) agent_store(&meet->arrived[1], 0u);
      for (int c = tid; c < (int)gridDim.x; c += SEL_THREADS) s_chunk[c] = agent_load(&chunk_kept[c]);
      __syncthreads();
      bool here = true, there = true;
      for (int m = 0; m < M; ++m) {
        here = here && (s_alive[m] != 1u || s_glisted[m] <= (uint32_t)CAP);
        there = there && (s_alive[m] != 1u || s_glisted[m] <= (uint32_t)gcap);
      }
      alone = !there;
      if (here)
        for (int m = 0; m < M; ++m)
          for (int e = tid; e < min((int)s_glisted[m], CAP); e += SEL_THREADS) list[m * CAP + e] = agent_load(glist + m * gcap + e);
      have = here ? 1 : there ? 2 : 0;
      __syncthreads();
      i_begin = 0; i_end = nc;                     // from here on the whole head is this workgroup's
    } else if (have != 1) {
      bool here = true;
      for (int m = 0; m < M; ++m) here = here && (s_alive[m] != 1u || s_listed[m] <= (uint32_t)CAP);
      have = here ? 1 : have;
    }
    bool few = have == 1;
    for (int m = 0; m < M; ++m) few = few && s_alive[m] != 2u && (s_alive[m] != 1u || s_listed[m] <= (uint32_t)SEL_RANK_MAX);
    if (few) {
      for (int e = tid; e < M * SEL_RANK_MAX; e += SEL_THREADS) rank[e] = 0u;
      __syncthreads();
      const bool mine = m_of < M && s_alive[min(m_of, M - 1)] == 1u;
      const int n = mine ? (int)s_listed[m_of] : 0;
      for (int i0 = 0; i0 < n; i0 += 64) {
        const unsigned long long x = list[m_of * CAP + min(i0 + lane, n - 1)];
        uint32_t above = 0u;
#pragma unroll 4
        for (int j = part; j < n; j += WPM) above += list[m_of * CAP + j] > x ? 1u : 0u;
        if (i0 + lane < n) atomicAdd(&rank[m_of * SEL_RANK_MAX + i0 + lane], above);
      }
      __syncthreads();
      if (mine) {
        const uint32_t need = s_need[m_of];
        for (int i = part * 64 + lane; i < n; i += WPM * 64) {
          const uint32_t above = rank[m_of * SEL_RANK_MAX + i];
          const unsigned long long x = list[m_of * CAP + i];
          if (above + 1u == need) { s_tau[m_of] = (uint32_t)(x >> 32); s_pos[m_of] = ~(uint32_t)x; }
        }
      }
      __syncthreads();
      ranked = true;
      break;
    }
    clear(tid);
    __syncthreads();
    auto add = [&](int m, uint32_t key) {
      const DescentRange r = s_range[m];
      if (key - r.lo <= r.hi - r.lo) atomicAdd(&cnt[m * BINS + (key >> r.sh) - r.sub], 1u);
    };
    if (have == 0) {
      for_key_groups(sc, mask, i_begin + 4 * tid, i_end, a.mpa_mode, [&](const KeyGroup& g, int i) {
        const uint32_t ids = mask4_ids<MM>(g.mw, top);
        for (int q = 0; q < 4; ++q)
          if (i + q < i_end) add((int)id_of<MM>(ids, q), float_key(q & 2 ? (q & 1 ? g.x[3] : g.x[2]) : (q & 1 ? g.x[1] : g.x[0])));
      });
    } else {
      for (int m = 0; m < M; ++m)
        for (int e = tid; e < (have == 1 ? listed(m) : glisted(m)); e += SEL_THREADS)
          add(m, (uint32_t)((have == 1 ? list[m * CAP + e] : agent_load(glist + m * gcap + e)) >> 32));
    }
    __syncthreads();
  }
  if (phase == 1 || (phase == 2 && ranked && !alone)) {        // hand over to the next launch
    if (tid0 < M) {
      meet->range[tid0] = s_range[tid0]; meet->need[tid0] = s_need[tid0]; meet->alive[tid0] = s_alive[tid0]; meet->tau[tid0] = s_tau[tid0];
      meet->pos[tid0] = s_pos[tid0];
    }
    if (tid0 == 0) meet->done = 0u;
    if (phase == 2) {
      // where the chunks begin: the sure ones of the chunks before, and what the head's list has of them.  (The list in memory
      // holds all candidates of the first crossing bins, those of a range that was narrowed since among them.)
      for (int m = 0; m < M; ++m)
        if (s_alive[m] == 1u)
          for (int e = tid0; e < (int)s_glisted[m]; e += SEL_THREADS) {
            const unsigned long long x = agent_load(glist + m * gcap + e);
            const uint32_t key = (uint32_t)(x >> 32), pos = ~(uint32_t)x;
            if (key > s_tau[m] || (key == s_tau[m] && (int)pos <= (int)s_pos[m])) atomicAdd(&s_chunk[pos / SEL_CHUNK], 1u);
          }
      __syncthreads();
      if (tid0 < 64) {                             // exclusive prefix over the chunks
        const uint32_t x = tid0 < (int)gridDim.x ? s_chunk[tid0] : 0u, incl = wave_incl_scan_u32(x);
        if (tid0 < (int)gridDim.x) chunk_kept[tid0] = incl - x;
      }
    }
    return;
  }
  if constexpr (PHASE != 1) {
  if (phase == 2 && tid0 == 0) meet->done = 1u;
  if (ranked) {
    const uint32_t end = write_kept<MM>(sc, mask, a.mpa_mode, out, 0, nc, top, s_tau, s_pos, 0u, &s_tot[0]);
    for (int r = tid0; r < a.W; r += SEL_THREADS) out[end + r] = nc + r;
    return;
  }

  // Many candidates share a threshold's bin: take every key > tau_m and the first ties_m keys == tau_m, 4096 candidates at a time.
  const int lane = tid0 & 63, wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  uint32_t tau[MM], ties[MM], run_eq[MM];
#pragma unroll
  for (int m = 0; m < MM; ++m) {
    tau[m] = m < M ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tau[m]) : 0xffffffffu;
    ties[m] = m < M ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_need[m]) : 0u;
    run_eq[m] = 0u;
  }
  uint32_t run_gt = 0u;
  constexpr int NF = MM == 2 ? 2 : 3;              // words of packed counts: {gt, eq0}, {eq1, eq2}, {eq3, -}
  KeyGroup next = load_keys(sc, mask, i_begin + 4 * tid0, i_end, a.mpa_mode);
  int buf = 0;
#pragma unroll 1
  for (int base = i_begin; base < i_end; base += 4 * SEL_THREADS, buf ^= 1) {
    const int i = base + 4 * tid0;
    const KeyGroup g = next;
    next = load_keys(sc, mask, i + 4 * SEL_THREADS, i_end, a.mpa_mode);
    const uint32_t ids = mask4_ids<MM>(g.mw, top);
    uint32_t gtbits = 0u, eqbits = 0u, pk[3] = {0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = (int)id_of<MM>(ids, q);
      const uint32_t key = float_key(g.x[q]), t = MM == 2 ? (m ? tau[1] : tau[0]) : s_tau[m];
      const bool ok = i + q < i_end, gt = ok && key > t, eq = ok && key == t && (MM == 2 ? (m ? ties[1] : ties[0]) : s_need[m]) > 0u;
      gtbits |= gt ? 1u << q : 0u;
      eqbits |= eq ? 1u << q : 0u;
      if (eq) {
        if (MM == 2) pk[m ? 1 : 0] += m ? 1u : 65536u;
        else { pk[0] += m == 0 ? 65536u : 0u; pk[1] += m == 1 ? 1u : (m == 2 ? 65536u : 0u); pk[2] += m == 3 ? 1u : 0u; }
      }
    }
    pk[0] += (uint32_t)__popc(gtbits);
    // exclusive prefix over the workgroup (4096 candidates: 16 bits hold every count)
    uint32_t ex[3] = {0u, 0u, 0u}, tot[3] = {0u, 0u, 0u};
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      ex[f] = wave_incl_scan_u32(pk[f]);
      if (lane == 63) s_tot[buf][f][wave] = ex[f];
      ex[f] -= pk[f];
    }
    __syncthreads();                               // (two buffers: a wave that is a trip ahead writes the other one)
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const uint32_t w = wave_incl_scan_u32(lane < NWAVES ? s_tot[buf][f][lane] : 0u);
      tot[f] = (uint32_t)__builtin_amdgcn_readlane((int)w, NWAVES - 1);
      ex[f] += wave ? (uint32_t)__builtin_amdgcn_readlane((int)w, wave - 1) : 0u;
    }
    {
      uint32_t rank[MM], pos = run_gt + (ex[0] & 0xffffu);
#pragma unroll
      for (int m = 0; m < MM; ++m) {
        rank[m] = run_eq[m] + (m == 0 ? ex[0] >> 16 : m == 1 ? ex[1] & 0xffffu : m == 2 ? ex[1] >> 16 : ex[2]);
        pos += min(rank[m], ties[m]);
      }
      if (gtbits | eqbits) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = (int)id_of<MM>(ids, q);
          const bool eq = (eqbits >> q) & 1u;
          if (((gtbits >> q) & 1u) || (eq && pick(rank, m) < (MM == 2 ? (m ? ties[1] : ties[0]) : s_need[m]))) out[pos++] = i + q;
#pragma unroll
          for (int mm = 0; mm < MM; ++mm) rank[mm] += eq && mm == m ? 1u : 0u;
        }
      }
    }
    run_gt += tot[0] & 0xffffu;
#pragma unroll
    for (int m = 0; m < MM; ++m) run_eq[m] += m == 0 ? tot[0] >> 16 : m == 1 ? tot[1] & 0xffffu : m == 2 ? tot[1] >> 16 : tot[2];
  }
  uint32_t kept = run_gt;
#pragma unroll
  for (int m = 0; m < MM; ++m) kept += min(run_eq[m], ties[m]);
  for (int r = tid0; r < a.W; r += SEL_THREADS) out[kept + r] = nc + r;
  }
  }
}

size_t select_split_bytes(int M, int nchunks) {
  return reinterpret_cast<size_t>(select_split(nullptr, M, nchunks).list + (size_t)M * nchunks * SEL_GLIST_PER_CHUNK);
}

size_t select_ws_bytes(const Dims& dm, const madakv_config& c) {
  long long per_batch_model = region_tokens_of(c);
  long long per_batch_call = (long long)dm.n * dm.H * ((long long)dm.L + c.max_new_tokens + 2 * c.page_rows);
  long long tokens = std::min(per_batch_model, per_batch_call);
  long long blocks = tokens / GATHER_ROWS + 2;
  return (size_t)dm.B * blocks * sizeof(int32_t) + (size_t)dm.B * 2 * sizeof(long long) + 64;
}

hipError_t launch_offsets(const Dims& dm, const madakv_config& c, int layer0, const int32_t* budgets,
                          int64_t* kv_off, int32_t* kv_len, int32_t* len1, long long* cursor_state, int32_t* layer_maxlen, void* ws,
                          const Paging& pg, int blocks_per_batch, hipStream_t st, const AllocArgs* alloc) {
  OffsetsArgs a;
  a.layer_maxlen = layer_maxlen;
  a.budgets = budgets; a.kv_off = kv_off; a.kv_len = kv_len; a.len1 = len1; a.cursor = cursor_state;
  a.call_range = reinterpret_cast<long long*>(ws);
  a.blk2head = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(ws) + ((size_t)dm.B * 2 * sizeof(long long) + 63) / 64 * 64);
  a.n = dm.n; a.B = dm.B; a.H = dm.H; a.L = dm.L; a.W = dm.W; a.layer0 = layer0; a.M = c.n_modalities;
  a.max_new = c.max_new_tokens; a.keep_all = c.budget >= c.ctx_len ? 1 : 0;
  a.blocks_per_batch = blocks_per_batch; a.region_tokens = pg.region_tokens; a.init_limit = pg.init_limit;
  a.page_rows = pg.page_rows; a.tbl_entries = pg.entries; a.page_tbl = pg.table; a.pool_top = pg.pool_top;
  if (alloc) hipLaunchKernelGGL((offsets_kernel<true>), dim3(dm.B), dim3(OFF_THREADS), 0, st, a, *alloc);
  else hipLaunchKernelGGL((offsets_kernel<false>), dim3(dm.B), dim3(OFF_THREADS), 0, st, a, AllocArgs{});
  return hipGetLastError();
}

template <int MM, int PHASE, bool SMALL = false>
static hipError_t launch_select_t(const SelectArgs& a, dim3 grid, hipStream_t st) {
  const size_t lds = PHASE == 3 ? 0 : select_front(a.M, SMALL) + (size_t)a.M * LIST_MAX<MM, SMALL> * sizeof(unsigned long long);
  if (lds > 48 * 1024) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel<MM, PHASE, SMALL>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((select_kernel<MM, PHASE, SMALL>), grid, dim3(SEL_THREADS), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_select(const Dims& dm, const madakv_config& c, const float* psi_pool, const uint8_t* mask,
                         const int32_t* budgets, const int64_t* kv_off, const int32_t* kv_len, int32_t* kept_idx,
                         hipStream_t st, const int32_t* seg_len, const uint8_t* rowmod, void* split_buf, size_t split_bytes, bool beside_gather) {
  SelectArgs a;
  a.seg_len = seg_len; a.rowmod = rowmod;
  a.psi_pool = psi_pool; a.mask = mask; a.budgets = budgets; a.kv_off = kv_off; a.kv_len = kv_len; a.kept_idx = kept_idx;
  a.B = dm.B; a.H = dm.H; a.L = dm.L; a.W = dm.W; a.nc = dm.nc; a.mpa_mode = c.mpa_mode;
  a.keep_all = (c.budget >= c.ctx_len && !seg_len) ? 1 : 0;
  a.select_mode = c.select_mode; a.sink_tokens = c.sink_tokens; a.M = c.n_modalities;
  a.split = nullptr; a.split_stride = 0;
  const int nchunks = split_chunks(dm);
  const dim3 whole(dm.heads), chunks(nchunks, dm.heads);
  const bool two = a.M == 2;
  if (nchunks && !seg_len && !a.keep_all && a.select_mode != 1 && split_buf &&
      split_bytes >= dm.heads * split_head_bytes(a.M, nchunks)) {
    a.split = static_cast<char*>(split_buf) + stats_split_bytes(a.M, nchunks);
    a.split_stride = (long long)split_head_bytes(a.M, nchunks);
    hipError_t e = two ? launch_select_t<2, 1>(a, chunks, st) : launch_select_t<4, 1>(a, chunks, st);
    if (e == hipSuccess) e = two ? launch_select_t<2, 2>(a, chunks, st) : launch_select_t<4, 2>(a, chunks, st);
    if (e == hipSuccess) e = two ? launch_select_t<2, 3>(a, chunks, st) : launch_select_t<4, 3>(a, chunks, st);
    return e;
  }
  if (beside_gather && a.nc <= SMALL_HEADS) return two ? launch_select_t<2, 0, true>(a, whole, st) : launch_select_t<4, 0, true>(a, whole, st);
  return two ? launch_select_t<2, 0>(a, whole, st) : launch_select_t<4, 0>(a, whole, st);
}

}  // namespace madakv
