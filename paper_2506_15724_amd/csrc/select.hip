// Eviction (paper Sec. 3.3, modality-specific eviction per attention head): for each head
// keep, per modality, the b_m candidates with the largest pooled score; equal scores go to
// the lower position.  Output: kept positions in ascending order, then the W window
// positions, written into the head's segment of the ragged index array.
//
// offsets_kernel   lays the segments out: batch item b owns a fixed region of the reduced
//                  cache, inside it layers and heads follow each other; a segment has
//                  kv_len = b_t + b_v + W rows plus max_new_tokens free rows.  It also fills
//                  a table "first head that overlaps each 64-row block" for the gather.
// select_kernel    one workgroup per head.  A radix descent (descent.h) over count histograms of the
//                  order-preserving keys finds, per modality, the threshold key tau_m and how many elements equal
//                  to tau_m are still needed; then key > tau_m is kept, and key == tau_m while
//                  its rank by position is below that number.  The last pass goes over the candidates in order, 4096 at
//                  a time; prefix sums over the workgroup give
//                  the ranks and the output slots, so the result is ascending by construction.
//                  Bound like the statistics (stats.hip) by latency and instruction issue; nothing unrolled over a
//                  thread's candidates, which are read again per level: 9 KB of code instead of 42, one scan instead of
//                  two in the last pass.  In the path, before -> after: 27.6 -> 11.3 us (8 heads of 1K candidates),
//                  29.5 -> 18.7 (32 of 8K), 35 -> 29 (128 of 16K), re-eviction's 1024 heads of 2K rows 87 -> 27.
#include "allocate.h"
#include "descent.h"

namespace madakv {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_CHUNK = 16384;                 // candidates per workgroup where a head's chunks have workgroups of their own
constexpr uint32_t SEL_SH1 = 21;                 // plain first digit of a 32-bit key

// what the walk of one level hands on, per head and modality, and what a chunk reports (phases 1-4 of select_kernel)
struct SelCarry { DescentRange range; uint32_t need, alive, tau, pad; };
struct SelChunk { uint32_t gt, pad; unsigned long long eq; };   // kept for sure; threshold-valued ones, 16 bits per modality

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
      // blocks whose first row lies inside this segment
      const long long b0 = (off + GATHER_ROWS - 1) / GATHER_ROWS, b1 = seg > 0 ? (off + seg - 1) / GATHER_ROWS : b0 - 1;
      for (long long blk = b0; blk <= b1; ++blk) {
        const long long t = blk - blk_base;
        if (t >= 0 && t < a.blocks_per_batch) a.blk2head[(long long)b * a.blocks_per_batch + t] = f;
      }
      if (f == 0 && (start % GATHER_ROWS) != 0 && 0 < a.blocks_per_batch)
        a.blk2head[(long long)b * a.blocks_per_batch] = 0;    // the call starts inside a block: its first head is head 0
    }
    carry = now_over ? used : carry + tot;
    overflowed = now_over;
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
  // Long heads on few heads (see launch_select): the chunks of a head go to workgroups of their own.
  // phase 0 = the whole head in one workgroup; 1 = count histogram of one chunk at `level`, added to the
  // head's histogram in memory; 2 = the walk over that histogram (one workgroup per head); 3 = a chunk's
  // numbers of kept and of threshold-valued candidates; 4 = a chunk's kept positions written behind those
  // of the chunks before it.
  int phase, level, heads, nchunks;
  uint32_t* gcnt;                 // [3 levels][heads][M][BINS]
  SelCarry* carry;                // [heads][4]
  SelChunk* chunkinfo;            // [heads][nchunks]
};

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

template <int MM>   // modalities the kernel is built for (2: the paper's text / image; 4: up to four)
__global__ __launch_bounds__(SEL_THREADS) __attribute__((amdgpu_waves_per_eu(MM == 2 ? 8 : 4))) void select_kernel(SelectArgs a) {
  constexpr int NWAVES = SEL_THREADS / 64;
  __shared__ __attribute__((aligned(16))) uint32_t cnt[MM][BINS];
  __shared__ DescentRange s_range[MM];
  __shared__ uint32_t s_need[MM], s_alive[MM], s_tau[MM], s_before[MM], s_bin[MM], s_part[MM][NWAVES];
  __shared__ uint32_t s_tot[2][3][NWAVES];
  const int M = a.M;
  const int tid0 = threadIdx.x;
  const int phase = a.phase;
  const bool per_chunk = phase == 1 || phase >= 3;             // grid (chunks, heads)
  const int head = per_chunk ? blockIdx.y : blockIdx.x;
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
  if (a.keep_all) {
    for (int i = tid0; i < a.L; i += SEL_THREADS) out[i] = i;
    return;
  }
  if (a.select_mode == 1) {
    // score-free baseline: the first `sink` candidates and the most recent ones, then the window
    uint32_t btot = 0;
    for (int m = 0; m < M; ++m) btot += (uint32_t)a.budgets[(long long)head * M + m];
    const int total = min((int)btot, nc);
    const int sink = min(a.sink_tokens, total);
    for (int j = tid0; j < total + a.W; j += SEL_THREADS)
      out[j] = j < sink ? j : (j < total ? nc - (total - j) : nc + (j - total));
    return;
  }
  const int i_begin = per_chunk ? (int)blockIdx.x * SEL_CHUNK : 0;
  const int i_end = per_chunk ? min(nc, i_begin + SEL_CHUNK) : nc;
  const uint32_t top = (uint32_t)(M - 1);
  uint32_t* gcnt = phase ? a.gcnt + ((size_t)(phase <= 2 ? a.level : 0) * a.heads + head) * (size_t)M * BINS : nullptr;
  SelCarry* carry = phase ? a.carry + (size_t)head * 4 : nullptr;
  if (tid0 < M) {
    if (phase != 0 && (phase >= 3 || a.level > 0)) {            // what the walks before left
      const SelCarry cy = carry[tid0];
      s_range[tid0] = cy.range; s_need[tid0] = cy.need; s_alive[tid0] = cy.alive; s_tau[tid0] = cy.tau;
    } else {
      s_range[tid0] = phase ? descent_plain<SEL_SH1>() : descent_first(1u);
      s_need[tid0] = (uint32_t)a.budgets[(long long)head * M + tid0]; s_alive[tid0] = 1u; s_tau[tid0] = 0xffffffffu;
    }
  }

  for (int level = phase ? a.level : 0; phase < 3; ++level) {
    // (addresses that depend on the thread are computed level by level: kept over the loop they would spill)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int e = tid; e < M * BINS / 4; e += SEL_THREADS) reinterpret_cast<uint4*>(&cnt[0][0])[e] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    DescentRange rg[MM];
#pragma unroll
    for (int m = 0; m < MM; ++m) rg[m] = descent_uniform(s_range[min(m, M - 1)]);
    if (phase == 2) {                              // the head's histogram of this level, gathered by the chunks' workgroups
      for (int e = tid; e < M * BINS; e += SEL_THREADS) (&cnt[0][0])[e] = gcnt[e];
    } else {
      const bool all = level == 0;                 // every key is in range
      const uint32_t span0 = rg[0].hi - rg[0].lo, span1 = rg[1].hi - rg[1].lo;
      KeyGroup next = load_keys(sc, mask, i_begin + 4 * tid, i_end, a.mpa_mode);
#pragma unroll 1
      for (int i = i_begin + 4 * tid; i < i_end; i += 4 * SEL_THREADS) {
        const KeyGroup g = next;
        next = load_keys(sc, mask, i + 4 * SEL_THREADS, i_end, a.mpa_mode);
        const uint32_t ids = mask4_ids<MM>(g.mw, top);
        if (all) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (i + q < i_end) atomicAdd(&cnt[id_of<MM>(ids, q)][descent_bin(rg[0], float_key(g.x[q]))], 1u);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t m = id_of<MM>(ids, q), key = float_key(g.x[q]);
            const uint32_t lo = MM == 2 ? (m ? rg[1].lo : rg[0].lo) : s_range[m].lo, sp = MM == 2 ? (m ? span1 : span0) : s_range[m].hi - lo;
            if (i + q < i_end && key - lo <= sp) {
              const uint32_t s1 = MM == 2 ? (m ? rg[1].sh : rg[0].sh) : s_range[m].sh;
              atomicAdd(&cnt[m][(key >> s1) - (MM == 2 ? (m ? rg[1].sub : rg[0].sub) : s_range[m].sub)], 1u);
            }
          }
        }
      }
    }
    __syncthreads();
    if (phase == 1) {                              // add the chunk's bins to the head's and leave
      for (int e = tid; e < M * BINS; e += SEL_THREADS) {
        const uint32_t x = (&cnt[0][0])[e];
        if (x) atomicAdd(&gcnt[e], x);
      }
      return;
    }
    // the walk from the top bin down, WPM waves per modality: lane 0 of the first of them has the top bins
    constexpr int WPM = NWAVES / MM, PER = BINS / (WPM * 64);
    const int m = wave / WPM, part = wave % WPM;
    const bool walks = m < M && s_alive[min(m, M - 1)] == 1u;
    const int tb = BINS - 1 - (part * 64 + lane) * PER;       // bins tb, tb - 1, ..., tb - PER + 1
    uint32_t share = 0u, incl = 0u;
    if (walks) {
#pragma unroll
      for (int j = 0; j < PER; ++j) share += cnt[m][tb - j];
      incl = wave_incl_scan_u32(share);
      if (lane == 63) s_part[m][part] = incl;
    }
    __syncthreads();
    uint32_t need = 0u;
    if (walks) {
      uint32_t total = 0u, before = incl - share;
#pragma unroll
      for (int w = 0; w < WPM; ++w) { const uint32_t x = s_part[m][w]; total += x; before += w < part ? x : 0u; }
      need = min(s_need[m], total);                // (first level: a budget above the candidate count keeps them all)
      if (before < need && before + share >= need) {          // one lane of one wave: the bin is among its own
        uint32_t bin = (uint32_t)tb;
#pragma unroll 1
        for (;;) {
          const uint32_t x = cnt[m][bin];
          if (before + x >= need) break;
          before += x; --bin;
        }
        s_before[m] = before; s_bin[m] = bin;
      }
    }
    __syncthreads();
    if (walks && part == 0 && lane == 0) {         // the next level's state (everybody has read this one's)
      if (need == 0u) { s_alive[m] = 0u; s_need[m] = 0u; s_range[m] = descent_none(); }     // nothing to keep: tau stays above every key
      else {
        const DescentRange r = s_range[m];
        s_need[m] = need - s_before[m];            // still needed from inside this bin
        if (r.sh == 0) { s_tau[m] = r.sub + s_bin[m]; s_alive[m] = 2u; s_range[m] = descent_none(); }
        else s_range[m] = descent_next<SEL_SH1>(r, s_bin[m]);
      }
    }
    __syncthreads();
    if (phase == 2) break;
    bool open = false;
    for (int mm = 0; mm < M; ++mm) open = open || s_alive[mm] == 1u;
    if (!open) break;
  }
  if (phase == 2) {                                // hand over to the next level, or to the chunks' compaction
    if (tid0 < M) {
      SelCarry cy;
      cy.range = s_range[tid0]; cy.need = s_need[tid0]; cy.alive = s_alive[tid0]; cy.tau = s_tau[tid0]; cy.pad = 0u;
      carry[tid0] = cy;
    }
    return;
  }
  if (phase >= 3) __syncthreads();

  // take every key > tau_m and the first ties_m keys == tau_m
  const int lane = tid0 & 63, wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  uint32_t tau[MM], ties[MM], run_eq[MM];
#pragma unroll
  for (int m = 0; m < MM; ++m) {
    tau[m] = m < M ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tau[m]) : 0xffffffffu;
    ties[m] = m < M ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_need[m]) : 0u;
    run_eq[m] = 0u;
  }
  uint32_t run_gt = 0u;
  if (phase == 4) {
    // what the chunks in front of this one have: sure ones and threshold-valued ones
    const SelChunk* ci = a.chunkinfo + (size_t)head * a.nchunks;
    for (int c = 0; c < (int)blockIdx.x; ++c) {
      const SelChunk x = ci[c];
      run_gt += x.gt;
#pragma unroll
      for (int m = 0; m < MM; ++m) run_eq[m] += (uint32_t)((x.eq >> (16 * m)) & 0xffffULL);
    }
  }
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
    if (phase != 3) {
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
  if (phase == 3) {                                // report and leave
    if (tid0 == 0) {
      SelChunk x;
      x.gt = run_gt; x.pad = 0u; x.eq = 0ULL;
#pragma unroll
      for (int m = 0; m < MM; ++m) x.eq |= (unsigned long long)run_eq[m] << (16 * m);
      a.chunkinfo[(size_t)head * a.nchunks + blockIdx.x] = x;
    }
    return;
  }
  if (per_chunk && i_end != nc) return;            // the window positions follow the last chunk's
  uint32_t kept = run_gt;
#pragma unroll
  for (int m = 0; m < MM; ++m) kept += min(run_eq[m], ties[m]);
  for (int r = tid0; r < a.W; r += SEL_THREADS) out[kept + r] = nc + r;
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

hipError_t launch_select(const Dims& dm, const madakv_config& c, const float* psi_pool, const uint8_t* mask,
                         const int32_t* budgets, const int64_t* kv_off, const int32_t* kv_len, int32_t* kept_idx,
                         hipStream_t st, const int32_t* seg_len, const uint8_t* rowmod, void* split_buf, size_t split_bytes) {
  SelectArgs a;
  a.seg_len = seg_len; a.rowmod = rowmod;
  a.psi_pool = psi_pool; a.mask = mask; a.budgets = budgets; a.kv_off = kv_off; a.kv_len = kv_len; a.kept_idx = kept_idx;
  a.B = dm.B; a.H = dm.H; a.L = dm.L; a.W = dm.W; a.nc = dm.nc; a.mpa_mode = c.mpa_mode;
  a.keep_all = (c.budget >= c.ctx_len && !seg_len) ? 1 : 0;
  a.select_mode = c.select_mode; a.sink_tokens = c.sink_tokens; a.M = c.n_modalities;
  a.phase = 0; a.level = 0; a.heads = dm.heads; a.nchunks = 0; a.gcnt = nullptr; a.carry = nullptr; a.chunkinfo = nullptr;
  const int nchunks = split_chunks(dm);
  if (nchunks && !seg_len && !a.keep_all && a.select_mode != 1 && split_buf &&
      split_bytes >= split_buffer_bytes(dm.heads, a.M, nchunks)) {
    // per level: the chunks' workgroups add their count histograms into the head's (in memory), one workgroup per head
    // walks it; then every chunk reports what it keeps and writes it behind the chunks in front of it
    const size_t hist = (size_t)3 * dm.heads * a.M * BINS;
    a.gcnt = reinterpret_cast<uint32_t*>(split_buf);
    a.carry = reinterpret_cast<SelCarry*>(a.gcnt + hist);
    a.chunkinfo = reinterpret_cast<SelChunk*>(a.carry + (size_t)dm.heads * 4);
    a.nchunks = nchunks;
    launch_split_zero(a.gcnt, (long long)hist, st);
    for (int step = 0; step < 8; ++step) {
      a.phase = step < 6 ? 1 + (step & 1) : step - 3;          // 1, 2, 1, 2, 1, 2, 3, 4
      a.level = step < 6 ? step / 2 : 0;
      const dim3 grid = a.phase == 2 ? dim3(dm.heads) : dim3(nchunks, dm.heads);
      if (a.M == 2) hipLaunchKernelGGL((select_kernel<2>), grid, dim3(SEL_THREADS), 0, st, a);
      else hipLaunchKernelGGL((select_kernel<4>), grid, dim3(SEL_THREADS), 0, st, a);
    }
    return hipGetLastError();
  }
  if (a.M == 2) hipLaunchKernelGGL((select_kernel<2>), dim3(dm.heads), dim3(SEL_THREADS), 0, st, a);
  else hipLaunchKernelGGL((select_kernel<4>), dim3(dm.heads), dim3(SEL_THREADS), 0, st, a);
  return hipGetLastError();
}

}  // namespace madakv
