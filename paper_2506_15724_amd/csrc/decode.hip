// Decode over the reduced, ragged cache (paper Sec. 3.1 Eq. 3-5): append the new K/V row to
// every head's segment (Eq. 4), then out = softmax(scale * q K_c^T) V_c over the rows the
// head kept (Eq. 5).  The G query heads of a KV head share one pass over its K_c and V_c.
//
// This is bandwidth work: 2 * len * d * sizeof(T) bytes per KV head and step, a few flops
// per byte.  A row is LPR lanes x 16 bytes; a wave reads 64 / LPR rows per load
// instruction and keeps UNROLL K rows and UNROLL V rows in flight.  The dot product is
// reduced over the LPR lanes of a row with DPP row operations, the softmax is the usual
// running max / running sum in the log2 domain with fp32 accumulation.  Each head's rows
// are cut into pieces of `chunk_rows` (one workgroup each): a single layer's 128 ragged heads
// become ~1100 pieces of work that the hardware scheduler spreads over 256 CUs.  The
// grid is (heads, most pieces a head is cut into by decode_plan, or the longest head's once the host knows it): workgroups past
// a head's real length exit at once, and since the piece index is the slow grid dimension they are dispatched
// after all the real work.  The pieces of a head meet inside the same launch (finish_piece): every one leaves its partial
// (max, sum, acc) in memory, has the stores acknowledged and counts itself at the head's counter, and whoever comes last
// merges them in piece order.  Nobody waits for another workgroup.  The appended row is taken from k_new / v_new by the
// workgroup whose piece holds it, which also stores it in the cache; kv_len is bumped by whoever finishes the head.
//
// Measured per layer call, with a merge kernel behind the attention kernel -> in one launch: 128 heads of ~2K bf16 rows,
// 135 MB, 28.6 -> 26.8 us (the rows alone take 21.7 at the rate of a large read), 8-bit rows 18.7 -> 16.6, 4 heads of 2K rows
// with 7 queries each 10.5 -> 8.8 (7.6 with the kernel as it is now).  What the end of a piece costs, from the last row to the output: 0.35 us among the lanes
// of a wave (row swaps and rotations; shuffles through LDS took 0.75), 0.4 among the waves, 0.6 for acknowledgement and
// arrival, 0.7-1.3 for reading the pieces, 0.3 for the output.  It is instructions as much as trips to memory: a merge by
// the whole workgroup with 8-byte accesses, polling for words not yet there instead of counting, took 3.5 us longer than
// this one on grouped queries and gained nothing over the merge kernel on single ones.  Counters that share a line cost
// as much as the merge kernel does: hence 128 bytes each.
// Cutting the rows of all heads, laid end to end, into equal stretches per workgroup, so that the launch has a single,
// perfectly balanced round of workgroups: 27.3 against 26.9 us for 128 heads of ~2K rows, the table of head starts every
// workgroup has to build first costs what the balance gains.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace madakv {

constexpr float DNEG_BIG = -1.0e30f;
constexpr int DEC_THREADS = 256;
typedef __attribute__((ext_vector_type(4))) unsigned int du32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned int du32x2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 dbf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 dbf16x2_t;
typedef __attribute__((ext_vector_type(4))) float df32x4_t;
typedef __attribute__((ext_vector_type(2))) float df32x2_t;
typedef __attribute__((ext_vector_type(4))) short ds16x4_t;

struct DecodeArgs {
  const void* q; const void* k_new; const void* v_new; void* k_c; void* v_c;
  const int64_t* kv_off; int32_t* kv_len; void* out;
  int B, H, G, chunk_rows, out_fp32, has_new;
  int max_chunks;       // most pieces a head is cut into (head_chunk_rows)
  int max_new;          // rows a segment has room for behind those of the eviction
  float* part;          // [heads][slots][G][d] partial results of the pieces of the call's heads
  float* part_ml;       // [heads][slots][G][2] their (max, sum)
  int slots;            // most pieces of a head
  uint32_t by_heads;    // ceil(2^32 / heads), likewise, where heads * (heads + pieces) < 2^32
  uint32_t by_chunk;    // ceil(2^32 / chunk_rows): quotients of numbers below 2^21, 0 where a head may be longer (see pieces_of)
  Meet meet;            // how they meet
  long long capacity;   // rows in k_c / v_c
  // paged cache (page_rows > 0): see struct Paging
  int page_rows, page_shift, tbl_entries;
  int32_t* page_tbl; unsigned long long* pool_top;
  long long region_pages;      // pages in one batch item's region
  long long head0;             // index of the call's first head in the whole model (layer0 * B * H)
  float scale_log2;
};

// 16 bytes that are read once per launch (cache rows): a non-temporal load, so that the stream
// does not push anything useful out of the caches.  Measured: 10-15% off the decode step.
typedef __attribute__((ext_vector_type(4))) unsigned int stream_u32x4_t;
__device__ __forceinline__ uint4 stream_load16(const void* p) {
  const stream_u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const stream_u32x4_t*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}

template <int LPR> __device__ __forceinline__ float row_sum(float x);
template <> __device__ __forceinline__ float row_sum<16>(float x) { return row16_sum(x); }
template <> __device__ __forceinline__ float row_sum<8>(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));
  return x;
}
template <> __device__ __forceinline__ float row_sum<4>(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));
  return x;
}
template <> __device__ __forceinline__ float row_sum<32>(float x) {
  x = row16_sum(x);
  return x + __shfl_xor(x, 16, 64);
}

template <typename T> struct Elems;
template <> struct Elems<uint16_t> {
  static constexpr int EPL = 8;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = bf16_lo(r.x); f[1] = bf16_hi(r.x); f[2] = bf16_lo(r.y); f[3] = bf16_hi(r.y);
    f[4] = bf16_lo(r.z); f[5] = bf16_hi(r.z); f[6] = bf16_lo(r.w); f[7] = bf16_hi(r.w);
  }
};
template <> struct Elems<uint8_t> {                  // E4M3 bytes of the 8-bit reduced cache
  static constexpr int EPL = 16;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {                     // the hardware conversion is exact (every code is a float)
      const f32x2_t lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], false);
      const f32x2_t hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], true);
      f[i * 4] = lo[0]; f[i * 4 + 1] = lo[1]; f[i * 4 + 2] = hi[0]; f[i * 4 + 3] = hi[1];
    }
  }
};
template <> struct Elems<float> {
  static constexpr int EPL = 4;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
};

// EPL consecutive elements of the caller's type T (Q, k_new, v_new) as floats
template <typename T, int EPL>
__device__ __forceinline__ void load_floats(const T* p, float* f) {
  constexpr int PER = 16 / sizeof(T);                 // elements per 16-byte load
#pragma unroll
  for (int j = 0; j < EPL / PER; ++j) Elems<T>::unpack(*reinterpret_cast<const uint4*>(p + j * PER), f + j * PER);
}

// ---- where row r of a head lives ---------------------------------------------------------
// Contiguous segments: at off + r.  Paged cache: the first init_rows rows (the head's initial pages,
// which follow each other) likewise; later rows in pages listed in the head's table.  `fresh`
// is the page this workgroup has just taken for the row being appended, if it had to take one
// (the table entry it wrote is not yet visible to its other threads).
struct RowMap {
  long long off;
  int init_rows;               // INT_MAX without paging
  const int32_t* tbl;          // the head's table (entries 1.. = pages taken later)
  int shift, fresh_slot;
  long long fresh_page;
  __device__ __forceinline__ long long operator()(int r) const {
    if (r < init_rows) return off + r;
    const int q = r - init_rows, j = q >> shift;
    const long long pg = (j == fresh_slot) ? fresh_page : (long long)tbl[1 + j];
    return (pg << shift) + (q & ((1 << shift) - 1));
  }
};

template <bool PAGED>
__device__ __forceinline__ bool can_append_to(const DecodeArgs& a, long long off, int len_old) {
  // an empty segment (its budgets did not fit the cache) stays empty; contiguous segments also end at the cache's end
  return a.has_new && len_old > 0 && (PAGED || off + len_old < a.capacity);
}

// All threads of the workgroup.  rows [r_begin, r_end) are the workgroup's; when the appended row is
// among them and starts a new page, thread 0 takes the next page from the top of the batch item's region.
template <bool PAGED>
__device__ __forceinline__ RowMap make_row_map(const DecodeArgs& a, long long hidx, long long off, int len_old, bool can_append,
                                               int r_begin, int r_end) {
  RowMap m;
  m.off = off; m.init_rows = 0x7fffffff; m.tbl = nullptr; m.shift = 0; m.fresh_slot = -1; m.fresh_page = 0;
  if (!PAGED) return m;
  __shared__ long long s_fresh;
  int32_t* tbl = a.page_tbl + (a.head0 + hidx) * a.tbl_entries;
  m.tbl = tbl; m.shift = a.page_shift;
  m.init_rows = tbl[0] << a.page_shift;
  const int q = len_old - m.init_rows;
  const bool takes = can_append && len_old >= r_begin && len_old < r_end && q >= 0 && (q & (a.page_rows - 1)) == 0;   // uniform
  if (takes) {
    if (threadIdx.x == 0) {
      const long long b = ((a.head0 + hidx) / a.H) % a.B;
      const unsigned long long nth = atomicAdd(a.pool_top + b, 1ULL);
      const long long page = (b + 1) * a.region_pages - 1 - (long long)nth;
      tbl[1 + (q >> a.page_shift)] = (int32_t)page;
      s_fresh = page;
    }
    __syncthreads();
    m.fresh_slot = q >> a.page_shift;
    m.fresh_page = s_fresh;
  }
  return m;
}

// Rows per piece of a head of `len` rows: a.chunk_rows, or for a head that would need more than max_chunks pieces a
// larger multiple of 32.  The grid then depends on the budget alone and not on the longest head a layer may have.  The
// host learns that length only once the eviction has run; sizing the grid for the whole context until then put 65
// instead of 17 workgroups per head in the grid (16K context, budget 2048), 5 of 36 us per layer call for
// workgroups that found nothing to do.
__device__ __forceinline__ int head_chunk_rows(const DecodeArgs& a, int len) {
  if (len <= a.chunk_rows * a.max_chunks) return a.chunk_rows;
  return ((len + a.max_chunks - 1) / a.max_chunks + 31) / 32 * 32;
}

// ceil(len / chunk_rows).  As a product: len + chunk_rows - 1 < 2^21 and chunk_rows <= 2^10, so what by_chunk is too large by
// (below chunk_rows / 2^32) stays below 1 in units of the next quotient.
__device__ __forceinline__ int pieces_of(const DecodeArgs& a, int len) {
  const uint32_t x = (uint32_t)(len + a.chunk_rows - 1);
  return a.by_chunk ? (int)__umulhi(x, a.by_chunk) : (int)(x / (uint32_t)a.chunk_rows);
}

// The head a workgroup works on.  Workgroups go to the 8 XCDs in turn; with the head as the fast grid dimension all
// pieces of a head would meet on one XCD (128 heads), and XCDs with long heads would finish last: the pieces of a head
// are rotated over the XCDs instead.
__device__ __forceinline__ int piece_head(const DecodeArgs& a) {
  const uint32_t x = blockIdx.x + blockIdx.y;
  if (x < gridDim.x) return (int)x;
  return (int)(x - (a.by_heads ? __umulhi(x, a.by_heads) : x / gridDim.x) * gridDim.x);
}

// The appended row of the 8-bit cache, encoded: written to the cache (Eq. 4) and left in LDS, K then V, for the tile it
// belongs to.  All threads; `row` is its place in the cache.  (Kept out of the load path of the tiles: the encoding,
// unrolled there, had made 48 KB of the grouped-query kernel, and by the wave of the tile, in its loop, it costs a single
// query head's calls 2%.)
template <int D>
__device__ __forceinline__ void stage_new_row(const DecodeArgs& a, long long hidx, long long row, uint8_t* s_new) {
  for (int e = threadIdx.x; e < 2 * D; e += (int)blockDim.x) {
    const bool is_k = e < D;
    const int c = is_k ? e : e - D;
    const uint8_t y = (uint8_t)f32_to_e4m3(bf16_bits_to_f32((reinterpret_cast<const uint16_t*>(is_k ? a.k_new : a.v_new))[hidx * D + c]));
    (reinterpret_cast<uint8_t*>(is_k ? a.k_c : a.v_c))[row * D + c] = y;
    s_new[e] = y;
  }
  __syncthreads();
}

// ---- the end of a piece ------------------------------------------------------------------------
// exp2 of something <= 0, a weight beside one of 1: the instruction itself (the library call spends seven more on keeping
// denormal results)
__device__ __forceinline__ float weight_of(float x) { return __builtin_amdgcn_exp2f(x); }

// The two values of lanes that are O apart (O = 4 ... 32: within a row by rotation, across rows by a swap of rows): the same
// pair in both lanes up to its order.  (Rotated by 4, lane i is paired with lane i - 4 and that one with i - 8: only the merge over 8
// that follows brings the four of a row together in every lane.)
template <int O>
__device__ __forceinline__ void lane_pair(float x, float& p, float& q) {
  const uint32_t u = __float_as_uint(x);
  if constexpr (O == 32) { const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false); p = __uint_as_float(r[0]); q = __uint_as_float(r[1]); }
  else if constexpr (O == 16) { const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false); p = __uint_as_float(r[0]); q = __uint_as_float(r[1]); }
  else { p = x; q = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, 0x120 + O, 0xF, 0xF, true)); }       // row_ror
}
// (max, sum, acc) of the lanes LPR, 2 LPR, ... apart merged, the result in all of them
template <int O, int N>
__device__ __forceinline__ void merge_lanes(float& m, float& l, float (&acc)[N]) {
  if constexpr (O < 64) {
    float m1, m2, l1, l2;
    lane_pair<O>(m, m1, m2);
    lane_pair<O>(l, l1, l2);
    m = fmaxf(m1, m2);
    const float c1 = weight_of(m1 - m), c2 = weight_of(m2 - m);
    l = l1 * c1 + l2 * c2;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      float a1, a2;
      lane_pair<O>(acc[e], a1, a2);
      acc[e] = a1 * c1 + a2 * c2;
    }
    merge_lanes<O * 2, N>(m, l, acc);
  }
}

// Workgroups of the grid that arrive at a head's counters: those whose piece may exist before the next eviction.  It follows
// from what only an eviction changes (len1: 1 + the rows it left; 0: this handle has not seen one) and not from the head's length,
// which the last one to arrive has replaced by the time a workgroup further back in the grid starts.
__device__ __forceinline__ int arrivals(const DecodeArgs& a, int len1) {
  if (len1 == 0) return (int)gridDim.y;
  return max(1, min((int)gridDim.y, pieces_of(a, len1 - 1 + a.max_new)));
}
// four neighbouring elements of the output
template <typename T>
__device__ __forceinline__ void store_out4(const DecodeArgs& a, long long o, float4 x, float ls) {
  x = make_float4(x.x / ls, x.y / ls, x.z / ls, x.w / ls);
  if (a.out_fp32 || sizeof(T) == 4) {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.out) + o) = x;
  } else {
    const df32x2_t lo = {x.x, x.y}, hi = {x.z, x.w};                    // (to nearest even, in one instruction each)
    const uint2 y = make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, dbf16x2_t)), __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, dbf16x2_t)));
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.out) + o) = y;
  }
}
// Partial results go past the caches that other XCDs do not see (the sc1 bit, which is what an agent-scope atomic access
// has; those move 8 bytes at most, and two per lane are twice the requests: 16 partial results of 7 query heads took 1.9 us
// to read instead of 1.3).
constexpr int AGENT = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t agent_buffer(void* p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00020000); }
constexpr int NOWHERE = 0x7ffffff0;      // past the end of any of them: a read gives zeros and touches nothing

// The NW waves' (max, sum, acc) of a piece merged in wave order: the output if the head is this one piece.  Otherwise the
// piece's partial result goes to the head's record in the workspace, and the last workgroup to arrive at the head's counter merges them all,
// in piece order, and stores the head's new length (everybody has read the old one).  Behind the barrier every wave works
// for itself, with counters of its own: 64 / (D / 4) query heads per wave, four elements per lane (a single query head:
// the first wave alone, whose lanes share the pieces); a wave has its stores acknowledged, arrives, and leaves unless it is
// the last.
// s_ml: [NW][GT] (max, sum); s_acc: a wave's results WS floats behind those of the wave before it, AR floats per query head.
template <typename T, int D, int NW, int GT, int WS, int AR>
__device__ __forceinline__ void finish_piece(const DecodeArgs& a, long long hidx, int chunk, int len, int rows, bool can_append, int arrive,
                                             const float (*s_ml)[GT][2], const float* s_acc) {
  constexpr int TL = D / 4, QW = 64 / TL;
  constexpr bool OWN = NW >= GT;                             // a query head per wave, whose lanes share the pieces
  constexpr int KP = OWN ? QW : 1, MB = OWN ? 8 : 16;        // MB: pieces in flight per lane
  constexpr int WK = OWN && (GT > 1 || NW == 8) ? KP : 1;    // and, of more than a few waves, their results
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave * (OWN ? 1 : QW) >= (GT == 1 ? 1 : a.G)) return;
  const int t = lane % TL, kp = OWN ? lane / TL : 0, g = OWN ? wave : wave * QW + lane / TL;
  const bool act = OWN ? kp == 0 : g < a.G;
  const int pieces = len <= rows ? 1 : rows == a.chunk_rows ? pieces_of(a, len) : (len + rows - 1) / rows;
  const long long o = (hidx * a.G + g) * D + 4 * t;
  // records of a head: [slots][G][D] accumulated elements, [slots][G] (max, sum)
  const int step = a.G * D * 4, step_ml = a.G * 8;
  const __amdgpu_buffer_rsrc_t rec = agent_buffer(a.part + hidx * a.slots * a.G * D, a.slots * step);
  const __amdgpu_buffer_rsrc_t rec_ml = agent_buffer(a.part_ml + hidx * a.slots * a.G * 2, a.slots * step_ml);
  if (chunk < pieces && (act || WK > 1)) {
    float mx = DNEG_BIG, ls = 0.f, av[4] = {0.f, 0.f, 0.f, 0.f};
    const int w0 = WK > 1 ? kp * (NW / WK) : 0;
#pragma unroll
    for (int w = 0; w < NW / WK; ++w) mx = fmaxf(mx, s_ml[w0 + w][g][0]);
#pragma unroll
    for (int w = 0; w < NW / WK; ++w) {
      const float c = weight_of(s_ml[w0 + w][g][0] - mx);
      const float4 x = *reinterpret_cast<const float4*>(s_acc + (w0 + w) * WS + g * AR + 4 * t);
      ls += s_ml[w0 + w][g][1] * c;
      av[0] += x.x * c; av[1] += x.y * c; av[2] += x.z * c; av[3] += x.w * c;
    }
    if (WK > 1) merge_lanes<TL, 4>(mx, ls, av);
    if (pieces == 1) {
      if (act) store_out4<T>(a, o, make_float4(av[0], av[1], av[2], av[3]), ls);
    } else if (act) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(du32x4_t, make_float4(av[0], av[1], av[2], av[3])), rec, (g * D + 4 * t) * 4, chunk * step, AGENT);
      if (t == 0) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(du32x2_t, make_float2(mx, ls)), rec_ml, g * 8, chunk * step_ml, AGENT);
    }
  }
  if (arrive > 1) {
    const long long head = a.head0 + hidx;
    uint32_t* count = a.meet.count + (GT == 1 ? head : head * a.G + wave) * MEET_COUNT_STRIDE;
    uint32_t arrived = 0u;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the wave's stores are where everybody sees them
    if (lane == 0) arrived = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)arrived);
    if (arrived + 1u != (uint32_t)arrive) return;
    if (lane == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (pieces > 1) {
      float m = DNEG_BIG, ls = 0.f, av[4] = {0.f, 0.f, 0.f, 0.f};
      const int gg = act || OWN ? g : 0;                       // (lanes without a query head read along)
      const int at = ((kp * a.G + gg) * D + 4 * t) * 4, at_ml = (kp * a.G + gg) * 8;
      const int left = min(pieces, a.slots);                   // (a head longer than the launch was sized for: what there is of it)
      const auto merge = [&](const float4 (&x)[MB], const float2 (&ml)[MB]) {
        float bm = m;
#pragma unroll
        for (int j = 0; j < MB; ++j) bm = fmaxf(bm, ml[j].x);
        const float sc = weight_of(m - bm);
        ls *= sc; av[0] *= sc; av[1] *= sc; av[2] *= sc; av[3] *= sc;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
          const float f = weight_of(ml[j].x - bm);
          ls = fmaf(ml[j].y, f, ls);
          av[0] = fmaf(x[j].x, f, av[0]); av[1] = fmaf(x[j].y, f, av[1]); av[2] = fmaf(x[j].z, f, av[2]); av[3] = fmaf(x[j].w, f, av[3]);
        }
        m = bm;
      };
      // Whole trips of KP * MB pieces, without masks (2 heads of 8K rows, 64 to 128 pieces each, took 1 us more per call with them) and
      // out of the way of the last one, which is the only one of most heads (0.2 us per call of 4 heads of 700 rows).
      int c0 = 0;
      if (__builtin_expect(left > KP * MB, 0)) {
        for (; c0 + KP * MB < left; c0 += KP * MB) {
          float4 x[MB]; float2 ml[MB];
#pragma unroll
          for (int j = 0; j < MB; ++j) {
            ml[j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rec_ml, at_ml, (c0 + j * KP) * step_ml, AGENT));
            x[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rec, at, (c0 + j * KP) * step, AGENT));
          }
          merge(x, ml);
        }
      }
      {
        float4 x[MB]; float2 ml[MB];
#pragma unroll
        for (int j = 0; j < MB; ++j) {
          const int c = c0 + j * KP;
          const bool mine = c + kp < left;
          ml[j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rec_ml, mine ? at_ml + c * step_ml : NOWHERE, 0, AGENT));
          x[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rec, mine ? at + c * step : NOWHERE, 0, AGENT));
        }
#pragma unroll
        for (int j = 0; j < MB; ++j) ml[j].x = c0 + j * KP + kp < left ? ml[j].x : 2.f * DNEG_BIG;     // weight 0, of zeros
        merge(x, ml);
      }
      if (KP > 1) merge_lanes<TL, 4>(m, ls, av);
      if (act) store_out4<T>(a, o, make_float4(av[0], av[1], av[2], av[3]), ls);
    }
  }
  if (can_append && threadIdx.x == 0) a.kv_len[hidx] = len;
}

template <typename T, typename CT, int LPR, int GT, int UNROLL, int NW, bool PAGED>   // T: Q / new rows / out; CT: cache elements
__global__ __launch_bounds__(NW * 64) void decode_attn_kernel(DecodeArgs a) {
  constexpr int EPL = Elems<CT>::EPL;
  constexpr int RPI = 64 / LPR;
  constexpr int D = LPR * EPL;
  __shared__ float s_ml[NW][GT][2];
  __shared__ __attribute__((aligned(16))) float s_acc[NW][GT][D];
  constexpr bool ENCODE = sizeof(CT) != sizeof(T);
  __shared__ __attribute__((aligned(16))) uint8_t s_new[ENCODE ? 2 * D : 16];

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane / LPR, piece = lane % LPR;
  const long long hidx = piece_head(a);               // (layer, batch, kv head) of the call
  const int chunk = blockIdx.y;                      // which piece of the head
  const int len1 = a.meet.len1[a.head0 + hidx], len_old = a.kv_len[hidx];
  const long long off = a.kv_off[hidx];
  // queries of the group (on their way while the length is), pre-multiplied by scale * log2(e) below
  float qf[GT][EPL];
  const T* qg = reinterpret_cast<const T*>(a.q) + hidx * a.G * D;
#pragma unroll
  for (int g = 0; g < GT; ++g) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) qf[g][e] = 0.f;
    if (g < a.G) load_floats<T, EPL>(qg + (long long)g * D + piece * EPL, qf[g]);
  }
  asm volatile("" :: "s"(len1), "s"(len_old), "s"((int)off));          // (all three in one trip)
  const int arrive = arrivals(a, len1);
  if (chunk >= arrive) return;                       // the grid is the same for all heads (decode_plan)
  // an empty segment (its budgets did not fit the cache) stays empty: no append, output 0/0 = NaN
  const bool can_append = can_append_to<PAGED>(a, off, len_old);
  const int len = len_old + (can_append ? 1 : 0);
  const int rows = head_chunk_rows(a, len);
  const int r_begin = chunk * rows;                  // (past the head's end: no rows, the workgroup only arrives)
  const int r_end = min(len, r_begin + rows);
  const RowMap at = make_row_map<PAGED>(a, hidx, off, len_old, can_append, r_begin, r_end);
  const bool has_fresh = can_append && len_old >= r_begin && len_old < r_end;   // uniform: the appended row is in this piece
  if constexpr (ENCODE) { if (has_fresh) stage_new_row<D>(a, hidx, at(len_old), s_new); }
  // the NW waves take turns on consecutive RPI * UNROLL-row slices, so that at any moment the
  // workgroup reads one contiguous stretch of K and one of V
  constexpr int WSTEP = RPI * UNROLL;

  float m[GT], l[GT], acc[GT][EPL];
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    m[g] = DNEG_BIG; l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) { acc[g][e] = 0.f; qf[g][e] *= a.scale_log2; }
  }

  // the piece's first row (64 bits: a head may take more than 4 GiB); the rows' offsets from it fit 32 bits
  const unsigned char* kc = reinterpret_cast<const unsigned char*>(a.k_c) + (PAGED ? 0 : (off + r_begin) * (LPR * 16));
  const unsigned char* vc = reinterpret_cast<const unsigned char*>(a.v_c) + (PAGED ? 0 : (off + r_begin) * (LPR * 16));

  for (int row0 = r_begin + wave * WSTEP; row0 < r_end; row0 += NW * WSTEP) {
    uint4 kraw[UNROLL], vraw[UNROLL];
    // rows past the end: the last row once more, masked below (no branch in the loads)
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int r = min(row0 + u * RPI + sub, r_end - 1);
      if (PAGED) {
        const long long o = (at(r) * LPR + piece) * 16;
        kraw[u] = stream_load16(kc + o); vraw[u] = stream_load16(vc + o);
      } else {
        const uint32_t o = (uint32_t)((r - r_begin) * LPR + piece) * 16u;
        kraw[u] = stream_load16(kc + o); vraw[u] = stream_load16(vc + o);
      }
    }
    if (has_fresh && row0 <= len_old && len_old < row0 + WSTEP) {        // the appended row (rows past it are masked)
      uint4 knew, vnew;
      if constexpr (ENCODE) {
        knew = *reinterpret_cast<const uint4*>(s_new + piece * EPL);
        vnew = *reinterpret_cast<const uint4*>(s_new + D + piece * EPL);
      } else {
        knew = *reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(a.k_new) + hidx * D + piece * EPL);
        vnew = *reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(a.v_new) + hidx * D + piece * EPL);
        if (sub == 0) {
          const long long o = at(len_old) * D + piece * EPL;
          *reinterpret_cast<uint4*>(reinterpret_cast<T*>(a.k_c) + o) = knew;
          *reinterpret_cast<uint4*>(reinterpret_cast<T*>(a.v_c) + o) = vnew;
        }
      }
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (row0 + u * RPI + sub >= len_old) { kraw[u] = knew; vraw[u] = vnew; }
    }
    if (row0 + WSTEP > r_end) {                                             // what is masked contributes 0 * 0
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (row0 + u * RPI + sub >= r_end) vraw[u] = make_uint4(0, 0, 0, 0);
    }
    float s[UNROLL][GT];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      float kf[EPL];
      Elems<CT>::unpack(kraw[u], kf);
      const bool valid = row0 + u * RPI + sub < r_end;
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) dot = fmaf(qf[g][e], kf[e], dot);
        dot = row_sum<LPR>(dot);
        s[u][g] = valid ? dot : 2.f * DNEG_BIG;                            // below every running maximum: exp2 gives 0
      }
    }
#pragma unroll
    for (int g = 0; g < GT; ++g) {
      float mx = m[g];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) mx = fmaxf(mx, s[u][g]);
      const float sc = weight_of(m[g] - mx);
      l[g] *= sc;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] *= sc;
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) { s[u][g] = weight_of(s[u][g] - mx); l[g] += s[u][g]; }
      m[g] = mx;
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      float vf[EPL];
      Elems<CT>::unpack(vraw[u], vf);
#pragma unroll
      for (int g = 0; g < GT; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(s[u][g], vf[e], acc[g][e]);
    }
  }

  // merge the RPI row groups of the wave, then the NW waves through LDS
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    merge_lanes<LPR, EPL>(m[g], l[g], acc[g]);
    if (sub == 0) {
      if (piece == 0) { s_ml[wave][g][0] = m[g]; s_ml[wave][g][1] = l[g]; }
#pragma unroll
      for (int e = 0; e < EPL; ++e) s_acc[wave][g][piece * EPL + e] = acc[g][e];
    }
  }
  __syncthreads();
  finish_piece<T, D, NW, GT, GT * D, D>(a, hidx, chunk, len, rows, can_append, arrive, s_ml, &s_acc[0][0][0]);
}

// ------------------------------------------------------------------------------------
// Grouped-query variant (bf16, G >= 2): both contractions run on the 16x16x32 bf16 MFMA, so
// that the G query heads of a KV head cost no more vector instructions than one.
//   S^T[key][q] = K_tile . Q^T     A = 16 keys x 32 dims read straight from the cache rows
//                                  (a lane takes 16 bytes of "its" key), B = Q, kept in registers
//   O^T[d][q]  += V_tile^T . P^T   contraction over 16 keys, twice: in S^T a lane holds 4 keys for
//                                  its query; as bf16 hi and lo parts, which keep fp32-level accuracy,
//                                  they are the lane's 8 entries of the B fragment (no cross-lane
//                                  movement), against the same 4 rows of V in both halves of the A
//                                  fragment: transposing LDS reads (four rows of 16 columns per 16
//                                  lanes) of a wave-private LDS tile that the V rows were written to
//                                  with coalesced 16-byte loads.
// The running max / sum live per query in the lanes of S^T, and so do the four neighbouring dims of one query that a
// lane has of O^T: rescaled by its own factor, left in LDS in 16-byte pieces.
// A layer of a grouped-query model has few KV heads and a few MB of cache: the kernel is bound by the latencies of
// one workgroup (start, length, rows, two contractions, merge), of which a wave's instructions, issued one per four
// cycles, are the larger part.  So a workgroup has eight waves with one tile of 16 rows each in the usual piece of 128: half
// of the instructions of a 32-row tile, a query head per wave in the merges, twice the loads in flight; the first tile adds
// to nothing and rescales nothing; the appended row is fetched from k_new / v_new in place of the cache row.
// The rows are read with ordinary loads: a K fragment takes half of a cache line, and a non-temporal load would fetch the
// line a second time for the other half.  Per layer call, four waves of 32 rows with non-temporal loads in a layout of O[q][d] -> this: 4
// heads of 2K rows, 7 queries, 8.8 -> 7.6 us (half of it the ordinary loads); 16 heads of 2K rows 11.4 -> 9.9; 32 heads of 4K rows, 4
// queries, 14.5 -> 11.5; 2 heads of 40K rows, 6 queries, 18.4 -> 12.6.  Launches that fill the chip: 64 heads of 8K rows 67 -> 62, 256 of 2K
// 71 -> 68, 128 of 16K 218 -> 218, 1024 of 2K 220 -> 217; 8-bit rows, 1024 heads of 1K, 84 -> 69.
// Rows of 64 dims have half the bytes for the same instructions per tile: with many of them in a launch it is four waves of 32-row
// tiles (the maxima, factors and rescaling once per 32 rows), in more workgroups at a time, and non-temporal loads of V, of which
// an instruction takes whole lines.  Old layout / eight waves of 16 rows / this, us: 64 heads of 4K rows 22.3 / 23.9 / 18.3, of 16K 64 / 68 / 54,
// 1024 of 2K 114 / 126 / 92; 8-bit rows, 128 heads of 4K 27 / 32 / 21, 1024 of 2K 78 / 83 / 58.  In pieces of 128 rows it is better from
// 256 heads on: 256 of 200 rows 8.9 / 11.1 / 8.7, 512 of 80 9.5 / 10.5 / 8.7, but 128 of 400 9.4 / 8.9 / 9.2, 4 of 2K 7.9 / 6.6 / 7.4.
// ------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) ds16x4_t* lds_s16x4_ptr_t;

// 4 E4M3 bytes -> 4 bf16 (exact: 3 mantissa bits fit bf16's 7), as two packed dwords
__device__ __forceinline__ du32x2_t e4m3x4_to_bf16x4(uint32_t w) {
  const df32x2_t a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
  du32x2_t o;
  o[0] = (__float_as_uint(a[0]) >> 16) | (__float_as_uint(a[1]) & 0xffff0000u);
  o[1] = (__float_as_uint(b[0]) >> 16) | (__float_as_uint(b[1]) & 0xffff0000u);
  return o;
}

template <int D, bool FP8, bool PAGED, int NW, int NB>   // FP8: the cache rows are E4M3 bytes, turned into bf16 operands on the fly; NW waves of tiles of 16 NB rows
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NB > 1 ? 5 : 4, NB > 1 ? 5 : 4))) void decode_gqa_kernel(DecodeArgs a) {
  constexpr int GT = 8;                // query heads per KV head supported (columns 8..15 of the MFMA tile are padding)
  constexpr int TR = 16 * NB;          // rows of a wave's tile
  constexpr int KS = D / 32;           // MFMA steps over the head dimension
  constexpr int DB = D / 16;           // 16-column blocks of the output
  constexpr int RS = D + 16;           // bf16 elements per LDS row of the V tile (rows 8 banks apart: the transposing reads of a wave do not collide)
  constexpr int AR = D + 4;            // floats per query head of a wave's results
  constexpr int CB = FP8 ? 1 : 2;      // bytes per cache element
  constexpr int LPR = D * CB / 16;     // lanes per row in a coalesced 16-byte load
  constexpr int VE = 16 / CB;          // V elements per lane and load
  constexpr int RPI = 64 / LPR;        // rows per load instruction
  constexpr int VL = TR / RPI;         // load instructions per V tile
  constexpr int WB = TR * RS * 2 > GT * AR * 4 ? TR * RS * 2 : GT * AR * 4;        // bytes of a wave's V tile, later of its results
  __shared__ float s_ml[NW][GT][2];
  __shared__ __attribute__((aligned(16))) unsigned char s_wave[NW][WB];
  __shared__ __attribute__((aligned(16))) uint8_t s_new[FP8 ? 2 * D : 16];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j16 = lane & 15, c = lane >> 4;
  const long long hidx = piece_head(a);
  const int chunk = blockIdx.y;
  const int len1 = a.meet.len1[a.head0 + hidx], len_old = a.kv_len[hidx];
  const long long off = a.kv_off[hidx];
  // Q as the B operand: lane (q = j16, c) holds dims [32 ks + 8 c, +8) of query q (padding columns: the last query once more)
  dbf16x8_t qb[KS];
  const uint16_t* qg = reinterpret_cast<const uint16_t*>(a.q) + hidx * a.G * D + min(j16, a.G - 1) * D + c * 8;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qb[ks] = __builtin_bit_cast(dbf16x8_t, *reinterpret_cast<const du32x4_t*>(qg + ks * 32));
  asm volatile("" :: "s"(len1), "s"(len_old), "s"((int)off));             // (all three in one trip)
  const int arrive = arrivals(a, len1);
  if (chunk >= arrive) return;                       // the grid is the same for all heads (decode_plan)
  const bool can_append = can_append_to<PAGED>(a, off, len_old);
  const int len = len_old + (can_append ? 1 : 0);
  const int rows = head_chunk_rows(a, len);
  const int r_begin = chunk * rows;
  const int r_end = min(len, r_begin + rows);
  const RowMap at = make_row_map<PAGED>(a, hidx, off, len_old, can_append, r_begin, r_end);
  const bool has_fresh = can_append && len_old >= r_begin && len_old < r_end;   // uniform: the appended row is in this piece

  // the piece's first row (cache rows of D * CB bytes); the rows' offsets from it fit 32 bits
  unsigned char* kc = reinterpret_cast<unsigned char*>(a.k_c) + (PAGED ? 0 : (off + r_begin) * (D * CB));
  unsigned char* vc = reinterpret_cast<unsigned char*>(a.v_c) + (PAGED ? 0 : (off + r_begin) * (D * CB));
  const unsigned char* kn = reinterpret_cast<const unsigned char*>(a.k_new) + hidx * (D * 2);
  const unsigned char* vn = reinterpret_cast<const unsigned char*>(a.v_new) + hidx * (D * 2);
  const int vsub = lane / LPR, vpiece = lane % LPR;
  const auto row_at = [&](unsigned char* base, int r) { return PAGED ? base + at(r) * (D * CB) : base + (uint32_t)(r - r_begin) * (uint32_t)(D * CB); };

  // K fragments and V rows of a tile; rows past the end of the piece: its last row once more, masked where they are used.
  // The appended row comes from k_new and v_new (8-bit rows: from LDS, encoded).
  du32x4_t kraw[NB][KS], vraw[VL];         // raw cache bytes (E4M3: 8 bytes of a K piece sit in .xy)
  const auto load_tile = [&](int t) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int r = min(t + nb * 16 + j16, r_end - 1);
      const unsigned char* kp = row_at(kc, r);
      if (!FP8 && has_fresh && r == len_old) kp = kn;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (FP8) { const du32x2_t t2 = *reinterpret_cast<const du32x2_t*>(kp + ks * 32 + c * 8); kraw[nb][ks] = du32x4_t{t2[0], t2[1], 0u, 0u}; }
        else kraw[nb][ks] = *reinterpret_cast<const du32x4_t*>(kp + ks * 64 + c * 16);
      }
    }
#pragma unroll
    for (int i = 0; i < VL; ++i) {
      const int r = min(t + i * RPI + vsub, r_end - 1);
      const unsigned char* vp = row_at(vc, r);
      if (!FP8 && has_fresh && r == len_old) vp = vn;
      const du32x4_t* at16 = reinterpret_cast<const du32x4_t*>(vp + vpiece * 16);
      vraw[i] = NB > 1 ? __builtin_nontemporal_load(at16) : *at16;
    }
  };
  const int first = r_begin + wave * TR;
  if (first < r_end) load_tile(first);
  if constexpr (FP8) { if (has_fresh) stage_new_row<D>(a, hidx, at(len_old), s_new); }       // (behind the loads)

  float m_run = DNEG_BIG, l_run = 0.f;       // for query j16 (every lane group c holds a copy of m, a share of l)
  df32x4_t oacc[DB];                         // O^T[d = 16 db + 4c + r][q = j16]
  uint16_t* vt = reinterpret_cast<uint16_t*>(s_wave[wave]);
  const auto tile = [&](auto is_first, int t0) {
    constexpr bool FIRST = decltype(is_first)::value;
    if (!FIRST) load_tile(t0);
    if (has_fresh && t0 <= len_old && len_old < t0 + TR) {          // the appended row, the last of the piece
      if constexpr (FP8) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          if (t0 + nb * 16 + j16 >= len_old) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) { const du32x2_t t2 = *reinterpret_cast<const du32x2_t*>(s_new + ks * 32 + c * 8); kraw[nb][ks] = du32x4_t{t2[0], t2[1], 0u, 0u}; }
          }
#pragma unroll
        for (int i = 0; i < VL; ++i)
          if (t0 + i * RPI + vsub >= len_old) vraw[i] = *reinterpret_cast<const du32x4_t*>(s_new + D + vpiece * VE);
      } else {                                                      // on its way to the cache
        unsigned char* kp = row_at(kc, len_old);
        unsigned char* vp = row_at(vc, len_old);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          if (t0 + nb * 16 + j16 == len_old)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<du32x4_t*>(kp + ks * 64 + c * 16) = kraw[nb][ks];
#pragma unroll
        for (int i = 0; i < VL; ++i)
          if (t0 + i * RPI + vsub == len_old) *reinterpret_cast<du32x4_t*>(vp + vpiece * 16) = vraw[i];
      }
    }
    // ---- S^T of the tile's keys, 16 at a time
    float p[NB][4];
    float tmax = DNEG_BIG;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      df32x4_t sacc = df32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        du32x4_t kb = kraw[nb][ks];
        if (FP8) {
          const du32x2_t c0 = e4m3x4_to_bf16x4(kraw[nb][ks][0]), c1 = e4m3x4_to_bf16x4(kraw[nb][ks][1]);
          kb = du32x4_t{c0[0], c0[1], c1[0], c1[1]};
        }
        sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dbf16x8_t, kb), qb[ks], sacc, 0, 0, 0);
      }
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int key = t0 + nb * 16 + 4 * c + rr;           // in S^T the lane holds keys 4c..4c+3
        p[nb][rr] = key < r_end ? sacc[rr] * a.scale_log2 : DNEG_BIG;
        tmax = fmaxf(tmax, p[nb][rr]);
      }
    }
    // ---- V rows parked in the wave's LDS tile
#pragma unroll
    for (int i = 0; i < VL; ++i) {
      if (FP8) {                                             // 16 bytes -> 16 bf16
        const du32x2_t c0 = e4m3x4_to_bf16x4(vraw[i][0]), c1 = e4m3x4_to_bf16x4(vraw[i][1]);
        const du32x2_t c2 = e4m3x4_to_bf16x4(vraw[i][2]), c3 = e4m3x4_to_bf16x4(vraw[i][3]);
        const du32x4_t b0 = {c0[0], c0[1], c1[0], c1[1]}, b1 = {c2[0], c2[1], c3[0], c3[1]};
        *reinterpret_cast<du32x4_t*>(vt + (i * RPI + vsub) * RS + vpiece * 16) = b0;
        *reinterpret_cast<du32x4_t*>(vt + (i * RPI + vsub) * RS + vpiece * 16 + 8) = b1;
      } else {
        *reinterpret_cast<du32x4_t*>(vt + (i * RPI + vsub) * RS + vpiece * 8) = vraw[i];
      }
    }
    float lo_m, hi_m;
    lane_pair<16>(tmax, lo_m, hi_m); tmax = fmaxf(lo_m, hi_m);
    lane_pair<32>(tmax, lo_m, hi_m); tmax = fmaxf(lo_m, hi_m);
    const float m_new = FIRST ? tmax : fmaxf(m_run, tmax);
    float psum = 0.f;
    dbf16x8_t pb[NB];                                        // P as bf16 hi + lo of the lane's 4 keys: the B fragment
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      uint32_t hi[2], lo[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const df32x2_t pv = {weight_of(p[nb][2 * e] - m_new), weight_of(p[nb][2 * e + 1] - m_new)};
        psum += pv[0] + pv[1];
        hi[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pv, dbf16x2_t));          // round to nearest even
        const df32x2_t rest = {pv[0] - bf16_lo(hi[e]), pv[1] - bf16_hi(hi[e])};
        lo[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, dbf16x2_t));
      }
      pb[nb] = __builtin_bit_cast(dbf16x8_t, du32x4_t{hi[0], hi[1], lo[0], lo[1]});
    }
    if (FIRST) {
      l_run = psum;
    } else {
      const float alpha = weight_of(m_run - m_new);
      l_run = l_run * alpha + psum;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) oacc[db][rr] *= alpha;
    }
    m_run = m_new;
    // the V tile must be complete before it is read with another lane mapping (same wave: in order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // A fragment: for dim 16 db + j16 the 4 keys of this lane group, twice (against the hi and the lo parts).  A transposing
    // read takes, per 16 lanes, four rows of 16 columns: lane j points at columns 4 (j & 3).. of row j >> 2 and gets
    // column j of the four rows.
    const uint16_t* vf = vt + (4 * c + (j16 >> 2)) * RS + 4 * (j16 & 3);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const ds16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr_t)(vf + nb * 16 * RS + db * 16));
        const dbf16x8_t va = __builtin_bit_cast(dbf16x8_t, __builtin_shufflevector(v, v, 0, 1, 2, 3, 4, 5, 6, 7));
        oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb[nb], FIRST && nb == 0 ? df32x4_t{0.f, 0.f, 0.f, 0.f} : oacc[db], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (first < r_end) {
    tile(std::true_type{}, first);
#pragma unroll 1
    for (int t0 = first + NW * TR; t0 < r_end; t0 += NW * TR) tile(std::false_type{}, t0);
    float x, y;                                              // the sums of the lane groups
    lane_pair<16>(l_run, x, y); l_run = x + y;
    lane_pair<32>(l_run, x, y); l_run = x + y;
  } else {
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = df32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // ---- per wave: everything to LDS in [q][d] form, where its V tile was
  if (j16 < GT) {                                            // (the padding columns 8..15 have nothing to leave)
    if (c == 0) { s_ml[wave][j16][0] = m_run; s_ml[wave][j16][1] = l_run; }
    float* acc = reinterpret_cast<float*>(s_wave[wave]) + j16 * AR + 4 * c;
#pragma unroll
    for (int db = 0; db < DB; ++db) *reinterpret_cast<df32x4_t*>(acc + db * 16) = oacc[db];
  }
  __syncthreads();
  finish_piece<uint16_t, D, NW, GT, WB / 4, AR>(a, hidx, chunk, len, rows, can_append, arrive, s_ml, reinterpret_cast<const float*>(s_wave));
}

// Rows per workgroup: small for a single layer (many short workgroups balance ragged heads and
// keep every CU streaming), larger when thousands of heads already fill the chip.
static int plan_chunk_rows(const Dims& dm, const madakv_config& c) {
  // Measured on MI355X: 256-row chunks for a single layer's ragged heads at a 16K context
  // (smaller chunks lose to per-workgroup start-up cost, one workgroup per head to the imbalance
  // of ragged lengths), growing to 1024 rows when the heads are long (un-evicted cache), so that
  // the chip sees about eight workgroups per CU; 512 rows once a call covers >= 1024 heads.
  if (dm.heads >= 1024) return 512;
  const long long typical = std::min(c.budget, c.ctx_len) + c.max_new_tokens;    // rows of an average head
  const long long per = ((long long)dm.heads * typical + 2047) / 2048;
  const long long by_len = typical / 64;                     // a long head is not cut into more than ~64 chunks
  return (int)std::min<long long>(1024, std::max<long long>(256, std::max(per, by_len) / 256 * 256));
}
static int plan_longest(const madakv_config& c, int longest_rows) { return std::max(1, std::min(longest_rows, c.ctx_len + c.max_new_tokens)); }

// The pieces of a launch.  A head is cut into pieces of chunk_rows and at most max_chunks of them, hcc_rho times what an
// average head takes (a demand is clamped to that; at least twice; longer heads: longer pieces, see head_chunk_rows).  With twice
// whatever hcc_rho is, 128 heads of which 8 hold half of the rows, 512 on average, took 21.3 us instead of 14.7, 512 heads of 256,
// 16 with half of the rows, 34 instead of 21.  Neither depends on what the host knows of the
// longest head, so that a call's result does not either; only the grid, at most max_chunks pieces, shrinks when it is known.
constexpr int SHORT_PIECES = 2000;             // most 128-row pieces of a launch: what the static scratch holds of 8 queries x 128 dims
static_assert((size_t)SHORT_PIECES * 8 * (128 + 2) * sizeof(float) <= MADAKV_STATIC_SCRATCH_BYTES, "short pieces must fit the static scratch");
DecodePlan decode_plan(const Dims& dm, const madakv_config& c, int longest_rows) {
  DecodePlan p;
  const int worst = plan_longest(c, c.ctx_len + c.max_new_tokens);
  const int base = plan_chunk_rows(dm, c);
  p.chunk_rows = base;
  const long long typical = std::min(c.budget, c.ctx_len) + (long long)c.max_new_tokens;
  // A launch that does not fill the chip with it: pieces of 128 rows, one trip of all waves to memory each, where a piece of 256 is
  // two (grouped queries) to four trips one behind the other.
  // Grouped queries up to 64K rows in all.  (Twice as far: 2 heads of 40K rows 12.6 -> 16.1 us; four times: 32 heads of 4K rows
  // 11.5 -> 13.4: the pieces to merge.)
  // Single ones on up to 128 heads, up to 64K rows in all while a head has few pieces to merge, fewer with more of them.  Us per call
  // (device), 256-row pieces / these: 8 heads of 300 rows 6.9 / 6.3, of 2K 9.1 / 7.8, of 4K 10.0 / 9.7, 32 of 600 9.2 / 7.6, of 1.5K 10.8 / 10.4,
  // of 1.7K fp32 rows 16.9 / 15.4, 64 of 300 9.4 / 8.0, of 700 10.7 / 10.3, 96 of 600 11.9 / 11.9, 128 of 200 9.5 / 8.5, of 450 11.6 / 11.8
  // (paged, of 400 12.6 / 11.6).  Beyond: 8 heads of 6K 11.4 / 11.6, 16 of 3K 11.0 / 11.0, of 4K 12.4 / 13.0, 32 of 2K 11.9 / 12.4, 64 of 1K 12.0 / 12.3;
  // more heads fill the chip with 256-row pieces: 192 of 300 rows 11.9 / 12.5, 256 of 200 10.9 / 11.4, 512 of 130 12.0 / 14.0.  Rows of less
  // than 256 bytes, of which a piece of 256 takes no more trips, lose: 20 heads of 400 8-bit rows 5.1 / 5.3.  Heads of hardly more
  // than one such piece keep the longer ones, which they fill alone: 32 of 140 rows and room 5.8 / 6.4, of 150 6.5 / 6.6, of 175 7.1 / 6.7.
  const long long rows = dm.heads * typical;
  const int row_bytes = dm.d * (c.cache_fp8 ? 1 : c.dtype == MADAKV_BF16 ? 2 : 4);
  const long long most = typical <= 160 ? 0 : typical <= 1024 ? 65536 : typical <= 2048 ? 57344 : typical <= 4096 ? 32768 : 0;
  const bool short_pieces = dm.G >= 2 ? dm.heads <= 512 && c.dtype == MADAKV_BF16 && rows <= 65536
                                      : dm.heads <= 128 && row_bytes >= 256 && rows <= most;
  if (short_pieces) p.chunk_rows = 128;
  long long want = std::max<long long>((std::max(2, c.hcc_rho) * typical + p.chunk_rows - 1) / p.chunk_rows, 512 / dm.heads);
  if (short_pieces) want = std::min<long long>(want, SHORT_PIECES / dm.heads);
  // never more partial results than a worst-case head cut into `base` rows has: what decode_ws_bytes is made for
  p.max_chunks = (int)std::min<long long>((worst + base - 1) / base, std::max<long long>(2, want));
  p.grid_chunks = std::min(p.max_chunks, (plan_longest(c, longest_rows) + p.chunk_rows - 1) / p.chunk_rows);
  // every head is known to be one piece: nobody has to arrive anywhere
  if (p.grid_chunks == 1) p.max_chunks = 1;
  return p;
}

// The partial results of the heads' pieces, as many per head as the longest one has.  (decode_part_bytes: those of a launch, in
// pieces of its own size; never more than decode_ws_bytes_for of the same head, since max_chunks is not, but for short pieces of
// fewer rows than `base`, of which there are SHORT_PIECES.)
size_t decode_part_bytes(const Dims& dm, const madakv_config& c, int longest_rows) {
  const DecodePlan p = decode_plan(dm, c, longest_rows);
  return p.max_chunks == 1 ? 0 : (size_t)dm.heads * p.grid_chunks * dm.G * (dm.d + 2) * sizeof(float);
}
size_t decode_ws_bytes_for(const Dims& dm, const madakv_config& c, int longest_rows) {
  const int base = plan_chunk_rows(dm, c);
  const int chunks = (plan_longest(c, longest_rows) + base - 1) / base;
  return (size_t)dm.heads * chunks * dm.G * (dm.d + 2) * sizeof(float) + 64;
}
size_t decode_ws_bytes(const Dims& dm, const madakv_config& c) { return decode_ws_bytes_for(dm, c, c.ctx_len + c.max_new_tokens); }

template <typename T, typename CT, int LPR, bool PAGED>
static hipError_t launch_decode_t(const Dims& dm, DecodeArgs& a, int grid_chunks, hipStream_t st) {
  constexpr int D = LPR * 16 / (int)sizeof(CT);
  dim3 grid(dm.heads, grid_chunks), block(DEC_THREADS);
  // Four rows in flight per lane; eight where the pieces are long (a cache that was hardly reduced: 128 heads of 16K bf16 rows
  // 5.42 -> 5.17 ms for 32 layer calls, 6.6 TB/s): with many trips per workgroup the loads in flight count, with one or two its
  // start and its instructions.  512-row pieces are in between: 128 heads of 8K rows 92 us with four, 90 with eight, 4096 heads
  // of 256 75 and 70, but 1024 heads of 512 45.6 and 47.6.  8-bit rows, of which a lane has twice the elements, take four always:
  // 128 heads of 16K rows 89.3 us with either at 128 dims, 50.6 and 52.9 at 64 (64 heads of 32K: 92.8 and 90.4, 50.4 and 48.0).
  constexpr int LONG_ROWS = sizeof(CT) == 1 ? 4 : 8;
  if (sizeof(T) == 2 && dm.G >= 2) {                                 // grouped queries in bf16: the MFMA kernel
    if constexpr (D == 64) if (a.chunk_rows > 128 || dm.heads > 128) {
      hipLaunchKernelGGL((decode_gqa_kernel<D, sizeof(CT) == 1, PAGED, 4, 2>), grid, dim3(256), 0, st, a);
      return hipGetLastError();
    }
    hipLaunchKernelGGL((decode_gqa_kernel<D, sizeof(CT) == 1, PAGED, 8, 1>), grid, dim3(512), 0, st, a);
  }
  else if (LPR >= 16 && dm.G == 1 && a.chunk_rows == 128) {          // eight waves, a piece in one trip
    if constexpr (LPR >= 16) hipLaunchKernelGGL((decode_attn_kernel<T, CT, LPR, 1, LPR / 4, 8, PAGED>), grid, dim3(512), 0, st, a);
  }
  else if (dm.G == 1 && a.chunk_rows > 512) hipLaunchKernelGGL((decode_attn_kernel<T, CT, LPR, 1, LONG_ROWS, 4, PAGED>), grid, block, 0, st, a);
  else if (dm.G == 1) hipLaunchKernelGGL((decode_attn_kernel<T, CT, LPR, 1, 4, 4, PAGED>), grid, block, 0, st, a);
  else if constexpr (sizeof(T) == 4) {
    if (dm.G == 2) hipLaunchKernelGGL((decode_attn_kernel<T, CT, LPR, 2, 4, 4, PAGED>), grid, block, 0, st, a);
    else if (dm.G <= 4) hipLaunchKernelGGL((decode_attn_kernel<T, CT, LPR, 4, 4, 4, PAGED>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((decode_attn_kernel<T, CT, LPR, 8, 2, 4, PAGED>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}
template <typename T, typename CT, int LPR>
static hipError_t launch_decode_p(const Dims& dm, DecodeArgs& a, int grid_chunks, hipStream_t st) {
  return a.page_rows ? launch_decode_t<T, CT, LPR, true>(dm, a, grid_chunks, st) : launch_decode_t<T, CT, LPR, false>(dm, a, grid_chunks, st);
}

hipError_t launch_decode(const Dims& dm, const madakv_config& c, const void* q, const void* k_new,
                         const void* v_new, void* k_c, void* v_c, const int64_t* kv_off, int32_t* kv_len,
                         void* out, const Meet& meet, void* ws, long long capacity_tokens, int longest_rows, const Paging& pg, int layer0, hipStream_t st) {
  DecodeArgs a;
  a.capacity = capacity_tokens;
  a.page_rows = pg.page_rows; a.tbl_entries = pg.entries; a.page_tbl = pg.table; a.pool_top = pg.pool_top;
  a.page_shift = 0;
  while (pg.page_rows && (1 << a.page_shift) < pg.page_rows) ++a.page_shift;
  a.region_pages = pg.page_rows ? pg.region_tokens / pg.page_rows : 0;
  a.head0 = (long long)layer0 * dm.B * dm.H;
  a.q = q; a.k_new = k_new; a.v_new = v_new; a.k_c = k_c; a.v_c = v_c; a.kv_off = kv_off; a.kv_len = kv_len;
  a.out = out; a.meet = meet; a.max_new = c.max_new_tokens;
  DecodePlan p = decode_plan(dm, c, longest_rows);
  a.B = dm.B; a.H = dm.H; a.G = dm.G; a.chunk_rows = p.chunk_rows; a.max_chunks = p.max_chunks;
  a.slots = p.grid_chunks;
  a.by_heads = dm.heads > 1 && (long long)dm.heads * (dm.heads + p.grid_chunks) < (1ll << 32) ? (uint32_t)(((1ull << 32) + dm.heads - 1) / dm.heads) : 0u;
  a.by_chunk = plan_longest(c, c.ctx_len + c.max_new_tokens) + (long long)c.max_new_tokens + a.chunk_rows < (1 << 21) ? (uint32_t)(((1ull << 32) + a.chunk_rows - 1) / a.chunk_rows) : 0u;
  a.part = reinterpret_cast<float*>(ws); a.part_ml = a.part + (long long)dm.heads * a.slots * dm.G * dm.d;
  a.out_fp32 = c.out_fp32; a.has_new = (k_new != nullptr) ? 1 : 0;
  const float scale = c.softmax_scale > 0.f ? c.softmax_scale : 1.0f / sqrtf((float)dm.d);
  a.scale_log2 = scale * 1.4426950408889634f;
  const int lpr = dm.d * (c.dtype == MADAKV_BF16 ? 2 : 4) / 16;
  if (c.dtype == MADAKV_BF16) {
    if (c.cache_fp8) {                                   // rows of d bytes: d / 16 lanes per row
      if (dm.d == 128) return launch_decode_p<uint16_t, uint8_t, 8>(dm, a, p.grid_chunks, st);
      if (dm.d == 64) return launch_decode_p<uint16_t, uint8_t, 4>(dm, a, p.grid_chunks, st);
    }
    if (lpr == 8) return launch_decode_p<uint16_t, uint16_t, 8>(dm, a, p.grid_chunks, st);
    if (lpr == 16) return launch_decode_p<uint16_t, uint16_t, 16>(dm, a, p.grid_chunks, st);
  } else {
    if (lpr == 16) return launch_decode_p<float, float, 16>(dm, a, p.grid_chunks, st);
    if (lpr == 32) return launch_decode_p<float, float, 32>(dm, a, p.grid_chunks, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace madakv
