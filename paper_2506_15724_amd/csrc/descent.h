// Radix descent shared by the statistics (mass histograms) and the selection (count histograms): from the largest key
// down, the key at which a running total reaches a target, without sorting.  Every level histograms the keys still in
// range and walks the bins from the top to the one where the total crosses the target.
//
// The first level has 64 bins per factor of two over 2^-16 .. 2^8, where the scores that matter are (column sums of softmax
// rows), and 16 over 2^-48 .. 2^-16, where a head may have all scores of a modality that it hardly looks at; everything below
// is in the lowest bin and everything above in the highest.  About a hundredth of the keys is left after it, and few lanes of a
// wave meet in one bin (an LDS atomic serialises over the lanes that hit the same address; the 8 bins per octave of a plain
// 11-bit digit made that most of the level's time).  (With 64 bins per octave down to 2^-24 and none below, one head in thirty
// of an 8K prompt had half of its keys in the lowest bin, and the launch waited 12 us for it.)  Then 11 and 6 or 8 bits.  A
// crossing in one of the two open bins restarts with plain digits of 11, 11 and the remaining bits.
#pragma once
#include "common.h"

namespace madakv {

constexpr int BINS = 2048;               // bins of a level
constexpr int LAST_BINS = 1024;          // most bins of the last level
constexpr uint32_t FIRST_SH = 17;        // shift of the first level, and of its lower bins
constexpr uint32_t LOW_SH = 19;
constexpr uint32_t LOW_BINS = 512;       // they end at 2^-16, 111 << 23
constexpr uint32_t FIRST_SUB = (111u << (23 - FIRST_SH)) - LOW_BINS, LOW_SUB = (111u << (23 - LOW_SH)) - LOW_BINS;

// keys [lo, hi] are in range; bin = (key >> sh) - sub, clamped
struct DescentRange { uint32_t lo, hi, sh, sub; };

// the first level: every key is in range (sh = FIRST_SH stands for it; sub = the sign bit's share of a key >> FIRST_SH)
__device__ __forceinline__ DescentRange descent_first(uint32_t sign) { return {0u, 0xffffffffu, FIRST_SH, sign << (31 - FIRST_SH)}; }
__device__ __forceinline__ int descent_first_bin(uint32_t key, uint32_t sign) {          // above the boundary the first is the larger, below the second
  const int hi = (int)(key >> FIRST_SH) - (int)(FIRST_SUB + (sign << (31 - FIRST_SH))), lo = (int)(key >> LOW_SH) - (int)(LOW_SUB + (sign << (31 - LOW_SH)));
  return min(max(hi, lo), BINS - 1);                                                       // (<= 0: the lowest)
}
__device__ __forceinline__ DescentRange descent_none() { return {1u, 1u, 1u, 0u}; }   // (over: only a key of the smallest denormal is still in range, and nobody looks)
// the same in every lane: into scalar registers
__device__ __forceinline__ DescentRange descent_uniform(const DescentRange& r) {
  return {(uint32_t)__builtin_amdgcn_readfirstlane((int)r.lo), (uint32_t)__builtin_amdgcn_readfirstlane((int)r.hi),
          (uint32_t)__builtin_amdgcn_readfirstlane((int)r.sh), (uint32_t)__builtin_amdgcn_readfirstlane((int)r.sub)};
}
// The range after a crossing in bin b (at sh == 0 the descent is over: the key is sub + b).  SH1: shift of the plain first digit.
template <uint32_t SH1>
__device__ __forceinline__ DescentRange descent_next(const DescentRange& r, uint32_t b) {
  DescentRange n;
  if (r.sh == FIRST_SH) {
    const bool low = b < LOW_BINS;
    const uint32_t sh = low ? LOW_SH : FIRST_SH, t = low ? (LOW_SUB + (r.sub >> (LOW_SH - FIRST_SH)) + b) << LOW_SH : (FIRST_SUB + r.sub + b) << FIRST_SH;
    const uint32_t end = t + ((1u << sh) - 1u);
    if (b > 0 && b < BINS - 1) return {t, end, sh - 11u, t >> (sh - 11u)};
    n.lo = b ? t : 0u; n.hi = b ? 0xffffffffu : end; n.sh = SH1; n.sub = 0u;
    return n;
  }
  const uint32_t t = (r.sub + b) << r.sh;
  n.lo = max(r.lo, t); n.hi = min(r.hi, t + ((1u << r.sh) - 1u));
  n.sh = r.sh == SH1 ? SH1 - 11u : 0u;
  n.sub = t >> n.sh;
  return n;
}

template <typename T, int N>
__device__ __forceinline__ T pick(const T (&x)[N], int m) {              // x[m] without indexing registers by m
  T r = x[0];
#pragma unroll
  for (int j = 1; j < N; ++j) r = (m == j) ? x[j] : r;
  return r;
}

// Entries that a workgroup's list has per modality.  Some hundredths of a head's candidates fall into the crossing bin; where they
// do not fit, another pass over all of them is due: 2048 for two modalities (192 heads of 128K: statistics 92 us, selection 99,
// with 1024 entries 127 and 141; 112 of 32K and 224 proxy rows 29 and 32, with 1024 39 and 32; of 16K 22 and 23, with 1024 23 and 24).
// SMALL: 1024, in a call over several layer groups for heads of up to SMALL_HEADS candidates: the workgroup has to find room on
// a compute unit beside a gather (launch_gather).
template <int MM, bool SMALL> constexpr int LIST_MAX = MM == 2 && !SMALL ? 2048 : 1024;
constexpr int SMALL_HEADS = 16384;

// Few lanes of a wave find something for a list now and then: they leave it in a buffer of the wave's own, which needs no
// atomic and waits for nothing, and the buffer goes to the list once it holds a wave's worth (push per entry).  All lanes of
// the wave take part in every call.
constexpr int WAVE_BUF = 64 + 256;               // entries: a rest, and a group of four of every lane
constexpr int WAVE_BUF_SMALL = 64 + 64;          // a rest, and one of every lane
template <typename E>
struct WaveBuf {
  E* buf;                                        // this wave's
  uint32_t n;
  __device__ __forceinline__ void put(bool in, E x) {
    const unsigned long long who = __ballot(in);
    if (who) {
      const uint32_t at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
      if (in) buf[at] = x;
      n += (uint32_t)__popcll(who);
    }
  }
  template <typename F> __device__ __forceinline__ void flush(int lane, F push) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t e = (uint32_t)lane; e < n; e += 64u) push(buf[e]);
    n = 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};

// ---- the chunks of a head meet
// All waves of the workgroup; the last workgroup of `parts` to arrive gets true.  What the others stored before is where it can
// be read (agent-scope accesses).
__device__ __forceinline__ bool arrive_last(uint32_t* count, uint32_t parts, uint32_t* s_flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) *s_flag = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == parts ? 1u : 0u;
  __syncthreads();
  return *s_flag != 0u;
}
template <typename T> __device__ __forceinline__ T agent_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ void agent_store(T* p, T x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// vectors of floats that are only 4-byte aligned (a head's scores start anywhere): one 16-byte access all the same
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any_t;
__device__ __forceinline__ uint32_t load_mask4(const uint8_t* p) { uint32_t w; __builtin_memcpy(&w, p, 4); return w; }
// modality ids of four candidates from their bytes, ids above `top` counting as top (two modalities: any other byte than 0 is 1)
template <int MM>
__device__ __forceinline__ uint32_t mask4_ids(uint32_t w, uint32_t top) {
  if (MM == 2) return (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u;
  return min(w & 0xffu, top) | (min((w >> 8) & 0xffu, top) << 8) | (min((w >> 16) & 0xffu, top) << 16) | (min(w >> 24, top) << 24);
}
template <int MM>
__device__ __forceinline__ uint32_t id_of(uint32_t ids, int q) { return MM == 2 ? (ids >> (8 * q + 7)) & 1u : (ids >> (8 * q)) & 0xffu; }

}  // namespace madakv
