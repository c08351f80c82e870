// Radix descent shared by the statistics (mass histograms) and the selection (count histograms): from the largest key
// down, the key at which a running total reaches a target, without sorting.  Every level histograms the keys still in
// range and walks the bins from the top to the one where the total crosses the target.
//
// The first level has 64 bins per factor of two over 2^-24 .. 2^8, where the scores are (column sums of softmax rows),
// with everything below in its lowest bin and everything above in its highest: about a hundredth of the keys is
// left after it, and few lanes of a wave meet in one bin (an LDS atomic serialises over the lanes that hit the same
// address; the 8 bins per octave of a plain 11-bit digit made that most of the level's time).  Then 11 and 6 bits.  A
// crossing in one of the two open bins restarts with plain digits of 11, 11 and the remaining bits.
#pragma once
#include "common.h"

namespace madakv {

constexpr int BINS = 2048;               // bins of a level
constexpr int LAST_BINS = 1024;          // most bins of the last level
constexpr uint32_t FIRST_SH = 17;        // shift of the first level
constexpr uint32_t FIRST_SUB = 6599;     // bits of 2^-24 (about) >> 17: (FIRST_SUB + 1) << 17 is a multiple of 2^20

// keys [lo, hi] are in range; bin = (key >> sh) - sub, clamped
struct DescentRange { uint32_t lo, hi, sh, sub; };

__device__ __forceinline__ DescentRange descent_first(uint32_t sign) { return {0u, 0xffffffffu, FIRST_SH, FIRST_SUB + (sign << (31 - FIRST_SH))}; }
template <uint32_t SH1> __device__ __forceinline__ DescentRange descent_plain() { return {0u, 0xffffffffu, SH1, 0u}; }
__device__ __forceinline__ DescentRange descent_none() { return {1u, 1u, 1u, 0u}; }   // (over: only a key of the smallest denormal is still in range, and nobody looks)
// the same in every lane: into scalar registers
__device__ __forceinline__ DescentRange descent_uniform(const DescentRange& r) {
  return {(uint32_t)__builtin_amdgcn_readfirstlane((int)r.lo), (uint32_t)__builtin_amdgcn_readfirstlane((int)r.hi),
          (uint32_t)__builtin_amdgcn_readfirstlane((int)r.sh), (uint32_t)__builtin_amdgcn_readfirstlane((int)r.sub)};
}
__device__ __forceinline__ uint32_t descent_bin(const DescentRange& r, uint32_t key) {
  return (uint32_t)min(max((int)((key >> r.sh) - r.sub), 0), BINS - 1);
}
// The range after a crossing in bin b (at sh == 0 the descent is over: the key is sub + b).  SH1: shift of the plain first digit.
template <uint32_t SH1>
__device__ __forceinline__ DescentRange descent_next(const DescentRange& r, uint32_t b) {
  DescentRange n;
  if (r.sh == FIRST_SH) {
    const uint32_t t = (r.sub + b) << FIRST_SH;
    if (b > 0 && b < BINS - 1) return {t, t + ((1u << FIRST_SH) - 1u), 6u, t >> 6};
    n.lo = b ? t : 0u; n.hi = b ? 0xffffffffu : t + ((1u << FIRST_SH) - 1u); n.sh = SH1; n.sub = 0u;
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
