// Proxy-token scores (paper Sec. 3.3 Eq. 7): psi[i] = sum over the G*W proxy rows of the
// causal softmax(scale * q k^T) they pay to key i.
//
// The softmax normaliser of a row needs the whole row, the column sum needs the
// normalisers, so the scores are produced in two sweeps over K:
//   sweep 1  per row: running max and sum of exp2 (log2 domain), per L-chunk
//   sweep 2  recompute the logits, p = exp2(s - (m + log2 l)), sum p over the rows
// Both sweeps are the same small-M contraction S^T = Q K^T (M = G*W rows, N = keys).
// Where a workgroup's logits fit in its registers one sweep does both (score_fused_kernel: bf16 up to 64 proxy rows, fp32 up
// to 32768 keys); more bf16 rows, longer heads and given normalisers take the two.
// bf16 inputs run on the 32x32x16 bf16 MFMA with fp32 accumulation, fp32 inputs on the 32x32x2 fp32 MFMA (a plain FMA kernel
// above 32768 keys and for given normalisers).  All reductions have a fixed
// order: psi feeds integer decisions downstream and must not change from run to run.
#include "common.h"

#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace madakv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) int i32x4_t;

constexpr float NEG_BIG = -1.0e30f;
constexpr int SCORE_THREADS = 256;
// types the keys of the one-sweep kernel come in: bf16, E4M3 bytes (rows of d bytes: the 8-bit reduced cache; the queries
// are bf16 then), fp32 (the queries too)
constexpr int K_BF16 = 0, K_E4M3 = 1, K_F32 = 2;

struct ScoreArgs {
  const void* q_win;   // [heads/H * Hq, W, d]
  const void* k;       // [heads, L, d]
  float* psi;          // [heads, L]
  float* rowstat;      // [heads, nsplit, mpad, 2]
  const float* lse;    // optional [heads/H * Hq, W]: natural log-sum-exp of each proxy row's scaled logits (sweep 1 not needed)
  float* sink;         // 32 floats nobody reads: keeps the psi store of sweep 2 unconditional (both half-waves
                       // store the same value; a store under a branch makes the load waits pessimistic)
  int H, G, d, L, W, M, mpad, nsplit, chunk;
  int nmerge;          // chunks whose row statistics sweep 2 still has to merge (1 after score_combine_kernel)
  // one-sweep kernel: row statistics of the head's chunks as (max, sum) pairs in one 64-bit word each,
  // [heads, fsplit, mpad], all ones = not yet there; status[0] != 0 = a workgroup gave up waiting.  (In the handle; those of
  // ragged heads in the workspace.)
  unsigned long long* xchg;
  int subtiles = 0;             // (host) of a wave, fp32
  bool xchg_clean = false;      // (host) its words are XCHG_EMPTY already
  int k_kind;             // type of the keys of the one-sweep kernel: K_BF16, K_E4M3 or K_F32
  int xgroups;            // 0: every workgroup reads every chunk's words; else the number of groups of XCHG_GROUP chunks (two levels)
  long long xstride;      // exchange words per head: (fsplit + xgroups) * mpad
  int* status;         // status[0]: workgroups of one-sweep launches that gave up waiting so far (diagnostic counter,
                       // the first word of the workspace; never cleared here)
  int fsplit;          // chunks per head of the one-sweep kernel
  const int64_t* seg_off;   // one-sweep kernel on ragged heads (null: every head has L keys at head * L): first row and
  const int32_t* seg_len;   // number of rows of each head in k; psi is indexed the same way
  // one-sweep kernel with more than 64 proxy rows: the rows are cut into rb_count blocks of 64, each handled
  // like a head of its own (grid.y = heads * rb_count); their column sums go to psi_part [rb][heads][L stride]
  // and are added in block order afterwards
  int rb_count;
  float* psi_part;
  long long psi_part_stride;   // floats between two row blocks' copies
  int spin_limit;      // polls a workgroup of the one-sweep kernel spends on one missing word before it goes its own way
  // one-sweep kernel on long heads whose chunks do not pack the chip's workgroup slots (see launch_fused): the last
  // nstrag chunks of every head come first in the grid (x < nstrag), leave their row statistics as exchange words
  // of the group level and their logits in `park`, and do not wait; the other chunks' workgroups leave the heads'
  // row offsets in offs_out, a small kernel finishes the parked chunks
  int nstrag = 0;
  float* park = nullptr;
  float* offs_out = nullptr;
  int head0;           // first head of this launch (grid.y indexes head0 + y)
  float scale_log2;    // softmax scale * log2(e)
};

__device__ __forceinline__ void merge_ml(float& m, float& l, float m2, float l2) {
  float mn = fmaxf(m, m2);
  l = l * exp2f(m - mn) + l2 * exp2f(m2 - mn);
  m = mn;
}

// ------------------------------------------------------------------------------------
// bf16 MFMA path.  One workgroup = 4 waves works on one (head, L-chunk); a wave streams
// 32-key subtiles of K:
//   D[i = proxy row][j = key] = sum_k A[i][k] * B[k][j],  A = 32-row block of Q, B = K subtile^T.
// HBM side: a subtile (32 rows of 256 B) is fetched with fully coalesced 16-byte loads (16
// lanes cover one row), PF subtiles ahead of the arithmetic, into registers.  That is
// what hides the HBM latency: a subtile's arithmetic takes a fraction of a microsecond.
// MFMA side: an operand lane needs the whole row of "its" key, a layout that would touch 64
// different cache lines per load instruction if read from global memory directly; so the
// subtile is parked in a wave-private LDS tile (rows padded by 16 bytes: the 128-bit reads of
// 32 different rows fall into different banks) and the B fragments are read from there.  The
// tile is private to the wave: no workgroup barrier in the loop, LDS operations of one wave
// execute in order.
// In D a lane holds one key column and 16 rows: the column sum is in-lane, the row
// statistics need one cross-lane merge at the end of the chunk.
// Every wave has its own keys and all (at most two) row blocks; more than 64 proxy rows take the
// kernels further down, whose waves share the keys and own row blocks.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }   // x <= ~0 here; tiny results may flush to 0

template <int OP>   // 0 = max, 1 = sum over the 32 lanes of a half-wave; every lane gets the result
__device__ __forceinline__ float half_reduce(float x) {
#define MADAKV_DPP(ctrl) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), ctrl, 0xF, 0xF, true))
  float y;
  y = MADAKV_DPP(0xB1);  x = OP ? x + y : fmaxf(x, y);     // quad_perm [1,0,3,2]
  y = MADAKV_DPP(0x4E);  x = OP ? x + y : fmaxf(x, y);     // quad_perm [2,3,0,1]
  y = MADAKV_DPP(0x141); x = OP ? x + y : fmaxf(x, y);     // row_half_mirror
  y = MADAKV_DPP(0x140); x = OP ? x + y : fmaxf(x, y);     // row_mirror
#undef MADAKV_DPP
  y = __shfl_xor(x, 16, 64); x = OP ? x + y : fmaxf(x, y); // the two 16-lane rows of the half
  return x;
}

// The same, in the same order, of 16 values: at each step a lane goes on with half of its values and takes what its
// partner had of them; lane i of a half-wave gets the result of x[i & 15].  (Half the instructions of 16 single
// reductions, one wide store instead of 16.)
template <int OP>   // 0 = max, 1 = sum
__device__ __forceinline__ float half_fold(const float (&x)[16], int lane) {
#define MADAKV_DPP(v, ctrl) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xF, 0xF, true))
  const auto both = [](float x, float y) { return OP ? x + y : fmaxf(x, y); };
  float a[8], b[4], c[2];
#pragma unroll
  for (int k = 0; k < 8; ++k) { const bool o = lane & 1; const float keep = o ? x[2 * k + 1] : x[2 * k], give = o ? x[2 * k] : x[2 * k + 1]; a[k] = both(keep, MADAKV_DPP(give, 0xB1)); }   // lane ^ 1
#pragma unroll
  for (int k = 0; k < 4; ++k) { const bool o = lane & 2; const float keep = o ? a[2 * k + 1] : a[2 * k], give = o ? a[2 * k] : a[2 * k + 1]; b[k] = both(keep, MADAKV_DPP(give, 0x4E)); }   // lane ^ 2
#pragma unroll
  for (int k = 0; k < 2; ++k) {                                                     // lane ^ 4: mirrored in 8, then in 4
    const bool o = lane & 4;
    const float keep = o ? b[2 * k + 1] : b[2 * k], give = o ? b[2 * k] : b[2 * k + 1];
    const float m = MADAKV_DPP(give, 0x141);
    c[k] = both(keep, MADAKV_DPP(m, 0x1B));
  }
  const bool o = lane & 8;
  const float keep = o ? c[1] : c[0], give = o ? c[0] : c[1];
  const float d = both(keep, MADAKV_DPP(give, 0x128));                                   // lane ^ 8: rotated by 8 in 16
#undef MADAKV_DPP
  return both(d, __shfl_xor(d, 16, 64));                                                 // the two 16-lane rows of the half
}

template <int D, int NRB, int PASS>
__global__ __launch_bounds__(SCORE_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void score_mfma_kernel(ScoreArgs a) {
  constexpr int KS = D / 16;                  // MFMA k-steps
  constexpr int RS = D + 8;                   // bf16 elements per LDS row (16 B pad)
  constexpr int KG = 4;                       // key groups: the waves
  constexpr int PPR = D / 8;                  // 16-byte pieces per row
  constexpr int LPS = 32 * PPR / 64;          // 16-byte loads per lane per subtile
  constexpr int PF = 2;                       // subtiles in flight per wave
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* qs = reinterpret_cast<uint16_t*>(smem);                       // [mpad][RS]
  uint16_t* kt_all = qs + (size_t)a.mpad * RS;                            // [4 waves][32][RS]
  float* fbuf = reinterpret_cast<float*>(kt_all + 4 * 32 * RS);           // pass 1: [KG][mpad][2]; pass 2: off[mpad]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = blockIdx.x;
  const int head = a.head0 + blockIdx.y;
  const int kvh = head % a.H;
  const long long lb = head / a.H;            // (layer, batch) index
  const uint16_t* qg = reinterpret_cast<const uint16_t*>(a.q_win) + (lb * a.H + kvh) * (long long)a.G * a.W * D;
  const uint16_t* kg = reinterpret_cast<const uint16_t*>(a.k) + (long long)head * a.L * D;
  const int chunk0 = split * a.chunk;
  const int chunk1 = min(a.L, chunk0 + a.chunk);
  const int nsub = (chunk1 - chunk0 + 31) / 32;
  const int niter = (nsub + KG - 1) / KG;
  const int kgid = wave;                      // subtiles of this wave: kgid, kgid + KG, ...
  uint16_t* kt = kt_all + (size_t)wave * 32 * RS;

  // PF subtiles of K on their way before anything else
  u32x4_t pre0[LPS], pre1[LPS];                // two register sets = PF subtiles in flight
  static_assert(PF == 2, "the loop body below is written out for two register sets");
#define MADAKV_LOAD_SUB(DST, IT)                                                                 \
  {                                                                                              \
    const int lt0 = chunk0 + ((IT) * KG + kgid) * 32;                                            \
    _Pragma("unroll") for (int i = 0; i < LPS; ++i) {                                            \
      const int idx = i * 64 + lane;                                                             \
      const int lkey = min(lt0 + idx / PPR, a.L - 1); /* past the end: a valid row, masked later */ \
      DST[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(kg + (long long)lkey * D + (idx % PPR) * 8)); \
    }                                                                                            \
  }
  MADAKV_LOAD_SUB(pre0, 0)
  MADAKV_LOAD_SUB(pre1, 1)

  // stage Q (the G*W rows of this KV head are contiguous), zero the padding rows
  for (int e = tid; e < a.mpad * PPR; e += SCORE_THREADS) {
    const int r = e / PPR, c = e % PPR;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (r < a.M) val = *reinterpret_cast<const uint4*>(qg + (long long)r * D + c * 8);
    *reinterpret_cast<uint4*>(qs + r * RS + c * 8) = val;
  }
  float* offs = fbuf;                          // pass 2 only
  if (PASS == 2) {
    const float* rs = a.rowstat + (long long)head * a.nsplit * a.mpad * 2;
    for (int r = tid; r < a.mpad; r += SCORE_THREADS) {
      float m = NEG_BIG, l = 0.f;
      if (a.lse) {                                               // the caller's prefill attention already has the row normalisers
        if (r < a.M) { m = a.lse[(lb * a.H + kvh) * (long long)a.G * a.W + r] * 1.4426950408889634f; l = 1.f; }
      } else {
        for (int s = 0; s < a.nmerge; ++s) merge_ml(m, l, rs[(s * a.mpad + r) * 2], rs[(s * a.mpad + r) * 2 + 1]);
      }
      offs[r] = (r < a.M) ? m + log2f(l) : __builtin_inff();     // padding rows contribute exp2(-inf) = 0
    }
  }
  __syncthreads();

  const int half = lane >> 5, col = lane & 31;
  const int first_masked = a.L - a.W + 1;      // keys below this are visible to every proxy row

  float st_m[NRB][16], st_l[NRB][16], off_r[NRB][16];
#pragma unroll
  for (int b = 0; b < NRB; ++b)
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      st_m[b][j] = NEG_BIG; st_l[b][j] = 0.f;
      const int row = min(b * 32 + (j >> 2) * 8 + half * 4 + (j & 3), a.mpad - 1);
      off_r[b][j] = (PASS == 2) ? offs[row] : 0.f;
    }
  // with a single row block per wave the Q fragments stay in registers (no LDS reads in the loop)
  bf16x8_t areg[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    areg[ks] = *reinterpret_cast<const bf16x8_t*>(qs + col * RS + half * (D / 2) + ks * 8);
  const int MB = a.mpad / 32;

  // one subtile per step: registers -> LDS tile -> MFMA -> statistics / column sums.
  // (Written as a macro applied to each register set: the sets must stay in registers, and
  // any indirection over them makes the compiler park them in scratch memory.)
#define MADAKV_STEP(SRC, IT)  {  const int it = (IT);  { \
_Pragma("unroll") \
    for (int i = 0; i < LPS; ++i) { \
      const int idx = i * 64 + lane; \
      *reinterpret_cast<u32x4_t*>(kt + (idx / PPR) * RS + (idx % PPR) * 8) = SRC[i]; \
    } \
    MADAKV_LOAD_SUB(SRC, it + PF) \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); \
    __builtin_amdgcn_wave_barrier(); \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); \
    const int t0 = chunk0 + (it * KG + kgid) * 32; \
    const int key = t0 + col; \
    const bool tail = (t0 + 32 > first_masked) || (t0 + 32 > chunk1); \
    const uint16_t* krow = kt + col * RS + half * (D / 2); \
    bf16x8_t bfrag[KS]; \
_Pragma("unroll") \
    for (int ks = 0; ks < KS; ++ks) bfrag[ks] = *reinterpret_cast<const bf16x8_t*>(krow + ks * 8); \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); \
    __builtin_amdgcn_wave_barrier(); \
    float colsum = 0.f; \
_Pragma("unroll") \
    for (int b = 0; b < NRB; ++b) { \
      const int rb = b; \
      if (rb < MB) { \
        f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; \
        const uint16_t* qrow = qs + (rb * 32 + col) * RS + half * (D / 2); \
_Pragma("unroll") \
        for (int ks = 0; ks < KS; ++ks) { \
          const bf16x8_t afrag = (NRB == 1) ? areg[ks] : *reinterpret_cast<const bf16x8_t*>(qrow + ks * 8); \
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, bfrag[ks], acc, 0, 0, 0); \
        } \
        if (!tail) { \
_Pragma("unroll") \
          for (int j = 0; j < 16; ++j) { \
            const float s2 = acc[j] * a.scale_log2; \
            if (PASS == 1) { \
              const float dlt = s2 - st_m[b][j]; \
              const float e = fast_exp2(-fabsf(dlt)); \
              st_l[b][j] = dlt > 0.f ? fmaf(st_l[b][j], e, 1.0f) : st_l[b][j] + e; \
              st_m[b][j] = fmaxf(st_m[b][j], s2); \
            } else { \
              colsum += fast_exp2(s2 - off_r[b][j]); \
            } \
          } \
        } else { \
_Pragma("unroll") \
          for (int j = 0; j < 16; ++j) { \
            const float s2 = acc[j] * a.scale_log2; \
            const int row = rb * 32 + (j >> 2) * 8 + half * 4 + (j & 3); \
            const int pos = a.L - a.W + (row % a.W); \
            const bool valid = (key < chunk1) && (key <= pos) && (row < a.M); \
            if (PASS == 1) { \
              const float dlt = s2 - st_m[b][j]; \
              const float e = fast_exp2(-fabsf(dlt)); \
              const float nl = dlt > 0.f ? fmaf(st_l[b][j], e, 1.0f) : st_l[b][j] + e; \
              st_l[b][j] = valid ? nl : st_l[b][j]; \
              st_m[b][j] = valid ? fmaxf(st_m[b][j], s2) : st_m[b][j]; \
            } else { \
              const float pr = fast_exp2(s2 - off_r[b][j]); \
              colsum += valid ? pr : 0.f; \
            } \
          } \
        } \
      } \
    } \
    if (PASS == 2) { \
      colsum += __shfl_xor(colsum, 32, 64); \
      { float* dst = (key < chunk1) ? a.psi + ((long long)head * a.L + key) : a.sink + col; __builtin_nontemporal_store(colsum, dst); } \
    } \
  } }
  // Four unconditional steps per trip; the step count is rounded up (a step past the end works on
  // clamped rows and is fully masked).  A step under a condition would leave the compiler unsure how
  // many loads are in flight after it, and it would then wait for all of them at every step.
  const int niter4 = (niter + 2 * PF - 1) / (2 * PF) * (2 * PF);
  for (int it0 = 0; it0 < niter4; it0 += 2 * PF) {
    MADAKV_STEP(pre0, it0)
    MADAKV_STEP(pre1, it0 + 1)
    MADAKV_STEP(pre0, it0 + 2)
    MADAKV_STEP(pre1, it0 + 3)
  }
#undef MADAKV_STEP
#undef MADAKV_LOAD_SUB

  if (PASS == 1) {
    // per row: maximum over the 32 key columns of the half, sums rescaled to it and added;
    // then the key groups meet in LDS
    float* part = fbuf;                        // [KG][mpad][2]
#pragma unroll
    for (int b = 0; b < NRB; ++b) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float m = half_reduce<0>(st_m[b][j]);
        const float l = half_reduce<1>(st_l[b][j] * fast_exp2(st_m[b][j] - m));
        const int rb = b;
        if (rb < MB && col == 0) {
          const int row = rb * 32 + (j >> 2) * 8 + half * 4 + (j & 3);
          part[(kgid * a.mpad + row) * 2] = m;
          part[(kgid * a.mpad + row) * 2 + 1] = l;
        }
      }
    }
    __syncthreads();
    float* rs = a.rowstat + ((long long)head * a.nsplit + split) * a.mpad * 2;
    for (int r = tid; r < a.mpad; r += SCORE_THREADS) {
      float m = NEG_BIG, l = 0.f;
      for (int g = 0; g < KG; ++g) merge_ml(m, l, part[(g * a.mpad + r) * 2], part[(g * a.mpad + r) * 2 + 1]);
      rs[r * 2] = m; rs[r * 2 + 1] = l;
    }
  }
}

// ------------------------------------------------------------------------------------
// More than 64 proxy rows (grouped queries: G*W up to 256), the same two sweeps.  The arithmetic per
// key grows with the rows and is what bounds these kernels (one exp2 per logit and sweep on the vector
// unit; the contraction is a fraction of that), so the layout serves the vector unit: a wave owns
// one or two blocks of 32 proxy rows for all keys of the workgroup's chunk and keeps their Q
// fragments in registers; the waves share the keys.  Sweep 1 needs no merge among the waves (a row's
// statistics over the chunk are complete in its wave) and multiplies the other way round, S^T = K Q^T:
// a lane then holds one row against 16 keys, the running (max, sum) of a row is one register pair and
// in-lane work.  Sweep 2 (S = Q K^T: a lane holds one key against 16 rows, the column sum is in-lane)
// adds the waves' partial column sums through LDS, in wave order, one tile behind the arithmetic.
// The keys are fetched straight into LDS (global_load_lds, 16 bytes per lane): no register holds a
// key on its way, so three tiles form a ring with two tiles in flight while the third is multiplied.
// A wave's load instruction fills 1 KB of consecutive LDS (lane i at base + 16 i), so rows cannot be
// padded; instead the 16-byte pieces of a row are stored permuted, piece c of row r at slot
// c ^ (r mod pieces per row): the lane that writes slot s of row r fetches piece s ^ (r mod ...) from
// memory (a row's pieces are still one contiguous stretch per 16 lanes), and the operand reads of 16
// lanes with consecutive rows fall into 16 different slots.
// The compiler cannot tell which LDS bytes such a load writes and would wait for ALL outstanding loads
// before every LDS access it sees; so inside the loop every LDS access and every wait is written out:
// loads are counted (they complete in order), "tile t is there" is s_waitcnt vmcnt(loads of one tile),
// and the barrier that follows also tells that everybody is done with the tile the next load overwrites.
// ------------------------------------------------------------------------------------
constexpr int DMA_NBUF = 3;
#ifndef MADAKV_P1_WPE
#define MADAKV_P1_WPE 3      // waves per SIMD of sweep 1 (its registers allow three)
#endif

typedef __attribute__((address_space(3))) void* lds_void_ptr_t;
typedef const __attribute__((address_space(1))) void* global_void_ptr_t;

// NW waves of NRB row blocks each; tiles of DMA_TK keys; the vector arithmetic runs on BS subtiles at a time.
// CLOSE (sweep 1 for the last-window attention, whose entries get their final value from these statistics): a row's sum is
// rescaled by the difference of the maxima as rounded, and the terms of a subtile are added among themselves first;
// log-sum-exp within 5e-6 instead of 1e-5, at the same speed.
template <int D, int NW, int NRB, int DMA_TK, int BS, int PASS, bool CLOSE = false>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(PASS == 1 ? MADAKV_P1_WPE : 2, PASS == 1 ? MADAKV_P1_WPE : 2))) void score_wide_dma_kernel(ScoreArgs a) {
  constexpr int NT = NW * 64;
  constexpr int KS = D / 16;                  // MFMA k-steps
  constexpr int PPR = D / 8;                  // 16-byte pieces per row
  constexpr int ROWB = D * 2;                 // bytes per row
  constexpr int LPT = DMA_TK * PPR / NT;              // load instructions per thread and tile (each fills 1 KB per wave)
  constexpr int NSUB = DMA_TK / 32;
  constexpr int TILEB = DMA_TK * ROWB;
  static_assert((LPT == 4 || LPT == 2 || LPT == 1) && NSUB % BS == 0 && (PASS == 1 || DMA_TK == 64), "the waits below are written for these");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* ring = smem;                                              // [DMA_NBUF][DMA_TK][ROWB], pieces permuted
  float* offs = reinterpret_cast<float*>(smem + DMA_NBUF * TILEB);         // sweep 2: [mpad]
  float* red = offs + a.mpad;                                              // sweep 2: [2][NW][DMA_TK]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = blockIdx.x;
  const int head = a.head0 + blockIdx.y;
  const int kvh = head % a.H;
  const long long lb = head / a.H;            // (layer, batch) index
  const uint16_t* qg = reinterpret_cast<const uint16_t*>(a.q_win) + (lb * a.H + kvh) * (long long)a.G * a.W * D;
  const unsigned char* kg = reinterpret_cast<const unsigned char*>(a.k) + (long long)head * a.L * ROWB;
  const int chunk0 = split * a.chunk;
  const int chunk1 = min(a.L, chunk0 + a.chunk);
  const int ntiles = (chunk1 - chunk0 + DMA_TK - 1) / DMA_TK;
  const int half = lane >> 5, col = lane & 31;
  const int MB = a.mpad / 32;
  // Row blocks of this wave: `role` and, with two per wave, role + NW.  Where the rows leave the second of some waves empty (160
  // rows: five blocks for four waves) it is left out, and the roles go round from workgroup to workgroup: wave w of all
  // workgroups of a compute unit is on the same SIMD, and the light ones would help only that.  (Score and
  // statistics calls over 32K keys: 64 heads of 160 rows 341 -> 305 us, 56 of 192 rows 343 -> 332, 112 of 224 rows 628 -> 608; a branch
  // per block instead of two pieces of code is 5% slower than that.)
  const int role = NRB == 1 ? wave : __builtin_amdgcn_readfirstlane((wave + (int)(blockIdx.x + blockIdx.y)) % NW);
  const bool second = NRB == 2 && (role + NW) * 32 < a.M;
  const int first_masked = a.L - a.W + 1;      // keys below this are visible to every proxy row

  // sweep 2: the rows' offsets (ordinary LDS traffic, so before the first key is on its way)
  // sweep 2: st_m holds the offsets of the 16 rows a lane has of each block.  Sweep 1 runs the contraction the
  // other way round (S^T = K Q^T: a lane holds ONE row and 16 keys of a subtile), so its running (max in
  // accumulator units, sum) is one pair per lane and block: row_m, row_l.
  float st_m[PASS == 2 ? NRB : 1][16];
  float row_m[NRB], row_ms[NRB], row_l[NRB];    // (row_ms: the maximum in logit units, as rounded)
  if (PASS == 2) {
    const float* rs = a.rowstat + (long long)head * a.nsplit * a.mpad * 2;
    for (int r = tid; r < a.mpad; r += NT) {
      float m = NEG_BIG, l = 0.f;
      if (a.lse) {                                               // the caller's prefill attention already has the row normalisers
        if (r < a.M) { m = a.lse[(lb * a.H + kvh) * (long long)a.G * a.W + r] * 1.4426950408889634f; l = 1.f; }
      } else {
        for (int s = 0; s < a.nmerge; ++s) merge_ml(m, l, rs[(s * a.mpad + r) * 2], rs[(s * a.mpad + r) * 2 + 1]);
      }
      offs[r] = (r < a.M) ? m + log2f(l) : __builtin_inff();     // padding rows contribute exp2(-inf) = 0
    }
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < NRB; ++b)
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int row = (role + b * NW) * 32 + (j >> 2) * 8 + half * 4 + (j & 3);     // (a block past the last: rows that count for nothing)
      if (PASS == 2) st_m[b][j] = row < a.mpad ? offs[row] : __builtin_inff();
    }
#pragma unroll
  for (int b = 0; b < NRB; ++b) { row_m[b] = NEG_BIG; row_ms[b] = 0.f; row_l[b] = 0.f; }
  __syncthreads();                             // (the last ordinary LDS access of the kernel)

  // tile T of the chunk -> ring slot T mod 3.  Load j of wave w fills bytes [(w LPT + j) 1024, + 1024) of the slot:
  // lane i writes piece P = (w LPT + j) 64 + i, i.e. slot P mod PPR of row P / PPR, and fetches that row's piece
  // (P mod PPR) ^ (row mod PPR).  Rows past the head's end: its last row (masked where it is used).
  const uint32_t ring_lds = (uint32_t)(uintptr_t)ring;
#define MADAKV_DMA_ISSUE(T)                                                                          \
  {                                                                                                  \
    const int tt = (T);                                                                              \
    const int lt0 = chunk0 + tt * DMA_TK;                                                            \
    const uint32_t slot_lds = ring_lds + (uint32_t)(tt % DMA_NBUF) * TILEB;                          \
    _Pragma("unroll") for (int j = 0; j < LPT; ++j) {                                                \
      const int piece = (wave * LPT + j) * 64 + lane;                                                \
      const int row = piece / PPR;                                                                   \
      const int lkey = min(lt0 + row, a.L - 1);                                                      \
      const unsigned char* src = kg + (long long)lkey * ROWB + (((piece % PPR) ^ (row % PPR)) * 16); \
      const uint32_t dst = __builtin_amdgcn_readfirstlane(slot_lds + (uint32_t)(wave * LPT + j) * 1024u); \
      __builtin_amdgcn_global_load_lds((global_void_ptr_t)(uintptr_t)src, (lds_void_ptr_t)(uintptr_t)dst, 16, 0, 0); \
    }                                                                                                \
  }
  MADAKV_DMA_ISSUE(0)
  MADAKV_DMA_ISSUE(min(1, ntiles - 1))

  // Q fragments of the wave's rows straight from memory (rows past M: zeros); a lane holds, for k-step ks,
  // elements [half * D/2 + ks * 8, + 8) of row `col` of the block
  bf16x8_t areg[NRB][KS];
#pragma unroll
  for (int b = 0; b < NRB; ++b) {
    const int row = (role + b * NW) * 32 + col;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 val = make_uint4(0, 0, 0, 0);
      if (row < a.M) val = *reinterpret_cast<const uint4*>(qg + (long long)row * D + half * (D / 2) + ks * 8);
      areg[b][ks] = __builtin_bit_cast(bf16x8_t, val);
    }
  }
  // where this lane's operand pieces of row `col` of a subtile sit, relative to the subtile's first byte
  uint32_t frag_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) frag_off[ks] = (uint32_t)(col * ROWB + (((half * KS + ks) ^ (col % PPR)) * 16));
  const uint32_t red_lds = (uint32_t)(uintptr_t)red;

  for (int t = 0; t < ntiles; ++t) {
    // tile t has landed (the loads of tile t + 1 may still be out), this wave's LDS stores of the last trip are
    // done; after the barrier that holds for every wave, and nobody reads tile t - 1 any more
    if (LPT == 4) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else if (LPT == 2) asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    MADAKV_DMA_ISSUE(min(t + 2, ntiles - 1))   // into the slot of tile t - 1 (past the end: the last tile once more, which keeps the count of loads in flight)
    if (PASS == 2 && t > 0 && tid < DMA_TK) {  // the column sums of tile t - 1, the waves' shares added in wave order
      const int key = chunk0 + (t - 1) * DMA_TK + tid;
      const uint32_t r4 = red_lds + (uint32_t)((((t - 1) & 1) * NW * DMA_TK + tid) * 4);
      static_assert(NW == 4 || PASS == 1, "sweep 2 adds four waves' shares");
      float c0, c1, c2, c3;
      asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:256\n\tds_read_b32 %2, %4 offset:512\n\tds_read_b32 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3) : "v"(r4) : "memory");
      if (key < chunk1) __builtin_nontemporal_store(((c0 + c1) + c2) + c3, a.psi + ((long long)head * a.L + key));
    }
    const uint32_t tile_lds = ring_lds + (uint32_t)(t % DMA_NBUF) * TILEB;
    const int tile_end = chunk0 + (t + 1) * DMA_TK;
    const bool tail = tile_end > first_masked || tile_end > chunk1;

    // Sweep 2's vector arithmetic runs on the BS logits a lane holds of every row after the contractions of BS
    // subtiles.  In a tail tile (it holds keys that some proxy row must not see: the last W - 1 keys of the head,
    // keys past the chunk's end) such logits become NEG_BIG, in both sweeps.
#define MADAKV_DMA_VECTOR(TAIL, NB)                                                                  \
    _Pragma("unroll") for (int b = 0; b < (NB); ++b) {                                               \
      _Pragma("unroll") for (int j = 0; j < 16; ++j) {                                               \
        float x[BS];                                                                                 \
        _Pragma("unroll") for (int u = 0; u < BS; ++u) {                                             \
          x[u] = acc[u][b][j];                                                                       \
          if (TAIL) {                                                                                \
            const int key = chunk0 + t * DMA_TK + (s0 + u) * 32 + col;                               \
            const int row = (role + b * NW) * 32 + (j >> 2) * 8 + half * 4 + (j & 3);                      \
            const int pos = a.L - a.W + (row % a.W);                                                 \
            const bool valid = (key < chunk1) && (key <= pos) && (row < a.M);                        \
            x[u] = valid ? x[u] : NEG_BIG;                                                           \
          }                                                                                          \
        }                                                                                            \
        _Pragma("unroll") for (int u = 0; u < BS; ++u) colsum[u] += fast_exp2(fmaf(x[u], a.scale_log2, -st_m[b][j])); \
      }                                                                                              \
    }
    // Sweep 1 on one subtile: S^T = K Q^T, so that D[key][row] leaves a lane with the logits of its own row
    // (row `col` of the block) against 16 keys: keys t0 + 8 (j >> 2) + 4 half + (j & 3).  The row's maximum and sum
    // are then in-lane work, one rescaling of the sum per subtile; the two halves of a row meet after the last tile.
    // The running maximum stays in accumulator units (scale > 0).  A row that has seen no key yet holds NEG_BIG and
    // a meaningless, finite sum, which the first real key (and any merge with real statistics) multiplies by
    // exp2(-huge) = 0.
#define MADAKV_DMA_ROWS(TAIL, NB)                                                                    \
    _Pragma("unroll") for (int b = 0; b < (NB); ++b) {                                               \
      f32x16_t xt = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; \
      _Pragma("unroll") for (int ks = 0; ks < KS; ++ks)                                              \
        xt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfrag[0][ks], areg[b][ks], xt, 0, 0, 0);        \
      if (TAIL) {                                                                                    \
        const int row = (role + b * NW) * 32 + col;                                                        \
        const int pos = a.L - a.W + (row % a.W);                                                     \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) {                                             \
          const int key = chunk0 + t * DMA_TK + s0 * 32 + 8 * (j >> 2) + 4 * half + (j & 3);         \
          xt[j] = ((key < chunk1) && (key <= pos) && (row < a.M)) ? xt[j] : NEG_BIG;                 \
        }                                                                                            \
      }                                                                                              \
      float mn = row_m[b];                                                                           \
      _Pragma("unroll") for (int j = 0; j < 16; ++j) mn = fmaxf(mn, xt[j]);                          \
      /* (no key of the row seen yet: every x is NEG_BIG too, and x * scale - round(NEG_BIG * scale) would be the   \
         product's rounding error, some 1e21 of either sign; against 0 the terms are exp2(-huge) = 0) */            \
      const float ms = mn > 0.5f * NEG_BIG ? mn * a.scale_log2 : 0.f;                                \
      float l;                                                                                       \
      if (CLOSE) {                                                                                   \
        l = row_m[b] > 0.5f * NEG_BIG ? row_l[b] * fast_exp2(row_ms[b] - ms) : 0.f;                  \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) xt[j] = fast_exp2(fmaf(xt[j], a.scale_log2, -ms)); \
        _Pragma("unroll") for (int o = 8; o >= 1; o >>= 1) { _Pragma("unroll") for (int j = 0; j < o; ++j) xt[j] += xt[j + o]; } \
        l += xt[0];                                                                                  \
      } else {                                                                                       \
        l = row_l[b] * fast_exp2((row_m[b] - mn) * a.scale_log2);                                    \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) l += fast_exp2(fmaf(xt[j], a.scale_log2, -ms)); \
      }                                                                                              \
      row_ms[b] = ms;                                                                                \
      row_m[b] = mn; row_l[b] = l;                                                                   \
    }
#pragma unroll 1
    for (int s0 = 0; s0 < NSUB; s0 += BS) {
      f32x16_t acc[BS][NRB];
      float colsum[BS];
#pragma unroll
      for (int u = 0; u < BS; ++u) colsum[u] = 0.f;
      bf16x8_t bfrag[BS][KS];
#pragma unroll
      for (int u = 0; u < BS; ++u) {
        const uint32_t sub_lds = tile_lds + (uint32_t)(s0 + u) * 32 * ROWB;
        if (KS == 8) {
          asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                       "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
                       "s_waitcnt lgkmcnt(0)"
                       : "=&v"(bfrag[u][0]), "=&v"(bfrag[u][1]), "=&v"(bfrag[u][2]), "=&v"(bfrag[u][3]), "=&v"(bfrag[u][4 % KS]), "=&v"(bfrag[u][5 % KS]), "=&v"(bfrag[u][6 % KS]), "=&v"(bfrag[u][7 % KS])
                       : "v"(sub_lds + frag_off[0]), "v"(sub_lds + frag_off[1]), "v"(sub_lds + frag_off[2]), "v"(sub_lds + frag_off[3]),
                         "v"(sub_lds + frag_off[4 % KS]), "v"(sub_lds + frag_off[5 % KS]), "v"(sub_lds + frag_off[6 % KS]), "v"(sub_lds + frag_off[7 % KS])
                       : "memory");
        } else {
          asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                       "s_waitcnt lgkmcnt(0)"
                       : "=&v"(bfrag[u][0]), "=&v"(bfrag[u][1]), "=&v"(bfrag[u][2]), "=&v"(bfrag[u][3])
                       : "v"(sub_lds + frag_off[0]), "v"(sub_lds + frag_off[1]), "v"(sub_lds + frag_off[2]), "v"(sub_lds + frag_off[3])
                       : "memory");
        }
        if (BS > 1) {                            // (a batch of several subtiles: its contractions as the fragments come)
#pragma unroll
          for (int b = 0; b < NRB; ++b) {
            acc[u][b] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
              acc[u][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(areg[b][ks], bfrag[u][ks], acc[u][b], 0, 0, 0);
          }
        }
      }
      // One subtile per batch: contractions and vector arithmetic of the subtile in one stretch of straight-line
      // code, so that the second row block's contraction can be issued between the first block's vector
      // instructions (a wave issues in order: what follows a matrix instruction that waits for its predecessor
      // waits with it).
#define MADAKV_DMA_CONTRACT(NB)                                                                      \
      if (BS == 1) {                                                                                 \
        _Pragma("unroll") for (int b = 0; b < (NB); ++b) {                                           \
          acc[0][b] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; \
          _Pragma("unroll") for (int ks = 0; ks < KS; ++ks)                                          \
            acc[0][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(areg[b][ks], bfrag[0][ks], acc[0][b], 0, 0, 0); \
        }                                                                                            \
      }
      if (PASS == 1) {
        static_assert(PASS == 2 || BS == 1, "sweep 1 takes one subtile at a time");
        (void)acc;
        if (tail) { MADAKV_DMA_ROWS(true, NRB) } else if (second) { MADAKV_DMA_ROWS(false, NRB) } else { MADAKV_DMA_ROWS(false, 1) }
      } else if (tail) {                         // (empty blocks count for nothing: offsets of +inf)
        MADAKV_DMA_CONTRACT(NRB)
        MADAKV_DMA_VECTOR(true, NRB)
      } else if (NRB == 2 && !second) {
        MADAKV_DMA_CONTRACT(1)
        MADAKV_DMA_VECTOR(false, 1)
      } else {
        MADAKV_DMA_CONTRACT(NRB)
        MADAKV_DMA_VECTOR(false, NRB)
        if (BS == 1 && NRB == 2 && PASS == 2 && KS == 8) {
          // the order asked of the compiler: the first block's eight matrix instructions, then each of the second
          // block's followed by four plain and two exp2 instructions of the first block's arithmetic
          __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
          }
        }
      }
#undef MADAKV_DMA_CONTRACT
      if (PASS == 2) {
#pragma unroll
        for (int u = 0; u < BS; ++u) {
          const float cs = colsum[u] + __shfl_xor(colsum[u], 32, 64);
          const uint32_t dst = red_lds + (uint32_t)((((t & 1) * NW + role) * DMA_TK + (s0 + u) * 32 + col) * 4);
          if (half == 0) asm volatile("ds_write_b32 %0, %1" :: "v"(dst), "v"(cs) : "memory");
        }
      }
    }
#undef MADAKV_DMA_VECTOR
#undef MADAKV_DMA_ROWS
  }
#undef MADAKV_DMA_ISSUE
  // nothing may still be on its way into this workgroup's LDS when it ends
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  if (PASS == 2) {
    if (tid < DMA_TK) {
      const int key = chunk0 + (ntiles - 1) * DMA_TK + tid;
      const uint32_t r4 = red_lds + (uint32_t)((((ntiles - 1) & 1) * NW * DMA_TK + tid) * 4);
      float c0, c1, c2, c3;
      asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:256\n\tds_read_b32 %2, %4 offset:512\n\tds_read_b32 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3) : "v"(r4) : "memory");
      if (key < chunk1) __builtin_nontemporal_store(((c0 + c1) + c2) + c3, a.psi + ((long long)head * a.L + key));
    }
  } else {
    // the two halves of a row (their keys interleave in groups of four) meet; lanes 0..31 hold rows 0..31 of a block
    float* rs = a.rowstat + ((long long)head * a.nsplit + split) * a.mpad * 2;
#pragma unroll
    for (int b = 0; b < NRB; ++b) {
      float m, l;                               // (m in logit units)
      if (CLOSE) {
        const float ms = row_m[b] > 0.5f * NEG_BIG ? row_ms[b] : NEG_BIG;
        const float m2 = __shfl_xor(ms, 32, 64), l2 = __shfl_xor(row_l[b], 32, 64);
        m = fmaxf(ms, m2);
        l = row_l[b] * fast_exp2(ms - m) + l2 * fast_exp2(m2 - m);
      } else {
        const float m2 = __shfl_xor(row_m[b], 32, 64), l2 = __shfl_xor(row_l[b], 32, 64);
        const float mx = fmaxf(row_m[b], m2);
        l = row_l[b] * fast_exp2((row_m[b] - mx) * a.scale_log2) + l2 * fast_exp2((m2 - mx) * a.scale_log2);
        m = mx * a.scale_log2;
      }
      if (role + b * NW < MB && half == 0) {
        const int row = (role + b * NW) * 32 + col;
        rs[row * 2] = m; rs[row * 2 + 1] = l;
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// One sweep over K (bf16 and 8-bit keys in at most two row blocks, G*W <= 64; fp32 in blocks of 64 rows).  The logits of a workgroup's
// keys, or their softmax terms against a reference, fit in its registers: a wave keeps the D tiles of its NS subtiles (NS * NRB * 16
// floats per lane) instead of reducing them on the fly.  After its last subtile a workgroup knows the
// (max, sum) of every proxy row over its own keys; the workgroups of a head exchange these
// through memory, every one merges all of them in the same fixed order, and the column sums
// come out of the registers: K is read once and multiplied once.
//
// The exchange: a (max, sum) pair is one 64-bit word, stored with a relaxed agent-scope atomic
// store and read with relaxed agent-scope atomic loads until it differs from the all-ones
// pattern the array is filled with before the launch; the word carries its own arrival, so no
// fence and no counter is needed.  A workgroup waits only for workgroups of its own head.  Those
// have consecutive workgroup ids (the chunk index is the fast grid dimension), workgroups are
// dispatched in id order, and a head has far fewer chunks than the chip has workgroup slots, so
// the workgroups waited for are already running or next in line for the slots that free up.
// The wait is bounded all the same: a workgroup that runs out of patience counts itself in
// status[0] and computes the row statistics of the whole head on its own with plain FMA code
// (slow, and its last bits differ from the exchanged ones, but it depends on nobody).
// ------------------------------------------------------------------------------------
// 4 E4M3 bytes -> 4 bf16 (exact: 3 mantissa bits fit bf16's 7), as two packed dwords
__device__ __forceinline__ u32x2_t e4m3x4_as_bf16x4(uint32_t w) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
  u32x2_t o;
  o[0] = (__float_as_uint(a[0]) >> 16) | (__float_as_uint(a[1]) & 0xffff0000u);
  o[1] = (__float_as_uint(b[0]) >> 16) | (__float_as_uint(b[1]) & 0xffff0000u);
  return o;
}

constexpr unsigned long long XCHG_EMPTY = ~0ULL;
constexpr int FUSED_SPIN_LIMIT = 1 << 16;     // default spin_limit: polls of ~1 us each

__global__ __launch_bounds__(256) void score_xchg_init_kernel(unsigned long long* xchg, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) xchg[i] = XCHG_EMPTY;
}

// Row statistics of a whole head by one workgroup, without matrix cores and without anybody
// else: wave w takes rows w, w + 4, ...; lanes stride over the keys the row sees.  Q comes from
// the staged tile.  Leaves offs[r] = max + log2(sum) (log2 domain), +inf for padding rows.
template <int D, int KIND = K_BF16>
__device__ __forceinline__ void score_head_stats_alone(const ScoreArgs& a, int Lh, int Mh, int rowbase, const uint16_t* kg, const uint16_t* qs, float* offs) {
  constexpr bool F8 = KIND == K_E4M3;
  constexpr int RS = (KIND == K_F32 ? 2 * D : D) + 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int r = wave; r < a.mpad; r += 4) {
    float m = NEG_BIG, l = 0.f;
    if (r < Mh) {
      const int pos = Lh - a.W + ((rowbase + r) % a.W);
      for (int key = lane; key <= pos; key += 64) {
        float sdot = 0.f;
        if (KIND == K_F32) {
          const f32x4_t* kr = reinterpret_cast<const f32x4_t*>(kg + (long long)key * 2 * D);
          const f32x4_t* qr = reinterpret_cast<const f32x4_t*>(qs + r * RS);
          for (int c = 0; c < D / 4; ++c) {
            const f32x4_t kk = kr[c], qq = qr[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) sdot = fmaf(kk[e], qq[e], sdot);
          }
        }
        for (int c = 0; c < (KIND == K_F32 ? 0 : D / 8); ++c) {
          uint4 kk;
          if (F8) {      // 8 of the row's D bytes -> 8 bf16
            const u32x2_t raw = *reinterpret_cast<const u32x2_t*>(reinterpret_cast<const unsigned char*>(kg) + (long long)key * D + c * 8);
            const u32x2_t lo = e4m3x4_as_bf16x4(raw[0]), hi = e4m3x4_as_bf16x4(raw[1]);
            kk = make_uint4(lo[0], lo[1], hi[0], hi[1]);
          } else {
            kk = *reinterpret_cast<const uint4*>(kg + (long long)key * D + c * 8);
          }
          const uint4 qq = *reinterpret_cast<const uint4*>(qs + r * RS + c * 8);
          sdot = fmaf(bf16_lo(kk.x), bf16_lo(qq.x), sdot); sdot = fmaf(bf16_hi(kk.x), bf16_hi(qq.x), sdot);
          sdot = fmaf(bf16_lo(kk.y), bf16_lo(qq.y), sdot); sdot = fmaf(bf16_hi(kk.y), bf16_hi(qq.y), sdot);
          sdot = fmaf(bf16_lo(kk.z), bf16_lo(qq.z), sdot); sdot = fmaf(bf16_hi(kk.z), bf16_hi(qq.z), sdot);
          sdot = fmaf(bf16_lo(kk.w), bf16_lo(qq.w), sdot); sdot = fmaf(bf16_hi(kk.w), bf16_hi(qq.w), sdot);
        }
        const float s2 = sdot * a.scale_log2;
        const float mn = fmaxf(m, s2);
        l = l * exp2f(m - mn) + exp2f(s2 - mn);
        m = mn;
      }
      for (int o = 1; o < 64; o <<= 1) {
        const float m2 = __shfl_xor(m, o, 64), l2 = __shfl_xor(l, o, 64);
        merge_ml(m, l, m2, l2);
      }
    }
    if (lane == 0) offs[r] = (r < Mh) ? m + log2f(l) : __builtin_inff();
  }
}

// After a workgroup has left the (max, sum) of every proxy row over its own keys in part[4 waves][mpad][2]
// (LDS, behind a barrier): the head-wide exchange described above, in two halves.  post_row_stats
// publishes this workgroup's words and waits for nobody; collect_row_stats gathers the head's words and
// leaves offs[r] = max + log2(sum) over all keys of the head (log2 domain; +inf for padding rows), and, if asked, max and
// 1 / sum (0 for padding rows) in norm[2 r], norm[2 r + 1], unless a workgroup had to go its own way (*s_fail).
// All threads call both; work that needs nobody else's statistics can sit between them.  The caller
// adds the barrier after collect_row_stats.
__device__ __forceinline__ void post_row_stats(const ScoreArgs& a, int head, int slot, int fs, const float* part) {   // slot: the chunk, or a word of the group level
  const int tid = threadIdx.x;
  if (fs == 1 || tid >= a.mpad) return;
  // a row none of whose keys here is visible has max NEG_BIG and a meaningless sum: merging it with
  // anything real scales it by exp2(NEG_BIG - m) = 0
  unsigned long long* xh = a.xchg + (long long)head * a.xstride;
  float m = NEG_BIG, l = 0.f;
  for (int w = 0; w < 4; ++w) merge_ml(m, l, part[(w * a.mpad + tid) * 2], part[(w * a.mpad + tid) * 2 + 1]);
  unsigned long long word = ((unsigned long long)__float_as_uint(l) << 32) | __float_as_uint(m);
  if (word == XCHG_EMPTY) word = 0x7fc000007fc00000ULL;            // cannot happen with finite inputs
  __hip_atomic_store(xh + (long long)slot * a.mpad + tid, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Thread (r, pt) of the workgroup merges, in order, its share of the `n` words base[item * mpad + r]
// (items [pt * cpp, (pt + 1) * cpp), cpp = ceil(n / parts)), waiting for each at most spin_limit polls,
// eight loads at a time; leaves (max, sum) in pm[(pt * mpad + r) * 2 ..] and raises *s_fail if a word stayed away.
__device__ __forceinline__ void poll_row_words(const ScoreArgs& a, const unsigned long long* base, int n, float* pm, int* s_fail) {
  const int tid = threadIdx.x;
  const int nparts = SCORE_THREADS / a.mpad;    // mpad is 32 or 64
  const int r = tid % a.mpad, pt = tid / a.mpad;
  const int cpp = (n + nparts - 1) / nparts;
  int s = min(pt * cpp, n);
  const int s1 = min(s + cpp, n);
  float m = NEG_BIG, l = 0.f;
  int patience = a.spin_limit;
  bool fail = false;
  while (s < s1) {
    unsigned long long v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = __hip_atomic_load(base + (long long)min(s + j, s1 - 1) * a.mpad + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int got = 0;
    bool open = true;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      open = open && (s + j < s1) && (v[j] != XCHG_EMPTY);
      if (open) { merge_ml(m, l, __uint_as_float((uint32_t)v[j]), __uint_as_float((uint32_t)(v[j] >> 32))); ++got; }
    }
    s += got;
    if (got == 0) {
      if (--patience == 0) { fail = true; break; }
      __builtin_amdgcn_s_sleep(8);
    }
  }
  if (fail) *s_fail = 1;
  pm[(pt * a.mpad + r) * 2] = m;
  pm[(pt * a.mpad + r) * 2 + 1] = l;
}

constexpr int XCHG_GROUP = 16;       // chunks per group when the exchange has two levels

template <int D, int KIND = K_BF16>
__device__ __forceinline__ void collect_row_stats(const ScoreArgs& a, int head, int split, int fs, int Lh, int Mh, int rowbase,
                                                  const uint16_t* kg, const uint16_t* qs, const float* part, float* offs, float* norm, float* pm, int* s_fail) {
  const int tid = threadIdx.x;
  const int nparts = SCORE_THREADS / a.mpad;
  const auto leave = [&](float m, float l) {
    offs[tid] = (tid < Mh) ? m + log2f(l) : __builtin_inff();
    if (norm) { norm[2 * tid] = m; norm[2 * tid + 1] = (tid < Mh) ? 1.f / l : 0.f; }
  };
  if (fs == 1) {
    if (tid < a.mpad) {
      float m = NEG_BIG, l = 0.f;
      for (int w = 0; w < 4; ++w) merge_ml(m, l, part[(w * a.mpad + tid) * 2], part[(w * a.mpad + tid) * 2 + 1]);
      leave(m, l);
    }
    return;
  }
  unsigned long long* xh = a.xchg + (long long)head * a.xstride;
  if (a.xgroups == 0) {
    poll_row_words(a, xh, fs, pm, s_fail);
  } else {
    // Two levels, so that a workgroup reads tens of words per row instead of one per chunk of a long head.
    // The workgroup of a group's last chunk (it starts after the group's others) merges the group's
    // words and leaves one word per row for the group; everybody merges the groups' words.
    unsigned long long* gw = xh + (long long)fs * a.mpad;
    const int g = split / XCHG_GROUP, c0 = g * XCHG_GROUP, c1 = min(c0 + XCHG_GROUP, fs);
    if (split == c1 - 1) {
      poll_row_words(a, xh + (long long)c0 * a.mpad, c1 - c0, pm, s_fail);
      __syncthreads();
      if (!*s_fail && tid < a.mpad) {
        float mm = NEG_BIG, ll = 0.f;
        for (int q = 0; q < nparts; ++q) merge_ml(mm, ll, pm[(q * a.mpad + tid) * 2], pm[(q * a.mpad + tid) * 2 + 1]);
        unsigned long long word = ((unsigned long long)__float_as_uint(ll) << 32) | __float_as_uint(mm);
        if (word == XCHG_EMPTY) word = 0x7fc000007fc00000ULL;
        __hip_atomic_store(gw + (long long)g * a.mpad + tid, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();                              // pm is written again below
    }
    if (!*s_fail) poll_row_words(a, gw, a.xgroups, pm, s_fail);   // (uniform: s_fail was read behind a barrier)
  }
  __syncthreads();
  if (__builtin_expect(*s_fail, 0)) {         // uniform over the workgroup
    if (tid == 0) atomicAdd(a.status, 1);
    score_head_stats_alone<D, KIND>(a, Lh, Mh, rowbase, kg, qs, offs);
  } else if (tid < a.mpad) {
    float mm = NEG_BIG, ll = 0.f;
    for (int q = 0; q < nparts; ++q) merge_ml(mm, ll, pm[(q * a.mpad + tid) * 2], pm[(q * a.mpad + tid) * 2 + 1]);
    leave(mm, ll);
  }
}

template <int D, int KIND = K_BF16>
__device__ __forceinline__ void exchange_row_stats(const ScoreArgs& a, int head, int split, int fs, int Lh, int Mh, int rowbase,
                                                   const uint16_t* kg, const uint16_t* qs, const float* part, float* offs, float* norm, float* pm, int* s_fail) {
  post_row_stats(a, head, split, fs, part);
  collect_row_stats<D, KIND>(a, head, split, fs, Lh, Mh, rowbase, kg, qs, part, offs, norm, pm, s_fail);
}

#ifndef MADAKV_FUSED_NS1      // tuning constants of the one-sweep kernel (measured on MI355X)
#define MADAKV_FUSED_NS1 8    // subtiles per wave with one row block
#define MADAKV_FUSED_NS2 6    // ... with two row blocks
#define MADAKV_FUSED_PF 2     // subtiles in flight per wave
#define MADAKV_FUSED_WPE 2    // waves per SIMD
#endif
#ifndef MADAKV_FUSED_MAX_SPLIT
#define MADAKV_FUSED_MAX_SPLIT 64   // most chunks per head the one-sweep kernel is used for
#endif
// KIND: E4M3 keys are turned into bf16 when parked in LDS.  fp32 keys and queries run on the 32x32x2 fp32 MFMA (fp32
// products and sums throughout, no conversion).  The plain FMA kernels they replace were bound by their loads (every lane
// walked a row of its own, one uncoalesced dword at a time): one layer of 8 heads x 1024 keys x 16 rows took 117 + 124 us in
// two sweeps, 17 us here (+ 2 us for the exchange words), most of it the latencies of one pass and the instruction stream.
// Between a workgroup's last key and its scores stand the row statistics, the exchange and the column sums, and all workgroups
// of a head go through them at about the same time, so the memory is idle meanwhile: with the logits in registers, two exp2 per
// logit and 32 or 64 row reductions of ten steps one behind the other.  With the softmax terms themselves there (below) it is additions,
// two folds and one product per logit, the exp2 (one) and everything else under the loads.  Score and statistics calls before /
// after, us: 32 heads of 128K keys, 32 rows 255 / 228, 64 rows 358 / 326, 64 rows and 64 dims 290 / 246; 32 of 32K 83 / 77; 128 of
// 16K 119 / 113.  (The polling is not what costs: one lane of a row polling for all changes nothing, nor does
// starting the heads one after the other.)  A row's terms are not used where
// - their sum over the wave's keys is no number, or beyond 2^120;
// - its reference is beyond 2^23, so that reference + exponent is exact (logits of 2^30 and more gave zeros and NaN without this).
// A term of more than 2^100 gives its row another reference (see the kernel).
constexpr float FAR_TERM = 0x1p100f, LATE_SUM = 0x1p120f, LATE_REF = 0x1p23f;
template <int D, int NRB, int NS, int KIND = K_BF16>
__global__ __launch_bounds__(SCORE_THREADS) __attribute__((amdgpu_waves_per_eu(KIND == K_F32 && D == 128 ? 1 : MADAKV_FUSED_WPE, KIND == K_F32 && D == 128 ? 1 : MADAKV_FUSED_WPE))) void score_fused_kernel(ScoreArgs a) {
  constexpr bool F8 = KIND == K_E4M3, F32 = KIND == K_F32;
  constexpr int PF = F32 && D == 128 ? 1 : (MADAKV_FUSED_PF < NS ? MADAKV_FUSED_PF : NS);   // (an fp32 subtile of 128 dims takes 64 registers)
  constexpr int KS = D / 16;                  // MFMA k-steps (bf16)
  constexpr int RU = F32 ? 2 * D : D;         // 2-byte units per row
  constexpr int RS = RU + 8;                  // 2-byte units per LDS row (16 B pad)
  constexpr int PPR = RU / 8;                 // 16-byte pieces per row
  constexpr int LPS = 32 * PPR / 64;          // 16-byte loads per lane per subtile
  constexpr int CK = 4 * NS * 32;             // keys per workgroup
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* qs = reinterpret_cast<uint16_t*>(smem);                       // [mpad][RS]
  uint16_t* kt_all = qs + (size_t)a.mpad * RS;                            // [4 waves][32][RS]
  float* part = reinterpret_cast<float*>(kt_all + 4 * 32 * RS);           // [4 waves][mpad][2]
  float* offs = part + 4 * a.mpad * 2;                                    // [mpad]
  float* pm = offs + a.mpad;                                              // [256 / mpad parts][mpad][2]
  float* refs = pm + 512;                                                 // [4 waves][mpad]
  float* norm = refs + 4 * a.mpad;                                        // [mpad][2]
  int* last = reinterpret_cast<int*>(norm + 2 * a.mpad);                  // [mpad] last key of the chunk that the row sees
  int* drops = last + a.mpad;                                             // [4 waves][NS][mpad]
  __shared__ int s_fail, s_late;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bx = blockIdx.x;                  // (the parked chunks first: split is set below, once fs is known)
  const int hv = a.head0 + blockIdx.y;        // head, or (head, block of 64 proxy rows) when there are more than 64
  const int head = hv / a.rb_count;
  const int rowbase = (hv % a.rb_count) * 64; // first proxy row of this workgroup's block
  const int Mh = min(a.M - rowbase, a.mpad);  // its rows
  const int kvh = head % a.H;
  const long long lb = head / a.H;            // (layer, batch) index
  const uint16_t* qg = reinterpret_cast<const uint16_t*>(a.q_win) + ((lb * a.H + kvh) * (long long)a.G * a.W + rowbase) * RU;
  // keys of this head: L rows at head * L, or (ragged: the rows of a reduced cache) seg_len rows at seg_off
  const int Lh = a.seg_len ? a.seg_len[head] : a.L;
  const long long base = a.seg_off ? a.seg_off[head] : (long long)head * a.L;
  const int fs = a.seg_len ? (Lh + CK - 1) / CK : a.fsplit;      // chunks of this head (the grid is sized for the longest)
  const int split = bx < a.nstrag ? fs + bx : bx - a.nstrag;
  if (split >= fs + a.nstrag) return;
  const bool parked = split >= fs;            // one of the head's last chunks, run ahead of the others
  // (F8: rows of D bytes; kg then counts in 2-byte units from a byte address that is base * D)
  const uint16_t* kg = F8 ? reinterpret_cast<const uint16_t*>(reinterpret_cast<const unsigned char*>(a.k) + base * D)
                          : reinterpret_cast<const uint16_t*>(a.k) + base * RU;
  const int chunk0 = split * CK;
  const int chunk1 = min(Lh, chunk0 + CK);
  uint16_t* kt = kt_all + (size_t)wave * 32 * RS;
  float* ref = refs + wave * a.mpad;
  int* drop = drops + wave * NS * a.mpad;
  if (tid == 0) s_fail = s_late = 0;

  // subtile `it` of this wave: keys chunk0 + (it * 4 + wave) * 32 ...; PF subtiles in flight
  constexpr int CPR = F8 ? PPR / 2 : PPR;      // 16-byte pieces per cached row
  constexpr int LPSK = F8 ? LPS / 2 : LPS;     // loads per lane and subtile
  u32x4_t pre[PF][LPSK];
  const int lrow = lane / CPR, lpiece = lane % CPR;     // of the lane's first load; the next is 64 / CPR rows further
#define MADAKV_FUSED_LOAD(SET, IT)                                                               \
  {                                                                                              \
    const int lt0 = chunk0 + ((IT) * 4 + wave) * 32 + lrow;                                      \
    _Pragma("unroll") for (int i = 0; i < LPSK; ++i) {                                           \
      const int lkey = min(lt0 + i * (64 / CPR), Lh - 1); /* past the end: a valid row, masked later */ \
      pre[SET][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(                 \
          reinterpret_cast<const unsigned char*>(kg) + (uint32_t)(lkey * CPR + lpiece) * 16u));  \
    }                                                                                            \
  }
#pragma unroll
  for (int it = 0; it < PF; ++it) MADAKV_FUSED_LOAD(it, it)

  // Q tile.  Padding rows count for nothing (their offset is +inf) unless they turn an infinite key element into NaN, as rows
  // of zeros do: fp32 takes the last row once more.  (bf16 keeps zeros: the other costs 2 of 320 us at 128K keys.)
  for (int e = tid; e < a.mpad * PPR; e += SCORE_THREADS) {
    const int r = e / PPR, c = e % PPR;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (F32 || r < Mh) val = *reinterpret_cast<const uint4*>(qg + (long long)(F32 ? min(r, Mh - 1) : r) * RU + c * 8);
    *reinterpret_cast<uint4*>(qs + r * RS + c * 8) = val;
  }
  if (tid < a.mpad) last[tid] = tid < Mh ? min(Lh - a.W + (rowbase + tid) % a.W, chunk1 - 1) : -1;
  __syncthreads();

  const int half = lane >> 5, col = lane & 31;
  const int first_masked = Lh - a.W + 1;      // keys below this are visible to every proxy row
  bf16x8_t areg[KS];                           // one row block: its Q fragments stay in registers
#pragma unroll
  for (int ks = 0; ks < (F32 || NRB > 1 ? 0 : KS); ++ks)
    areg[ks] = *reinterpret_cast<const bf16x8_t*>(qs + col * RS + half * (D / 2) + ks * 8);

  // (padding rows need no mask: their offset is +inf)
  const auto mask = [&](float (&x)[16], int b, int it, float none) __attribute__((always_inline)) {
    const int t0 = chunk0 + (it * 4 + wave) * 32, key = t0 + col;
    if (t0 + 32 <= first_masked && t0 + 32 <= chunk1) return;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const i32x4_t to = *reinterpret_cast<const i32x4_t*>(last + b * 32 + half * 4 + c * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[c * 4 + e] = key <= to[e] ? x[c * 4 + e] : none;
    }
  };
  // a subtile's keys from their registers to the wave's tile
  const auto park = [&](const u32x4_t (&keys)[LPSK]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPSK; ++i) {
      uint16_t* kw = kt + lrow * RS + lpiece * (F8 ? 16 : 8) + i * (64 / CPR) * RS;
      if (F8) {                                   // 16 bytes of a row -> 16 bf16
        const u32x4_t raw = keys[i];
        const u32x2_t c0 = e4m3x4_as_bf16x4(raw[0]), c1 = e4m3x4_as_bf16x4(raw[1]), c2 = e4m3x4_as_bf16x4(raw[2]), c3 = e4m3x4_as_bf16x4(raw[3]);
        *reinterpret_cast<u32x4_t*>(kw) = u32x4_t{c0[0], c0[1], c1[0], c1[1]};
        *reinterpret_cast<u32x4_t*>(kw + 8) = u32x4_t{c2[0], c2[1], c3[0], c3[1]};
      } else {
        *reinterpret_cast<u32x4_t*>(kw) = keys[i];
      }
    }
  };
  const auto contract = [&](f32x16_t (&acc)[NRB]) __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t* krow = kt + col * RS + half * (RU / 2);
    const uint16_t* qrow = qs + col * RS + half * (RU / 2);
#pragma unroll
    for (int b = 0; b < NRB; ++b) acc[b] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (F32) {                                    // step s contracts dims s and D/2 + s: a lane's operands are consecutive floats
#pragma unroll
      for (int b = 0; b < NRB; ++b) {
#pragma unroll 4
        for (int c = 0; c < D / 8; ++c) {
          const f32x4_t qv = *reinterpret_cast<const f32x4_t*>(qrow + b * 32 * RS + c * 8), kv = *reinterpret_cast<const f32x4_t*>(krow + c * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(qv[e], kv[e], acc[b], 0, 0, 0);
        }
      }
    }
    if (NRB == 1) {
      bf16x8_t bfrag[KS];
#pragma unroll
      for (int ks = 0; ks < (F32 ? 0 : KS); ++ks) bfrag[ks] = *reinterpret_cast<const bf16x8_t*>(krow + ks * 8);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int ks = 0; ks < (F32 ? 0 : KS); ++ks) acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(areg[ks], bfrag[ks], acc[0], 0, 0, 0);
    } else {                                      // (a key fragment at a time: all of them would spill)
#pragma unroll
      for (int ks = 0; ks < (F32 ? 0 : KS); ++ks) {
        const bf16x8_t bfrag = *reinterpret_cast<const bf16x8_t*>(krow + ks * 8);
#pragma unroll
        for (int b = 0; b < NRB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(qrow + b * 32 * RS + ks * 8), bfrag, acc[b], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");                // (the tile is free)
    __builtin_amdgcn_wave_barrier();
  };

  float* psi = (a.rb_count > 1 ? a.psi_part + (hv % a.rb_count) * a.psi_part_stride : a.psi) + base;
  const auto store = [&](int it, float colsum) __attribute__((always_inline)) {
    colsum += __shfl_xor(colsum, 32, 64);
    const int key = chunk0 + (it * 4 + wave) * 32 + col;
    if (half == 0 && key < chunk1) __builtin_nontemporal_store(colsum, psi + key);
  };
  // What stays in registers of a (row, key) pair is its softmax term against the wave's reference of the row, the
  // largest logit of the wave's first subtile (a whole number, so that nothing is rounded but the difference).  The
  // terms are formed under the loads of the keys that follow; behind the last subtile the row sums are additions and the column
  // sums products with one factor per row and wave.
  // A subtile with a term beyond FAR_TERM gives the rows their largest logit so far as a reference; by how much the terms before it are
  // too large, an exponent, goes to LDS and into them behind the last subtile.  (A second sweep over the workgroup's keys with the logits
  // instead, which all workgroups of the head wait for, is what such keys had cost: queries four times as long as those of the workloads put a
  // wave's first keys that far below others in 20 to 60% of the workgroups.  Us per call with logits in registers / with that second sweep / now: 128
  // heads of 16K keys, 32 rows, all workgroups 128 / 210 / 125, 32 of 128K, 64 rows, all 354 / 530 / 360, 64 fp32 heads of 4K, long queries 37.0 / 41.7 /
  // 36.7.  The check costs nothing that runs do not differ by, 64 dims gain, 60 -> 57 (112 heads of 8K, 40 rows); one per block instead costs two
  // blocks of 128 dims 2-3%.  The scaling in the branch itself, the logits of both blocks before the terms of either, or unrolled
  // contractions there spilled 40 to 190 registers in the ordinary path of two blocks of 128 dims: 341 -> 356-400 us.)
  // In a workgroup in which a row's terms or reference pass their limits (above), and in the parked chunks: the logits themselves,
  // and all row maxima and two exp2 per logit between the last key and the scores.
  float x[NS][NRB][16];
  bool moved = false;                             // a reference did
  const auto settle = [&]() __attribute__((always_inline)) {             // (what the wave's lanes leave each other in LDS)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const auto form = [&](const f32x16_t& acc, int b, int it) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4_t m = *reinterpret_cast<const f32x4_t*>(ref + b * 32 + half * 4 + c * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[it][b][c * 4 + e] = fast_exp2(fmaf(acc[c * 4 + e], a.scale_log2, -m[e]));
    }
    mask(x[it][b], b, it, 0.f);
  };
  // a block of the subtile that is still in the wave's tile once more
  const auto again = [&](int b) __attribute__((always_inline)) {
    const uint16_t* krow = kt + col * RS + half * (RU / 2);
    const uint16_t* qrow = qs + (b * 32 + col) * RS + half * (RU / 2);
    f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int c = 0; c < (F32 ? D / 8 : KS); ++c) {
      if (F32) {
        const f32x4_t qv = *reinterpret_cast<const f32x4_t*>(qrow + c * 8), kv = *reinterpret_cast<const f32x4_t*>(krow + c * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qv[e], kv[e], acc, 0, 0, 0);
      } else {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(qrow + c * 8), *reinterpret_cast<const bf16x8_t*>(krow + c * 8), acc, 0, 0, 0);
      }
    }
    settle();
    return acc;
  };
  const int frow = half * 4 + (col >> 2) * 8 + (col & 3);                // the row of a block whose fold this lane (of the first 16) gets
  const auto move = [&](int b, int it) __attribute__((always_inline)) {
    if (!moved)
      for (int e = lane; e < NS * a.mpad; e += 64) drop[e] = 0;
    moved = true;
    settle();
    {
      const f32x16_t acc = again(b);
#pragma unroll
      for (int j = 0; j < 16; ++j) x[it][b][j] = acc[j] * a.scale_log2;
    }
    mask(x[it][b], b, it, NEG_BIG);
    const float mx = half_fold<0>(x[it][b], lane);
    if (col < 16) {
      const float old = ref[b * 32 + frow], now = fmaxf(old, floorf(mx));
      const int up = (int)fminf(now - old, 1e6f);
      ref[b * 32 + frow] = now;
#pragma unroll 1
      for (int i = 0; i < it; ++i) drop[i * a.mpad + b * 32 + frow] += up;
    }
    settle();
    form(again(b), b, it);
  };
  const auto sweep = [&](auto terms_t) __attribute__((always_inline)) {
    constexpr bool T = decltype(terms_t)::value;
    if (!T) {
#pragma unroll
      for (int it = 0; it < PF; ++it) MADAKV_FUSED_LOAD(it, it)
    }
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      park(pre[it % PF]);
      if (it + PF < NS) MADAKV_FUSED_LOAD(it % PF, it + PF)
      f32x16_t acc[NRB];
      contract(acc);
      uint32_t top = 0u;
#pragma unroll
      for (int b = 0; b < NRB; ++b) {
        if (!T) {
#pragma unroll
          for (int j = 0; j < 16; ++j) x[it][b][j] = acc[b][j] * a.scale_log2;
          mask(x[it][b], b, it, NEG_BIG);
          continue;
        }
        if (it == 0) {
          float lg[16];
#pragma unroll
          for (int j = 0; j < 16; ++j) lg[j] = acc[b][j] * a.scale_log2;
          mask(lg, b, it, NEG_BIG);
          const float mx = half_fold<0>(lg, lane);
          if (col < 16) ref[b * 32 + frow] = mx == NEG_BIG ? 0.f : floorf(mx);
          settle();
        }
        form(acc[b], b, it);
        if (it > 0) {                             // (no term is negative: the largest has the largest bits)
#pragma unroll
          for (int j = 0; j < 16; ++j) top = max(top, __float_as_uint(x[it][b][j]));
          if (b == NRB - 1 && __builtin_expect(__any(top > __float_as_uint(FAR_TERM)), 0)) {
#pragma unroll
            for (int o = 0; o < NRB; ++o) move(o, it);
          }
        }
      }
    }
  };
  bool terms = !parked;
  if (terms) {
    sweep(std::true_type{});
    if (__builtin_expect(moved, 0)) {
#pragma unroll
      for (int it = 0; it + 1 < NS; ++it)
#pragma unroll
        for (int b = 0; b < NRB; ++b)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const i32x4_t n = *reinterpret_cast<const i32x4_t*>(drop + it * a.mpad + b * 32 + half * 4 + c * 8);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[it][b][c * 4 + e] = ldexpf(x[it][b][c * 4 + e], -n[e]);
          }
    }
    // ---- (reference, sum) of every row over this workgroup's keys: lanes, then waves (fixed order)
#pragma unroll
    for (int b = 0; b < NRB; ++b) {
      float sum[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        sum[j] = x[0][b][j];
#pragma unroll
        for (int it = 1; it < NS; ++it) sum[j] += x[it][b][j];
      }
      const float l = half_fold<1>(sum, lane);
      if (col < 16) {
        const int row = b * 32 + (col >> 2) * 8 + half * 4 + (col & 3);
        const float rf = ref[row];
        if (!(l <= LATE_SUM) || fabsf(rf) > LATE_REF) s_late = 1;         // (NaN too)
        const int e = l > 0.f ? __builtin_amdgcn_frexp_expf(l) : 0;
        part[(wave * a.mpad + row) * 2] = l > 0.f ? rf + (float)e : NEG_BIG;
        part[(wave * a.mpad + row) * 2 + 1] = ldexpf(l, -e);
      }
    }
    __syncthreads();
    terms = s_late == 0;                        // the same in the whole workgroup
  }
  if (!terms) {
    sweep(std::false_type{});
    // ---- (max, sum) the same way
#pragma unroll
    for (int b = 0; b < NRB; ++b) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        float mx = x[0][b][j];
        if (F32) mx = fmaxf(mx, NEG_BIG);       // (a row whose logits here are all -Inf: against NEG_BIG its sum is 0)
#pragma unroll
        for (int it = 1; it < NS; ++it) mx = fmaxf(mx, x[it][b][j]);
        const float m = half_reduce<0>(mx);
        float sm = 0.f;
#pragma unroll
        for (int it = 0; it < NS; ++it) sm += fast_exp2(x[it][b][j] - m);   // masked entries against a real maximum: 0
        const float l = half_reduce<1>(sm);
        if (col == 0) {
          const int row = b * 32 + (j >> 2) * 8 + half * 4 + (j & 3);
          part[(wave * a.mpad + row) * 2] = m;
          part[(wave * a.mpad + row) * 2 + 1] = l;
        }
      }
    }
    __syncthreads();
    if (parked) {
      // its statistics as a word of the group level (behind the groups' own), its logits to memory; nobody is waited for
      post_row_stats(a, hv, fs + (a.xgroups - a.nstrag) + (split - fs), fs, part);
      float* pk = a.park + ((long long)hv * a.nstrag + (split - fs)) * (NS * NRB * 16 * SCORE_THREADS);
#pragma unroll
      for (int it = 0; it < NS; ++it)
#pragma unroll
        for (int b = 0; b < NRB; ++b)
#pragma unroll
          for (int j = 0; j < 16; ++j) __builtin_nontemporal_store(x[it][b][j], pk + ((it * NRB + b) * 16 + j) * SCORE_THREADS + tid);
      return;
    }
  }
  exchange_row_stats<D, KIND>(a, hv, split, fs, Lh, Mh, rowbase, kg, qs, part, offs, norm, pm, &s_fail);
  __syncthreads();
  if (a.offs_out && split == 0 && tid < a.mpad) a.offs_out[(long long)hv * a.mpad + tid] = offs[tid];

  // ---- column sums from the registers
  const auto column_sums = [&](const float* per_row, auto entry) __attribute__((always_inline)) {
    float f[NRB][16];
#pragma unroll
    for (int b = 0; b < NRB; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) f[b][j] = per_row[b * 32 + (j >> 2) * 8 + half * 4 + (j & 3)];
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      float colsum = 0.f;
#pragma unroll
      for (int b = 0; b < NRB; ++b)
#pragma unroll
        for (int j = 0; j < 16; ++j) colsum = entry(colsum, x[it][b][j], f[b][j]);
      store(it, colsum);
    }
  };
  if (!terms) {
    column_sums(offs, [](float sum, float lg, float off) { return sum + fast_exp2(lg - off); });
    return;
  }
  // a row's factor, exp2(reference - max) / sum (a wave has not more than 64 rows; a row that sees none of the wave's keys has
  // a reference of 0 and no terms)
  const int r = min(lane, a.mpad - 1);
  const float dist = ref[r] - (s_fail ? offs[r] : norm[2 * r]), inv = s_fail ? 1.f : norm[2 * r + 1];
  const float rel = dist > 0.f ? 0.f : dist;                 // (a normaliser that is no number stays one: fminf would lose it)
  // Where the wave's reference is far below the head's maximum, the factor alone would flush to zero and its product
  // with a large term would not: two factors then.
  const bool small = __any(rel < -100.f && inv > 0.f);
  if (lane < a.mpad) ref[lane] = small ? fast_exp2(0.5f * rel) * sqrtf(inv) : fast_exp2(rel) * inv;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (__builtin_expect(small, 0)) column_sums(ref, [](float sum, float p, float f) { return fmaf(p * f, f, sum); });
  else column_sums(ref, [](float sum, float p, float f) { return fmaf(p, f, sum); });
}
#undef MADAKV_FUSED_LOAD

// The parked chunks' column sums, from their logits and the heads' row offsets: the arithmetic (and its order) of the
// kernel's own last step on logits.  Grid (parked chunk, head).
template <int NRB, int NS>
__global__ __launch_bounds__(SCORE_THREADS) void score_fused_finish_kernel(ScoreArgs a) {
  constexpr int CK = 4 * NS * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int hv = a.head0 + blockIdx.y, sidx = blockIdx.x;
  const int chunk0 = (a.fsplit + sidx) * CK;
  const int chunk1 = min(a.L, chunk0 + CK);
  const float* pk = a.park + ((long long)hv * a.nstrag + sidx) * (NS * NRB * 16 * SCORE_THREADS);
  const float* offs = a.offs_out + (long long)hv * a.mpad;
  float off_r[NRB][16];
#pragma unroll
  for (int b = 0; b < NRB; ++b)
#pragma unroll
    for (int j = 0; j < 16; ++j) off_r[b][j] = offs[b * 32 + (j >> 2) * 8 + half * 4 + (j & 3)];
#pragma unroll
  for (int it = 0; it < NS; ++it) {
    float colsum = 0.f;
#pragma unroll
    for (int b = 0; b < NRB; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) colsum += fast_exp2(__builtin_nontemporal_load(pk + ((it * NRB + b) * 16 + j) * SCORE_THREADS + tid) - off_r[b][j]);
    colsum += __shfl_xor(colsum, 32, 64);
    const int key = chunk0 + (it * 4 + wave) * 32 + col;
    if (half == 0 && key < chunk1) __builtin_nontemporal_store(colsum, a.psi + ((long long)hv * a.L + key));
  }
}

// ------------------------------------------------------------------------------------
// The prefill attention of the last W prompt positions (paper Sec. 3.1 Eq. 5 for the proxy rows of
// Sec. 3.3) with the proxy-token scores of Eq. 7 as a by-product: out = softmax(scale Q K^T) V for
// a block of up to 32 of the G*W proxy rows of a KV head (more rows: more blocks, each with a pass of its own over
// K and V, their column sums added in block order afterwards, or window_wide_kernel below, see win_one_pass), their log-sum-exp, and psi = the column sums of the same
// softmax rows.  A model's prefill runs this attention anyway; taking psi from it removes the
// eviction's own sweep over K.
// Same structure as score_fused_kernel (a workgroup's logits stay in registers while the row
// statistics travel among the head's workgroups), with the contraction transposed: S^T = K Q^T, so a
// lane holds one proxy row and 16 keys of a subtile.  Row statistics are then in-lane, the
// column sums of Eq. 7 one half-wave reduction per key, and P is already laid out as the A
// operand of O += P V: the contraction index of that product is numbered so that a lane's
// eight keys of a 16-key step are the eight it holds.  V subtiles are streamed through the same
// wave-private LDS tile as K was; a B fragment (eight keys of one output column) is read
// from it by two transposing reads.  P goes in as bf16 hi + lo parts (two MFMAs), which keeps
// fp32-level accuracy.  The V sweep does not wait for the exchange: it exponentiates against the
// wave's own row maxima, and the head-wide statistics, collected after it, enter as one factor per
// row (for O and for the column sums alike).  Every workgroup leaves its share of O, normalised
// that way, in memory; window_attn_reduce_kernel adds the shares in chunk order.
// ------------------------------------------------------------------------------------
struct WinArgs {
  ScoreArgs s;
  const void* v;       // [heads, L, d]
  float* opart;        // [heads, fsplit, 32, d] shares of O
  float* lse;          // optional [heads/H * Hq, W] natural log-sum-exp of every proxy row
  void* out;           // [heads/H * Hq, W, d]
  int out_fp32;
};

typedef __attribute__((ext_vector_type(2))) float win_f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 win_bf16x2_t;
typedef __attribute__((ext_vector_type(4))) short win_s16x4_t;
typedef __attribute__((address_space(3))) win_s16x4_t* win_lds_s16x4_ptr_t;
template <int D, int NS>
__global__ __launch_bounds__(SCORE_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void window_attn_kernel(WinArgs wa) {
  const ScoreArgs& a = wa.s;
  constexpr int KS = D / 16, RS = D + 8, PPR = D / 8, LPS = 32 * PPR / 64, CK = 4 * NS * 32, PF = 2, DB = D / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* qs = reinterpret_cast<uint16_t*>(smem);                       // [32][RS]
  uint16_t* kt_all = qs + 32 * RS;                                        // [4 waves][32][RS]
  float* part = reinterpret_cast<float*>(kt_all + 4 * 32 * RS);           // [4 waves][32][2]
  float* offs = part + 4 * 32 * 2;                                        // [32]
  float* pm = offs + 32;                                                  // [8 parts][32][2]
  __shared__ int s_fail;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = blockIdx.x;
  const int hv = a.head0 + blockIdx.y;        // head, or (head, block of 32 proxy rows) when there are more than 32
  const int head = hv / a.rb_count;
  const int rowbase = (hv % a.rb_count) * 32; // first proxy row of this workgroup's block
  const int Mh = min(a.M - rowbase, 32);      // its rows
  const int kvh = head % a.H;
  const long long lb = head / a.H;
  const uint16_t* qg = reinterpret_cast<const uint16_t*>(a.q_win) + ((lb * a.H + kvh) * (long long)a.G * a.W + rowbase) * D;
  const uint16_t* kg = reinterpret_cast<const uint16_t*>(a.k) + (long long)head * a.L * D;
  const uint16_t* vg = reinterpret_cast<const uint16_t*>(wa.v) + (long long)head * a.L * D;
  const int Lh = a.L, fs = a.fsplit;
  const int chunk0 = split * CK;
  const int chunk1 = min(Lh, chunk0 + CK);
  uint16_t* kt = kt_all + (size_t)wave * 32 * RS;
  if (tid == 0) s_fail = 0;

  u32x4_t pre[PF][LPS];
#define MADAKV_WIN_LOAD(BASE, SET, IT)                                                           \
  {                                                                                              \
    const int lt0 = chunk0 + ((IT) * 4 + wave) * 32;                                             \
    _Pragma("unroll") for (int i = 0; i < LPS; ++i) {                                            \
      const int idx = i * 64 + lane;                                                             \
      const int lkey = min(lt0 + idx / PPR, Lh - 1); /* past the end: a valid row, masked */     \
      pre[SET][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(BASE + (long long)lkey * D + (idx % PPR) * 8)); \
    }                                                                                            \
  }
#define MADAKV_WIN_PARK(SET)                                                                     \
  _Pragma("unroll") for (int i = 0; i < LPS; ++i) {                                              \
    const int idx = i * 64 + lane;                                                               \
    *reinterpret_cast<u32x4_t*>(kt + (idx / PPR) * RS + (idx % PPR) * 8) = pre[SET][i];          \
  }
#pragma unroll
  for (int it = 0; it < PF; ++it) MADAKV_WIN_LOAD(kg, it, it)

  for (int e = tid; e < 32 * PPR; e += SCORE_THREADS) {                   // Q tile, padding rows zero
    const int r = e / PPR, c = e % PPR;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (r < Mh) val = *reinterpret_cast<const uint4*>(qg + (long long)r * D + c * 8);
    *reinterpret_cast<uint4*>(qs + r * RS + c * 8) = val;
  }
  __syncthreads();

  const int half = lane >> 5, col = lane & 31;            // col = this lane's proxy row (of the block)
  const int first_masked = Lh - a.W + 1;
  const int pos = Lh - a.W + ((rowbase + col) % a.W);     // last key the row sees
  bf16x8_t qfrag[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qfrag[ks] = *reinterpret_cast<const bf16x8_t*>(qs + col * RS + half * (D / 2) + ks * 8);

  // ---- S^T = K Q^T: lg[it][j] = scaled logit of row `col` and key t0 + 8 (j >> 2) + 4 half + (j & 3)
  float lg[NS][16];
#pragma unroll
  for (int it = 0; it < NS; ++it) {
    MADAKV_WIN_PARK(it % PF)
    if (it + PF < NS) MADAKV_WIN_LOAD(kg, it % PF, it + PF)
    else MADAKV_WIN_LOAD(vg, it % PF, it + PF - NS)          // V's first subtiles: the loads don't pause for the statistics
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int t0 = chunk0 + (it * 4 + wave) * 32;
    const bool tail = (t0 + 32 > first_masked) || (t0 + 32 > chunk1) || (Mh < 32);
    const uint16_t* krow = kt + col * RS + half * (D / 2);
    f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8_t kfrag = *reinterpret_cast<const bf16x8_t*>(krow + ks * 8);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag, qfrag[ks], acc, 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int key = t0 + 8 * (j >> 2) + 4 * half + (j & 3);
      const bool valid = !tail || ((key < chunk1) && (key <= pos) && (col < Mh));
      lg[it][j] = valid ? acc[j] * a.scale_log2 : NEG_BIG;
    }
  }

  // ---- (max, sum) of the lane's row over this wave's keys: in-lane, then the two halves
  float mx = NEG_BIG;
#pragma unroll
  for (int it = 0; it < NS; ++it)
#pragma unroll
    for (int j = 0; j < 16; ++j) mx = fmaxf(mx, lg[it][j]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float mloc = mx > NEG_BIG ? mx : 0.f;              // NEG_BIG: the row sees none of this wave's keys
  {
    float sm = 0.f;
#pragma unroll
    for (int it = 0; it < NS; ++it)
#pragma unroll
      for (int j = 0; j < 16; ++j) sm += fast_exp2(lg[it][j] - mx);
    sm += __shfl_xor(sm, 32, 64);
    if (half == 0) { part[(wave * 32 + col) * 2] = mx; part[(wave * 32 + col) * 2 + 1] = sm; }
  }
  __syncthreads();
  post_row_stats(a, hv, split, fs, part);

  // ---- O += P V with p taken against the wave's own row maxima, so that nothing here waits for the
  // other workgroups of the head; the head-wide statistics come in as one factor per row afterwards
  // where this lane's transposing reads start: per 16 lanes four rows of 16 columns, lane j pointing at columns 4 (j & 3).. of row
  // j >> 2 and getting column j of the four.  (For 32 heads of 8K keys, 40 us with eight single
  // 2-byte reads per operand and P rounded in integer instructions, 34 us so; 31 us with V's first loads under the statistics
  // and the column sums folded.  K and V alone take 24 us at the rate of a copy.)
  const uint16_t* vtr = kt + (4 * half + ((lane & 15) >> 2)) * RS + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  f32x16_t oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int it = 0; it < NS; ++it) {
    MADAKV_WIN_PARK(it % PF)
    if (it + PF < NS) MADAKV_WIN_LOAD(vg, it % PF, it + PF)
#pragma unroll
    for (int j = 0; j < 16; ++j) lg[it][j] = fast_exp2(lg[it][j] - mloc);   // masked: exp2(NEG_BIG) = 0
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int st = 0; st < 2; ++st) {                       // two 16-key steps of the subtile
      uint32_t hi[4], lo[4];                               // round to nearest even, in pairs
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const win_f32x2_t pv = {lg[it][8 * st + 2 * i], lg[it][8 * st + 2 * i + 1]};
        hi[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pv, win_bf16x2_t));
        const win_f32x2_t rest = {pv[0] - bf16_lo(hi[i]), pv[1] - bf16_hi(hi[i])};
        lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, win_bf16x2_t));
      }
      const bf16x8_t pa_hi = __builtin_bit_cast(bf16x8_t, u32x4_t{hi[0], hi[1], hi[2], hi[3]});
      const bf16x8_t pa_lo = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], lo[2], lo[3]});
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        // V[key of contraction index 8 half + i][32 db + col], keys 16 st + 8 (i >> 2) + 4 half + (i & 3): transposing reads
        const win_s16x4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((win_lds_s16x4_ptr_t)(vtr + 16 * st * RS + db * 32));
        const win_s16x4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((win_lds_s16x4_ptr_t)(vtr + (16 * st + 8) * RS + db * 32));
        const bf16x8_t vb = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa_hi, vb, oacc[db], 0, 0, 0);
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa_lo, vb, oacc[db], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
#undef MADAKV_WIN_LOAD
#undef MADAKV_WIN_PARK

  // ---- the head-wide statistics (by now the other workgroups have normally posted theirs)
  collect_row_stats<D>(a, hv, split, fs, Lh, Mh, rowbase, kg, qs, part, offs, nullptr, pm, &s_fail);
  __syncthreads();
  if (split == 0 && wa.lse && tid < Mh) wa.lse[(lb * a.H + kvh) * (long long)a.G * a.W + rowbase + tid] = offs[tid] * 0.6931471805599453f;
  const float mxw = part[(wave * 32 + col) * 2];           // the wave's own row maximum again
  const float rs = mxw > NEG_BIG ? fast_exp2(mxw - offs[col]) : 0.f;   // this wave's p times rs = the softmax entry

  // ---- Eq. 7 column sums
#pragma unroll
  for (int it = 0; it < NS; ++it) {
    const int t0 = chunk0 + (it * 4 + wave) * 32;
    float cs[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) cs[j] = lg[it][j] * rs;
    const float sum = half_fold<1>(cs, lane);                 // over the 32 rows: psi of the key that this lane (of the first 16) has
    const int key = t0 + 8 * ((lane & 15) >> 2) + 4 * half + (lane & 3);
    // (more than 32 proxy rows: the block's share of psi, added to the other blocks' in block order afterwards)
    float* psi_dst = a.rb_count > 1 ? a.psi_part + (hv % a.rb_count) * a.psi_part_stride : a.psi;
    if (col < 16 && key < chunk1) psi_dst[(long long)head * a.L + key] = sum;
  }
  // ---- O rows take their factor: row m of the tile sits in lane m's rs
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const float f = __shfl(rs, 8 * (j >> 2) + 4 * half + (j & 3), 64);
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db][j] *= f;
  }

  // ---- the four waves' shares of O, added in wave order, CR output columns at a time through the K/V tiles' space
  constexpr int DPR = D == 128 ? 2 : 1, CR = 32 * DPR;     // 4 waves x 32 rows x CR floats fit the four tiles
  static_assert(4 * 32 * CR * sizeof(float) <= 4 * 32 * RS * sizeof(uint16_t), "the shares must fit the tiles");
  float* fl = reinterpret_cast<float*>(kt_all);           // [4 waves][32 rows][CR]
  float* op = wa.opart + ((long long)hv * fs + split) * 32 * D;
  for (int rd = 0; rd < DB / DPR; ++rd) {
    __syncthreads();
#pragma unroll
    for (int dd = 0; dd < DPR; ++dd)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int m = 8 * (j >> 2) + 4 * half + (j & 3);   // O[row m][column 32 db + col] sits in oacc[db][j]
        fl[(wave * 32 + m) * CR + dd * 32 + col] = oacc[rd * DPR + dd][j];
      }
    __syncthreads();
    for (int e = tid; e < 32 * CR; e += SCORE_THREADS) {
      const int m = e / CR, c = e % CR;
      op[m * D + rd * CR + c] = ((fl[(0 * 32 + m) * CR + c] + fl[(1 * 32 + m) * CR + c]) + fl[(2 * 32 + m) * CR + c]) + fl[(3 * 32 + m) * CR + c];
    }
  }
}

// ------------------------------------------------------------------------------------
// The same for more than 64 proxy rows (grouped queries) in calls that fill the chip (win_one_pass): one pass over K and V for
// all of them instead of one per block of 32.  The row statistics come from sweep 1 of the wide scoring kernels (a pass over K of its own), so the softmax
// entries are final when they are formed: nothing is exchanged, O is never rescaled, and a workgroup may take as many keys
// as suits the chip.  Wave w owns the rows of block w (Q fragments and 32 x d of O in registers), the waves share the keys:
// tiles of K and V come straight into a ring of three (global_load_lds, as in score_wide_dma_kernel, all LDS traffic of the
// loop written out for the same reason).  Per 32 keys: S^T = K Q^T (a lane holds one row against 16 keys), exp2, the
// row-wise sums for psi over the lanes, P as bf16 hi + lo parts straight from those registers into O += P V, the V
// fragments through transposing LDS reads (four keys of 16 columns per 16 lanes).  The 16-byte pieces of a row are permuted
// in the tile so that both kinds of reads are spread over all banks (tile_swizzle).
// Per logit one exp2, two conversions and 3 instructions of the sum over rows; 24 matrix instructions per 32 keys and block (more
// with third parts), one after the other in a wave; two waves per SIMD overlap them in part: by the counters the matrix unit
// is busy 36% of the time, a wave issues vector or matrix instructions in 28% of its cycles and waits in 25%; K and V
// are fetched once.
// 28 layers x 4 heads of 32K keys with 224 rows: 2.73 ms in seven passes -> 1.22 ms for the whole call (sweep 1 0.34, this
// kernel 0.80: K and V once is 1.9 GB, 0.3 ms; the matrix instructions alone 0.35 ms).
// ------------------------------------------------------------------------------------
template <int D> __device__ __forceinline__ int tile_swizzle(int row) {       // piece c of a row sits in slot c ^ tile_swizzle(row)
  return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : ((row & 2) << 1) | ((row >> 2) & 3);
}

// sums over the 32 lanes of a half wave of 16 values each, except for the last step: lanes 16 apart keep their halves.
// Lane c (its low four bits) ends with value c.  Fixed order.
__device__ __forceinline__ float lanes_sum16(const float (&v)[16], int lane) {
#define MADAKV_XCHG(ctrl, x) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), ctrl, 0xF, 0xF, true))
  float a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) { const bool u = lane & 8; const float send = u ? v[i] : v[i + 8]; a[i] = (u ? v[i + 8] : v[i]) + MADAKV_XCHG(0x140, send); }   // row_mirror
#pragma unroll
  for (int i = 0; i < 4; ++i) { const bool u = lane & 4; const float send = u ? a[i] : a[i + 4]; b[i] = (u ? a[i + 4] : a[i]) + MADAKV_XCHG(0x141, send); }   // row_half_mirror
#pragma unroll
  for (int i = 0; i < 2; ++i) { const bool u = lane & 2; const float send = u ? b[i] : b[i + 2]; c[i] = (u ? b[i + 2] : b[i]) + MADAKV_XCHG(0x1B, send); }    // quad_perm [3,2,1,0]
  const bool u = lane & 1;
  const float send = u ? c[0] : c[1];
  return (u ? c[1] : c[0]) + MADAKV_XCHG(0xB1, send);                                                                                                          // quad_perm [1,0,3,2]
#undef MADAKV_XCHG
}

constexpr float WINDOW_THIRD_PART_FROM = 0.0625f;
template <int D, int NW>   // NW waves of one row block each
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void window_wide_kernel(WinArgs wa) {
  const ScoreArgs& a = wa.s;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  constexpr int NT = NW * 64, TK = NW * 8;    // keys per tile
  constexpr int KS = D / 16, DB = D / 32, PPR = D / 8, ROWB = D * 2;
  constexpr int TILEB = TK * ROWB;            // one of K, one of V per ring slot
  constexpr int LPT = 2 * TK * PPR / NT;      // load instructions per thread and tile
  constexpr int NPART = 2 * NW;               // shares of a key's psi: per wave one of rows 0-15 and one of rows 16-31 of its block
  static_assert(LPT == 4 || LPT == 2, "the wait below is written for these");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const uint32_t ring_lds = (uint32_t)(uintptr_t)smem, red_lds = ring_lds + DMA_NBUF * 2 * TILEB;    // red: [2][NPART][TK] floats

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = blockIdx.x, head = a.head0 + blockIdx.y, kvh = head % a.H;
  const long long lb = head / a.H;
  const uint16_t* qg = reinterpret_cast<const uint16_t*>(a.q_win) + (lb * a.H + kvh) * (long long)a.G * a.W * D;
  const unsigned char* kg = reinterpret_cast<const unsigned char*>(a.k) + (long long)head * a.L * ROWB;
  const unsigned char* vg = reinterpret_cast<const unsigned char*>(wa.v) + (long long)head * a.L * ROWB;
  const int chunk0 = split * a.chunk, chunk1 = min(a.L, chunk0 + a.chunk);
  const int ntiles = (chunk1 - chunk0 + TK - 1) / TK;
  const int half = lane >> 5, col = lane & 31;
  const int row = wave * 32 + col;            // this lane's proxy row
  const bool active = wave < a.rb_count;      // (uniform) the wave has a block
  const int first_masked = a.L - a.W + 1;     // keys below this are visible to every proxy row
  const int pos = a.L - a.W + (row % a.W);    // last key the row sees

#define MADAKV_WW_ISSUE(T)                                                                           \
  {                                                                                                  \
    const int tt = (T);                                                                              \
    const int lt0 = chunk0 + tt * TK;                                                                \
    const uint32_t slot_lds = ring_lds + (uint32_t)(tt % DMA_NBUF) * (2 * TILEB);                    \
    _Pragma("unroll") for (int j = 0; j < LPT; ++j) {                                                \
      const int first = __builtin_amdgcn_readfirstlane((wave * LPT + j) * 64);                       \
      const bool is_v = first >= TK * PPR;                                                           \
      const int piece = first - (is_v ? TK * PPR : 0) + lane;                                        \
      const int r = piece / PPR;                                                                     \
      const int lkey = min(lt0 + r, a.L - 1);                                                        \
      const unsigned char* src = (is_v ? vg : kg) + (long long)lkey * ROWB + (((piece % PPR) ^ tile_swizzle<D>(r)) * 16); \
      const uint32_t dst = __builtin_amdgcn_readfirstlane(slot_lds + (uint32_t)first * 16u);         \
      __builtin_amdgcn_global_load_lds((global_void_ptr_t)(uintptr_t)src, (lds_void_ptr_t)(uintptr_t)dst, 16, 0, 0); \
    }                                                                                                \
  }
  // the row's offset (max + log2 sum over all its keys) and its Q fragments: before the first key is on its way
  // (maximum and 1 / sum kept apart: max + log2(sum) rounds to 1e-6 of every entry)
  float rmax = __builtin_inff(), rinv = 0.f;  // padding rows: exp2(-inf) = 0
  bf16x8_t qfrag[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    // (padding rows: the last row once more; zeros would turn an infinite key element into NaN, which the key's psi takes in)
    qfrag[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qg + (long long)min(row, a.M - 1) * D + half * (D / 2) + ks * 8));
  }
  if (row < a.M) {
    const float* rs = a.rowstat + (long long)head * a.nsplit * a.mpad * 2 + row * 2;
    rmax = rs[0]; rinv = 1.0f / rs[1];
    if (split == 0 && half == 0 && wa.lse) wa.lse[(lb * a.H + kvh) * (long long)a.G * a.W + row] = (rs[0] + log2f(rs[1])) * 0.6931471805599453f;
  }
  MADAKV_WW_ISSUE(0)
  MADAKV_WW_ISSUE(min(1, ntiles - 1))

  // where this lane's operand pieces sit, relative to a 32-key subtile's first byte
  uint32_t koff[KS], voff[2][DB];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) koff[ks] = (uint32_t)(col * ROWB + (((half * KS + ks) ^ tile_swizzle<D>(col)) * 16));
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const int r = 8 * e + 4 * half + ((lane >> 2) & 3), c = 4 * db + 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
      voff[e][db] = (uint32_t)(r * ROWB + ((c ^ tile_swizzle<D>(r)) * 16) + (lane & 1) * 8);
    }
  f32x16_t oacc[DB];                          // O[row 8 (j >> 2) + 4 half + (j & 3) of the block][column 32 db + col]
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // psi of the keys of tile T: their shares added in wave order
#define MADAKV_WW_PSI(T)                                                                             \
  if (tid < TK) {                                                                                    \
    const int key = chunk0 + (T) * TK + tid;                                                         \
    const uint32_t r4 = red_lds + (uint32_t)((((T) & 1) * NPART * TK + tid) * 4);                    \
    float sum = 0.f;                                                                                 \
    _Pragma("unroll") for (int w = 0; w < NPART; w += 4) {                                           \
      float c0, c1, c2, c3;                                                                          \
      asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %5\n\tds_read_b32 %2, %6\n\tds_read_b32 %3, %7\n\ts_waitcnt lgkmcnt(0)" \
                   : "=&v"(c0), "=&v"(c1), "=&v"(c2), "=&v"(c3)                                      \
                   : "v"(r4 + w * TK * 4), "v"(r4 + (w + 1) * TK * 4), "v"(r4 + (w + 2) * TK * 4), "v"(r4 + (w + 3) * TK * 4) : "memory"); \
      sum = (((sum + c0) + c1) + c2) + c3;                                                           \
    }                                                                                                \
    if (key < chunk1) __builtin_nontemporal_store(sum, a.psi + ((long long)head * a.L + key));       \
  }

  for (int t = 0; t < ntiles; ++t) {
    // tile t has landed (the loads of tile t + 1 may still be out), this wave's LDS accesses of the last trip are
    // done; after the barrier that holds for every wave, and nobody reads tile t - 1 any more
    if (LPT == 4) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    MADAKV_WW_ISSUE(min(t + 2, ntiles - 1))    // into the slot of tile t - 1 (past the end: the last tile once more, which keeps the count of loads in flight)
    if (t > 0) { MADAKV_WW_PSI(t - 1) }
    const uint32_t tile_lds = ring_lds + (uint32_t)(t % DMA_NBUF) * (2 * TILEB);
    const int tile_end = chunk0 + (t + 1) * TK;
    const bool tail = tile_end > first_masked || tile_end > chunk1;
    if (active) {
#pragma unroll 1
      for (int s0 = 0; s0 < TK / 32; ++s0) {
        const uint32_t kb = tile_lds + (uint32_t)s0 * 32 * ROWB, vb0 = kb + TILEB;
        bf16x8_t kfrag[KS];
        if constexpr (KS == 8) {
          asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                       "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
                       "s_waitcnt lgkmcnt(0)"
                       : "=&v"(kfrag[0]), "=&v"(kfrag[1]), "=&v"(kfrag[2]), "=&v"(kfrag[3]), "=&v"(kfrag[4 % KS]), "=&v"(kfrag[5 % KS]), "=&v"(kfrag[6 % KS]), "=&v"(kfrag[7 % KS])
                       : "v"(kb + koff[0]), "v"(kb + koff[1]), "v"(kb + koff[2]), "v"(kb + koff[3]),
                         "v"(kb + koff[4 % KS]), "v"(kb + koff[5 % KS]), "v"(kb + koff[6 % KS]), "v"(kb + koff[7 % KS]) : "memory");
        } else {
          asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                       : "=&v"(kfrag[0]), "=&v"(kfrag[1]), "=&v"(kfrag[2]), "=&v"(kfrag[3])
                       : "v"(kb + koff[0]), "v"(kb + koff[1]), "v"(kb + koff[2]), "v"(kb + koff[3]) : "memory");
        }
        f32x16_t x = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag[ks], qfrag[ks], x, 0, 0, 0);
        // V fragments of both 16-key steps, under the contraction: vr[st][e][db] = keys 16 st + 8 e + 4 half .. + 3 of column 32 db + col
        u32x2_t vr[2][2][DB];
        if constexpr (DB == 4) {
          asm volatile("ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %17\n\tds_read_b64_tr_b16 %2, %18\n\tds_read_b64_tr_b16 %3, %19\n\t"
                       "ds_read_b64_tr_b16 %4, %20\n\tds_read_b64_tr_b16 %5, %21\n\tds_read_b64_tr_b16 %6, %22\n\tds_read_b64_tr_b16 %7, %23\n\t"
                       "ds_read_b64_tr_b16 %8, %16 offset:4096\n\tds_read_b64_tr_b16 %9, %17 offset:4096\n\tds_read_b64_tr_b16 %10, %18 offset:4096\n\tds_read_b64_tr_b16 %11, %19 offset:4096\n\t"
                       "ds_read_b64_tr_b16 %12, %20 offset:4096\n\tds_read_b64_tr_b16 %13, %21 offset:4096\n\tds_read_b64_tr_b16 %14, %22 offset:4096\n\tds_read_b64_tr_b16 %15, %23 offset:4096\n\t"
                       "s_waitcnt lgkmcnt(0)"
                       : "=&v"(vr[0][0][0]), "=&v"(vr[0][0][1]), "=&v"(vr[0][0][2 % DB]), "=&v"(vr[0][0][3 % DB]),
                         "=&v"(vr[0][1][0]), "=&v"(vr[0][1][1]), "=&v"(vr[0][1][2 % DB]), "=&v"(vr[0][1][3 % DB]),
                         "=&v"(vr[1][0][0]), "=&v"(vr[1][0][1]), "=&v"(vr[1][0][2 % DB]), "=&v"(vr[1][0][3 % DB]),
                         "=&v"(vr[1][1][0]), "=&v"(vr[1][1][1]), "=&v"(vr[1][1][2 % DB]), "=&v"(vr[1][1][3 % DB])
                       : "v"(vb0 + voff[0][0]), "v"(vb0 + voff[0][1]), "v"(vb0 + voff[0][2 % DB]), "v"(vb0 + voff[0][3 % DB]),
                         "v"(vb0 + voff[1][0]), "v"(vb0 + voff[1][1]), "v"(vb0 + voff[1][2 % DB]), "v"(vb0 + voff[1][3 % DB]) : "memory");
        } else {
          asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %9\n\tds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %3, %11\n\t"
                       "ds_read_b64_tr_b16 %4, %8 offset:2048\n\tds_read_b64_tr_b16 %5, %9 offset:2048\n\tds_read_b64_tr_b16 %6, %10 offset:2048\n\tds_read_b64_tr_b16 %7, %11 offset:2048\n\t"
                       "s_waitcnt lgkmcnt(0)"
                       : "=&v"(vr[0][0][0]), "=&v"(vr[0][0][1]), "=&v"(vr[0][1][0]), "=&v"(vr[0][1][1]),
                         "=&v"(vr[1][0][0]), "=&v"(vr[1][0][1]), "=&v"(vr[1][1][0]), "=&v"(vr[1][1][1])
                       : "v"(vb0 + voff[0][0]), "v"(vb0 + voff[0][1]), "v"(vb0 + voff[1][0]), "v"(vb0 + voff[1][1]) : "memory");
        }
        if (tail) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int key = chunk0 + t * TK + s0 * 32 + 8 * (j >> 2) + 4 * half + (j & 3);
            x[j] = key < chunk1 && key <= pos ? x[j] : NEG_BIG;
          }
        }
        float pv[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) pv[j] = fast_exp2(fmaf(x[j], a.scale_log2, -rmax));
        // Two bf16 parts leave 2^-18 of an entry, which shows where the entry is large (the row's largest is 1): there a third
        // part goes in as well, so that the error against 64 bits stays below what exponentiating against every wave's own
        // maximum gave (32K keys: 0.75e-6 of the result, two parts 1.13e-6, the kernel above 1.04e-6; from 1/4 on 0.78e-6, from 1/64
        // on 0.74e-6, a few per cent of the time apart).
        float big = pv[0];
#pragma unroll
        for (int j = 1; j < 16; ++j) big = fmaxf(big, pv[j]);
        const bool three = __any(big > WINDOW_THIRD_PART_FROM);
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          uint32_t hi[4], lo[4];
          f32x2_t left[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const f32x2_t p2 = {pv[8 * st + 2 * i], pv[8 * st + 2 * i + 1]};
            hi[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(p2, bf16x2_t));          // round to nearest even
            const f32x2_t rest = {p2[0] - bf16_lo(hi[i]), p2[1] - bf16_hi(hi[i])};
            lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2_t));
            left[i] = f32x2_t{rest[0] - bf16_lo(lo[i]), rest[1] - bf16_hi(lo[i])};
          }
          const bf16x8_t ph = __builtin_bit_cast(bf16x8_t, u32x4_t{hi[0], hi[1], hi[2], hi[3]}), pl = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], lo[2], lo[3]});
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, u32x4_t{vr[st][0][db][0], vr[st][0][db][1], vr[st][1][db][0], vr[st][1][db][1]});
            oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ph, vf, oacc[db], 0, 0, 0);
            oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pl, vf, oacc[db], 0, 0, 0);
          }
          if (three) {
            uint32_t ll[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) ll[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(left[i], bf16x2_t));
            const bf16x8_t p3 = __builtin_bit_cast(bf16x8_t, u32x4_t{ll[0], ll[1], ll[2], ll[3]});
#pragma unroll
            for (int db = 0; db < DB; ++db) {
              const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, u32x4_t{vr[st][0][db][0], vr[st][0][db][1], vr[st][1][db][0], vr[st][1][db][1]});
              oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p3, vf, oacc[db], 0, 0, 0);
            }
          }
        }
        // Eq. 7: this wave's shares of the 32 keys' psi (lane c of a 16-lane row: the key of accumulator register c)
#pragma unroll
        for (int j = 0; j < 16; ++j) pv[j] *= rinv;
        const float cs = lanes_sum16(pv, lane);
        const int c16 = lane & 15;
        const uint32_t dst = red_lds + (uint32_t)((((t & 1) * NPART + wave * 2 + ((lane >> 4) & 1)) * TK + s0 * 32 + 8 * (c16 >> 2) + 4 * half + (c16 & 3)) * 4);
        asm volatile("ds_write_b32 %0, %1" :: "v"(dst), "v"(cs) : "memory");
      }
    } else {                                    // a wave without rows: nothing to add
      for (int x = lane; x < 2 * TK; x += 64) {
        const uint32_t dst = red_lds + (uint32_t)((((t & 1) * NPART + wave * 2) * TK + x) * 4);
        asm volatile("ds_write_b32 %0, %1" :: "v"(dst), "v"(0.f) : "memory");
      }
    }
  }
#undef MADAKV_WW_ISSUE
  // nothing may still be on its way into this workgroup's LDS when it ends
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  MADAKV_WW_PSI(ntiles - 1)
#undef MADAKV_WW_PSI
  if (active) {                                 // this chunk's share of O
    float* op = wa.opart + (((long long)head * a.rb_count + wave) * a.fsplit + split) * 32 * D;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int m = 8 * (j >> 2) + 4 * half + (j & 3);
      const float f = __shfl(rinv, m, 64);      // the factor of row m sits in lane m
#pragma unroll
      for (int db = 0; db < DB; ++db) op[m * D + db * 32 + col] = oacc[db][j] * f;
    }
  }
}

// out[row][c] = sum over the head's chunks, in chunk order, of their shares.  Grid (head, slice of
// 256 float4 of the 32 x d tile); eight shares in flight per thread.
__global__ __launch_bounds__(256) void window_attn_reduce_kernel(WinArgs wa) {
  const ScoreArgs& a = wa.s;
  const int hv = a.head0 + blockIdx.x;
  const int head = hv / a.rb_count, rowbase = (hv % a.rb_count) * 32;
  const int kvh = head % a.H;
  const long long lb = head / a.H;
  const int e4 = blockIdx.y * 256 + threadIdx.x;           // float4 index in the [32][d] tile
  const int tile4 = 32 * a.d / 4;
  if (e4 >= min(a.M - rowbase, 32) * a.d / 4) return;
  const f32x4_t* op = reinterpret_cast<const f32x4_t*>(wa.opart) + (long long)hv * a.fsplit * tile4 + e4;
  f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
  int sp = 0;
  for (; sp + 8 <= a.fsplit; sp += 8) {
    f32x4_t x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = __builtin_nontemporal_load(op + (long long)(sp + j) * tile4);
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += x[j];
  }
  for (; sp < a.fsplit; ++sp) sum += __builtin_nontemporal_load(op + (long long)sp * tile4);
  const long long o = ((lb * a.H + kvh) * (long long)a.G * a.W + rowbase) * a.d + (long long)e4 * 4;
  if (wa.out_fp32) *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(wa.out) + o) = sum;
  else {
    u32x2_t pk;
    pk[0] = (uint32_t)f32_to_bf16_rne(sum[0]) | ((uint32_t)f32_to_bf16_rne(sum[1]) << 16);
    pk[1] = (uint32_t)f32_to_bf16_rne(sum[2]) | ((uint32_t)f32_to_bf16_rne(sum[3]) << 16);
    *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(wa.out) + o) = pk;
  }
}

// ------------------------------------------------------------------------------------
// Plain FMA path: fp32 heads of more than FUSED_MAX_SPLIT chunks, and fp32 with given normalisers.  Same two sweeps.
// Sweep 1: wave w takes rows w, w+4, ...; lanes stride over the keys of the chunk.
// Sweep 2: one thread per key, loop over the rows.
// ------------------------------------------------------------------------------------
template <int PASS>
__global__ __launch_bounds__(SCORE_THREADS) void score_simple_kernel(ScoreArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* qs = reinterpret_cast<float*>(smem);          // [M][d]
  float* offs = qs + a.M * a.d;                        // [M]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = blockIdx.x;
  const int head = a.head0 + blockIdx.y;
  const int kvh = head % a.H;
  const long long lb = head / a.H;
  const float* qg = reinterpret_cast<const float*>(a.q_win) + (lb * a.H + kvh) * (long long)a.G * a.W * a.d;
  const float* kg = reinterpret_cast<const float*>(a.k) + (long long)head * a.L * a.d;
  for (int e = tid; e < a.M * a.d; e += SCORE_THREADS) qs[e] = qg[e];
  if (PASS == 2) {
    const float* rs = a.rowstat + (long long)head * a.nsplit * a.mpad * 2;
    for (int r = tid; r < a.M; r += SCORE_THREADS) {
      float m = NEG_BIG, l = 0.f;
      if (a.lse) { m = a.lse[(lb * a.H + kvh) * (long long)a.G * a.W + r] * 1.4426950408889634f; l = 1.f; }
      else for (int s = 0; s < a.nmerge; ++s) merge_ml(m, l, rs[(s * a.mpad + r) * 2], rs[(s * a.mpad + r) * 2 + 1]);
      offs[r] = m + log2f(l);
    }
  }
  __syncthreads();
  const int chunk0 = split * a.chunk, chunk1 = min(a.L, chunk0 + a.chunk);
  if (PASS == 1) {
    float* rs = a.rowstat + ((long long)head * a.nsplit + split) * a.mpad * 2;
    for (int r = wave; r < a.mpad; r += 4) {
      float m = NEG_BIG, l = 0.f;
      if (r < a.M) {
        const int pos = a.L - a.W + (r % a.W);
        for (int key = chunk0 + lane; key < chunk1 && key <= pos; key += 64) {
          float s = 0.f;
          for (int e = 0; e < a.d; ++e) s = fmaf(qs[r * a.d + e], kg[(long long)key * a.d + e], s);
          float s2 = s * a.scale_log2;
          float mn = fmaxf(m, s2);
          l = l * exp2f(m - mn) + exp2f(s2 - mn);
          m = mn;
        }
        for (int o = 1; o < 64; o <<= 1) {
          float m2 = __shfl_xor(m, o, 64), l2 = __shfl_xor(l, o, 64);
          merge_ml(m, l, m2, l2);
        }
      }
      if (lane == 0) { rs[r * 2] = m; rs[r * 2 + 1] = l; }
    }
  } else {
    for (int key = chunk0 + tid; key < chunk1; key += SCORE_THREADS) {
      float sum = 0.f;
      for (int r = 0; r < a.M; ++r) {
        const int pos = a.L - a.W + (r % a.W);
        if (key > pos) continue;
        float s = 0.f;
        for (int e = 0; e < a.d; ++e) s = fmaf(qs[r * a.d + e], kg[(long long)key * a.d + e], s);
        sum += exp2f(s * a.scale_log2 - offs[r]);
      }
      a.psi[(long long)head * a.L + key] = sum;
    }
  }
}

// ------------------------------------------------------------------------------------
// With many chunks per head every sweep-2 workgroup would redo the same merge of the chunks' row
// statistics: this small kernel does it once per head and leaves the result in the first chunk's slot.
__global__ __launch_bounds__(256) void score_combine_kernel(ScoreArgs a) {
  const int head = a.head0 + blockIdx.x;
  float* rs = a.rowstat + (long long)head * a.nsplit * a.mpad * 2;
  for (int r = threadIdx.x; r < a.mpad; r += blockDim.x) {
    float m = NEG_BIG, l = 0.f;
    for (int s = 0; s < a.nsplit; ++s) merge_ml(m, l, rs[(s * a.mpad + r) * 2], rs[(s * a.mpad + r) * 2 + 1]);
    rs[r * 2] = m; rs[r * 2 + 1] = l;
  }
}

// chunks per head from which the merge is hoisted out of sweep 2
constexpr int COMBINE_FROM = 8;
#ifndef MADAKV_WIDE_WGS
#define MADAKV_WIDE_WGS 768
#endif
constexpr int WIDE_WGS = MADAKV_WIDE_WGS;       // workgroups the chunking of sweep 1 aims at with more than 64 proxy rows

static bool use_mfma(const Dims& dm, int dtype) { return dtype == MADAKV_BF16 && (dm.d == 64 || dm.d == 128); }

ScorePlan score_plan(const Dims& dm, int dtype) {
  (void)dtype;
  ScorePlan p;
  p.mpad = (dm.M + 31) / 32 * 32;
  // Both sweeps run over all heads of the call in one launch each, at most 65535 heads at a
  // time (the grid's y limit).  (Splitting a call into groups of heads whose K fits the 256 MB
  // memory-side cache, so that the second sweep finds its data there, was measured slower at
  // every group size.)
  p.group_heads = std::min(dm.heads, 65535);
  // enough workgroups per launch to fill 256 CUs several times over; chunks are a multiple
  // of 128 keys (4 waves x 32-key tiles) and at least 256 keys long
  int want = std::max(1, (2048 + p.group_heads - 1) / p.group_heads);
  int max_split = std::max(1, dm.L / 256);
  // (more than 64 proxy rows: the arithmetic per key is several times larger and a workgroup's start, its Q
  // fragments and first tile, costs more, so about two workgroups per CU with long chunks)
  if (p.mpad > 64) { want = std::max(1, (WIDE_WGS + p.group_heads / 2) / p.group_heads); max_split = std::max(1, dm.L / 1024); }
  int ns = std::min(std::min(want, max_split), 128);
  int chunk = ((dm.L + ns - 1) / ns + 127) / 128 * 128;
  p.nsplit = (dm.L + chunk - 1) / chunk;
  p.chunk = chunk;
  return p;
}

// One sweep when the logits of a workgroup's keys fit in registers (at most two row blocks) and a
// head has few enough chunks that all its workgroups are certain to be on the chip together.
constexpr int FUSED_NS1 = MADAKV_FUSED_NS1, FUSED_NS2 = MADAKV_FUSED_NS2;
constexpr int FUSED_MAX_SPLIT = MADAKV_FUSED_MAX_SPLIT;
static int fused_blocks(const Dims& dm) { return dm.M <= 64 ? 1 : (dm.M + 63) / 64; }   // blocks of 64 proxy rows handled like heads
// fp32: half the keys per workgroup, since a wave takes 4-8 times as long over a subtile; where even a call over the whole model
// leaves most of the chip idle, a quarter or an eighth.  (By the model and not by the call: psi depends on it in the last bits, and
// is the same layer by layer and in one call.)  Scores and statistics, 4 / 2 / 1 subtiles per wave: 8 heads of 1K keys and 64 dims
// 23.6 / 20.5 / 18.7 us, 64 of them 24.8 / 22.1 / 21.4, 256 33 / 43 / 56; 32 heads of 1K and 128 dims 29 / 24 / 22, of 4K 33 / 42 / 57.
constexpr int FUSED_NS_F32 = 4;
static int fused_subtiles(const Dims& dm, int dtype) {
  if (dtype != MADAKV_FP32) return dm.M <= 32 ? FUSED_NS1 : FUSED_NS2;
  for (int ns = 1; ns < FUSED_NS_F32; ns *= 2) {
    const int chunks = (dm.L + 128 * ns - 1) / (128 * ns);
    if (chunks <= FUSED_MAX_SPLIT && (long long)dm.model_heads * fused_blocks(dm) * chunks <= (dm.d == 64 ? 512 : 256)) return ns;
  }
  return FUSED_NS_F32;
}
static int fused_chunk(const Dims& dm, int dtype) { return 4 * 32 * fused_subtiles(dm, dtype); }
static int fused_split(const Dims& dm, int dtype) { return (dm.L + fused_chunk(dm, dtype) - 1) / fused_chunk(dm, dtype); }
static int fused_mpad(const Dims& dm) { return dm.M <= 32 ? 32 : 64; }
// exchange levels: one up to FUSED_MAX_SPLIT chunks per head, two (groups of XCHG_GROUP chunks) up to
// FUSED_MAX_SPLIT_2L.  All workgroups of a head wait for each other, so a head must never need more
// workgroups than the chip holds at once (512 of this kernel): half of that is the limit.
constexpr int FUSED_MAX_SPLIT_2L = 256;
static int xchg_groups(int split) { return split <= FUSED_MAX_SPLIT ? 0 : (split + XCHG_GROUP - 1) / XCHG_GROUP; }
// (More than 64 proxy rows: the prompt's keys take the two-sweep kernels above, which are bound by their vector
// arithmetic either way and twice as fast as one sweep per block of 64 rows; the ragged rows of a reduced cache
// still go through the one-sweep kernel in blocks.)
// Long heads whose chunks pack the workgroup slots badly.  A workgroup keeps its slot until its whole head is
// through; the chip holds FUSED_SLOTS workgroups of the kernel; k = slots / chunks heads fit at once, and when a
// few chunks fewer per head would let k + 1 fit (171 chunks at a 128K context: 3 x 171 = 513), every (k + 1)-th
// head's last chunk waits for a slot while its head-mates hold theirs idle.  Those few last chunks per head then
// run ahead of the launch of the others (ScoreArgs::nstrag).  Returns their number (0: nothing to gain).
constexpr int FUSED_SLOTS = 512, FUSED_MAX_PARKED = 8;
static int fused_parked_chunks(int split) {
  if (split <= FUSED_MAX_SPLIT) return 0;                 // (the parked chunks' words live at the group level)
  const int k = FUSED_SLOTS / split, fewer = FUSED_SLOTS / (k + 1);
  const int n = split - fewer;
  return (fewer > FUSED_MAX_SPLIT && n >= 1 && n <= FUSED_MAX_PARKED && k * split * 10 < FUSED_SLOTS * 9) ? n : 0;
}
static size_t fused_park_bytes(const Dims& dm, int dtype);
static bool fused_fits(const Dims& dm, int dtype) {
  // fp32: more than 64 proxy rows in blocks of 64 (the alternative is the plain FMA kernels); its LDS holds one or two workgroups
  // per compute unit, so only heads of up to FUSED_MAX_SPLIT chunks (32768 keys) are certain to be on the chip as a whole
  if (dtype == MADAKV_FP32) return fused_split(dm, dtype) <= FUSED_MAX_SPLIT && (long long)dm.heads * fused_blocks(dm) <= 65535;
  return use_mfma(dm, dtype) && dm.M <= 64 && fused_split(dm, dtype) <= FUSED_MAX_SPLIT_2L && dm.heads <= 65535;
}
static bool use_fused(const Dims& dm, int dtype) {
  const char* e = getenv("MADAKV_SCORE_TWO_SWEEPS");      // diagnostic switch: the two-sweep kernels everywhere
  const bool off = e && atoi(e) != 0;
  return !off && fused_fits(dm, dtype);
}

static size_t rowstat_bytes(const Dims& dm, int dtype) {
  ScorePlan p = score_plan(dm, dtype);
  return ((size_t)dm.heads * p.nsplit * p.mpad * 2 * sizeof(float) + 255) / 256 * 256;
}
static size_t xchg_bytes(const Dims& dm, int dtype) {
  const size_t per_head = (size_t)(fused_split(dm, dtype) + xchg_groups(fused_split(dm, dtype))) * fused_mpad(dm);
  return fused_fits(dm, dtype) ? ((size_t)dm.heads * fused_blocks(dm) * per_head * 8 + 255) / 256 * 256 : 0;
}
static size_t fused_park_bytes(const Dims& dm, int dtype) {
  if (!fused_fits(dm, dtype)) return 0;
  const int n = fused_parked_chunks(fused_split(dm, dtype));
  const int ns = fused_subtiles(dm, dtype), nrb = fused_mpad(dm) / 32;
  // the parked logits (one float per thread and logit register) and the heads' row offsets
  return n ? ((size_t)dm.heads * n * ns * nrb * 16 * SCORE_THREADS * sizeof(float) + (size_t)dm.heads * fused_mpad(dm) * sizeof(float) + 255) / 256 * 256 : 0;
}
size_t score_ws_bytes(const Dims& dm, int dtype) {
  // the counter of lone workgroups, the row statistics of the two sweeps, the store sink, the one-sweep kernel's
  // per-row-block copies of psi when there are more than 64 proxy rows, its parked chunks.  (The size is that of the time when it
  // held the exchange words too, 0.1% of the keys: without that room the caches that a program allocates behind it end up elsewhere,
  // and where K and V are relative to each other decides up to 13% of a decode call over 32 heads of 4K rows, 13.7 to 15.7 us;
  // 1175 -> 1218 us for a generation at 128K.)
  const size_t part = fused_fits(dm, dtype) && fused_blocks(dm) > 1 ? (size_t)fused_blocks(dm) * dm.heads * dm.L * sizeof(float) : 0;
  return 256 + rowstat_bytes(dm, dtype) + 256 + xchg_bytes(dm, dtype) + part + fused_park_bytes(dm, dtype);
}

// psi = the row blocks' column sums added in block order (more than 64 proxy rows)
__global__ __launch_bounds__(256) void score_blocks_sum_kernel(const float* part, long long stride, int blocks, float* psi, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float acc = part[i];
  for (int b = 1; b < blocks; ++b) acc += part[b * stride + i];
  psi[i] = acc;
}

template <int D, int NRB, int NS, int KIND>
static void launch_fused_kernel(const ScoreArgs& a, dim3 grid, hipStream_t st) {
  constexpr int RS = (KIND == K_F32 ? 2 * D : D) + 8;
  const size_t lds = ((size_t)a.mpad + 4 * 32) * RS * 2 + ((size_t)4 * a.mpad * 3 + 4 * a.mpad + 512 + (size_t)4 * NS * a.mpad) * sizeof(float);
  if (lds > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&score_fused_kernel<D, NRB, NS, KIND>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((score_fused_kernel<D, NRB, NS, KIND>), grid, dim3(SCORE_THREADS), lds, st, a);
}
template <int D>
static void launch_fused_by_kind(const ScoreArgs& a, dim3 grid, hipStream_t st) {
  const bool one = a.mpad == 32;
  if (a.k_kind == K_F32) {
    if (a.subtiles == 1) { if (one) launch_fused_kernel<D, 1, 1, K_F32>(a, grid, st); else launch_fused_kernel<D, 2, 1, K_F32>(a, grid, st); }
    else if (a.subtiles == 2) { if (one) launch_fused_kernel<D, 1, 2, K_F32>(a, grid, st); else launch_fused_kernel<D, 2, 2, K_F32>(a, grid, st); }
    else { if (one) launch_fused_kernel<D, 1, FUSED_NS_F32, K_F32>(a, grid, st); else launch_fused_kernel<D, 2, FUSED_NS_F32, K_F32>(a, grid, st); }
  }
  else if (a.k_kind == K_E4M3) { if (one) launch_fused_kernel<D, 1, FUSED_NS1, K_E4M3>(a, grid, st); else launch_fused_kernel<D, 2, FUSED_NS2, K_E4M3>(a, grid, st); }
  else { if (one) launch_fused_kernel<D, 1, FUSED_NS1, K_BF16>(a, grid, st); else launch_fused_kernel<D, 2, FUSED_NS2, K_BF16>(a, grid, st); }
}

// the one-sweep kernel over `heads` heads (each cut into a.rb_count blocks of proxy rows)
template <int D>
static void launch_fused(const ScoreArgs& a, int heads, hipStream_t st) {
  const int vheads = heads * a.rb_count;
  const long long nx = (long long)vheads * a.xstride;
  if (a.fsplit > 1 && !a.xchg_clean)
    hipLaunchKernelGGL(score_xchg_init_kernel, dim3((unsigned)((nx + 255) / 256)), dim3(256), 0, st,
                       a.xchg + (long long)a.head0 * a.rb_count * a.xstride, nx);
  ScoreArgs b = a;
  b.head0 = a.head0 * a.rb_count;
  // (a.nstrag > 0: a.fsplit counts the chunks that wait for each other; the parked ones are the first in the grid)
  launch_fused_by_kind<D>(b, dim3(a.nstrag + a.fsplit, vheads), st);
  if (a.nstrag) {
    if (a.mpad == 32) hipLaunchKernelGGL((score_fused_finish_kernel<1, FUSED_NS1>), dim3(a.nstrag, vheads), dim3(SCORE_THREADS), 0, st, b);
    else hipLaunchKernelGGL((score_fused_finish_kernel<2, FUSED_NS2>), dim3(a.nstrag, vheads), dim3(SCORE_THREADS), 0, st, b);
  }
  if (a.rb_count > 1) {
    const long long n = (long long)heads * a.L;
    hipLaunchKernelGGL(score_blocks_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       a.psi_part + (long long)a.head0 * a.L, a.psi_part_stride, a.rb_count, a.psi + (long long)a.head0 * a.L, n);
  }
}

template <int D, int NRB>
static void launch_mfma_pair(const ScoreArgs& a0, int heads, size_t lds1, size_t lds2, hipStream_t st) {
  ScoreArgs a = a0;
  dim3 grid(a.nsplit, heads);
  if (lds1 > 48 * 1024 || lds2 > 48 * 1024) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&score_mfma_kernel<D, NRB, 1>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds1);
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&score_mfma_kernel<D, NRB, 2>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds2);
  }
  if (!a.lse) {
    hipLaunchKernelGGL((score_mfma_kernel<D, NRB, 1>), grid, dim3(SCORE_THREADS), lds1, st, a);
    if (a.nsplit >= COMBINE_FROM) { hipLaunchKernelGGL(score_combine_kernel, dim3(heads), dim3(256), 0, st, a); a.nmerge = 1; }
  }
  hipLaunchKernelGGL((score_mfma_kernel<D, NRB, 2>), grid, dim3(SCORE_THREADS), lds2, st, a);
}

// More than 64 proxy rows (up to 128 with WIDE8 = false, else up to 256).  Both sweeps: four waves of one or two row blocks,
// tiles of 64 keys.  Sweep 1 leaves every row's (max, sum) over the head's keys in the first chunk's slot.
template <int D, bool WIDE8, bool CLOSE>
static void launch_wide_sweep1(const ScoreArgs& a, int heads, hipStream_t st) {
  constexpr int NRB1 = WIDE8 ? 2 : 1;
  const size_t lds1 = (size_t)DMA_NBUF * 64 * D * 2;
  if (lds1 > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&score_wide_dma_kernel<D, 4, NRB1, 64, 1, 1, CLOSE>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds1);
  hipLaunchKernelGGL((score_wide_dma_kernel<D, 4, NRB1, 64, 1, 1, CLOSE>), dim3(a.nsplit, heads), dim3(256), lds1, st, a);
  hipLaunchKernelGGL(score_combine_kernel, dim3(heads), dim3(256), 0, st, a);
}
// Keys per chunk of sweep 2: what costs least, counted in tiles of a workgroup.  The chip holds two workgroups per compute unit;
// a last round that leaves compute units with one of them takes some 0.6 of a full one, a workgroup's start about a tile.
// 112 heads of 32K keys and 224 rows (statistics kernel included): 4 chunks per head (448 workgroups) 325 us, 5 (560, what "about
// 512" had meant) 389-442, 7 (784) 359, 9 (1008) 318, 14 (1568) 341, 16 (1792) 305, 27 (3024) 322; of 4K keys: 4 chunks 60, 5
// 70, 11 64; 128 heads of 16K and 128 rows: 4 chunks (512) 137, 5 170, 7 148, 8 138.  Few heads: flat (4 of 32K: 45-51 from
// 128 to 1800 workgroups).  psi does not depend on it.
static int wide_chunk2(int L, int heads) {
  constexpr int SLOTS = 512, TILE = 64;
  int best = 0; double least = 0.;
  const int most = std::max(1, std::min(L / 512, (2048 + heads - 1) / heads));
  for (int ns = 1; ns <= most; ++ns) {
    const int chunk = ((L + ns - 1) / ns + TILE - 1) / TILE * TILE;
    const long long wgs = (long long)heads * ((L + chunk - 1) / chunk);
    const int left = (int)(wgs % SLOTS);
    const double rounds = (double)(wgs / SLOTS) + (left == 0 ? 0. : left <= SLOTS / 2 ? 0.6 : 1.);
    const double cost = rounds * (chunk / TILE + 1);
    if (!best || cost < least) { best = chunk; least = cost; }
  }
  return best;
}
template <int D, bool WIDE8>
static void launch_wide_pair(const ScoreArgs& a0, int heads, hipStream_t st) {
  ScoreArgs a = a0;
  constexpr int NRB2 = WIDE8 ? 2 : 1;
  constexpr int BS2 = WIDE8 ? 1 : 2;            // (sweep 2: what the registers hold)
  const size_t lds2 = (size_t)DMA_NBUF * 64 * D * 2 + ((size_t)a.mpad + 2 * 4 * 64) * sizeof(float);
  static size_t allowed[64] = {};               // (per instantiation and device; set again only when a call needs more)
  int dev = 0;
  (void)hipGetDevice(&dev);
  size_t& allowed2 = allowed[dev & 63];
  if (lds2 > allowed2) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&score_wide_dma_kernel<D, 4, NRB2, 64, BS2, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds2);
    allowed2 = lds2;
  }
  if (!a.lse) {
    launch_wide_sweep1<D, WIDE8, false>(a, heads, st);
    a.nmerge = 1;
  }
  // sweep 2 in chunks of its own; a.nsplit stays what the row statistics are laid out by
  a.chunk = wide_chunk2(a.L, heads);
  dim3 grid2((a.L + a.chunk - 1) / a.chunk, heads);
  hipLaunchKernelGGL((score_wide_dma_kernel<D, 4, NRB2, 64, BS2, 2>), grid2, dim3(SCORE_THREADS), lds2, st, a);
}

// ---- the one-sweep kernel on ragged heads: the rows of a reduced cache, scored against the most recent queries
static int ragged_split(const Dims& dm, int longest_rows) { const int ck = fused_chunk(dm, MADAKV_BF16); return (std::max(longest_rows, 1) + ck - 1) / ck; }
bool score_ragged_supported(const Dims& dm, const madakv_config& c, int longest_rows) {
  return use_mfma(dm, c.dtype) && dm.M <= 256 && ragged_split(dm, longest_rows) <= FUSED_MAX_SPLIT &&
         (long long)dm.heads * fused_blocks(dm) <= 65535;
}
static size_t ragged_xchg_bytes(const Dims& dm, int longest_rows) {
  return ((size_t)dm.heads * fused_blocks(dm) * ragged_split(dm, longest_rows) * fused_mpad(dm) * 8 + 255) / 256 * 256;
}
// cache_rows: rows of the whole reduced cache (psi_c is indexed like it; so are the row blocks' copies)
size_t score_ragged_ws_bytes(const Dims& dm, const madakv_config& c, int longest_rows, long long cache_rows) {
  (void)c;
  return 256 + ragged_xchg_bytes(dm, longest_rows) + (fused_blocks(dm) > 1 ? (size_t)fused_blocks(dm) * cache_rows * sizeof(float) : 0);
}
hipError_t launch_score_ragged(const Dims& dm, const madakv_config& c, const void* q_recent, const void* k_c,
                               const int64_t* seg_off, const int32_t* seg_len, int longest_rows, long long cache_rows,
                               float* psi_c, void* ws, hipStream_t st) {
  ScoreArgs a;
  a.lse = nullptr; a.q_win = q_recent; a.k = k_c; a.psi = psi_c;
  a.status = reinterpret_cast<int*>(ws);
  a.rowstat = nullptr; a.sink = nullptr;
  a.xchg = reinterpret_cast<unsigned long long*>(static_cast<char*>(ws) + 256);
  a.seg_off = seg_off; a.seg_len = seg_len;
  a.H = dm.H; a.G = dm.G; a.d = dm.d; a.L = dm.L; a.W = dm.W; a.M = dm.M;
  a.mpad = fused_mpad(dm); a.nsplit = 0; a.nmerge = 0; a.chunk = 0; a.head0 = 0;
  a.fsplit = ragged_split(dm, longest_rows);
  a.xgroups = 0; a.xstride = (long long)a.fsplit * fused_mpad(dm);
  a.k_kind = c.cache_fp8 ? K_E4M3 : K_BF16;       // the reduced cache is what is scored here
  const char* spin = getenv("MADAKV_SCORE_SPIN_LIMIT");
  a.spin_limit = spin && atoi(spin) > 0 ? atoi(spin) : FUSED_SPIN_LIMIT;
  const float scale = c.softmax_scale > 0.f ? c.softmax_scale : 1.0f / sqrtf((float)dm.d);
  a.scale_log2 = scale * 1.4426950408889634f;
  a.rb_count = fused_blocks(dm);
  a.psi_part = reinterpret_cast<float*>(static_cast<char*>(ws) + 256 + ragged_xchg_bytes(dm, longest_rows));
  a.psi_part_stride = cache_rows;
  if (a.rb_count == 1) {
    if (dm.d == 128) launch_fused<128>(a, dm.heads, st); else launch_fused<64>(a, dm.heads, st);
  } else {
    // the kernel writes the row blocks' copies at the rows' own places; they are added over the whole cache
    // (rows outside the call's segments hold old values of the workspace and are not read by anybody)
    const ScoreArgs& b = a;
    const int vheads = dm.heads * a.rb_count;
    const long long nx = (long long)vheads * a.fsplit * a.mpad;
    if (a.fsplit > 1) hipLaunchKernelGGL(score_xchg_init_kernel, dim3((unsigned)((nx + 255) / 256)), dim3(256), 0, st, a.xchg, nx);
    const dim3 grid(a.fsplit, vheads);
    if (dm.d == 128) launch_fused_by_kind<128>(b, grid, st); else launch_fused_by_kind<64>(b, grid, st);
    hipLaunchKernelGGL(score_blocks_sum_kernel, dim3((unsigned)((cache_rows + 255) / 256)), dim3(256), 0, st,
                       a.psi_part, a.psi_part_stride, a.rb_count, psi_c, cache_rows);
  }
  return hipGetLastError();
}

// ---- the last-window attention with the scores as a by-product
constexpr int WIN_NS_128 = 4, WIN_NS_64 = 6;             // subtiles per wave (registers: logits + the O tile)
static int win_split(const Dims& dm) { const int ck = 4 * 32 * (dm.d == 128 ? WIN_NS_128 : WIN_NS_64); return (dm.L + ck - 1) / ck; }
static int win_blocks(const Dims& dm) { return (dm.M + 31) / 32; }   // blocks of 32 proxy rows, each handled like a head of its own
bool window_attn_supported(const Dims& dm, const madakv_config& c) {
  return use_mfma(dm, c.dtype) && dm.M <= 256 && win_split(dm) <= FUSED_MAX_SPLIT_2L;
}
static size_t win_xchg_bytes(const Dims& dm) {
  return ((size_t)dm.heads * win_blocks(dm) * (win_split(dm) + xchg_groups(win_split(dm))) * 32 * 8 + 255) / 256 * 256;
}
static size_t win_opart_bytes(const Dims& dm) { return ((size_t)dm.heads * win_blocks(dm) * win_split(dm) * 32 * dm.d * sizeof(float) + 255) / 256 * 256; }
size_t window_attn_ws_bytes(const Dims& dm, const madakv_config& c) {
  if (!window_attn_supported(dm, c)) return 256;
  // the counter of lone workgroups, the workgroups' shares of O, the row blocks' shares of psi
  return 256 + win_opart_bytes(dm) + (win_blocks(dm) > 1 ? (size_t)win_blocks(dm) * dm.heads * dm.L * sizeof(float) : 0);
}
// More than 64 proxy rows: window_wide_kernel, in one pass for all rows but behind a sweep over K of its own (four launches,
// one or two workgroups per compute unit, each walking its tiles one after the other), or the kernel above, block by block
// of 32 rows (three launches, 512 workgroups at a time, 512 or 768 keys each).  With few of the latter's workgroups the chip
// is not full either way and its shorter chain wins; with more than two rounds of them its repeated passes over K and V cost
// more.  Measured per call, blocks / one pass, by the number of the blocks' workgroups: head_dim 128, 5-8 blocks of rows, 512
// (8K keys) 58 / 90 us, 1024 (8K) 84 / 92, 1344 (2K) 109 / 89, 1536 (32K) 132 / 118, 3072 (128K) 286 / 192; up to 4 blocks,
// whose waves share a compute unit with another workgroup, 512 (8K) 57 / 74, 768 (2K) 75 / 70, 768 (32K) 94 / 100, 2048 (32K)
// 156 / 116; head_dim 64 516 (32K) 95 / 106, 616 (8K) 81 / 82, 704 (8K) 81 / 72, 1032 (32K) 124 / 106.
static bool win_one_pass(const Dims& dm) {
  if (dm.M <= 64 || dm.L < 64) return false;              // (below 64 keys the row statistics do not fit where they go)
  const long long block_wgs = (long long)dm.heads * win_blocks(dm) * win_split(dm);
  return block_wgs > ((dm.L > 16384 || (dm.d == 128 && win_blocks(dm) > 4)) ? 1024 : 640);
}
// Keys per chunk of window_wide_kernel: what costs least, counted in tiles of a workgroup.  A call takes as many rounds of
// workgroups as the chip holds of them (one of eight waves per compute unit, two of four), a round its tiles and about one of 64
// keys for its start; every chunk leaves a share of O, 32 d floats per block of rows written and read again, 6.5 ns at 128 dims
// against 2.8 us for a tile of eight waves and 1.7 for one of four (1.2 where a workgroup has its compute unit to itself).  Over 92
// measured shapes (1-224 heads, 96-256 rows, 2K-128K keys) the choice is within 3% of the best number of chunks.  112 heads
// of 32K keys and 224 rows: 9 chunks, 16 or 32 are 4-9% slower; one head of 128K keys and 256 rows: 16 chunks 549 us, 64
// 237, 256 174; 4 heads of 128K and 224 rows: 16 chunks 564, 64 266, 256 316; 112 heads of 8K: 2 chunks 348, 9 376, 16 405.
// (At most win_split chunks, for which the workspace is made.)
static int win_wide_chunk(const Dims& dm, bool wide8) {
  const int slots = wide8 ? 256 : 512, tile = wide8 ? 64 : 32;
  const double start = wide8 ? 1.0 : 2.0, share = (wide8 ? 0.002 : 0.004) * dm.d / 128 * win_blocks(dm);
  int best = 0; double least = 0.;
  for (int ns = 1; ns <= win_split(dm); ++ns) {
    const int chunk = ((dm.L + ns - 1) / ns + 63) / 64 * 64;
    const long long wgs = (long long)dm.heads * ((dm.L + chunk - 1) / chunk), rounds = (wgs + slots - 1) / slots;
    const double tiles = (double)((chunk + tile - 1) / tile) * (!wide8 && wgs <= 256 ? 0.7 : 1.0);
    const double cost = (double)rounds * (tiles + start) + share * (double)wgs;
    if (!best || cost < least) { best = chunk; least = cost; }
  }
  return best;
}
template <int D, int NW>
static void launch_win_wide(const WinArgs& wa, int heads, hipStream_t st) {
  const size_t lds = (size_t)DMA_NBUF * 2 * (NW * 8) * D * 2 + (size_t)2 * 2 * NW * (NW * 8) * sizeof(float);
  if (lds > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&window_wide_kernel<D, NW>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((window_wide_kernel<D, NW>), dim3(wa.s.fsplit, heads), dim3(NW * 64), lds, st, wa);
}
template <int D>
static void launch_win_many_rows(WinArgs& wa, const Dims& dm, const madakv_config& c, hipStream_t st) {
  ScoreArgs& a = wa.s;
  const ScorePlan p = score_plan(dm, c.dtype);
  const bool wide8 = p.mpad > 128;
  // the row statistics go where the row blocks' copies of psi would be (32 rb = mpad rows): 2 nsplit mpad <= 2 max(1, L / 1024) 32 rb
  // floats per head against L rb
  a.rowstat = a.psi_part;
  a.mpad = p.mpad; a.nsplit = p.nsplit; a.nmerge = 1;
  const int chunk2 = win_wide_chunk(dm, wide8);
  a.fsplit = (dm.L + chunk2 - 1) / chunk2;
  for (int h0 = 0; h0 < dm.heads; h0 += 65535) {
    const int nh = std::min(65535, dm.heads - h0);
    a.head0 = h0;
    a.chunk = p.chunk;
    if (wide8) launch_wide_sweep1<D, true, true>(a, nh, st); else launch_wide_sweep1<D, false, true>(a, nh, st);
    a.chunk = chunk2;
    if (wide8) launch_win_wide<D, 8>(wa, nh, st); else launch_win_wide<D, 4>(wa, nh, st);
    a.head0 = h0 * a.rb_count;
    hipLaunchKernelGGL(window_attn_reduce_kernel, dim3(nh * a.rb_count, (32 * D / 4 + 255) / 256), dim3(256), 0, st, wa);
  }
}
hipError_t launch_window_attn(const Dims& dm, const madakv_config& c, const void* q_win, const void* k, const void* v,
                              void* out, float* row_lse, float* psi, void* ws, Exchange& x, hipStream_t st) {
  WinArgs wa;
  ScoreArgs& a = wa.s;
  a.lse = nullptr; a.q_win = q_win; a.k = k; a.psi = psi;
  a.status = reinterpret_cast<int*>(ws);
  a.rowstat = nullptr; a.sink = nullptr; a.seg_off = nullptr; a.seg_len = nullptr;
  a.xchg = x.words; a.xchg_clean = true;
  a.H = dm.H; a.G = dm.G; a.d = dm.d; a.L = dm.L; a.W = dm.W; a.M = dm.M;
  a.mpad = 32; a.nsplit = 0; a.nmerge = 0; a.chunk = 0; a.head0 = 0;
  const int rb = win_blocks(dm);
  a.rb_count = rb;
  a.psi_part = reinterpret_cast<float*>(static_cast<char*>(ws) + 256 + win_opart_bytes(dm));
  a.psi_part_stride = (long long)dm.heads * dm.L;
  a.fsplit = win_split(dm);
  a.xgroups = xchg_groups(a.fsplit); a.xstride = (long long)(a.fsplit + a.xgroups) * 32; a.k_kind = K_BF16;   // (two exchange levels above 64 chunks)
  const char* spin = getenv("MADAKV_SCORE_SPIN_LIMIT");
  a.spin_limit = spin && atoi(spin) > 0 ? atoi(spin) : FUSED_SPIN_LIMIT;
  const float scale = c.softmax_scale > 0.f ? c.softmax_scale : 1.0f / sqrtf((float)dm.d);
  a.scale_log2 = scale * 1.4426950408889634f;
  wa.v = v; wa.lse = row_lse; wa.out = out; wa.out_fp32 = c.out_fp32;
  wa.opart = reinterpret_cast<float*>(static_cast<char*>(ws) + 256);
  if (win_one_pass(dm)) {
    if (dm.d == 128) launch_win_many_rows<128>(wa, dm, c, st); else launch_win_many_rows<64>(wa, dm, c, st);
    return hipGetLastError();
  }
  x.per_head = rb * a.xstride;
  const size_t lds = ((size_t)32 + 4 * 32) * (dm.d + 8) * 2 + ((size_t)4 * 32 * 2 + 32 + 512) * sizeof(float);
  const int vheads = dm.heads * rb, step = 65535 / rb * rb;       // whole heads per launch (the grid's y limit)
  for (int h0 = 0; h0 < vheads; h0 += step) {
    const int nh = std::min(step, vheads - h0);
    a.head0 = h0;
    if (dm.d == 128) hipLaunchKernelGGL((window_attn_kernel<128, WIN_NS_128>), dim3(a.fsplit, nh), dim3(SCORE_THREADS), lds, st, wa);
    else hipLaunchKernelGGL((window_attn_kernel<64, WIN_NS_64>), dim3(a.fsplit, nh), dim3(SCORE_THREADS), lds, st, wa);
    hipLaunchKernelGGL(window_attn_reduce_kernel, dim3(nh, (32 * dm.d / 4 + 255) / 256), dim3(256), 0, st, wa);
  }
  if (rb > 1) {
    const long long n = (long long)dm.heads * dm.L;
    hipLaunchKernelGGL(score_blocks_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a.psi_part, a.psi_part_stride, rb, psi, n);
  }
  return hipGetLastError();
}

// Words the workgroups of a layer's heads may exchange in, whichever of the kernels takes the call.  They are the handle's, a
// layer's at a place of its own, and XCHG_EMPTY between calls: the statistics kernel, which every scoring call runs behind the
// scores, empties them again (a launch of its own for that took 2 to 5 us of every call).
size_t xchg_layer_words(const madakv_config& c, const Dims& one) {
  size_t n = xchg_bytes(one, c.dtype);
  if (window_attn_supported(one, c) && !win_one_pass(one)) n = std::max(n, win_xchg_bytes(one));
  return n / 8;
}
hipError_t launch_xchg_clear(unsigned long long* words, size_t n, hipStream_t st) {
  if (n) hipLaunchKernelGGL(score_xchg_init_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, words, (long long)n);
  return hipGetLastError();
}

hipError_t launch_score(const Dims& dm, const madakv_config& c, const void* q_win, const void* k, const float* row_lse,
                        float* psi, void* ws, Exchange& x, hipStream_t st) {
  ScorePlan p = score_plan(dm, c.dtype);
  ScoreArgs a;
  a.lse = row_lse;
  a.q_win = q_win; a.k = k; a.psi = psi;
  a.status = reinterpret_cast<int*>(ws);
  a.rowstat = reinterpret_cast<float*>(static_cast<char*>(ws) + 256);
  a.sink = reinterpret_cast<float*>(static_cast<char*>(ws) + 256 + rowstat_bytes(dm, c.dtype));
  a.xchg = x.words; a.xchg_clean = true;
  a.rb_count = fused_blocks(dm);
  a.psi_part = reinterpret_cast<float*>(static_cast<char*>(ws) + 256 + rowstat_bytes(dm, c.dtype) + 256);
  a.psi_part_stride = (long long)dm.heads * dm.L;
  a.fsplit = (!row_lse && use_fused(dm, c.dtype)) ? fused_split(dm, c.dtype) : 0;
  a.nstrag = a.fsplit ? fused_parked_chunks(a.fsplit) : 0;
  if (getenv("MADAKV_SCORE_NO_PARKED_CHUNKS")) a.nstrag = 0;                      // (measurement switch)
  a.fsplit -= a.nstrag;                                                            // the chunks of the main launch
  a.xgroups = xchg_groups(a.fsplit) + a.nstrag; a.xstride = (long long)(a.fsplit + a.xgroups) * fused_mpad(dm);
  a.k_kind = c.dtype == MADAKV_FP32 ? K_F32 : K_BF16;
  {
    char* pk = static_cast<char*>(ws) + 256 + rowstat_bytes(dm, c.dtype) + 256 +
               (fused_fits(dm, c.dtype) && fused_blocks(dm) > 1 ? (size_t)fused_blocks(dm) * dm.heads * dm.L * sizeof(float) : 0);
    a.offs_out = a.nstrag ? reinterpret_cast<float*>(pk) : nullptr;
    a.park = a.nstrag ? reinterpret_cast<float*>(pk) + (size_t)dm.heads * fused_mpad(dm) : nullptr;
  }
  a.seg_off = nullptr; a.seg_len = nullptr;
  // (a test can force the lone-workgroup path of the one-sweep kernel from the host with a spin limit of 1)
  const char* spin = getenv("MADAKV_SCORE_SPIN_LIMIT");
  a.spin_limit = spin && atoi(spin) > 0 ? atoi(spin) : FUSED_SPIN_LIMIT;
  a.H = dm.H; a.G = dm.G; a.d = dm.d; a.L = dm.L; a.W = dm.W; a.M = dm.M;
  a.mpad = p.mpad; a.nsplit = p.nsplit; a.nmerge = p.nsplit; a.chunk = p.chunk; a.head0 = 0;
  float scale = c.softmax_scale > 0.f ? c.softmax_scale : 1.0f / sqrtf((float)dm.d);
  a.scale_log2 = scale * 1.4426950408889634f;
  if (a.fsplit > 0) {                                      // one sweep (heads * row blocks fit one launch)
    a.mpad = fused_mpad(dm); a.subtiles = fused_subtiles(dm, c.dtype);
    x.per_head = a.rb_count * a.xstride;
    if (dm.d == 128) launch_fused<128>(a, dm.heads, st); else launch_fused<64>(a, dm.heads, st);
    return hipGetLastError();
  }
  for (int h0 = 0; h0 < dm.heads; h0 += p.group_heads) {
    int nh = std::min(p.group_heads, dm.heads - h0);
    a.head0 = h0;
    if (use_mfma(dm, c.dtype)) {
      // row blocks of 32 proxy rows: 1-2 -> every wave its own keys and all rows; 3-8 -> the waves share the
      // keys and own row blocks (the kernels with the LDS ring)
      const int MB = p.mpad / 32;
      const size_t qbytes = ((size_t)p.mpad + 4 * 32) * (dm.d + 8) * 2;      // Q tile + one K subtile per wave
      const size_t lds1 = qbytes + (size_t)4 * p.mpad * 2 * sizeof(float);
      const size_t lds2 = qbytes + (size_t)p.mpad * sizeof(float);
#define MADAKV_SCORE_CASE(DD, NN) launch_mfma_pair<DD, NN>(a, nh, lds1, lds2, st)
#define MADAKV_SCORE_BY_MB(DD) \
      if (MB == 1) MADAKV_SCORE_CASE(DD, 1); else if (MB == 2) MADAKV_SCORE_CASE(DD, 2); \
      else if (MB <= 4) launch_wide_pair<DD, false>(a, nh, st); else launch_wide_pair<DD, true>(a, nh, st)
      if (dm.d == 128) { MADAKV_SCORE_BY_MB(128); } else { MADAKV_SCORE_BY_MB(64); }
#undef MADAKV_SCORE_BY_MB
#undef MADAKV_SCORE_CASE
    } else {
      size_t lds = ((size_t)dm.M * dm.d + dm.M) * sizeof(float);
      dim3 grid(a.nsplit, nh);
      if (!a.lse) hipLaunchKernelGGL((score_simple_kernel<1>), grid, dim3(SCORE_THREADS), lds, st, a);
      hipLaunchKernelGGL((score_simple_kernel<2>), grid, dim3(SCORE_THREADS), lds, st, a);
    }
  }
  return hipGetLastError();
}

}  // namespace madakv
