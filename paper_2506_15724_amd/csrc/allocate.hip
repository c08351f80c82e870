// Budget allocation (paper Sec. 3.3): Eq. 10-11 layer compensation in integers, then the
// Eq. 8 modality split per head.
//
// One wavefront per batch item, one lane per KV head (H <= 64), layers in sequence; the split by the whole workgroup.
// The recurrence phi^{l+1} = phi^l - K^l / (layers left) is carried as an integer pool R of
// candidate tokens for all remaining layers and heads: nominal per-head budget
// phi^l = R / (H * rem).  A head's demand is its Eq. 9 count k_t + k_v clamped to
// [phi/rho, rho*phi]; the layer draws the sum of demands, clamped so that every later layer
// can still get between beta_floor and n_cand tokens per head; the last layer draws what is
// left.  Heads share the layer total by largest remainder (ties to the lower head), scaled
// by demand when it has to shrink and by head-room when it has to grow.  All cross-head
// sums and ranks are wavefront shuffles; arithmetic is 64-bit integer except the double
// multiply (and, with more than two modalities, the subtraction) of the Eq. 8 share.  Those
// must round after every operation, as the reference arithmetic does: a fused multiply-add
// keeps the exact product and changes which of two nearly equal fractional parts is the
// larger, so contraction is switched off for them.
#include "allocate.h"

namespace madakv {

__global__ __launch_bounds__(256) void allocate_kernel(AllocArgs a) {
  if (threadIdx.x < 64) allocate_wave(a, blockIdx.x, threadIdx.x);
  __syncthreads();
  split_totals(a, blockIdx.x, threadIdx.x, blockDim.x);
}

AllocArgs alloc_args(const Dims& dm, const madakv_config& c, int layer0, const void* stats, const int32_t* n_mod, int32_t* budgets, long long* pool_state) {
  AllocArgs a;
  a.M = c.n_modalities;
  a.stats = stats; a.n_mod = n_mod; a.budgets = budgets; a.pool = pool_state;
  a.n = dm.n; a.B = dm.B; a.H = dm.H; a.NL = c.n_layers; a.layer0 = layer0; a.nc = dm.nc;
  a.beta = c.budget - c.window; a.rho = c.hcc_rho; a.mpa_mode = c.mpa_mode; a.hcc_mode = c.hcc_mode;
  a.keep_all = c.budget >= c.ctx_len ? 1 : 0;
  return a;
}

hipError_t launch_allocate(const Dims& dm, const madakv_config& c, int layer0, const void* stats,
                           const int32_t* n_mod, int32_t* budgets, long long* pool_state, hipStream_t st) {
  hipLaunchKernelGGL(allocate_kernel, dim3(dm.B), dim3(dm.n == 1 ? 64 : 256), 0, st, alloc_args(dm, c, layer0, stats, n_mod, budgets, pool_state));
  return hipGetLastError();
}

}  // namespace madakv
