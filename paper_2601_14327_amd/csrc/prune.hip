// LAEP prune mask for one layer and one counted batch (laep_prune_mask), and
// Algorithm 1 over a recorded window (laep_expert_pruning).
//
// Section 3.2, Eqs. (1)-(2), as carried out by the marking step of
// Algorithm 1: rank experts by (load, index) ascending, accumulate the
// loads inclusively in that order, prune an expert iff
//     running < total * beta   and   load < (total * alpha) / E
// with both sides evaluated in IEEE double.  One workgroup, one thread per
// expert (E <= 256).
#include "common.hpp"
#include "internal.hpp"

namespace laep {
namespace {

constexpr int kPruneThreads = 256;

// The marking rule for expert e among loads[0, E): its place in the
// (load, index) order needs no sort, since the inclusive running sum there is
// the sum over every expert that is not after it (exact in integers, in any
// order).
__device__ __forceinline__ bool marked(const long long* loads, int E, int e, double beta_thr,
                                       double alpha_thr) {
  const long long c = loads[e];
  long long running = 0;
#pragma unroll 8
  for (int j = 0; j < E; ++j) {
    const long long cj = loads[j];
    // (bitwise: a select, where || and && branch around every load of the loop)
    running += ((int)(cj < c) | ((int)(cj == c) & (int)(j <= e))) ? cj : 0ll;
  }
  return (double)running < beta_thr && (double)c < alpha_thr;
}

// The same in 32 bits, for loads below kNarrowLoad (their sum over 256 experts
// stays below 2^31): (load, index) is one key, so an expert costs a compare,
// a select and an add instead of about a dozen 64-bit steps.
constexpr int kNarrowLoad = 1 << 23;
struct KeyLoad {
  int key, load;  // load * 256 + index, load
};
__device__ __forceinline__ KeyLoad key_load(int load, int e) { return {load * 256 + e, load}; }
__device__ __forceinline__ bool marked(const KeyLoad* loads, int E, int e, double beta_thr,
                                       double alpha_thr) {
  const KeyLoad c = loads[e];
  int running = 0;
#pragma unroll 16
  for (int j = 0; j < E; ++j) {
    const KeyLoad cj = loads[j];
    running += cj.key <= c.key ? cj.load : 0;
  }
  return (double)running < beta_thr && (double)c.load < alpha_thr;
}
union LoadSlot {
  long long wide;
  KeyLoad narrow;
};

__global__ __launch_bounds__(kPruneThreads) void prune_kernel(const int32_t* __restrict__ counts,
                                                              int E, long long total, double alpha,
                                                              double beta,
                                                              uint8_t* __restrict__ alive,
                                                              int32_t* __restrict__ n_pruned) {
  __shared__ LoadSlot s_c[kPruneThreads];
  const int tid = threadIdx.x;
  const int c = tid < E ? counts[tid] : 0;
  const bool wide = __syncthreads_or(c < 0 || c >= kNarrowLoad);
  if (wide) s_c[tid].wide = c;
  else s_c[tid].narrow = key_load(c, tid);
  __syncthreads();
  bool pruned = false;
  if (tid < E) {
    const double beta_thr = (double)total * beta;
    const double alpha_thr = ((double)total * alpha) / (double)E;
    pruned = wide ? marked(&s_c[0].wide, E, tid, beta_thr, alpha_thr)
                  : marked(&s_c[0].narrow, E, tid, beta_thr, alpha_thr);
    alive[tid] = pruned ? 0 : 1;
  }
  const int n = __syncthreads_count(pruned);
  if (tid == 0) *n_pruned = n;
}

// Algorithm 1 over a window of ITER recorded iterations (Appendix), one
// workgroup per layer, one thread per (iteration, expert): the iterations
// are independent up to their integer sums, so kWindowThreads / E of them run
// at once.  (One thread per expert walking the window through a rank sort and
// a scan each took 59 us for 16 iterations of 64 experts; now 12.)
//   Step 2: per iteration, the marking rule above on ETN[iter, layer, :] with
//           the layer's alpha; Marker[e] counts the iterations that marked e
//           and Exp_dis the marks of all experts.
//   Step 3: N = floor(Exp_dis / ITER + 0.5) experts are pruned: the most
//           marked, ties to the lower mean load, then the lower index.  All
//           means share the divisor ITER, so they are compared as exact
//           int64 window sums (same order as the float64 means while the
//           sums stay below 2^52).
struct LayerAlphas {
  double a[kMaxLayers];
};

constexpr int kWindowThreads = 1024;

__global__ __launch_bounds__(kWindowThreads) void expert_pruning_kernel(
    const long long* __restrict__ etn, int ITER, int L, int E, long long total,
    const LayerAlphas alpha, double beta, uint8_t* __restrict__ alive,
    int32_t* __restrict__ n_pruned, int32_t* __restrict__ marker_out) {
  __shared__ LoadSlot s_c[kWindowThreads];  // [group][E]
  __shared__ int s_mark[kPruneThreads];
  __shared__ long long s_sum[kPruneThreads];
  const int tid = threadIdx.x;
  const int layer = blockIdx.x;
  const double a = alpha.a[layer];
  const double beta_thr = (double)total * beta;
  const double alpha_thr = ((double)total * a) / (double)E;
  if (tid < kPruneThreads) {
    s_mark[tid] = 0;
    s_sum[tid] = 0;
  }
  const int groups = kWindowThreads / E;  // iterations at once
  const int g = tid / E, e = tid % E;
  long long exp_dis = 0;
  for (int it0 = 0; it0 < ITER; it0 += groups) {
    const bool on = g < groups && it0 + g < ITER;
    const long long c = on ? etn[((size_t)(it0 + g) * L + layer) * E + e] : 0;
    const bool wide = __syncthreads_or(c < 0 || c >= kNarrowLoad);
    if (wide) s_c[tid].wide = c;
    else s_c[tid].narrow = key_load((int)c, e);
    __syncthreads();
    bool m = false;
    if (on) {
      m = wide ? marked(&s_c[g * E].wide, E, e, beta_thr, alpha_thr)
               : marked(&s_c[g * E].narrow, E, e, beta_thr, alpha_thr);
      if (m) atomicAdd(&s_mark[e], 1);  // integer sums: any order gives the same
      atomicAdd(reinterpret_cast<unsigned long long*>(&s_sum[e]), (unsigned long long)c);
    }
    exp_dis += __syncthreads_count(m);  // (and s_c may be refilled)
  }
  const long long n_dis = (long long)floor((double)exp_dis / (double)ITER + 0.5);
  if (tid < E) {
    const int m = s_mark[tid];
    const long long sm = s_sum[tid];
    int rank = 0;  // position in (marker desc, window load asc, index asc)
#pragma unroll 8
    for (int j = 0; j < E; ++j) {
      const int mj = s_mark[j];
      const long long sj = s_sum[j];
      rank += (int)(mj > m) |
              ((int)(mj == m) & ((int)(sj < sm) | ((int)(sj == sm) & (int)(j < tid))));
    }
    alive[(size_t)layer * E + tid] = rank < n_dis ? 0 : 1;
    if (marker_out) marker_out[(size_t)layer * E + tid] = m;
  }
  if (tid == 0) n_pruned[layer] = (int32_t)(n_dis < E ? n_dis : E);
}

}  // namespace

hipError_t launch_prune(const int32_t* counts, int E, int64_t total, double alpha, double beta,
                        uint8_t* alive, int32_t* n_pruned, hipStream_t s) {
  hipLaunchKernelGGL(prune_kernel, dim3(1), dim3(kPruneThreads), 0, s, counts, E,
                     (long long)total, alpha, beta, alive, n_pruned);
  return hipGetLastError();
}

hipError_t launch_expert_pruning(const int64_t* etn, int iters, int L, int E, int64_t total,
                                 const double* alpha, double beta, uint8_t* alive,
                                 int32_t* n_pruned, int32_t* marker, hipStream_t s) {
  LayerAlphas la;
  for (int l = 0; l < kMaxLayers; ++l) la.a[l] = l < L ? alpha[l] : 0.0;
  hipLaunchKernelGGL(expert_pruning_kernel, dim3(L), dim3(kWindowThreads), 0, s,
                     reinterpret_cast<const long long*>(etn), iters, L, E, (long long)total, la,
                     beta, alive, n_pruned, marker);
  return hipGetLastError();
}

}  // namespace laep
