// Physical expert compaction after pruning (Section 3.2: pruned experts are
// removed from the model, which is the parameter reduction LAEP reports).
//
//   expert_map_kernel: per layer, the surviving experts keep their order and
//     take consecutive slots: map[e] = #{alive j < e} if e is alive, else -1.
//   repack_kernel: copies each surviving expert's parameter block (a W_r row,
//     a [2f, d] gate/up matrix, a [d, f] down matrix, or an optimizer state of
//     the same shape) from its logical index to its slot; a pure HBM copy.
#include "common.hpp"
#include "internal.hpp"
#include "tiles.hpp"

namespace laep {
namespace {

// One workgroup per layer, one thread per expert (E <= 256).
__global__ __launch_bounds__(kTableThreads) void expert_map_kernel(
    const uint8_t* __restrict__ alive, int E, int32_t* __restrict__ expert_map,
    int32_t* __restrict__ n_alive) {
  __shared__ int s_tmp[4];
  const int layer = blockIdx.x;
  const int e = threadIdx.x;
  const int a = (e < E && alive[(size_t)layer * E + e] != 0) ? 1 : 0;
  const int slot = block_excl_scan_256(a, s_tmp);
  if (e < E) expert_map[(size_t)layer * E + e] = a ? slot : -1;
  if (e == kTableThreads - 1) n_alive[layer] = slot + a;
}

// All of an expert's tensors in one launch: workgroup (chunk, expert), the
// chunks of up to three tensors one after the other, kRepackVecs 16-byte
// vectors per thread in flight; the first chunk's workgroup also copies the
// bias entry.  Workgroups of an expert that is pruned, or whose slot is not
// below n_out, copy nothing.  STREAM: non-temporal accesses, for tensors past
// what the 256 MB last-level cache holds (30 of 64 experts kept, d 2048, d_ff
// 1024: 187 us in three launches with four plain vectors in flight, 182 with
// eight streamed ones, 126 with two: more workgroups; 6.0 TB/s); smaller layers
// stay cached for their next use.
constexpr int kRepackThreads = 256;
constexpr int kRepackVecs = 2;
constexpr int kRepackChunk = kRepackThreads * kRepackVecs;
constexpr int kRepackTensors = 3;
struct RepackParams {
  const u32x4_t* src[kRepackTensors];
  u32x4_t* dst[kRepackTensors];
  long long vecs[kRepackTensors];   // 16-byte vectors per expert (0: absent)
  long long first[kRepackTensors];  // first chunk of the tensor
  const float* bias;
  float* bias_out;
};

template <bool STREAM>
__global__ __launch_bounds__(kRepackThreads) void repack_kernel(
    const int32_t* __restrict__ expert_map, int n_out, RepackParams p) {
  const int e = blockIdx.y;
  const int slot = expert_map[e];
  if (slot < 0 || slot >= n_out) return;
  const long long b = blockIdx.x;
  if (b == 0 && threadIdx.x == 0 && p.bias != nullptr) p.bias_out[slot] = p.bias[e];
  int t = 0;
#pragma unroll
  for (int i = 1; i < kRepackTensors; ++i)
    if (b >= p.first[i]) t = i;
  const long long n = p.vecs[t];
  const u32x4_t* in = p.src[t] + (size_t)e * n;
  u32x4_t* out = p.dst[t] + (size_t)slot * n;
  const long long i0 = (b - p.first[t]) * kRepackChunk + threadIdx.x;
  u32x4_t v[kRepackVecs];
#pragma unroll
  for (int u = 0; u < kRepackVecs; ++u) {
    const long long i = i0 + (long long)u * kRepackThreads;
    if (i < n) v[u] = STREAM ? ld_stream(in + i) : in[i];
  }
#pragma unroll
  for (int u = 0; u < kRepackVecs; ++u) {
    const long long i = i0 + (long long)u * kRepackThreads;
    if (i < n) {
      if (STREAM) st_stream(out + i, v[u]);
      else out[i] = v[u];
    }
  }
}

}  // namespace

hipError_t launch_expert_map(const uint8_t* alive, int L, int E, int32_t* expert_map,
                             int32_t* n_alive, hipStream_t s) {
  hipLaunchKernelGGL(expert_map_kernel, dim3(L), dim3(kTableThreads), 0, s, alive, E, expert_map,
                     n_alive);
  return hipGetLastError();
}

hipError_t launch_repack(const int32_t* expert_map, int E, int n_out, const void* const* src,
                         void* const* dst, const size_t* bytes_per_expert, int n_tensors,
                         const float* bias, float* bias_out, hipStream_t s) {
  RepackParams p = {};
  long long chunks = 0;
  size_t bytes = 0;
  for (int i = 0; i < kRepackTensors; ++i) {
    p.first[i] = chunks;
    if (i >= n_tensors || src[i] == nullptr) continue;
    p.src[i] = static_cast<const u32x4_t*>(src[i]);
    p.dst[i] = static_cast<u32x4_t*>(dst[i]);
    p.vecs[i] = (long long)(bytes_per_expert[i] / 16);
    chunks += (p.vecs[i] + kRepackChunk - 1) / kRepackChunk;
    bytes += bytes_per_expert[i];
  }
  p.bias = bias;
  p.bias_out = bias_out;
  if (chunks == 0) {
    if (bias == nullptr) return hipSuccess;
    chunks = 1;
  }
  const int kept = n_out < E ? n_out : E;
  const auto kernel = 2 * bytes * kept > (size_t(256) << 20) ? repack_kernel<true>
                                                             : repack_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)chunks, (unsigned)E), dim3(kRepackThreads), 0, s,
                     expert_map, n_out, p);
  return hipGetLastError();
}

}  // namespace laep
