// Backward of router scoring and gating (moe_route_bwd), with the top-k
// selection held fixed (it is piecewise constant in the logits):
//   dl[t, e] = dLoss/dlogits[t, e] from dgate (the softmax Jacobian),
//   dx[t]   (+)= sum_e dl[t, e] W_r[e]
//   dW_r[e]   = sum_t dl[t, e] x[t],   db[e] = sum_t dl[t, e]
// Renormalised gates make dl zero outside the k selected experts, so dx is a
// k-term weighted sum of W_r rows (like the combine) and dW_r[e] a weighted
// sum over the expert's routed rows, which moe_expert_counts already lists
// in expert order (row_src); with few experts, or many slots, the dense product
// over all tokens is faster than gathering them.  Full-softmax gates make dl
// dense over the alive experts; dx then sums over all E experts and dW_r over all
// T tokens.
// Every sum runs in a fixed order: results are deterministic.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "tiles.hpp"

namespace laep {
namespace {

constexpr int kDlThreads = 256;

// Waves in two grid dimensions (one holds less than 2^32 threads).
inline dim3 dl_grid(int T, int tokens_per_wave) {
  const unsigned per = (kDlThreads / 64) * (unsigned)tokens_per_wave;
  const unsigned n = ((unsigned)T + per - 1) / per, x = n < 1u << 20 ? n : 1u << 20;
  return dim3(x, (n + x - 1) / x);
}
__device__ __forceinline__ unsigned dl_wave() {
  return __builtin_amdgcn_readfirstlane((blockIdx.y * gridDim.x + blockIdx.x) * (kDlThreads / 64) +
                                        (threadIdx.x >> 6));
}

// Renormalised gates: dl_slot[t, j] = g_j (dg_j - sum_i g_i dg_i) (0 for
// unrouted slots).  dl_dense and dlogits (both optional) get the dense [T, E]
// gradient.  One wave per token: lane j holds slot j (then j + 64, ...), lane e
// writes experts e, e + 64, ..., so the slots are loaded and the rows written in
// whole lines and the sum is still taken in slot order.
__global__ __launch_bounds__(kDlThreads) void route_bwd_dl_kernel(
    const float* __restrict__ dgate, const int32_t* __restrict__ idx,
    const float* __restrict__ gate, int T, int E, int k, float* __restrict__ dl_out,
    float* __restrict__ dl_dense, float* __restrict__ dlogits) {
  const unsigned t = dl_wave();
  if (t >= (unsigned)T) return;
  const int lane = threadIdx.x & 63;
  const size_t s0 = (size_t)t * k;
  auto from_lane = [](float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
  };
  float s = 0.0f;
  for (int j0 = 0; j0 < k; j0 += 64) {
    const int n = min(64, k - j0);
    float p = 0.0f;
    if (lane < n && idx[s0 + j0 + lane] >= 0)
      p = gate[s0 + j0 + lane] * dgate[s0 + j0 + lane];
    for (int j = 0; j < n; ++j) s += from_lane(p, j);
  }
  constexpr int EPL = 4;  // at most 256 experts
  float row[EPL] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int j0 = 0; j0 < k; j0 += 64) {
    const int n = min(64, k - j0);
    int e = -1;
    float v = 0.0f;
    if (lane < n) {
      e = idx[s0 + j0 + lane];
      v = e >= 0 ? gate[s0 + j0 + lane] * (dgate[s0 + j0 + lane] - s) : 0.0f;
      dl_out[s0 + j0 + lane] = v;
    }
    if (dl_dense || dlogits)
      for (int j = 0; j < n; ++j) {
        const int ej = __builtin_amdgcn_readlane(e, j);
        const float vj = from_lane(v, j);
#pragma unroll
        for (int u = 0; u < EPL; ++u) row[u] = ej == lane + 64 * u ? vj : row[u];
      }
  }
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    const int e = lane + 64 * u;
    if (e >= E) continue;
    if (dl_dense) dl_dense[(size_t)t * E + e] = row[u];
    if (dlogits) dlogits[(size_t)t * E + e] = row[u];
  }
}

// The same for the slots alone, at most 64: `lanes` lanes per token (the power of
// two from k up), 64 / lanes tokens per wave.  (A wave per token for one slot took
// 9 us at 40000 tokens; a thread per token, each reading its slots alone, 7 us at
// 1000 tokens of 8 slots; here 3 and 3.)
inline int dl_lanes(int k) {
  int lanes = 1;
  while (lanes < k) lanes *= 2;
  return lanes;
}
__global__ __launch_bounds__(kDlThreads) void route_bwd_dl_slots_kernel(
    const float* __restrict__ dgate, const int32_t* __restrict__ idx,
    const float* __restrict__ gate, int T, int k, int lanes, float* __restrict__ dl_out) {
  const int lane = threadIdx.x & 63;
  const int sub = lane & (lanes - 1), group = lane - sub;
  const unsigned t = dl_wave() * (64u / lanes) + (unsigned)(lane / lanes);
  const bool on = t < (unsigned)T && sub < k;
  const size_t at = (size_t)t * k + sub;
  int e = -1;
  float g = 0.0f, dg = 0.0f;
  if (on) {
    e = idx[at];
    g = gate[at];
    dg = dgate[at];
  }
  const float p = e >= 0 ? g * dg : 0.0f;
  float s = 0.0f;
  for (int j = 0; j < k; j += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __shfl(p, group + ((j + u) & (lanes - 1)), kWave);
#pragma unroll
    for (int u = 0; u < 8; ++u) s += j + u < k ? v[u] : 0.0f;
  }
  if (on) dl_out[at] = e >= 0 ? g * (dg - s) : 0.0f;
}

// Full-softmax gates: dl_full[t, e] = p_e (q_e - sum_j g_j dg_j) over alive e,
// p = softmax of the alive logits, q_e = dg_j at e = idx[t, j].  One wave per
// token, lane l owning experts l, l + 64, ...: the logits are read and dl
// written in whole lines (one thread per token walked its row alone, every
// load touching 64 lines: 103 us at 4096 tokens over 128 experts).  PACKED: up to
// 32 experts, `lanes` lanes per token (the power of two from E up), 64 / lanes
// tokens per wave, lane e its expert e (a wave per token took 14 us at 40000
// tokens, now 5).
template <bool PACKED>
__global__ __launch_bounds__(kDlThreads) void route_bwd_dl_full_kernel(
    const float* __restrict__ dgate, const int32_t* __restrict__ idx,
    const float* __restrict__ gate, const float* __restrict__ logits,
    const uint8_t* __restrict__ alive, int T, int E, int k, int lanes,
    float* __restrict__ dl_out, float* __restrict__ dlogits) {
  const int in_wave = threadIdx.x & 63;
  const unsigned t = PACKED ? dl_wave() * (64u / lanes) + (unsigned)(in_wave / lanes) : dl_wave();
  if (t >= (unsigned)T) return;  // (whole groups)
  const int lane = PACKED ? in_wave & (lanes - 1) : in_wave;
  const int width = PACKED ? lanes : 64;
  auto sum = [&](float v) {  // over the token's lanes
#pragma unroll
    for (int off = PACKED ? 16 : 32; off >= 1; off >>= 1)
      if (off < width) v += __shfl_xor(v, off, kWave);
    return v;
  };
  const size_t s0 = (size_t)t * k;
  float s = 0.0f;
  for (int j = lane; j < k; j += width)
    if (idx[s0 + j] >= 0) s += gate[s0 + j] * dgate[s0 + j];
  s = sum(s);
  constexpr int EPL = PACKED ? 1 : 4;  // at most 256 experts
  float l[EPL], q[EPL];
  bool a[EPL];
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    const int e = lane + 64 * u;
    a[u] = e < E && (alive == nullptr || alive[e]);
    l[u] = a[u] ? logits[(size_t)t * E + e] : -INFINITY;
    q[u] = 0.0f;
    m = fmaxf(m, l[u]);
  }
#pragma unroll
  for (int off = PACKED ? 16 : 32; off >= 1; off >>= 1)
    if (off < width) m = fmaxf(m, __shfl_xor(m, off, kWave));
  for (int j = 0; j < k; ++j) {  // (one address per token)
    const int ej = idx[s0 + j];
    const float dg = dgate[s0 + j];
#pragma unroll
    for (int u = 0; u < EPL; ++u) q[u] = ej == lane + 64 * u ? dg : q[u];
  }
  float z = 0.0f;
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    l[u] = a[u] ? __expf(l[u] - m) : 0.0f;
    z += l[u];
  }
  z = sum(z);
  const float inv = z > 0.0f ? 1.0f / z : 0.0f;
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    const int e = lane + 64 * u;
    if (e >= E) continue;
    const float v = a[u] ? l[u] * inv * (q[u] - s) : 0.0f;
    dl_out[(size_t)t * E + e] = v;
    if (dlogits) dlogits[(size_t)t * E + e] = v;
  }
}

// dx[t] (+)= sum over slots of w * W_r[row], row ids from `ids` ([T, slots], -1 =
// none) or the slot itself (ids == NULL: full-softmax gates of few experts),
// weights dl [T, slots].  One wave per token (its ids and weights are wave-uniform
// loads); each lane owns the 8-column vectors lane, lane + 64, ...
template <typename T>
__global__ __launch_bounds__(256) void route_bwd_dx_kernel(
    const T* __restrict__ w_router, const int32_t* __restrict__ ids,
    const float* __restrict__ dl, int n_tok, int slots, int d, int accumulate,
    T* __restrict__ dx) {
  const int t = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (int)(threadIdx.x >> 6));
  if (t >= n_tok) return;
  const int lane = threadIdx.x & 63;
  const int vec_per_row = d / 8;
  const size_t o = (size_t)t * slots;
  for (int v = lane; v < vec_per_row; v += 64) {
    float acc[8];
    if (accumulate) {
      Elem<T>::load8(dx + (size_t)t * d + (size_t)v * 8, acc);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[q] = 0.0f;
    }
    // slot order, in groups of 8 whose row loads are all issued before the sums
    float sum[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) sum[q] = 0.0f;
    for (int s0 = 0; s0 < slots; s0 += 8) {
      int r[8];
      float w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int s = s0 + u;
        r[u] = -1;
        w[u] = 0.0f;
        if (s < slots) {
          r[u] = ids ? ids[o + s] : s;
          w[u] = dl[o + s];
        }
        if (w[u] == 0.0f) r[u] = -1;
      }
      float val[8][8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (r[u] >= 0) {
          Elem<T>::load8(w_router + (size_t)r[u] * d + (size_t)v * 8, val[u]);
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) val[u][q] = 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (r[u] >= 0) {
#pragma unroll
          for (int q = 0; q < 8; ++q) sum[q] += w[u] * val[u][q];
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] += sum[q];
    Elem<T>::store8(dx + (size_t)t * d + (size_t)v * 8, acc);
  }
}

// Dense products of the full-softmax gates (every alive expert carries a
// gradient), on the fp32 matrix cores: dl stays fp32, and x and W_r are
// widened exactly, so a product and its sum are fp32 as in a plain loop.
//   kDx:  dx[t, c] (+)= sum_e dl[t, e] W_r[e, c]        (K = E)
//   kDw:  part[s][e, c] = sum_{t in split s} dl[t, e] x[t, c], and the
//         split's bias sums                             (K = T / splits)
// 64 x 128 output tiles, 4 waves of 32 x 64 (v_mfma_f32_32x32x2_f32, operands
// swapped: a lane owns one row and 4 consecutive columns per register quad),
// 32 k at a time through LDS as [k][row], [k][column], the next 32 loaded into
// registers beside the MFMAs.  dW_r has only E x d outputs, so its tokens are
// split over enough workgroups to fill the chip twice and the partial tiles
// summed in order by a second kernel.  (Before: one wave per token walking all
// E rows of W_r for dx, one workgroup per (expert, 256 columns) reading all of
// x, E times in all, for dW_r: 74 + 198 us at 4096 tokens, 128 experts, d 1024;
// now 17 + 18 + 4 with the
// sum of the partial tiles.)
enum { kDx = 0, kDw = 1 };
constexpr int kDenseBM = 64, kDenseBN = 128, kDenseKC = 32;

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(bf16_t v) { return lo_bf16(v); }

template <typename T> struct Wide8;  // 8 consecutive elements -> fp32
template <> struct Wide8<bf16_t> {
  u32x4_t r;
  __device__ __forceinline__ void zero() { r = u32x4_t{0u, 0u, 0u, 0u}; }
  __device__ __forceinline__ void drop_nonfinite() {  // infinities and NaNs to zero
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool lo = (r[i] & 0x7f80u) == 0x7f80u, hi = (r[i] & 0x7f800000u) == 0x7f800000u;
      r[i] &= (lo ? 0xffff0000u : ~0u) & (hi ? 0xffffu : ~0u);
    }
  }
  __device__ __forceinline__ void load(const bf16_t* p) {
    r = *reinterpret_cast<const u32x4_t*>(p);
  }
  __device__ __forceinline__ void put(float* d) const {
    *reinterpret_cast<f32x4_t*>(d) = f32x4_t{lo_bf16(r[0]), hi_bf16(r[0]), lo_bf16(r[1]), hi_bf16(r[1])};
    *reinterpret_cast<f32x4_t*>(d + 4) = f32x4_t{lo_bf16(r[2]), hi_bf16(r[2]), lo_bf16(r[3]), hi_bf16(r[3])};
  }
};
template <> struct Wide8<float> {
  f32x4_t a, b;
  __device__ __forceinline__ void zero() { a = b = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
  __device__ __forceinline__ void drop_nonfinite() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = fabsf(a[i]) < INFINITY ? a[i] : 0.0f;
      b[i] = fabsf(b[i]) < INFINITY ? b[i] : 0.0f;
    }
  }
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4_t*>(p);
    b = *reinterpret_cast<const f32x4_t*>(p + 4);
  }
  __device__ __forceinline__ void put(float* d) const {
    *reinterpret_cast<f32x4_t*>(d) = a;
    *reinterpret_cast<f32x4_t*>(d + 4) = b;
  }
};

// Mrows: rows of the output (tokens for kDx, experts for kDw); K: the
// reduction length; k_per: its length per split (a multiple of 32).
// An infinite or NaN element of B must not reach the outputs whose dl is 0.  A tile
// whose sums are not all finite is formed again without such elements (the other
// sums keep their bits), and they are added afterwards, in the order of k, by the
// lanes that own the sums.
//   kDx: to the tokens whose dl is not 0 (an expert of probability 0 carries none,
//        whatever its row of W_r holds);
//   kDw, SPARSE (dl is 0 outside each token's selected experts, idx [T, k]): to the
//        experts that the token selected.
// kDw of full-softmax gates needs neither: every alive expert sees every token.
template <typename T, int MODE, bool SPARSE = false>
__global__ __launch_bounds__(256) void route_bwd_dense_kernel(
    const float* __restrict__ dl, const T* __restrict__ B, const uint8_t* __restrict__ alive,
    int Mrows, int K, int k_per, int E, int d, int accumulate, T* __restrict__ dx, float* __restrict__ part,
    float* __restrict__ part_b, const int32_t* __restrict__ idx, int k) {
  constexpr int BM = kDenseBM, BN = kDenseBN, KC = kDenseKC;
  constexpr int LDA = BM + 33, LDB = BN + 4;  // LDA odd: transposed writes spread over the banks
  __shared__ float sA[KC * LDA];
  __shared__ __attribute__((aligned(16))) float sB[KC * LDB];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int k0 = blockIdx.z * k_per, k1 = min(K, k0 + k_per);

  static_assert(!SPARSE || MODE == kDw, "dx reads every alive expert's row");
  constexpr bool APART = SPARSE || MODE == kDx;
  float ra[BM * KC / 256];
  Wide8<T> rb[KC * BN / 8 / 256];
  auto load = [&](int kb) {
#pragma unroll
    for (int i = 0; i < BM * KC / 256; ++i) {
      const int q = i * 256 + tid;
      // kDx: dl rows are tokens, k contiguous; kDw: dl rows are k, experts contiguous
      const int m = m0 + (MODE == kDx ? q / KC : q % BM);
      const int kk = kb + (MODE == kDx ? q % KC : q / BM);
      const bool ok = m < Mrows && kk < k1;
      const size_t at = MODE == kDx ? (size_t)m * E + kk : (size_t)kk * E + m;
      ra[i] = ok ? dl[at] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < KC * BN / 8 / 256; ++i) {
      const int q = i * 256 + tid;
      const int kk = kb + q / (BN / 8), c = n0 + (q % (BN / 8)) * 8;
      // kDx: a pruned expert's row of W_r is not read (its dl is 0, its weights anything)
      const bool row_ok = kk < k1 && (MODE == kDw || alive == nullptr || alive[kk] != 0);
      if (row_ok && c < d) rb[i].load(B + (size_t)kk * d + c);
      else rb[i].zero();
    }
  };
  auto store = [&](auto finite_only) {
#pragma unroll
    for (int i = 0; i < BM * KC / 256; ++i) {
      const int q = i * 256 + tid;
      if (MODE == kDx) sA[(q % KC) * LDA + q / KC] = ra[i];
      else sA[(q / BM) * LDA + q % BM] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < KC * BN / 8 / 256; ++i) {
      const int q = i * 256 + tid;
      if constexpr (decltype(finite_only)::value) rb[i].drop_nonfinite();
      rb[i].put(sB + (q / (BN / 8)) * LDB + (q % (BN / 8)) * 8);
    }
  };
  f32x16_t acc[2];
  const bool sums_bias = MODE == kDw && part_b != nullptr && blockIdx.y == 0 && tid < BM;
  float bias;

  const int lr = lane & 31, h = lane >> 5;
  auto product = [&](auto finite_only) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
    bias = 0.0f;
    if (k0 < k1) load(k0);
    for (int kb = k0; kb < k1; kb += KC) {
      store(finite_only);
      __syncthreads();
      if (kb + KC < k1) load(kb + KC);
#pragma unroll
      for (int s = 0; s < KC / 2; ++s) {
        const float a = sA[(2 * s + h) * LDA + wm * 32 + lr];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float b = sB[(2 * s + h) * LDB + wn * 64 + j * 32 + lr];
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b, a, acc[j], 0, 0, 0);
        }
      }
      if (sums_bias)
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) bias += sA[kk * LDA + tid];
      __syncthreads();
    }
  };
  product(std::false_type{});

  const int row = m0 + wm * 32 + lr;
  auto column = [&](int j, int q) { return n0 + wn * 64 + j * 32 + q * 8 + h * 4; };
  if constexpr (APART) {
    float any = 0.0f;  // stays 0 while every sum is finite
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) any = fmaf(acc[j][r], 0.0f, any);
    if (__syncthreads_or(any != 0.0f ? 1 : 0)) {
      product(std::true_type{});
      for (int kk = k0; kk < (row < Mrows ? k1 : k0); ++kk) {
        const float w = MODE == kDx ? dl[(size_t)row * E + kk] : dl[(size_t)kk * E + row];
        bool seen = MODE == kDx && w != 0.0f;  // (0 for a pruned expert)
        for (int s = 0; SPARSE && s < k; ++s) seen |= idx[(size_t)kk * k + s] == row;
        if (!seen) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = column(j, r >> 2) + (r & 3);
            const float v = c < d ? widen(B[(size_t)kk * d + c]) : 0.0f;
            if (!(fabsf(v) < INFINITY)) acc[j][r] += w * v;
          }
      }
    }
  }
  if (row < Mrows) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = column(j, q);
        if (c >= d) continue;
        f32x4_t v = {acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
        if constexpr (MODE == kDw) {
          *reinterpret_cast<f32x4_t*>(part + ((size_t)blockIdx.z * Mrows + row) * d + c) = v;
        } else if constexpr (sizeof(T) == 4) {
          f32x4_t* p = reinterpret_cast<f32x4_t*>(dx + (size_t)row * d + c);
          if (accumulate) v = *p + v;
          *p = v;
        } else {
          u32x2_t* p = reinterpret_cast<u32x2_t*>(dx + (size_t)row * d + c);
          if (accumulate) {
            const u32x2_t o = *p;
            v = f32x4_t{lo_bf16(o[0]), hi_bf16(o[0]), lo_bf16(o[1]), hi_bf16(o[1])} + v;
          }
          *p = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        }
      }
  }
  if (sums_bias && m0 + tid < Mrows) part_b[(size_t)blockIdx.z * Mrows + m0 + tid] = bias;
}

// dW_r = sum of the splits' partial tiles in split order, db likewise.  One
// output per thread: the E x d outputs are few, so wider vectors would leave
// the chip short of loads in flight.
__global__ __launch_bounds__(256) void route_bwd_dense_reduce_kernel(
    const float* __restrict__ part, const float* __restrict__ part_b, int splits, int E, int d,
    float* __restrict__ dw, float* __restrict__ db) {
  const size_t n = (size_t)E * d;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  auto sum = [&](const float* p, size_t stride) {
    float acc = 0.0f;
    for (int s0 = 0; s0 < splits; s0 += 16) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = s0 + u < splits ? p[(s0 + u) * stride] : 0.0f;
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += v[u];
    }
    return acc;
  };
  if (i < n) dw[i] = sum(part + i, n);
  if (db != nullptr && i < (size_t)E) db[i] = sum(part_b + i, E);
}

// Token splits of the dense dW_r: enough workgroups to fill the chip twice,
// each with at least two 32-token steps.
struct DenseSplit {
  int n, per;
};
inline DenseSplit dense_split(int T, int E, int d) {
  int tiles = ((E + kDenseBM - 1) / kDenseBM) * ((d + kDenseBN - 1) / kDenseBN);
  if (tiles < 1) tiles = 1;
  int n = (512 + tiles - 1) / tiles;
  const int most = (T + 2 * kDenseKC - 1) / (2 * kDenseKC);
  if (n > most) n = most;
  if (n < 1) n = 1;
  const int per = ((T + n - 1) / n + kDenseKC - 1) / kDenseKC * kDenseKC;
  return {per > 0 ? (T + per - 1) / per : 0, per};
}

// Renormalised gates of many experts, weight gradient in two deterministic passes.
// Pass 1: one workgroup per 128-row segment of an expert's routed rows (the
// row-tile table); the segment's (token, weight) pairs go to LDS first, then
// every x row is read whole (each thread one 8-column vector, eight rows in
// flight) and the segment's partial dW_r row and bias sum are written.
constexpr int kSegRows = 128;
template <typename T, int VPT>
__global__ __launch_bounds__(256) void route_bwd_dw_seg_kernel(
    const T* __restrict__ x, const float* __restrict__ dl, const int32_t* __restrict__ row_src,
    const TileEntry* __restrict__ table, const int* __restrict__ n_entries, int k, int d,
    float* __restrict__ part, float* __restrict__ part_b) {
  __shared__ int s_tok[kSegRows];
  __shared__ float s_w[kSegRows];
  const int entry = blockIdx.x;
  if (entry >= *n_entries) return;
  const TileEntry te = table[entry];
  const int tid = threadIdx.x;
  if (tid < te.rows) {
    const int sl = row_src[te.row0 + tid];
    s_tok[tid] = sl / k;
    s_w[tid] = dl[sl];
  }
  __syncthreads();
  const int nvec = d / 8;
  float* out = part + (size_t)entry * d;
  for (int v0 = 0; v0 < nvec; v0 += 256 * VPT) {
    float acc[VPT][8];
#pragma unroll
    for (int u = 0; u < VPT; ++u)
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[u][q] = 0.0f;
    for (int r0 = 0; r0 < te.rows; r0 += 8) {
      float val[8][VPT][8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
          const int v = v0 + u * 256 + tid;
          if (r0 + i < te.rows && v < nvec) {
            Elem<T>::load8(x + (size_t)s_tok[r0 + i] * d + (size_t)v * 8, val[i][u]);
          } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) val[i][u][q] = 0.0f;
          }
        }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float w = r0 + i < te.rows ? s_w[r0 + i] : 0.0f;
#pragma unroll
        for (int u = 0; u < VPT; ++u)
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[u][q] += w * val[i][u][q];
      }
    }
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const int v = v0 + u * 256 + tid;
      if (v < nvec) Elem<float>::store8(out + (size_t)v * 8, acc[u]);
    }
  }
  // the segment's bias sum, in row order
  float b = 0.0f;
  if (tid < 64) {
    for (int r = tid; r < te.rows; r += 64) b += s_w[r];
    b = wave_sum(b);
  }
  if (tid == 0) part_b[entry] = b;
}

// Pass 2: dW_r[e] = sum of the expert's segment partials in table order.
__global__ __launch_bounds__(256) void route_bwd_dw_reduce_kernel(
    const float* __restrict__ part, const float* __restrict__ part_b,
    const TileEntry* __restrict__ table, const int* __restrict__ n_entries, int E, int d,
    float* __restrict__ dw, float* __restrict__ db) {
  // the expert's segments are consecutive in the table; find them in parallel
  __shared__ int s_first, s_count;
  const int e = blockIdx.x;
  if (threadIdx.x == 0) {
    s_first = INT_MAX;
    s_count = 0;
  }
  __syncthreads();
  const int n = *n_entries;
  for (int i = threadIdx.x; i < n; i += 256)
    if (table[i].expert == e) {
      atomicMin(&s_first, i);
      atomicAdd(&s_count, 1);
    }
  __syncthreads();
  const int first = s_first, count = s_count;
  for (int c = blockIdx.y * 256 + threadIdx.x; c < d; c += gridDim.y * 256) {
    float acc = 0.0f;
    for (int i = 0; i < count; ++i) acc += part[(size_t)(first + i) * d + c];
    dw[(size_t)e * d + c] = acc;
  }
  if (db != nullptr && blockIdx.y == 0 && threadIdx.x == 0) {
    float acc = 0.0f;
    for (int i = 0; i < count; ++i) acc += part_b[first + i];
    db[e] = acc;
  }
}

__global__ void fill_zero_kernel(float* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0.0f;
}

}  // namespace

// ws: dl by slot, dl by expert; then the segment table, partial rows and sums, or
// the dense product's partial tiles and sums.
inline int seg_max(int T, int k, int E) { return (int)(((int64_t)T * k + kSegRows - 1) / kSegRows) + E; }

// Renormalised gates, dW_r: the dense product over all tokens and experts (dl is
// zero outside the k selected ones) or the segment sums over the routed rows.  The
// dense product multiplies a token's x by 64 experts at a time and reads it as
// often, the segments read it k times, but gather it and, with few rows an expert,
// wait for their loads more than they use them.  So: dense from 8 slots per 64
// experts, and for less than that while x is small; the line grows with k, and
// steeply, since with one slot the segments read x once, in order.  Whole
// weights-only call, dense / segments, us, bf16, d 2048 (x of 33.6 MB at 8192
// tokens):
//             experts, slots   8, 1       64, 1      64, 2      64, 8      128, 8
//     1000 tokens            15 / 38    16 / 17    16 / 20    16 / 40    23 / 28
//     8192 tokens            30 / 56    34 / 55    37 / 58    38 / 69    60 / 67
//    40000 tokens           115 / 76   118 / 64   126 / 71   130 / 202  227 / 197
// Over 1863 sizes (64 to 100000 tokens, d 256 to 4096, 4 to 256 experts, both
// types) eight are more than 3 % behind the segments, 22 % and 4 us at most.
inline bool renorm_dw_dense(int T, int E, int k, int d, int elem_bytes) {
  const int tiles = (E + kDenseBM - 1) / kDenseBM;
  const double bytes = (double)T * d * elem_bytes;
  if (k >= 8 * tiles) return true;
  return tiles == 1 ? bytes <= 12e6 * k * k : E <= 16 * k && bytes <= 16e6;
}

// dx of full-softmax gates: over few experts the dense product's tiles hold little
// work beside their rows of dx, which a wave per token reads and writes in whole
// lines; with few tokens that is one long wait.  By rows / dense, us, accumulated,
// bf16: 8192 tokens, d 2048, 4 experts 25 / 47, 8 31 / 47, 16 48 / 47, 32 80 / 47;
// 40000 tokens 90 / 139, 116 / 140, 184 / 143; 1000 tokens of 8 experts 15 / 12.
inline bool dx_by_rows(int T, int E) { return E <= 8 && T >= 400 * E && T < 1 << 26; }

size_t route_bwd_ws_bytes(int T, int k, int E, int d) {
  const int m = seg_max(T, k, E);
  const size_t seg = table_bytes(m) + align_up((size_t)m * d * sizeof(float), 256) +
                     align_up((size_t)m * sizeof(float), 256);
  // not the dense product's own splits, whose number falls where a split gains a
  // step or the output a tile, but bounds that grow with every size, so that a
  // workspace for the largest call serves the smaller ones: at most 512 and T / 64
  // splits (rounded up), and less than 512 tiles of 64 x 128 beyond one output
  const size_t n = (size_t)(T + 63) / 64 < 512 ? (size_t)(T + 63) / 64 : 512;
  auto least = [](size_t a, size_t b) { return a < b ? a : b; };
  const size_t dense =
      align_up(least(n * E * d, (size_t)512 * kDenseBM * kDenseBN + (size_t)E * d) * sizeof(float), 256) +
      align_up(least(n * E, (size_t)512 * kDenseBM + E) * sizeof(float), 256);
  return align_up((size_t)T * k * sizeof(float), 256) + align_up((size_t)T * E * sizeof(float), 256) +
         (seg > dense ? seg : dense);
}

namespace {

// dW_r (and db) from the dense dl [T, E]
template <typename T, bool SPARSE>
void launch_dense_dw(const float* dl, const T* x, int T_, int E, int d, char* base,
                     float* dw_router, float* dbias, const int32_t* idx, int k, hipStream_t s) {
  const DenseSplit sp = dense_split(T_, E, d);
  const bool one = sp.n == 1;  // its partial tiles are dW_r
  float* part = one ? dw_router : reinterpret_cast<float*>(base);
  float* part_b = one ? dbias : reinterpret_cast<float*>(
                                    base + align_up((size_t)sp.n * E * d * sizeof(float), 256));
  hipLaunchKernelGGL((route_bwd_dense_kernel<T, kDw, SPARSE>),
                     dim3((unsigned)((E + kDenseBM - 1) / kDenseBM),
                          (unsigned)((d + kDenseBN - 1) / kDenseBN), (unsigned)sp.n),
                     dim3(256), 0, s, dl, x, nullptr, E, T_, sp.per, E, d, 0,
                     static_cast<T*>(nullptr), part, dbias ? part_b : nullptr, idx, k);
  if (one) return;
  const size_t n = (size_t)E * d;  // >= E
  hipLaunchKernelGGL(route_bwd_dense_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256),
                     0, s, part, part_b, sp.n, E, d, dw_router, dbias);
}

template <typename T>
hipError_t launch_route_bwd_t(const float* dgate, const int32_t* idx, const float* gate,
                              const float* logits, const uint8_t* alive, const T* x,
                              const T* w_router, const int32_t* offsets, const int32_t* row_src,
                              int T_, int d, int E, int k, int renorm, float* dlogits,
                              float* dw_router, float* dbias, T* dx, int accumulate_dx, void* ws,
                              hipStream_t s) {
  float* dl = static_cast<float*>(ws);  // [T, k]
  float* dl_dense = reinterpret_cast<float*>(static_cast<char*>(ws) +
                                             align_up((size_t)T_ * k * sizeof(float), 256));
  char* base = reinterpret_cast<char*>(dl_dense) + align_up((size_t)T_ * E * sizeof(float), 256);
  if (!renorm) {
    const int lanes = E <= 32 ? dl_lanes(E) : 64;
    const auto dl_full = lanes < 64 ? route_bwd_dl_full_kernel<true> : route_bwd_dl_full_kernel<false>;
    hipLaunchKernelGGL(dl_full, dl_grid(T_, 64 / lanes), dim3(kDlThreads), 0, s, dgate, idx, gate,
                       logits, alive, T_, E, k, lanes, dl_dense, dlogits);
    if (dx && dx_by_rows(T_, E))
      hipLaunchKernelGGL(route_bwd_dx_kernel<T>, dim3((unsigned)((T_ + 3) / 4)), dim3(256), 0, s,
                         w_router, static_cast<const int32_t*>(nullptr), dl_dense, T_, E, d,
                         accumulate_dx, dx);
    else if (dx)
      hipLaunchKernelGGL((route_bwd_dense_kernel<T, kDx>),
                         dim3((unsigned)((T_ + kDenseBM - 1) / kDenseBM),
                              (unsigned)((d + kDenseBN - 1) / kDenseBN)),
                         dim3(256), 0, s, dl_dense, w_router, alive, T_, E, E, E, d, accumulate_dx,
                         dx, nullptr, nullptr, nullptr, 0);
    if (dw_router) launch_dense_dw<T, false>(dl_dense, x, T_, E, d, base, dw_router, dbias, idx, k, s);
    return hipGetLastError();
  }
  const bool dense = dw_router && renorm_dw_dense(T_, E, k, d, (int)sizeof(T));
  if (!dense && !dlogits && k <= 64) {
    const int lanes = dl_lanes(k);
    hipLaunchKernelGGL(route_bwd_dl_slots_kernel, dl_grid(T_, 64 / lanes), dim3(kDlThreads), 0, s,
                       dgate, idx, gate, T_, k, lanes, dl);
  } else {
    hipLaunchKernelGGL(route_bwd_dl_kernel, dl_grid(T_, 1), dim3(kDlThreads), 0, s, dgate, idx,
                       gate, T_, E, k, dl, dense ? dl_dense : nullptr, dlogits);
  }
  if (dx)
    hipLaunchKernelGGL(route_bwd_dx_kernel<T>, dim3((unsigned)((T_ + 3) / 4)), dim3(256), 0, s,
                       w_router, idx, dl, T_, k, d, accumulate_dx, dx);
  if (dense) {
    launch_dense_dw<T, true>(dl_dense, x, T_, E, d, base, dw_router, dbias, idx, k, s);
  } else if (dw_router) {
    // segment table of the routed rows (pass 1 + 2)
    const int m = seg_max(T_, k, E);
    TableWs tw = carve_table(base, m);
    float* part = reinterpret_cast<float*>(base + table_bytes(m));
    float* part_b = reinterpret_cast<float*>(base + table_bytes(m) + align_up((size_t)m * d * 4, 256));
    hipLaunchKernelGGL(build_table_kernel, dim3(1), dim3(kTableThreads), 0, s, offsets, nullptr, E,
                       kSegRows, 0, m, tw.n_entries, tw.table);
    hipLaunchKernelGGL((route_bwd_dw_seg_kernel<T, 1>), dim3(m), dim3(256), 0, s, x, dl, row_src,
                       tw.table, tw.n_entries, k, d, part, part_b);
    const dim3 gred(E, (d + 255) / 256 < 8 ? (d + 255) / 256 : 8);
    hipLaunchKernelGGL(route_bwd_dw_reduce_kernel, gred, dim3(256), 0, s, part, part_b, tw.table,
                       tw.n_entries, E, d, dw_router, dbias);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_route_bwd(const float* dgate, const int32_t* idx, const float* gate,
                            const float* logits, const uint8_t* alive, const void* x,
                            const void* w_router, const int32_t* offsets, const int32_t* row_src,
                            int dtype, int T_, int d, int E, int k, int renorm, float* dlogits,
                            float* dw_router, float* dbias, void* dx, int accumulate_dx, void* ws,
                            hipStream_t s) {
  if (T_ == 0) {
    // no tokens: zero weight gradients (dx has no rows)
    if (dw_router)
      hipLaunchKernelGGL(fill_zero_kernel, dim3(64), dim3(256), 0, s, dw_router, (size_t)E * d);
    if (dbias) hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, s, dbias, (size_t)E);
    return hipGetLastError();
  }
  if (dtype == kDtypeBf16)
    return launch_route_bwd_t(dgate, idx, gate, logits, alive, static_cast<const bf16_t*>(x),
                              static_cast<const bf16_t*>(w_router), offsets, row_src, T_, d, E, k,
                              renorm, dlogits, dw_router, dbias, static_cast<bf16_t*>(dx),
                              accumulate_dx, ws, s);
  return launch_route_bwd_t(dgate, idx, gate, logits, alive, static_cast<const float*>(x),
                            static_cast<const float*>(w_router), offsets, row_src, T_, d, E, k,
                            renorm, dlogits, dw_router, dbias, static_cast<float*>(dx),
                            accumulate_dx, ws, s);
}

}  // namespace laep
