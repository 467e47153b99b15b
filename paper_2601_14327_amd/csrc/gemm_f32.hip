// Grouped SwiGLU expert FFN, forward, in fp32 (moe_grouped_ffn_fwd with
// LAEP_F32): the full-precision variant for small layers, on the fp32 matrix
// cores (v_mfma_f32_32x32x2_f32: fp32 products and sums).
//
// At these sizes (a few hundred rows, d and d_ff of a few hundred) the call
// is a chain of latencies, not of flops: 32 x 32 output tiles give enough
// workgroups, the four waves of a workgroup split K and load their operands
// straight into registers, U k-steps of 8 in flight with the next U behind
// them, and one LDS round sums the four partial tiles in wave order.  No tile
// table: every workgroup finds its tile from the expert offsets.  (Before: a
// fused-multiply-add loop staging 16 k at a time through LDS with nothing in
// flight, 2.7 + 21.6 + 35.4 us for the table and the two products at 512 rows,
// d 128, d_ff 256, 8 experts; now 7.3 + 6.6.)
//
// The gate/up pass computes the same 32 f-columns of gate and up in one tile,
// so the SwiGLU epilogue needs no second pass: act_save = A, H = silu(A_g) * A_u.
#include "common.hpp"
#include "internal.hpp"
#include "tiles.hpp"

namespace laep {
namespace {

constexpr int kT = 32;     // rows and columns per tile
constexpr int kF32Threads = 256;
constexpr int kF32Waves = kF32Threads / 64;

// GU: B holds gate rows [0, f) and up rows [f, 2f), out = H, out2 = act_save or
// NULL.  Else out = Y.  K % 64 == 0 (two 8-k steps per wave at least).
template <bool GU>
__global__ __launch_bounds__(kF32Threads) void gemm_f32_kernel(
    const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
    long long strideB, int K, int f, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ expert_map, int E, int n_tiles_n, unsigned grid_x,
    float* __restrict__ out, int ldo, float* __restrict__ out2) {
  constexpr int NB = GU ? 2 : 1;   // column blocks of a tile: gate and up, or one
  constexpr int U = GU ? 4 : 8;    // 8-k steps in flight
  constexpr int LD = kT + 4;       // floats per staged row
  __shared__ __attribute__((aligned(16))) float s_part[kF32Waves * NB * kT * LD];
  FoundTile te;
  if (!find_tile(blockIdx.y * grid_x + blockIdx.x, offsets, expert_map, E, kT, n_tiles_n,
                 reinterpret_cast<char*>(s_part), te))
    return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int lr = lane & 31, h = lane >> 5;
  const int n0 = te.nt * kT;

  // lane (lr, h) feeds row lr, k = 8 step + 4 h + i to the i-th MFMA of a step
  const int steps = K / (8 * kF32Waves);
  const int row = lr < te.rows ? lr : te.rows - 1;  // rows past the expert: any valid row
  const size_t k0 = (size_t)wave * steps * 8 + h * 4;
  const float* pa = A + (size_t)(te.row0 + row) * lda + k0;
  const float* pb[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
    pb[b] = B + (size_t)te.phys * strideB + (size_t)(b * f + n0 + lr) * ldb + k0;

  f32x16_t acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;
  f32x4_t va[U], vb[U][NB], na[U], nb[U][NB];
  auto load = [&](int s0, f32x4_t* a, f32x4_t (*b)[NB]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < steps) {
        a[u] = *reinterpret_cast<const f32x4_t*>(pa + (s0 + u) * 8);
#pragma unroll
        for (int c = 0; c < NB; ++c)
          b[u][c] = *reinterpret_cast<const f32x4_t*>(pb[c] + (s0 + u) * 8);
      }
  };
  load(0, va, vb);
  for (int s0 = 0; s0 < steps; s0 += U) {
    load(s0 + U, na, nb);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < steps)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < NB; ++c)
            acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(vb[u][c][i], va[u][i], acc[c], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      va[u] = na[u];
#pragma unroll
      for (int c = 0; c < NB; ++c) vb[u][c] = nb[u][c];
    }
  }
  // partial tiles: the lane owns row lr and columns 8q + 4h .. +3 per quad
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4_t*>(s_part + ((wave * NB + c) * kT + lr) * LD + q * 8 + h * 4) =
          f32x4_t{acc[c][4 * q], acc[c][4 * q + 1], acc[c][4 * q + 2], acc[c][4 * q + 3]};
  __syncthreads();
  const int r = tid >> 3, col = (tid & 7) * 4;
  if (r >= te.rows) return;
  f32x4_t v[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    v[c] = *reinterpret_cast<const f32x4_t*>(s_part + (c * kT + r) * LD + col);
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w)
      v[c] += *reinterpret_cast<const f32x4_t*>(s_part + ((w * NB + c) * kT + r) * LD + col);
  }
  const size_t grow = (size_t)te.row0 + r;
  if constexpr (GU) {
    f32x4_t hv;
#pragma unroll
    for (int i = 0; i < 4; ++i) hv[i] = (v[0][i] / (1.0f + expf(-v[0][i]))) * v[1][i];
    *reinterpret_cast<f32x4_t*>(out + grow * f + n0 + col) = hv;
    if (out2) {
      *reinterpret_cast<f32x4_t*>(out2 + grow * 2 * f + n0 + col) = v[0];
      *reinterpret_cast<f32x4_t*>(out2 + grow * 2 * f + f + n0 + col) = v[1];
    }
  } else {
    *reinterpret_cast<f32x4_t*>(out + grow * ldo + n0 + col) = v[0];
  }
}

}  // namespace

hipError_t launch_ffn_fwd_f32(const void* x_perm, const void* w_gu, const void* w_d,
                              const int32_t* offsets, const int32_t* expert_map, int E, int d,
                              int f, int64_t R, void* y_perm, void* act_save, void* ws,
                              hipStream_t s) {
  if (R <= 0) return hipSuccess;
  float* H = static_cast<float*>(ws);
  // sum of ceil(rows / kT) over the experts with rows, to a multiple of 8 (the
  // tile search takes one range per XCD); in two dimensions, since one holds
  // less than 2^32 threads
  const int64_t rows = R / kT + (R < E ? R : E);
  auto grid = [&](int n_tiles_n) {
    const int64_t blocks = (rows * n_tiles_n + 7) / 8 * 8, x = blocks < 1 << 20 ? blocks : 1 << 20;
    return dim3((unsigned)x, (unsigned)((blocks + x - 1) / x));
  };
  const int nt_gu = f / kT, nt_d = d / kT;
  const dim3 gu = grid(nt_gu), dn = grid(nt_d);
  hipLaunchKernelGGL((gemm_f32_kernel<true>), gu, dim3(kF32Threads), 0, s,
                     static_cast<const float*>(x_perm), d, static_cast<const float*>(w_gu), d,
                     (long long)2 * f * d, d, f, offsets, expert_map, E, nt_gu, gu.x, H, f,
                     static_cast<float*>(act_save));
  hipLaunchKernelGGL((gemm_f32_kernel<false>), dn, dim3(kF32Threads), 0, s, H, f,
                     static_cast<const float*>(w_d), f, (long long)d * f, f, f, offsets,
                     expert_map, E, nt_d, dn.x, static_cast<float*>(y_perm), d, nullptr);
  return hipGetLastError();
}

}  // namespace laep
