// Forward grouped bf16 GEMMs for few rows per expert (decode batches, short
// prompts, small micro-batches): the same two products as gemm_bf16.hip.
//
// With a few dozen rows per expert every weight byte is used once, so the
// products are bound by streaming the weights from HBM, and 256-row tiles do
// that badly: each k-step moves as many (repeated) activation rows through
// LDS as weight rows, one workgroup fills a CU, and 64 experts x 4-8 column
// blocks leave an uneven last wave.  Here a tile is BM x 128 (BM = 32, 64 or
// 128) in a workgroup of 4 waves, with a ring of NST k-steps of 64 in at most
// 80 KB of LDS, so two workgroups share a CU and each keeps NST - 1 steps of
// weights in flight.
// No tile list: every workgroup finds its tile from the expert offsets.
//
// The k order and the MFMA are those of the 256-row kernels, so the results
// have the same bits.
#include <cmath>
#include <type_traits>

#include "gemm_common.hpp"

namespace laep {
namespace {

constexpr int kSmallThreads = 256;
constexpr int kSmallBN = 128;
static_assert(kSmallThreads == kTableThreads, "one thread per expert in find_tile");

struct SmallParams {
  const bf16_t* A;
  long long lda;
  const bf16_t* B;
  long long ldb, strideB;
  int N, K, f;
  const int32_t* offsets;
  const int32_t* expert_map;
  int E;
  int n_tiles_n;
  bf16_t* out;
  long long ldo;
  bf16_t* act;              // gate/up: pre-activations [R, 2f] or NULL
  const int32_t* row_src;   // gathered A rows; or the scatter's token rows
  int slots_k;
  const float* gate;        // scatter (one slot per token)
  bf16_t* out_tok;
  int stream;               // weights read once are past what the caches hold
};

template <int BM, int NST, int EPI, bool GATHER>
__global__ __launch_bounds__(kSmallThreads) void gemm_small_kernel(SmallParams p) {
  constexpr int BN = kSmallBN, NT = kSmallThreads;
  constexpr int NWM = BM == 128 ? 2 : 1, NWN = 4 / NWM;
  constexpr int WTM = BM / NWM, WTN = BN / NWN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int ROWB = 128;                    // bytes per LDS row (64 k)
  constexpr int ABYTES = BM * ROWB, STAGE = (BM + BN) * ROWB;
  constexpr int NA = BM * 8 / NT, NB = BN * 8 / NT, NC = NA + NB;
  constexpr int PITCH = BN * 2 + 16;           // bytes per staged output row
  constexpr int SMEM = NST * STAGE;
  static_assert(BM * PITCH <= SMEM, "the output tile is staged in the ring");
  static_assert(NST >= 2 && NST <= 5, "the wait dispatch below covers 0..3 steps in flight");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  FoundTile te;
  if (!find_tile(p.offsets, p.expert_map, p.E, BM, p.n_tiles_n, smem, te)) return;
  const int nt = te.nt;

  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave / NWN, wn = wave % NWN;

  // byte offsets of the chunks this thread copies (k-step 0): A from the
  // tile's first row (gathered: from x), B from the expert's weights
  uint32_t a_voff[NA], b_voff[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int q = i * NT + tid, r = q >> 3;
    const int lc = (q & 7) ^ swz8(r);
    const int rr = r < te.rows ? r : te.rows - 1;  // rows past the expert: any valid row
    const long long arow = GATHER ? (long long)(p.row_src[te.row0 + rr] / p.slots_k) : rr;
    a_voff[i] = (uint32_t)((arow * p.lda + lc * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int q = i * NT + tid, r = q >> 3;
    const int lc = (q & 7) ^ swz8(r);
    int row;
    if (EPI == EPI_GU) {  // 16 gate rows, then the same 16 f-columns' up rows, per 32
      const int fcol = nt * (BN / 2) + (r >> 5) * 16 + (r & 15);
      row = (r & 16) ? p.f + fcol : fcol;
    } else {
      row = nt * BN + r;
      row = row < p.N ? row : p.N - 1;
    }
    b_voff[i] = (uint32_t)(((long long)row * p.ldb + lc * 8) * 2);
  }
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(GATHER ? p.A : p.A + (long long)te.row0 * p.lda), 0, -1, kBufferFlags);
  const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.B + (long long)te.phys * p.strideB), 0, -1, kBufferFlags);
  const int nk = p.K / 64;
  // weights that only this row tile reads stream past the caches
  const bool stream = p.stream && te.expert_rows <= BM;
  auto issue = [&](int kt) {
    char* dst = smem + (kt % NST) * STAGE;
    if (stream) dma_chunks<NB, NT, kDmaStream>(dst + ABYTES, b_rsrc, b_voff, kt * 128, wave_s);
    else dma_chunks<NB, NT>(dst + ABYTES, b_rsrc, b_voff, kt * 128, wave_s);
    dma_chunks<NA, NT>(dst, a_rsrc, a_voff, kt * 128, wave_s);
  };

  // fragment byte offsets within a stage for k16 sub-step 0 (sub-step s: ^ 32 s)
  int a_off[TM], b_off[TN];
  const int lc0 = lane >> 5;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = wm * WTM + i * 32 + (lane & 31);
    a_off[i] = r * ROWB + ((lc0 ^ swz8(r)) << 4);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int r = wn * WTN + j * 32 + (lane & 31);
    b_off[j] = ABYTES + r * ROWB + ((lc0 ^ swz8(r)) << 4);
  }
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < nk) issue(t);
  for (int kt = 0; kt < nk; ++kt) {
    // step kt has landed: the steps issued after it (at most NST - 2) may
    // still be in flight; past the barrier that holds for every thread, and
    // every thread has read step kt - 1, whose stage takes step kt + NST - 1
    const int ahead = min(nk - 1 - kt, NST - 2);
    if (ahead >= 3) wait_vmcnt<3 * NC>();
    else if (ahead == 2) wait_vmcnt<2 * NC>();
    else if (ahead == 1) wait_vmcnt<NC>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    if (kt + NST - 1 < nk) issue(kt + NST - 1);
    const char* st = smem + (kt % NST) * STAGE;
    u32x4_t fa[4][TM], fb[4][TN];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[s][j] = *reinterpret_cast<const u32x4_t*>(st + (b_off[j] ^ (s << 5)));
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[s][i] = *reinterpret_cast<const u32x4_t*>(st + (a_off[i] ^ (s << 5)));
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8_t, fb[s][j]), __builtin_bit_cast(bf16x8_t, fa[s][i]),
              acc[i][j], 0, 0, 0);
    // the reads of this step are in registers before the next barrier frees it
    wait_lgkm0();
  }
  __builtin_amdgcn_s_barrier();  // every wave's reads are done: the ring is free for staging

  // ---- epilogue: lane owns row lane % 32 of each block and 4 consecutive columns
  // per register quad; staged through LDS so that whole row segments are written
  const int lrow = lane & 31;
  const int lcol = (lane >> 5) * 4;
  auto stage = [&](int row, int col, float a, float b, float c, float d) {
    u32x2_t w = {pack_bf16x2(a, b), pack_bf16x2(c, d)};
    *reinterpret_cast<u32x2_t*>(smem + row * PITCH + col * 2) = w;
  };
  auto sync = [&]() {
    wait_lgkm0();
    __builtin_amdgcn_s_barrier();
  };
  // staged columns [scol0, scol0 + 8 * CPR) -> dst + (te.row0 + row) * ld
  auto flush = [&](auto cpr_tag, bf16_t* dst, long long ld, int ncols, int scol0) {
    constexpr int CPR = decltype(cpr_tag)::value;
#pragma unroll
    for (int c = tid; c < BM * CPR; c += NT) {
      const int r = c / CPR, cc = c % CPR;
      if (r < te.rows && cc * 8 < ncols)
        *reinterpret_cast<u32x4_t*>(dst + (te.row0 + r) * ld + cc * 8) =
            *reinterpret_cast<const u32x4_t*>(smem + r * PITCH + (scol0 + cc * 8) * 2);
    }
  };
  if constexpr (EPI == EPI_GU) {
    const int f = p.f, fbase = nt * (BN / 2);  // f % 64 == 0: every column block is whole
    using Half = std::integral_constant<int, BN / 16>;
    auto each = [&](auto fn) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            fn(wm * WTM + i * 32 + lrow, ((wn * WTN) / 32 + j) * 16 + q * 8 + lcol, acc[i][j], q);
    };
    if (p.act) {
      each([&](int r, int c, const f32x16_t& a, int q) {
        stage(r, c, a[q * 4], a[q * 4 + 1], a[q * 4 + 2], a[q * 4 + 3]);
        stage(r, BN / 2 + c, a[8 + q * 4], a[9 + q * 4], a[10 + q * 4], a[11 + q * 4]);
      });
      sync();
      flush(Half{}, p.act + fbase, 2LL * f, BN / 2, 0);
      flush(Half{}, p.act + f + fbase, 2LL * f, BN / 2, BN / 2);
      sync();
    }
    each([&](int r, int c, const f32x16_t& a, int q) {
      float h[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) h[u] = fast_silu(a[q * 4 + u]) * a[8 + q * 4 + u];
      stage(r, c, h[0], h[1], h[2], h[3]);
    });
    sync();
    flush(Half{}, p.out + fbase, f, BN / 2, 0);
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          stage(wm * WTM + i * 32 + lrow, wn * WTN + j * 32 + q * 8 + lcol, acc[i][j][q * 4],
                acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]);
    sync();
    const int ncols = min(BN, p.N - nt * BN);
    if (!p.out_tok) {
      flush(std::integral_constant<int, BN / 8>{}, p.out + nt * BN, p.ldo, ncols, 0);
      return;
    }
    // scatter (one slot per token), with the combine's arithmetic
    constexpr int CPR = BN / 8;
#pragma unroll
    for (int c = tid; c < BM * CPR; c += NT) {
      const int r = c / CPR, cc = c % CPR;
      if (r < te.rows && cc * 8 < ncols) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(smem + r * PITCH + cc * 16);
        const long long row = (long long)te.row0 + r;
        if (p.out) *reinterpret_cast<u32x4_t*>(p.out + row * p.ldo + nt * BN + cc * 8) = v;
        const int src = p.row_src[row];
        const float g = p.gate[src];
        u32x4_t o;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          float lo = 0.0f, hi = 0.0f;
          lo += g * lo_bf16(v[w]);
          hi += g * hi_bf16(v[w]);
          o[w] = pack_bf16x2(lo, hi);
        }
        *reinterpret_cast<u32x4_t*>(p.out_tok + (long long)(src / p.slots_k) * p.ldo + nt * BN +
                                    cc * 8) = o;
      }
    }
  }
}

template <int BM, int NST, int EPI, bool GATHER>
hipError_t launch_small(const SmallParams& p, int64_t R, hipStream_t s) {
  // sum of ceil(rows / BM) over the experts with rows
  const int64_t tiles = (R / BM + (R < p.E ? R : p.E)) * p.n_tiles_n;
  if (tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((gemm_small_kernel<BM, NST, EPI, GATHER>), dim3(round8((int)tiles)),
                     dim3(kSmallThreads), 0, s, p);
  return hipGetLastError();
}

template <int BM, int NST>
hipError_t launch_small_pair(SmallParams g, SmallParams dn, int64_t R, bool gather,
                             hipStream_t s) {
  const hipError_t err = gather ? launch_small<BM, NST, EPI_GU, true>(g, R, s)
                                : launch_small<BM, NST, EPI_GU, false>(g, R, s);
  return err != hipSuccess ? err : launch_small<BM, NST, EPI_STORE, false>(dn, R, s);
}

}  // namespace

// Row-tile height by estimated time, root of the sum of squares of two parts:
//  - the weights' stream from HBM, at the rate each kernel reaches with few
//    rows (64 experts of 12.6 MB: 4.1 TB/s at 256 rows, 5.3-5.5 below);
//  - the k-steps a CU works through, each at its measured time: 0.275 / 0.40 /
//    0.64 us per tile at 32 / 64 / 128 rows (two or more workgroups sharing a
//    CU; 0.45 / 0.5 / 0.72 for one alone), and 1.9 us per full 256-row tile
//    (256 columns wide; a part of it for part of the rows, 0.8 more for each
//    further, partly filled tile, 1.0 at least).  The 256-row kernels hold one
//    workgroup per CU, so under two rounds of tiles whole rounds count.
// The experts' rows are taken as even (the host does not know them); where
// most loads no longer fit a whole number of tiles half a tile is added.
// Measured, us for both products (estimates within 20 %, the choice within
// 10 % of the best; d = 2048, f = 1024, E = 64, then d = f = 1024, E = 16):
//   rows each   32 / 64 / 128 / 256-row tiles    rows each
//     1         105 / 112 / 138 / 163              8          21 /  23 /  29 / 42
//    32         161 / 163 / 186 / 199             64          29 /  27 /  32 / 43
//    64         205 / 184 / 193 / 206            128          42 /  37 /  34 / 48
//    96         248 / 214 / 198 / 214            512         116 /  90 /  79 / 90
//   128         297 / 250 / 255 / 221            768         173 / 131 / 111 / 100
int small_fwd_bm(int64_t R, int E, int d, int f) {
  struct Kernel {
    int bm;           // returned as 0 for the 256-row kernels
    int cols_gu, cols_d;
    double step_us, alone_us, stream_bytes_per_us;
  };
  const Kernel kernels[] = {
      {256, ceil_div(f, 128), ceil_div(d, 256), 1.9, 1.0, 4.1e6},
      {128, f / 64, ceil_div(d, 128), 0.64, 0.72, 5.3e6},
      {64, f / 64, ceil_div(d, 128), 0.40, 0.5, 5.4e6},
      {32, f / 64, ceil_div(d, 128), 0.275, 0.45, 5.5e6},
  };
  constexpr double kCUs = 256, kPartTile = 0.8;
  const double rows = (double)R / E;
  // experts that R rows spread at random reach
  const double live = E * (1.0 - std::pow(1.0 - 1.0 / E, (double)R));
  int best = 0;
  double best_us = 0.0;
  for (const Kernel& kn : kernels) {
    const double r = rows / kn.bm;
    const double over = r < 0.75 ? 0.0 : r < 1.0 ? 2.0 * (r - 0.75) : 0.5;
    const double tiles = r + over > 1.0 ? r + over : 1.0;  // of one expert
    auto product = [&](int cols, int K) {
      const double per_cu = live * cols / kCUs;  // experts' column blocks
      double us = kn.step_us * tiles * per_cu;
      if (kn.bm == 256) {
        us = (kn.step_us * r + kPartTile * (tiles - (r > 1.0 ? r : 1.0))) * per_cu;
        const double rounds = tiles * per_cu;
        if (rounds < 2.0) us *= std::ceil(rounds) / rounds;
      }
      return K / 64 * (us > kn.alone_us ? us : kn.alone_us);
    };
    const double us = std::hypot(live * 6.0 * d * f / kn.stream_bytes_per_us,
                                 product(kn.cols_gu, d) + product(kn.cols_d, f));
    if (best_us == 0.0 || us < best_us) {
      best_us = us;
      best = kn.bm;
    }
  }
  return best == 256 ? 0 : best;
}

hipError_t launch_ffn_fwd_small(int bm, const void* x, const void* w_gu, const void* w_d,
                                const int32_t* offsets, const int32_t* expert_map, int E, int d,
                                int f, int64_t R, void* y_perm, void* act_save, void* H,
                                hipStream_t s, const int32_t* row_src, int slots_k,
                                const float* gate, void* out_tok) {
  SmallParams g = {};
  g.offsets = offsets;
  g.expert_map = expert_map;
  g.E = E;
  g.f = f;
  g.slots_k = slots_k;
  SmallParams dn = g;
  g.A = static_cast<const bf16_t*>(x);
  g.lda = d;
  g.B = static_cast<const bf16_t*>(w_gu);
  g.ldb = d;
  g.strideB = (long long)2 * f * d;
  g.N = 2 * f;
  g.K = d;
  g.n_tiles_n = f / (kSmallBN / 2);
  g.out = static_cast<bf16_t*>(H);
  g.ldo = f;
  g.act = static_cast<bf16_t*>(act_save);
  g.row_src = row_src;
  dn.A = static_cast<const bf16_t*>(H);
  dn.lda = f;
  dn.B = static_cast<const bf16_t*>(w_d);
  dn.ldb = f;
  dn.strideB = (long long)d * f;
  dn.N = d;
  dn.K = f;
  dn.n_tiles_n = ceil_div(d, kSmallBN);
  dn.out = static_cast<bf16_t*>(y_perm);
  dn.ldo = d;
  dn.row_src = out_tok ? row_src : nullptr;
  dn.gate = gate;
  dn.out_tok = static_cast<bf16_t*>(out_tok);
  // Streaming reads of the weights move 6.0 TB/s against 5.4 (64 experts of
  // 12.6 MB: 151 -> 136 us at 12 rows each, 105 -> 95 us at one).  Not below
  // what the 256 MB last-level cache can hold, where an earlier pass may have
  // left them there (16 experts of 6.3 MB: 21 -> 22 us), and not where several
  // row tiles of an expert read them (32-row tiles at 32 rows each: 152 -> 167).
  const int64_t live = R < E ? R : E;
  g.stream = dn.stream = live * 6 * d * f > ((int64_t)256 << 20);
  const bool gather = row_src != nullptr;
  if (bm == 32) return launch_small_pair<32, 4>(g, dn, R, gather, s);
  if (bm == 64) return launch_small_pair<64, 3>(g, dn, R, gather, s);
  return launch_small_pair<128, 2>(g, dn, R, gather, s);
}

}  // namespace laep
