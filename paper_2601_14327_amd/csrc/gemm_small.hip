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
  if (!find_tile(blockIdx.x, p.offsets, p.expert_map, p.E, BM, p.n_tiles_n, smem, te)) return;
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

// Row-tile height of a forward call.  The 256-row kernels take whole CUs for
// tiles of few rows; the short tiles fill the chip with little work, but need
// more time for the same rows once it is full: with all rows in one expert,
// 1.4 / 1.7 / 2.3 times at 128 / 64 / 32 rows.  The host does not know the
// loads, and with few of many experts taking most rows the tiles are full
// however few rows an expert has on average.  So the line lies where all rows,
// in 128-row tiles on a full chip (busy), take less than the 256-row kernels
// need for their own latency (alone: two k-loops of one tile each, the second's
// share larger where d is narrow and its tiles are few): there the short tiles
// win or tie whatever the loads.  32 rows only for a fraction of that, 128
// where the experts fill them.
// Measured, us for both products, rows in 256 / 32 / 64 / 128-row tiles; 64
// experts, d 2048, d_ff 1024:
//    rows  even loads              normal(0, 2) router bias  one expert
//     512  185 / 135 / 141 / 163    67 /  53 /  55 /  62     63 /  24 /  27 /  37
//    2048  189 / 146 / 149 / 171    72 / 100 /  72 /  62     66 /  60 /  41 /  44
//    3072  193 / 194 / 168 / 179    79 / 118 /  92 / 102     69 /  88 /  65 /  51
//    8192  215 / 303 / 243 / 234   155 / 260 / 197 / 165     98 / 214 / 149 / 131
// and 16 experts, d = d_ff = 1024:
//     512   40 /  24 /  24 /  32    49 /  23 /  21 /  27     48 /  18 /  21 /  26
//    2048   44 /  43 /  35 /  34    51 /  43 /  35 /  32     50 /  34 /  26 /  31
//    8192   80 / 115 /  86 /  77    81 / 121 /  92 /  91     63 / 112 /  83 /  70
// Over 13 widths (d 64-4096, d_ff 64-2048), 1-256 experts, 8-100000 rows and
// five kinds of load the rule's choice is at most 10 % behind the 256-row
// kernels (not behind the ones that staged their output), and takes 0.67 of
// their time on average.
int ffn_fwd_row_tile(int64_t R, int E, int d, int f) {
  // k-steps of one row tile over both products, two more for a tile's two ends;
  // 0.64 us each for 128 rows x 128 columns, two tiles sharing a CU of 256
  const double steps = (f / 64) * (d / 64 + 2.0) + ceil_div(d, 128) * (f / 64 + 2.0);
  const double busy_us = (double)R / 128 * steps * 0.64 / 256;
  const double alone_us = (d + 2.0 * f) / 96 + 15;
  if (busy_us > 0.8 * alone_us) return 256;
  if (busy_us <= 0.15 * alone_us) return 32;
  return R > 96 * (int64_t)E && busy_us > 0.4 * alone_us ? 128 : 64;
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
