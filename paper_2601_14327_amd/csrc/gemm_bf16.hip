// Forward grouped bf16 GEMMs of the SwiGLU expert FFN (moe_grouped_ffn_fwd)
// on the gfx950 matrix cores:
//   gate/up   A = X_e [M_e, d]  x W_gu[p]^T [2f, d]  -> SwiGLU epilogue (H, act_save)
//   down      A = H_e [M_e, f]  x W_d[p]^T  [d, f]   -> Y
// Both operands are K-contiguous, so global -> LDS moves are LDS-DMA
// (buffer_load_dwordx4 with the LDS flag, no register staging): one wave instruction fills
// 1 KB of LDS contiguously, lane i at +16 i, so any LDS swizzle is applied on
// the global side (each lane fetches the chunk that belongs in its slot).
//
// MFMA v_mfma_f32_32x32x16_bf16: each lane ends up owning one fragment column and
// 4 consecutive rows per register quad:
// acc[tm][tn][4q + i] = C[m = tm*32 + 8q + 4(lane/32) + i][n = (tn, lane%32)],
// where the weight rows are laid out in LDS so that the two fragments of a wave
// hold gate and up columns, or even and odd ones.
//
// Ragged expert rows come from a device-side tile table built from the
// expert offsets, so the host never learns the per-expert row counts.
// Workgroup ids are remapped so that each of the 8 XCDs walks a contiguous
// range of tiles (same expert, same weight blocks -> its own L2).
//
// Main loop: 256 x 256 tiles, 8 waves (2 x 4, each 128 x 64), k-steps of 64,
// so every row segment a step loads is one whole 128-byte line.  The L2 -> CU
// feed is bound by cache-line requests (about half a line per clock per CU,
// measured with LDS-DMA), so whole lines double the bytes per request against
// the 64-byte half lines of 32-wide k-steps.  One operand's k-step is a 32 KB
// "half"; the LDS is a ring of five halves (A0 B0 A1 B1 A2 | B2 A3 ...), so
// while step i computes, both halves of step i+1 are in flight, and from its last
// sub-steps on the A half of step i+2: every half has about one k-step (2048 MFMA
// cycles per SIMD) to land.
//
// The order of issue inside a k-step is written out MFMA by MFMA: one fragment
// read of the next k16 sub-step beside each MFMA, the wave's four copies of B one
// per MFMA right after the step boundary, those of A one per two MFMAs in the
// sub-step before it.  Issued in one burst after the boundary, the 64 copies of
// the eight waves queue behind each other in the address unit (16 clocks each)
// ahead of the MFMAs that follow them.  Layer forward, us: burst / B and A one per
// two MFMAs after the boundary / as it is: 8192 tokens top-8, d 2048, d_ff 1024
// 888 / 850 / 831; after pruning 853 / 821 / 814; 32768 rows, 16 experts, d 4096,
// d_ff 2048 1528 / 1478 / 1461.  Others: one copy per four MFMAs over the whole
// k-step 895 and 1545 (first and last); one per MFMA, all after the boundary, 877
// and 1503.  Four waves of 128 x 128, a third fewer fragment reads, run the k-loop
// no faster, and their epilogue spills.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "tiles.hpp"
#include "gemm_common.hpp"


namespace laep {
namespace {

// Weight row feeding B-tile row r of output block nt.  Down: the even columns of 64,
// then the odd ones, so a lane's two fragments are neighbours.  Gate/up: the tile's
// BN rows are BN/2 f-columns of W_gate and the same BN/2 of W_up, interleaved
// per 32 (rows 64g .. 64g+31 gate, 64g+32 .. 64g+63 up), so the SwiGLU pairs
// sit in one wave's accumulators.
template <int BN, bool GU_ROWS>
__device__ __forceinline__ int weight_row(const GemmParams& p, int nt, int r) {
  if (GU_ROWS) {
    const int grp = r >> 6, w = r & 63;
    int fcol = nt * (BN / 2) + grp * 32 + (w & 31);
    fcol = fcol < p.f ? fcol : p.f - 1;
    return (w < 32) ? fcol : p.f + fcol;
  }
  const int w = r & 63;  // LDS rows 64g .. 64g+31: even columns, 64g+32 .. 64g+63: odd ones
  const int row = nt * BN + (r & ~63) + 2 * (w & 31) + (w >> 5);
  return row < p.N ? row : p.N - 1;
}

// ---------------------------------------------------------------------------
// Epilogue: 32 rows of a wave's accumulators straight to the output.  A lane owns
// one fragment column (lane % 32) and, per register quad q, rows 8q + 4 (lane / 32)
// + 0..3.  Stores go through a buffer descriptor that ends with the tile's valid
// rows of these 32, so rows past the expert's end are dropped by the range check
// and every wave issues the same number of stores (kStoresGU, kStoresSave,
// kStoresDown), which the next tile's vmcnt waits count on.
// ---------------------------------------------------------------------------
constexpr uint32_t kDropped = 0x80000000u;  // an offset no descriptor reaches
constexpr int kStoresGU = 8, kStoresSave = 16, kStoresDown = 16;

__device__ __forceinline__ void buf_store(uint32_t v, __amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b32(v, rsrc, (int)off, 0, 0);
}

// Two rows of one column in every lane (low half: row r, high half: row r + 1)
// become two columns of one row: an even lane ends up with columns (c, c + 1) of
// row r, the odd lane beside it with the same columns of row r + 1.
__device__ __forceinline__ uint32_t pair_columns(uint32_t v, uint32_t sel) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
  return __builtin_amdgcn_perm(o, v, sel);
}

// Gate/up, 32-row block i: H = silu(gate) * up and, when training, both
// pre-activations.  A wave holds 32 columns of each, so a store covers 4 rows of
// 64 contiguous bytes.
__device__ __forceinline__ void store_gate_up(const GemmParams& p, const TileEntry& te, int row_lo,
                                              int wn, int lane, const f32x16_t& g,
                                              const f32x16_t& u) {
  const int rows = min(32, max(0, te.rows - row_lo));
  const int f = p.f, fbase = te.nt * 128 + wn * 32;
  const long long row = (long long)te.row0 + row_lo;
  const uint32_t sel = lane & 1 ? 0x03020706u : 0x05040100u;
  const uint32_t lrow = 4 * (lane >> 5) + (lane & 1), lcol = lane & 30;
  const bool in = fbase < p.f;  // f: a multiple of 64
  // the descriptor ends at the last valid row's end (from its column fbase on)
  auto rsrc_of = [&](bf16_t* base, long long ld) {
    return __builtin_amdgcn_make_buffer_rsrc(base + row * ld + fbase, 0,
                                             in ? (int)(max(0LL, rows * ld - fbase) * 2) : 0,
                                             kBufferFlags);
  };
  if (p.out2) {
    const __amdgpu_buffer_rsrc_t r2 = rsrc_of(p.out2, 2LL * f);
    const uint32_t off = (lrow * 2u * f + lcol) * 2u;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const uint32_t at = off + (q * 8 + r) * 4u * f;
        buf_store(pair_columns(pack_bf16x2(g[4 * q + r], g[4 * q + r + 1]), sel), r2, at);
        buf_store(pair_columns(pack_bf16x2(u[4 * q + r], u[4 * q + r + 1]), sel), r2, at + 2u * f);
      }
  }
  const __amdgpu_buffer_rsrc_t rh = rsrc_of(p.out, f);
  const uint32_t off = (lrow * f + lcol) * 2u;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
      const float a = fast_silu(g[4 * q + r]) * u[4 * q + r];
      const float b = fast_silu(g[4 * q + r + 1]) * u[4 * q + r + 1];
      buf_store(pair_columns(pack_bf16x2(a, b), sel), rh, off + (q * 8 + r) * 2u * f);
    }
}

// Down, 32-row block: fragments 0 and 1 hold the even and odd columns, so a lane's
// pair is one dword and a store writes two rows' whole 128-byte lines.  With
// p.out_tok (one slot per token) each row also goes, times its gate, to its token's
// row, with the combine's arithmetic (fp32 0 + g * y, one rounding); tok and gate
// are the tile's tables in LDS (tok: byte offset of the token row, kDropped for rows
// past the expert's end).
__device__ __forceinline__ void store_down(const GemmParams& p, const TileEntry& te, int row_lo,
                                           int wn, int lane, const f32x16_t& even,
                                           const f32x16_t& odd, const uint32_t* tok,
                                           const float* gate) {
  const int col = te.nt * 256 + wn * 64;
  const bool in = col < p.N;  // N: a multiple of 64
  const long long row = (long long)te.row0 + row_lo;
  const int rows = min(32, max(0, te.rows - row_lo));
  const uint32_t ld = (uint32_t)p.ldo;
  const uint32_t lcol = (lane & 31) * 4u, lrow = 4 * (lane >> 5);
  if (p.out) {
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        p.out + row * p.ldo + col, 0, in ? (int)(max(0LL, rows * p.ldo - col) * 2) : 0,
        kBufferFlags);
    const uint32_t off = lrow * ld * 2u + lcol;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        buf_store(pack_bf16x2(even[4 * q + r], odd[4 * q + r]), ro, off + (q * 8 + r) * ld * 2u);
  }
  if (!p.out_tok) return;
  const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(
      p.out_tok + col, 0, in ? (int)(kDropped - 2u * (uint32_t)col) : 0, kBufferFlags);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const u32x4_t t4 = *reinterpret_cast<const u32x4_t*>(tok + row_lo + q * 8 + lrow);
    const f32x4_t g4 = *reinterpret_cast<const f32x4_t*>(gate + row_lo + q * 8 + lrow);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t y = pack_bf16x2(even[4 * q + r], odd[4 * q + r]);
      float lo = 0.0f, hi = 0.0f;
      lo += g4[r] * lo_bf16(y);
      hi += g4[r] * hi_bf16(y);
      buf_store(pack_bf16x2(lo, hi), rt, t4[r] + lcol);
    }
  }
}

// ---------------------------------------------------------------------------
// Persistent kernel: one workgroup per CU walks its XCD's contiguous tile range,
// taking tiles from a per-XCD counter (so uneven tiles balance as the hardware
// dispatcher would, without a workgroup launch per tile; the counter's address is
// uniform, so the compiler adds once per wave and reads the reply at once: wave 0 waits
// for it, and for all that it has in flight, at the start of each k-loop).  Main loop:
// 256 x 256 tiles, 8 waves (2 x 4, each 128 x 64), k-steps of 64 in a ring of five 32 KB
// halves.  When a tile's k-loop ends, half of its rows are stored while the next
// tile's entry and gathered row ids load, then the next tile's first four halves are
// issued into the free ring, then the other half is stored: the operands' latency
// and the stores' both run under the epilogue, which needs no LDS and no barrier.
// (Staged through 64 KB of the ring for 16-byte stores, with the copies of the last
// half behind the flush, it took 7 us of a tile: 53 us for gate/up and 31 for down at
// d 2048, d_ff 1024.  Layer forward staged / direct: 8192 tokens top-8 815 / 806 us,
// after pruning 798 / 786, the 32768-row shard 1432 / 1401.)  The gate/up product
// that also writes act_save takes the same kernel; staged, that epilogue spilled
// beside the next tile's copies and kept a kernel of its own.
// ---------------------------------------------------------------------------
template <int NWM, int NWN, int EPI, bool GU_ROWS, bool GATHER>
__global__ __launch_bounds__(64 * NWM * NWN) void gemm_nt_persist_kernel(GemmParams p) {
  constexpr int BM = 256, BN = 256;
  constexpr int NT = 64 * NWM * NWN;
  constexpr int WTM = BM / NWM, WTN = BN / NWN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int ROWB = 128;                 // bytes per LDS row (64 k)
  constexpr int HALF = BM * ROWB;           // one operand's k-step, 32 KB
  constexpr int NSLOT = 5;
  constexpr int NH = BM * 8 / NT;           // 16-byte chunks per thread per half
  constexpr int SMEM = NSLOT * HALF;
  static_assert(BM == BN, "ring slots hold either operand");
  static_assert(EPI != EPI_GU || (TN % 2 == 0), "SwiGLU epilogue pairs gate/up blocks");
  static_assert(TM == 4, "the ragged-tile dispatch below covers 0..4 row blocks");
  static_assert(TN == 2, "the epilogue pairs a wave's two column fragments");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave / NWN, wn = wave % NWN;
  // thread 0's value to every thread through the first LDS word, while no copy
  // is in flight; the second barrier keeps it until every thread has read it.
  // The result is made wave-uniform (readfirstlane), so the tile's table
  // entry is a scalar load and its buffer descriptors stay in SGPRs (a
  // per-lane descriptor would put every LDS-DMA in a waterfall loop).
  auto bcast = [&](int v) {
    if (tid == 0) *reinterpret_cast<volatile int*>(smem) = v;
    __syncthreads();
    const int r = *reinterpret_cast<volatile int*>(smem);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(r);
  };

  // this XCD's contiguous range of the tile list (block i runs on XCD i % 8)
  const int n_valid = *p.n_entries;  // one tile per entry
  const int per = (n_valid + 7) >> 3;
  const int xcd = blockIdx.x & 7;
  const int t_lo = xcd * per, t_hi = min(t_lo + per, n_valid);
  int* const ctr = p.tile_ctr + xcd;
  // the first tile and the one after it
  const int L = t_lo + bcast(tid == 0 ? atomicAdd(ctr, 1) : 0);
  if (L >= t_hi) return;  // (uniform)

  // per-tile operand addressing, in two steps: the tile's rows (through
  // row_src for gathered A rows; rows past the expert: any valid row), then,
  // once they have arrived, the copies' offsets and descriptors
  TileEntry te;
  // the entry through the scalar cache (the table was complete before the launch;
  // a vector load would be waited for together with the stores around it)
  auto load_entry = [&](int at) {
    const auto* t = (const __attribute__((address_space(4))) int*)(uintptr_t)(p.table + at);
    TileEntry e;
    e.row0 = t[0];
    e.rows = t[1];
    e.expert = 0;  // (not read here)
    e.phys = t[3];
    e.nt = t[4];
    return e;
  };
  uint32_t a_voff[NH], b_voff[NH];
  __amdgpu_buffer_rsrc_t a_rsrc, b_rsrc;
  auto load_rows = [&](const TileEntry& t, uint32_t* raw) {
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      const int r = (i * NT + tid) >> 3;
      const int rr = r < t.rows ? r : t.rows - 1;
      raw[i] = GATHER ? (uint32_t)p.row_src[t.row0 + rr] : (uint32_t)rr;
    }
  };
  auto finish_tile = [&](const uint32_t* raw) {
    const char* a_base = GATHER ? reinterpret_cast<const char*>(p.A)
                                : reinterpret_cast<const char*>(p.A + (long long)te.row0 * p.lda);
    const char* b_base = reinterpret_cast<const char*>(p.B + (long long)te.phys * p.strideB);
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      const int q = i * NT + tid;
      const int r = q >> 3;
      const int lc = (q & 7) ^ swz8(r);
      const long long arow = GATHER ? (long long)(raw[i] / (uint32_t)p.slots_k) : (long long)raw[i];
      a_voff[i] = (uint32_t)((arow * p.lda + lc * 8) * 2);
      b_voff[i] = (uint32_t)(((long long)weight_row<BN, GU_ROWS>(p, te.nt, r) * p.ldb + lc * 8) * 2);
    }
    a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(a_base), 0, -1, kBufferFlags);
    b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(b_base), 0, -1, kBufferFlags);
  };
  const int nk = p.K / 64;
  // half h of the current tile: A of k-step h/2 (h even) or B (h odd), in
  // slot h % 5.  Past the end the last k-step is loaded again (never read),
  // so every iteration issues the same number of loads and one constant
  // vmcnt serves every wait.
  auto issue_half = [&](int h) {
    const int ks = min(h >> 1, nk - 1);
    char* dst = smem + (h % NSLOT) * HALF;
    if (h & 1) dma_chunks<NH, NT>(dst, b_rsrc, b_voff, ks * 128, wave);
    else dma_chunks<NH, NT>(dst, a_rsrc, a_voff, ks * 128, wave);
  };
  auto issue_chunk = [&](int h, int i) {  // chunk i of half h
    const int ks = min(h >> 1, nk - 1);
    char* dst = smem + (h % NSLOT) * HALF + i * NT * 16;
    if (h & 1) dma_chunks<1, NT>(dst, b_rsrc, b_voff + i, ks * 128, wave);
    else dma_chunks<1, NT>(dst, a_rsrc, a_voff + i, ks * 128, wave);
  };

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
    b_off[j] = r * ROWB + ((lc0 ^ swz8(r)) << 4);
  }
  f32x16_t acc[TM][TN];

  // The k-loop of one tile, its halves 0 .. 3 already issued, for a wave
  // whose first TMV 32-row blocks hold rows of the expert.  Thread 0 takes
  // the next tile from the counter at its start; the reply is used after the
  // loop, but waited for here (all of wave 0's loads and stores with it).
  int next_raw = 0;
  auto main_loop = [&](auto tmv_tag) {
    constexpr int TMV = decltype(tmv_tag)::value;
    constexpr int NRD = TMV > 0 ? TMV + TN : 0;
    constexpr int NMM = TMV * TN;
    u32x4_t fa0[TM], fb0[TN], fa1[TM], fb1[TN];
    // reads in the order the MFMAs consume them (B0 A0 B1 A1 ...)
    auto read_frag = [&](const char* sa, const char* sb, int s, u32x4_t* fa, u32x4_t* fb, int n) {
      const int pairs = TMV < TN ? TMV : TN;
      const bool is_b = n < 2 * pairs ? (n & 1) == 0 : TN > TMV;
      const int i = n < 2 * pairs ? n >> 1 : n - pairs;
      if (is_b) fb[i] = *reinterpret_cast<const u32x4_t*>(sb + (b_off[i] ^ (s << 5)));
      else fa[i] = *reinterpret_cast<const u32x4_t*>(sa + (a_off[i] ^ (s << 5)));
    };
    // One k16 sub-step: the MFMAs on (fa, fb), and beside them, in this order,
    // the fragment reads (ga, gb) of the next sub-step and the copies of half h,
    // one every `every` MFMAs (0: none).
    auto sub_step = [&](const u32x4_t* fa, const u32x4_t* fb, const char* sa, const char* sb,
                        int s, u32x4_t* ga, u32x4_t* gb, auto every_tag, int h) {
      constexpr int EVERY = decltype(every_tag)::value;
      static_assert(EVERY >= 0 && EVERY <= 2, "none, one per MFMA or one per two");
      constexpr int SLOTS = EVERY * NH, WORK = NMM > NRD ? NMM : NRD;
      constexpr int MOST = WORK > SLOTS ? WORK : SLOTS;
#pragma unroll
      for (int n = 0; n < MOST; ++n) {
        if (n < NMM) {
          const int i = n / TN, j = n % TN;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8_t, fa[i]), __builtin_bit_cast(bf16x8_t, fb[j]), acc[i][j],
              0, 0, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        if (n < NRD) {
          read_frag(sa, sb, s, ga, gb, n);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (n < SLOTS && (EVERY != 2 || n % 2 == 1)) {
          issue_chunk(h, EVERY == 2 ? n / 2 : n);
          __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        }
      }
    };
    using Every0 = std::integral_constant<int, 0>;
    using Every1 = std::integral_constant<int, 1>;
    using Every2 = std::integral_constant<int, 2>;

    // the fragment offsets are made opaque here, so the offsets each
    // instantiation derives from them are not hoisted out of the tile loop
    // (five instantiations' worth would stay live across every tile)
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(a_off[i]));
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(b_off[j]));
    // halves 0 and 1 (step 0) have landed (the caller waited)
    __builtin_amdgcn_s_barrier();
    if (tid == 0) next_raw = atomicAdd(ctr, 1);
    int ia = 0, ib = 1;
#pragma unroll
    for (int n = 0; n < NRD; ++n) read_frag(smem, smem + HALF, 0, fa0, fb0, n);
    wait_lgkm0();  // nothing pending at the loop's entry: its waits then count its own reads
    for (int kt = 0; kt < nk; ++kt) {
      const char* sa = smem + ia * HALF;
      const char* sb = smem + ib * HALF;
      sub_step(fa0, fb0, sa, sb, 1, fa1, fb1, Every0{}, 0);
      sub_step(fa1, fb1, sa, sb, 2, fa0, fb0, Every0{}, 0);
      sub_step(fa0, fb0, sa, sb, 3, fa1, fb1, Every2{}, 2 * kt + 4);
      wait_vmcnt_lgkm0<NH>();
      __builtin_amdgcn_s_barrier();
      ia = ia + 2 >= NSLOT ? ia + 2 - NSLOT : ia + 2;
      ib = ib + 2 >= NSLOT ? ib + 2 - NSLOT : ib + 2;
      sub_step(fa1, fb1, smem + ia * HALF, smem + ib * HALF, 0, fa0, fb0, Every1{}, 2 * kt + 5);
    }
  };

  // One tile ahead: thread 0 asks the counter for the next tile at the start
  // of each k-loop; after the loop its index reaches every thread.  Loading the
  // next tile's entry and rows during the k-loop instead (vector loads at the first
  // two step boundaries) measured no faster.
  uint32_t raw[NH];
  te = load_entry(L);
  load_rows(te, raw);
  finish_tile(raw);
#pragma unroll
  for (int h = 0; h < NSLOT - 1; ++h) issue_half(h);
  wait_vmcnt<2 * NH>();
  // the scatter's tables, in slot 4: free from a k-loop's end to the next one's
  // first copy of step 2, a barrier after the epilogue
  uint32_t* const tok = reinterpret_cast<uint32_t*>(smem + 4 * HALF);
  float* const tok_gate = reinterpret_cast<float*>(smem + 4 * HALF + BM * 4);
  const bool scatter = EPI == EPI_STORE && p.out_tok != nullptr;
  uint32_t src = 0;  // row tid of the tile: its slot and gate
  float src_gate = 0.0f;
  auto load_src = [&]() {
    if (scatter && tid < te.rows) src = (uint32_t)p.row_src[te.row0 + tid];
  };
  auto load_gate = [&]() {
    if (scatter && tid < te.rows) src_gate = p.gate[src];
  };
  load_src();
  load_gate();
  while (true) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    const int tmv = min(TM, max(0, (te.rows - wm * WTM + 31) >> 5));
    if (tmv >= TM) main_loop(std::integral_constant<int, TM>{});
    else if (tmv == 3) main_loop(std::integral_constant<int, 3>{});
    else if (tmv == 2) main_loop(std::integral_constant<int, 2>{});
    else if (tmv == 1) main_loop(std::integral_constant<int, 1>{});
    else main_loop(std::integral_constant<int, 0>{});
    // every copy into the ring has landed and every fragment read is done
    wait_vmcnt<0>();
    wait_lgkm0();
    if (tid == 0) *reinterpret_cast<volatile int*>(smem) = next_raw;
    __syncthreads();
    const int next =
        t_lo + __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(smem));
    if (scatter && tid < BM) {
      tok[tid] = tid < te.rows ? src / (uint32_t)p.slots_k * (uint32_t)p.ldo * 2u : kDropped;
      tok_gate[tid] = src_gate;
    }
    __syncthreads();
    const TileEntry cur = te;
    const bool more = next < t_hi;
    if (more) {
      te = load_entry(next);
      load_rows(te, raw);
      load_src();
    }
    auto store_block = [&](int i) {
      const int row_lo = wm * WTM + i * 32;
      if constexpr (EPI == EPI_GU)
        store_gate_up(p, cur, row_lo, wn, lane, acc[i][0], acc[i][1]);
      else
        store_down(p, cur, row_lo, wn, lane, acc[i][0], acc[i][1], tok, tok_gate);
    };
#pragma unroll
    for (int i = 0; i < TM / 2; ++i) store_block(i);
    if (more) {
      finish_tile(raw);
#pragma unroll
      for (int h = 0; h < NSLOT - 1; ++h) issue_half(h);
      load_gate();
    }
    __builtin_amdgcn_sched_barrier(0);  // the count below: these stores after the copies
#pragma unroll
    for (int i = TM / 2; i < TM; ++i) store_block(i);
    if (!more) break;
    __builtin_amdgcn_sched_barrier(0);
    // halves 0 and 1 have landed: at most halves 2 and 3 and the stores after them
    // in flight (the counter holds 63)
    constexpr int S = EPI == EPI_GU ? kStoresGU : kStoresDown;
    constexpr int S2 = EPI == EPI_GU ? S + kStoresSave : 2 * S;
    constexpr int W = 2 * NH + (TM / 2) * S, W2 = 2 * NH + (TM / 2) * S2;
    const bool both = EPI == EPI_GU ? p.out2 != nullptr : (p.out != nullptr && scatter);
    if (both) wait_vmcnt<(W2 < 63 ? W2 : 63)>();
    else wait_vmcnt<(W < 63 ? W : 63)>();
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// The products run persistent: one workgroup per CU, a multiple of 8 so every XCD
// gets the same number, each walking its XCD's tile range through p.tile_ctr.
template <int EPI, bool GU, bool GATHER = false>
hipError_t launch_fwd(const GemmParams& p, int max_tiles, hipStream_t s) {
  if (max_tiles <= 0) return hipSuccess;
  int dev = 0, cus = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err == hipSuccess) err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (err != hipSuccess) return err;
  const int grid = max(8, cus / 8 * 8);
  hipLaunchKernelGGL((gemm_nt_persist_kernel<2, 4, EPI, GU, GATHER>), dim3(grid), dim3(512), 0, s,
                     p);
  return hipGetLastError();
}

constexpr int kFwdBM = 256, kFwdBN = 256;

}  // namespace

// bf16 workspace: H [R, f], then the per-tile lists of the two products
namespace {
inline int fwd_list_max(int64_t R, int E, int n_tiles) { return (ceil_div(R, kFwdBM) + E) * n_tiles; }
}  // namespace

size_t ffn_fwd_ws_bytes(int64_t R, int E, int d, int f, int dtype) {
  if (dtype == kDtypeBf16)
    return align_up((size_t)R * f * 2, 256) +
           table_bytes(fwd_list_max(R, E, ceil_div(f, kFwdBN / 2))) +
           table_bytes(fwd_list_max(R, E, ceil_div(d, kFwdBN)));
  return align_up((size_t)R * f * 4, 256);  // fp32: H
}

namespace {

// the two products of the forward FFN (and the tile lists), on s
hipError_t launch_ffn_fwd_products(const void* x_perm, const void* w_gu, const void* w_d,
                                   const int32_t* offsets, const int32_t* expert_map, int E,
                                   int d, int f, int64_t R, void* y_perm, void* act_save,
                                   bf16_t* H, void* ws, hipStream_t s, const int32_t* row_src,
                                   int slots_k, const float* gate, void* out_tok) {
  const int bm = ffn_fwd_row_tile(R, E, d, f);
  if (bm != kFwdBM)
    return launch_ffn_fwd_small(bm, x_perm, w_gu, w_d, offsets, expert_map, E, d, f, R, y_perm,
                                act_save, H, s, row_src, slots_k, gate, out_tok);
  const int nt_gu = ceil_div(f, kFwdBN / 2), nt_d = ceil_div(d, kFwdBN);
  const int max_gu = fwd_list_max(R, E, nt_gu), max_d = fwd_list_max(R, E, nt_d);
  char* tables = static_cast<char*>(ws) + align_up((size_t)R * f * 2, 256);
  TableWs tgu = carve_table(tables, max_gu);
  TableWs td = carve_table(tables + table_bytes(max_gu), max_d);
  const int group = kFwdTileGroup;
  TileList lgu = {nt_gu, group, max_gu, tgu.n_entries, tgu.table};
  TileList ld = {nt_d, group, max_d, td.n_entries, td.table};
  const int list_blocks = ceil_div(max_gu > max_d ? max_gu : max_d, kTableThreads);
  hipLaunchKernelGGL(build_tile_lists_kernel, dim3(list_blocks), dim3(kTableThreads), 0, s,
                     offsets, expert_map, E, kFwdBM, lgu, ld);
  GemmParams g = {};
  g.table = tgu.table;
  g.n_entries = tgu.n_entries;
  g.tile_ctr = tgu.n_entries + kTileCtrOffset;
  g.f = f;
  // gate/up + SwiGLU: B rows interleaved gate/up per 32, BN/2 f-columns per tile
  g.A = static_cast<const bf16_t*>(x_perm);
  g.lda = d;
  g.B = static_cast<const bf16_t*>(w_gu);
  g.ldb = d;
  g.strideB = (long long)2 * f * d;
  g.N = 2 * f;
  g.K = d;
  g.out = H;
  g.ldo = f;
  g.out2 = static_cast<bf16_t*>(act_save);
  g.row_src = row_src;
  g.slots_k = slots_k;
  hipError_t err = row_src ? launch_fwd<EPI_GU, true, true>(g, max_gu, s)
                           : launch_fwd<EPI_GU, true>(g, max_gu, s);
  if (err != hipSuccess) return err;
  // down projection
  g.table = td.table;
  g.n_entries = td.n_entries;
  g.tile_ctr = td.n_entries + kTileCtrOffset;
  g.A = H;
  g.lda = f;
  g.B = static_cast<const bf16_t*>(w_d);
  g.ldb = f;
  g.strideB = (long long)d * f;
  g.N = d;
  g.K = f;
  g.out = static_cast<bf16_t*>(y_perm);
  g.ldo = d;
  g.out2 = nullptr;
  g.row_src = out_tok ? row_src : nullptr;  // the scatter's token rows (A is H here)
  g.gate = gate;
  g.out_tok = static_cast<bf16_t*>(out_tok);
  return launch_fwd<EPI_STORE, false>(g, max_d, s);
}

}  // namespace

hipError_t launch_ffn_fwd_bf16(const void* x_perm, const void* w_gu, const void* w_d,
                               const int32_t* offsets, const int32_t* expert_map, int E, int d,
                               int f, int64_t R, void* y_perm, void* act_save, void* ws,
                               hipStream_t s, const int32_t* row_src, int slots_k,
                               const float* gate, void* out_tok, void* x_perm_out) {
  bf16_t* H = static_cast<bf16_t*>(ws);
  // x_perm for the weight gradient: written on the side stream beside the FFN
  // (HBM-bound copy against MFMA-bound products), joined before returning
  std::unique_lock<std::mutex> lock;
  SideStream* side = nullptr;
  if (x_perm_out && row_src) {
    hipError_t e = side_stream_acquire(side, lock);
    if (e == hipSuccess) e = side_stream_fork(*side, s);
    if (e == hipSuccess) e = launch_gather_rows(x_perm, row_src, slots_k, R, d, 2, x_perm_out,
                                                side->stream);
    if (e != hipSuccess) {
      if (side) side_stream_join(*side, s);
      return e;
    }
  }
  const hipError_t err = launch_ffn_fwd_products(x_perm, w_gu, w_d, offsets, expert_map, E, d, f,
                                                 R, y_perm, act_save, H, ws, s, row_src, slots_k,
                                                 gate, out_tok);
  if (side) {
    const hipError_t jerr = side_stream_join(*side, s);
    return err != hipSuccess ? err : jerr;
  }
  return err;
}

}  // namespace laep
