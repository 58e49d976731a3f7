// LM heads of small batches: one product of the activations' high part, K whole and at least 16 stages of 64 k long, in tiles of 16 MT
// rows by 64 NF columns (operand formats and columns: gemm_tile.h; which launch takes it: gemm_k64.hip).
//
// Bound: the copies -- the weight stream from HBM and, behind it, the activations out of L2.  So everything else has to stay out of
// their way:
//   * four wavefronts only copy: a stage's place is asked for again the moment it has been read, not behind MFMAs;
//   * eight multiply, two per SIMD, in turns: while the even halves of the stages' K are read and widened the odd ones'
//     MFMAs run, and the other way round.  A wavefront owns half of a stage's K x half of the rows x half of the columns: at
//     128 rows 0.8 of the bytes out of LDS that four wavefronts with all rows and a quarter of the columns each read;
//   * as many stages as fit the LDS (up to six);
//   * tile rows of 128 bytes: whole cache lines, which are asked for once and need not be kept (GemmArgs::once);
//   * blocks start at different k (GemmArgs::rotate).
// LM head at 32 / 64 / 128 / 256 rows, 8B 61.6 / 64.2 / 68.8 / 119 -> 43.3 / 46.1 / 55 / 100 us, 70B 112 / 116 / 128 / 228 -> 85 / 88 / 105
// / 187 (before: the tile of gemm_tile.h).
//
// The two K halves are added through LDS at the end, the even half first, and a row's sum may start at another k: an order of its own.
// The logits move by 5e-7 of their norm; nothing that is rounded follows.  (Gate/up in this order moved the K and V rows behind it by
// 1e-4 of the norm in the 8B shape, 4e-4 in the 70B: bf16 roundings that fall the other way.)
#include "gemm_k64.h"

template <int MT, int NF>
__global__ __launch_bounds__(768) void whole_k_kernel(GemmArgs g) {
  constexpr int BM = 16 * MT, BN = 64 * NF, BK = 64, CPR = 8;
  constexpr int R = BM + BN, STAGE = R * BK * 2;                 // rows [A | W] of 128 bytes
  constexpr int FIT = 163840 / STAGE, DEPTH = FIT < 6 ? FIT : 6;
  static_assert(DEPTH >= 3, "three stages have to fit the 160 KB of LDS");
  constexpr int A_INS = BM / 8;                                  // copies (8 rows, 1 KB) of a stage, and per wavefront
  constexpr int A_IPW = (A_INS + 3) / 4, W_IPW = BN / 32, IPW = A_IPW + W_IPW;
  constexpr int MB = (MT + 1) / 2, NFW = 2 * NF;                 // 16-row blocks and 16-column fragments of a wavefront
  __shared__ __attribute__((aligned(16))) unsigned char lds[DEPTH * STAGE];
  static_assert(8 * MB * NFW / 2 * 1024 <= DEPTH * STAGE, "the exchange of the K halves reuses the stages");

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rh = wave & 1, ch = (wave >> 1) & 1, kh = wave >> 2; // halves of the rows, the columns, the stage's K
  // blocks and tiles as in gemm_tile.h: the M tiles of one N tile follow one another on one XCD
  const int m_tiles = (g.M + BM - 1) / BM, n_tiles = g.N / BN;
  const int xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
  const int n_tile = (within / m_tiles) * 8 + xcd;
  if (n_tile >= n_tiles) return;
  const int m0 = (within % m_tiles) * BM, n0 = n_tile * BN;
  const int K = g.K, M = g.M;
  const int n_steps = K / BK;

#define SY_BARRIER asm volatile("s_barrier" ::: "memory")
  if (wave >= 8) {                                               // ---- the four wavefronts that copy
    const uint16_t* src[IPW];                                      // as in gemm_tile.h: uniform base, byte offset of the lane
    uint32_t off[IPW], dst[IPW];
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
      int grp;                                                     // group of 8 rows of the stage
      if (j < A_IPW) {
        grp = wave - 8 + 4 * j;
        grp = grp < A_INS ? grp : A_INS - 1;                       // same bytes to the same place: harmless
      } else {
        grp = A_INS + (wave - 8) * W_IPW + (j - A_IPW);
      }
      const int r = grp * 8 + lane / CPR;
      const int chunk = (lane % CPR) ^ (((r >> 1) & 3) << 1);      // swz16<8>, on the global side
      dst[j] = grp * 1024;
      if (j < A_IPW) {
        const int am = m0 + r < M ? m0 + r : M - 1;                // rows past M are copied (clamped) and never stored
        src[j] = g.a + (size_t)m0 * K;
        off[j] = (uint32_t)(am - m0) * (uint32_t)(2 * K) + chunk * 16;
      } else {
        const int col = grp * 8 - BM;
        int wrow = n0 + col;
        const bf16_t* wbase = g.w[0];
        if (wrow >= g.w_rows[0]) {
          wrow -= g.w_rows[0];
          wbase = g.w[1];
          if (wrow >= g.w_rows[1]) {
            wrow -= g.w_rows[1];
            wbase = g.w[2];
          }
        }
        src[j] = wbase + (size_t)wrow * K;
        off[j] = (uint32_t)(lane / CPR) * (uint32_t)(2 * K) + chunk * 16;
      }
    }
    const int turn = g.rotate ? (int)((unsigned)n_tile * 3u % (unsigned)n_steps) : 0;
    const uint32_t base = lds_addr_of(lds);
    // copy j of the stage of step s (past the end, of the last one again: never read, but the wait counts stay constants)
    auto issue = [&](int j, int s, int slot) {
      int at = (s < n_steps ? s : n_steps - 1) + turn;
      if (at >= n_steps) at -= n_steps;
      const uint16_t* from = src[j] + (size_t)at * BK;
      const uint32_t to = base + slot * STAGE + dst[j];
      if (j >= A_IPW && g.once) glds16_once(from, off[j], to);
      else glds16_at(from, off[j], to);
    };

    auto fill = [&](int s, int slot) {
#pragma unroll
      for (int j = 0; j < IPW; ++j) issue(j, s, slot);
    };
#define SY_LANDED asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DEPTH - 2) * IPW) : "memory")
#pragma unroll
    for (int s = 0; s < DEPTH - 1; ++s) fill(s, s);
    SY_LANDED;
    SY_BARRIER;
    int free_slot = DEPTH - 1;
    for (int s = 0; s < n_steps; ++s) {
      fill(s + DEPTH - 1, free_slot);
      SY_BARRIER;
      SY_LANDED;
      SY_BARRIER;
      free_slot = free_slot + 1 == DEPTH ? 0 : free_slot + 1;
    }
#undef SY_LANDED
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // (the surplus copies, before LDS is reused)
    __syncthreads();
    __syncthreads();
    return;
  }

  f32x4 acc[MB][NFW];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NFW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int l16 = lane & 15, kc = lane >> 4;
  // byte offsets inside a stage; + i * 16 rows, + j * 16 rows.  With MT odd the last block of the second half lies behind the
  // activations' rows, still inside the stage, and is never stored.
  const int frag = swz16<CPR>(l16, 4 * kh + kc) * 2;
  const int a_off = rh * MB * 16 * BK * 2 + frag, w_off = (BM + ch * 16 * NFW) * BK * 2 + frag;

  u32x4 w[NFW], act[MB];
  auto read = [&](int slot) {                                    // this wavefront's fragments of a stage, widened
    const unsigned char* stage = lds + slot * STAGE;
#pragma unroll
    for (int j = 0; j < NFW; ++j) w[j] = *reinterpret_cast<const u32x4*>(stage + w_off + j * 16 * BK * 2);
#pragma unroll
    for (int i = 0; i < MB; ++i) act[i] = *reinterpret_cast<const u32x4*>(stage + a_off + i * 16 * BK * 2);
#pragma unroll
    for (int j = 0; j < NFW; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) w[j][q] = widen_weights(w[j][q]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  auto multiply = [&] {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NFW; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w[j]), __builtin_bit_cast(f16x8, act[i]),
                                                           acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Phases 2 s and 2 s + 1 of step s end with a barrier each.  Phase 2 s: the even half reads the stage, the odd one multiplies what
  // it read of the stage before; phase 2 s + 1: the other way round.  Stage s - 1 has been read by all when phase 2 s begins: its place
  // is then filled for step s + DEPTH - 1; before phase 2 s + 2 all copies of stage s + 1 have landed.
  SY_BARRIER;
  int slot = 0;
  if (kh == 0) {
    for (int s = 0; s < n_steps; ++s) {
      read(slot);
      SY_BARRIER;
      multiply();
      SY_BARRIER;
      slot = slot + 1 == DEPTH ? 0 : slot + 1;
    }
  } else {
    SY_BARRIER;
    read(0);
    SY_BARRIER;
    for (int s = 1; s < n_steps; ++s) {
      slot = slot + 1 == DEPTH ? 0 : slot + 1;
      multiply();
      SY_BARRIER;
      read(slot);
      SY_BARRIER;
    }
    multiply();
  }
#undef SY_BARRIER

  // ---- the two halves of K: each wavefront hands half of its columns to its partner and finishes the other half
  __syncthreads();
  constexpr int HALF = NFW / 2;
  const float os = g.out_scale;
  const int nq = kc * 4;                                         // this lane's 4 consecutive columns of a fragment
  auto finish = [&](auto KH) {
    constexpr int KEEP = decltype(KH)::value * HALF, GIVE = HALF - KEEP;
    f32x4* mine = reinterpret_cast<f32x4*>(lds) + (size_t)wave * MB * HALF * 64;
    const f32x4* other = reinterpret_cast<const f32x4*>(lds) + (size_t)(wave ^ 4) * MB * HALF * 64;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < HALF; ++j) mine[(i * HALF + j) * 64 + lane] = acc[i][GIVE + j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = (rh * MB + i) * 16 + l16, m = m0 + row;
      if (row >= BM || m >= M) continue;
      float* c = reinterpret_cast<float*>(g.c) + (size_t)m * g.N + n0 + (ch * NFW + KEEP) * 16 + nq;
#pragma unroll
      for (int j = 0; j < HALF; ++j)
        *reinterpret_cast<f32x4*>(c + j * 16) = (acc[i][KEEP + j] + other[(i * HALF + j) * 64 + lane]) * os;
    }
  };
  if (kh == 0) finish(std::integral_constant<int, 0>{});
  else finish(std::integral_constant<int, 1>{});
}

hipError_t launch_proj_k64_whole(int mt, int nf, GemmArgs g, hipStream_t s) {
  // At the same k all blocks ask the same memory channels; starting at different ones spreads them, but every XCD then reads all
  // activations at any time: up to 3 MB of them stay in its 4 MB of L2.  LM head at 32 / 64 / 128 rows, 8B 59.8 / 62.9 / 63.8 ->
  // 43.3 / 44.7 / 53.0 us, 70B 114 / 116 / 127 -> 85 / 88 / 102.
  g.rotate = g.M <= 16 * mt && (size_t)g.M * g.K * 2 <= ((size_t)3 << 20) && g.K >= 2048;
  // Several tiles of rows want the same weight lines out of one XCD's L2: 200 rows with lines marked as not wanted again 8B 97.1 -> 101.8
  // us, 70B 184.9 -> 192.8; 224 to 280 rows the same within 1 %.
  g.once = g.once && g.M <= 16 * mt;
  return with_short_tile(mt, nf, [&](auto MT, auto NF) {
    constexpr int mt_ = decltype(MT)::value, nf_ = decltype(NF)::value;
    const int m_tiles = (g.M + 16 * mt_ - 1) / (16 * mt_), n_tiles = g.N / (64 * nf_);
    whole_k_kernel<mt_, nf_><<<8 * ((n_tiles + 7) / 8) * m_tiles, 768, 0, s>>>(g);
    return hipGetLastError();
  });
}
