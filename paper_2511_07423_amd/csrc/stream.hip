// The decoder's projections for batches of up to SY_STREAM_ROWS rows, C[M][N] = A[M][K] W[N][K]^T with the operand formats of
// gemm_tile.h (bf16 weights widened to fp16 in registers, activations as an fp16 (hi, lo) pair), fp32 accumulation, and
// with the small kernels around them folded in: such a call is bound by its weight stream, and every kernel between two
// projections is time in which no weights move.
//
//   QKV       A = RMSNorm(x), made here from the residual; the rotary embedding and the cache append are its epilogue
//   residual  A = a pair from the attention / SwiGLU; x += product in place, and the sum of squares of the block's columns
//             of every row, from which the next projection's blocks form the row's RMS
//   SwiGLU    A = RMSNorm(x); writes the pair SiLU(gate) up
//   LM head   A = RMSNorm(selected rows of x)
//
// A block takes 8 h consecutive weight rows, with h so that about 256 blocks cover the matrix, over all of K: nothing is
// left to add for another kernel.  Its eight wavefronts split K: wavefront w takes every eighth stage of 128 k with a ring
// of 4 KB units of LDS of its own, refilled unit by unit as it is read (global_load_lds_dwordx4), so that about 100 KB per
// block is on its way at any time and no barrier stands in the loop; the partial tiles are added at the end, in
// wavefront order.  (Two wavefronts per SIMD: with one, the reads, widening and norm of a unit were not hidden by another's.)
// A unit is 16 weight rows or 8 activation rows of one stage.  One copy moves 4 rows x 256 bytes; the blocks start at
// different stages.  Both matter to HBM: copies alone of the 8B gate/up matrix (235 MB) take 43.9 us with 8 rows x 128
// bytes and every block at the same k, 38.2 us in this form (6.2 TB/s).
//
// Up to 8 rows the low parts are rows 8 .. 15 of the MFMA's activation operand: one MFMA for both.
//
// Measured, 8B shape, one request of 5 rows, per layer: QKV 13.2, output 9.0, gate/up 40.3, down 22.0 us (5.2 TB/s over the
// four), where the tile kernels, with RMSNorm and the rotary kernel, took 12, 10, 49.9, 21 and 18.8 us.
#include "common.h"
#include <utility>

namespace {
constexpr int UNIT = 4096, STAGE_K = 128, WAVES = 8;
constexpr int SPARE = 32768;                       // LDS beside the rings of a kernel that normalises: gains, row sums

__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
// (The instruction's own offset field is not used: it moves the LDS address along with the global one.)
__device__ __forceinline__ void copy16(const void* base, uint32_t lane_off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(lane_off), "s"(base) : "memory", "m0");
}
// The four copies of a unit.  Off, they move nothing but still count as four: the waits of a
// wavefront's last units are then those of all others.  Called with all lanes active.  ONCE: the lines are marked as not
// wanted again (nt), for weights that no cache holds until the next call; one block reads them, whole lines at a time.  Loads alone
// of the 8B gate/up matrix then run at 6.4 instead of 5.6 TB/s, the kernel at 5 rows takes 40.3 instead of 42.8 us, the LM head's
// 42.0 instead of 45.6.
#define SY_UNIT_COPIES(MOD)                                                                                          \
  asm volatile(                                                                                                      \
      "s_mov_b32 m0, %0\n\ts_mov_b32 exec_lo, %7\n\ts_mov_b32 exec_hi, %7\n\tglobal_load_lds_dwordx4 %1, %5" MOD "\n\t" \
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %5" MOD "\n\t"                             \
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %6" MOD "\n\t"                             \
      "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %6" MOD "\n\t"                             \
      "s_mov_b64 exec, -1" ::"s"(lds), "v"(o0), "v"(o1), "v"(o2), "v"(o3), "s"(base0), "s"(base1), "s"(mask)         \
      : "memory", "m0", "scc")
template <bool ONCE>
__device__ __forceinline__ void copy_unit(const void* base0, const void* base1, uint32_t o0, uint32_t o1, uint32_t o2, uint32_t o3,
                                          uint32_t lds, bool on) {
  const uint32_t mask = __builtin_amdgcn_readfirstlane(on ? ~0u : 0u);
  if (ONCE) SY_UNIT_COPIES(" nt");
  else SY_UNIT_COPIES("");
}
#undef SY_UNIT_COPIES
template <int... P, class F>
__device__ __forceinline__ void each(std::integer_sequence<int, P...>, F&& f) {
  (f(std::integral_constant<int, P>{}), ...);
}
}  // namespace

// NF: 16-row weight units per block; NA: 8-row activation units (1: M <= 8, 2: M <= 16).
template <int NF, int NA, int EPI, bool ONCE>
__global__ __launch_bounds__(64 * WAVES) void stream_kernel(StreamArgs g) {
  constexpr bool NORM = EPI != STREAM_ADD;
  constexpr int UPS = NA + NF;                     // units per stage
  constexpr int RING = NORM ? 4 : 5;
  __shared__ __attribute__((aligned(16))) unsigned char lds[WAVES * RING * UNIT + (NORM ? SPARE : 0)];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = g.K, M = g.M, h = g.half_units, row0 = blockIdx.x * 8 * h;
  const int all = K / STAGE_K;
  const int n = all > wave ? (all - wave + WAVES - 1) / WAVES : 0;    // this wavefront's stages: wave, wave + 8, ..., from the turn'th on
  const int turn = n ? (int)(blockIdx.x * 3u % (unsigned)n) : 0;
  unsigned char* ring = lds + wave * RING * UNIT;
  const uint32_t ring_at = lds_address(ring);
  unsigned char *gains = lds + WAVES * RING * UNIT + wave * (SPARE / 2 / WAVES), *sums_at = lds + WAVES * RING * UNIT + SPARE / 2;
  const int l16 = lane & 15, kc = lane >> 4;

  // ---- row sums and gains first: everything waits for them
  if (NORM) {
    // row r of the batch is row `src` of x; its sum of squares arrives in g.ss_parts parts
    for (int r = wave; r < M; r += WAVES) {
      const int src = EPI == STREAM_LOGITS ? g.rows[r] : r;      // uniform
      copy16(g.ss + (size_t)__builtin_amdgcn_readfirstlane(src) * SY_STREAM_PARTS, lane * 16, lds_address(sums_at) + r * 1024);
    }
    // gains of stage list entry j (stage wave + 8 j) at j x 256 bytes
    for (int j = 0; j < n; j += 4)
      copy16(g.gain + wave * STAGE_K, (uint32_t)min(j + kc, n - 1) * (WAVES * STAGE_K * 2) + l16 * 16, lds_address(gains) + j * 256);
  }

  // ---- sources.  A unit's rows of 16-byte chunks are permuted within the row so that fragment reads of 8 (16) rows at the
  // same k fall on different banks: position p of row r holds chunk p ^ r (activations: p ^ (r % 8)).
  const char* w_half[2 * NF];                      // the 8-row halves of the units
#pragma unroll
  for (int q = 0; q < 2 * NF; ++q) {
    if (EPI == STREAM_SWIGLU) {                    // a unit is 8 gate rows and the 8 up rows of the same columns
      const int row = min(row0 / 2 + (q / 2) * 8, g.N / 2 - 8);
      w_half[q] = reinterpret_cast<const char*>(g.w[q & 1]) + (size_t)row * K * 2;
    } else {
      // past the block's rows, and past the matrix: some rows again, never stored
      int row = min(row0 + min(q, h - 1) * 8, g.N - 8);
      const bf16_t* base = g.w[0];
      if (row >= g.w_rows[0]) {
        row -= g.w_rows[0];
        base = g.w[1];
        if (row >= g.w_rows[1]) {
          row -= g.w_rows[1];
          base = g.w[2];
        }
      }
      w_half[q] = reinterpret_cast<const char*>(base) + (size_t)row * K * 2;
    }
    w_half[q] += wave * (STAGE_K * 2);
  }
  uint32_t w_lane[4], a_lane[4 * NA];
#pragma unroll
  for (int c = 0; c < 4; ++c)                      // rows 4 c .. 4 c + 3 of the unit, relative to their half
    w_lane[c] = (uint32_t)((c & 1) * 4 + kc) * 2 * K + ((l16 ^ (4 * c + kc)) * 16);
#pragma unroll
  for (int c = 0; c < 4 * NA; ++c) {               // rows 2 c and 2 c + 1 of the batch
    const int r = 2 * c + (lane >> 5);
    const int m = min(r, M - 1);                   // rows past M: never stored
    const int src = EPI == STREAM_LOGITS ? g.rows[m] : m;
    a_lane[c] = (uint32_t)src * 4 * K + (((lane & 31) ^ (r & 7)) * 16);
  }
  const char* a_src = reinterpret_cast<const char*>(g.a) + wave * (STAGE_K * 4);

  // the copies of the unit at position P of list entry i's stage (none, but counted, where on is false)
  auto issue = [&](auto P, int i, uint32_t at, bool on) {
    constexpr int p = decltype(P)::value;
    int j = turn + i;
    if (j >= n) j -= n;
    if constexpr (p < NA) {
      const char* src = a_src + (size_t)j * (WAVES * STAGE_K * 4);
      copy_unit<false>(src, src, a_lane[p * 4], a_lane[p * 4 + 1], a_lane[p * 4 + 2], a_lane[p * 4 + 3], at, on);
    } else {
      const size_t k = (size_t)j * (WAVES * STAGE_K * 2);
      copy_unit<ONCE>(w_half[2 * (p - NA)] + k, w_half[2 * (p - NA) + 1] + k, w_lane[0], w_lane[1], w_lane[2], w_lane[3], at, on);
    }
  };
  each(std::make_integer_sequence<int, RING>{}, [&](auto T) {
    constexpr int t = decltype(T)::value;
    issue(std::integral_constant<int, t % UPS>{}, t / UPS, ring_at + t * UNIT, t / UPS < n);
  });

  // ---- 1 / RMS of the rows (x SY_Y_SCALE)
  float inv = 0.f;                                 // of row l16 (NA 1: l16 % 8)
  if (NORM) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * RING) : "memory");
    float* sums = reinterpret_cast<float*>(sums_at);
    for (int r = wave; r < M; r += WAVES) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(sums + r * 256 + lane * 4);
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) s += lane * 4 + i < g.ss_parts ? v[i] : 0.f;
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
      if (lane == 0) sums[r * 256] = s;            // (after every lane's read: the sum depends on them)
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    inv = rsqrtf(sums[min(NA == 1 ? l16 & 7 : l16, M - 1) * 256] / (float)K + g.eps) * SY_Y_SCALE;
  }
  // what the epilogue will need: wavefront f finishes fragment f, lane = row l16, columns 4 kc .. 4 kc + 3.  (Loads that no
  // branch guards: a register that two paths meet in would be waited for here.)
  const int m = min(l16, M - 1), f_mine = min(wave, NF - 1), col = row0 + f_mine * 16 + kc * 4;
  f32x4 ahead;
  uint32_t at_slot;
  if (EPI == STREAM_ADD) ahead = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.c) + (size_t)m * g.N + min(col, g.N - 4));
  if (EPI == STREAM_QKV) {
    ahead = *reinterpret_cast<const f32x4*>(g.cs + (size_t)m * (g.hd / 2) + min(col, g.N - 4) % g.hd / 2);   // (cos, sin) of two adjacent pairs
    at_slot = g.meta.tok_slot[m];
  }

  // ---- the stages
  f32x4 acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  int slot = 0, left = n * UPS;                    // ring position of the next unit; units not yet read
  const bool low_half = l16 < 8;
  for (int i = 0; i < n; ++i) {
    f16x8 hi[4], lo[4];                            // activation fragments of the stage's four steps of 32 k
    // ---- activations
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (RING - NA)) : "memory");
    const int slot1 = slot + 1 == RING ? 0 : slot + 1;
    const unsigned char* a = ring + (NA == 1 || low_half ? slot : slot1) * UNIT + (l16 & 7) * 512;
    if (NORM) {
      int j = turn + i;
      if (j >= n) j -= n;
      const unsigned char* gn = gains + j * 256 + kc * 16;
      if (NA == 1) {
        // lanes of rows r and r + 8 hold the same row: each normalises four of its eight values, then the high parts
        // gather in the one and the low parts in the other
        f32x4 v[4];
        uint2 gv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          v[s] = *reinterpret_cast<const f32x4*>(a + ((s * 8 + 2 * kc + (low_half ? 0 : 1)) ^ (l16 & 7)) * 16);
          gv[s] = *reinterpret_cast<const uint2*>(gn + s * 64 + (low_half ? 0 : 8));
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          uint32_t h0, h1, l0, l1;
          split_f16x2(v[s][0] * inv * bf2f(gv[s].x & 0xFFFF), v[s][1] * inv * bf2f(gv[s].x >> 16), h0, l0);
          split_f16x2(v[s][2] * inv * bf2f(gv[s].y & 0xFFFF), v[s][3] * inv * bf2f(gv[s].y >> 16), h1, l1);
          const uint32_t keep0 = low_half ? h0 : l0, keep1 = low_half ? h1 : l1;
          const uint32_t got0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(low_half ? l0 : h0), 0x128, 0xF, 0xF, true);   // row_ror:8
          const uint32_t got1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(low_half ? l1 : h1), 0x128, 0xF, 0xF, true);
          const u32x4 e = {low_half ? keep0 : got0, low_half ? keep1 : got1, low_half ? got0 : keep0, low_half ? got1 : keep1};
          hi[s] = __builtin_bit_cast(f16x8, e);
        }
      } else {
        f32x4 v[4][2];
        u32x4 gv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          v[s][0] = *reinterpret_cast<const f32x4*>(a + ((s * 8 + 2 * kc) ^ (l16 & 7)) * 16);
          v[s][1] = *reinterpret_cast<const f32x4*>(a + ((s * 8 + 2 * kc + 1) ^ (l16 & 7)) * 16);
          gv[s] = *reinterpret_cast<const u32x4*>(gn + s * 64);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          u32x4 eh, el;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            uint32_t a_hi, a_lo;
            split_f16x2(v[s][q / 2][q % 2 * 2] * inv * bf2f(gv[s][q] & 0xFFFF), v[s][q / 2][q % 2 * 2 + 1] * inv * bf2f(gv[s][q] >> 16), a_hi, a_lo);
            eh[q] = a_hi;
            el[q] = a_lo;
          }
          hi[s] = __builtin_bit_cast(f16x8, eh);
          lo[s] = __builtin_bit_cast(f16x8, el);
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int first = s * 8 + (NA == 1 && !low_half ? 4 : 0) + kc;
        hi[s] = *reinterpret_cast<const f16x8*>(a + (first ^ (l16 & 7)) * 16);
        if (NA == 2) lo[s] = *reinterpret_cast<const f16x8*>(a + ((first + 4) ^ (l16 & 7)) * 16);
      }
    }
    // what was read is in registers: refill its places
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    auto refill = [&](auto P) {                    // position P of this stage, RING units on
      constexpr int q = decltype(P)::value + RING;
      issue(std::integral_constant<int, q % UPS>{}, i + q / UPS, ring_at + slot * UNIT, left > RING);
      slot = slot + 1 == RING ? 0 : slot + 1;
      --left;
    };
    each(std::make_integer_sequence<int, NA>{}, refill);
    // ---- weights
    each(std::make_integer_sequence<int, NF>{}, [&](auto F) {
      constexpr int f = decltype(F)::value;
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (RING - 1)) : "memory");
      const unsigned char* w = ring + slot * UNIT + l16 * 256;
      u32x4 raw[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) raw[s] = *reinterpret_cast<const u32x4*>(w + ((s * 4 + kc) ^ l16) * 16);
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(raw[0]), "+v"(raw[1]), "+v"(raw[2]), "+v"(raw[3])::"memory");
      refill(std::integral_constant<int, NA + f>{});
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 wide;
#pragma unroll
        for (int q = 0; q < 4; ++q) wide[q] = widen_weights(raw[s][q]);
        const f16x8 wf = __builtin_bit_cast(f16x8, wide);
        acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, hi[s], acc[f], 0, 0, 0);
        if (NA == 2) acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, lo[s], acc[f], 0, 0, 0);
      }
    });
  }

  // ---- the partial tiles, added in wavefront order
  __syncthreads();
#pragma unroll
  for (int f = 0; f < NF; ++f) *reinterpret_cast<f32x4*>(lds + (wave * NF + f) * 1024 + lane * 16) = acc[f];
  __syncthreads();
  float* squares = reinterpret_cast<float*>(lds + WAVES * NF * 1024);     // [NF][16]
  if (wave < NF) {                                 // wavefront-uniform
    auto sum = [&](int ln) {
      f32x4 v[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        v[0] += *reinterpret_cast<const f32x4*>(lds + (w * NF + f_mine) * 1024 + ln * 16);
        if (NA == 1) v[1] += *reinterpret_cast<const f32x4*>(lds + (w * NF + f_mine) * 1024 + (ln ^ 8) * 16);
      }
      return v[0] + v[1];                          // NA 1: rows 8 .. 15 are the low parts of rows 0 .. 7
    };
    const float os = g.out_scale;
    if (EPI == STREAM_SWIGLU) {
      // lanes 0..31 hold 8 gate columns, lanes 32..63 the up columns of the same places
      const f32x4 gate = sum(lane & 31), up = sum(32 + (lane & 31));
      const int out = row0 / 2 + f_mine * 8 + kc * 4;
      if (lane < 32 && l16 < M && out < g.N / 2) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float gr = gate[r] * os, ur = up[r] * os;
          v[r] = gr / (1.0f + __expf(-gr)) * ur * g.c_scale;
        }
        uint32_t h0, l0, h1, l1;
        split_f16x2(v[0], v[1], h0, l0);
        split_f16x2(v[2], v[3], h1, l1);
        uint16_t* to = reinterpret_cast<uint16_t*>(g.c) + (size_t)l16 * g.N + pair_col(out);
        *reinterpret_cast<uint2*>(to) = make_uint2(h0, h1);
        *reinterpret_cast<uint2*>(to + 32) = make_uint2(l0, l1);
      }
    } else {
      f32x4 v = sum(lane);
      const bool mine = l16 < M && col < row0 + 8 * h && col < g.N;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] *= os;
      if (EPI == STREAM_ADD) {
        v += ahead;
        float s = mine ? v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3] : 0.f;
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (kc == 0) squares[f_mine * 16 + l16] = s;
      }
      if (EPI != STREAM_QKV) {
        if (mine) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.c) + (size_t)l16 * g.N + col) = v;
      } else if (mine) {
        const uint32_t page = at_slot / SY_PAGE, in_page = at_slot % SY_PAGE;
        const int head = col / g.hd, dim = col % g.hd;
        if (head < g.Hq + g.Hkv) {
          float r0, r1, r2, r3;
          rotate_pair(v[0], v[1], ahead[0], ahead[1], r0, r1);
          rotate_pair(v[2], v[3], ahead[2], ahead[3], r2, r3);
          const uint32_t p0 = pack_bf2(r0, r1), p1 = pack_bf2(r2, r3);
          if (head < g.Hq) {
            const size_t to = ((size_t)l16 * g.Hq + head) * g.hd + dim;
            *reinterpret_cast<uint2*>(g.q + to) = make_uint2(p0, p1);
            *reinterpret_cast<uint2*>(g.q_lo + to) = make_uint2(pack_bf2(r0 - bf2f(p0 & 0xFFFF), r1 - bf2f(p0 >> 16)),
                                                                pack_bf2(r2 - bf2f(p1 & 0xFFFF), r3 - bf2f(p1 >> 16)));
          } else {
            *reinterpret_cast<uint2*>(g.k_layer + (((size_t)page * g.Hkv + head - g.Hq) * SY_PAGE + in_page) * g.hd + dim) = make_uint2(p0, p1);
          }
        } else {
          bf16_t* to = g.v_layer + (((size_t)page * g.Hkv + head - g.Hq - g.Hkv) * g.hd + dim) * SY_PAGE + in_page;
#pragma unroll
          for (int r = 0; r < 4; ++r) to[r * SY_PAGE] = (bf16_t)f2bf(v[r]);
        }
      }
    }
  }
  if (EPI == STREAM_ADD && g.ss_out) {
    __syncthreads();
    if (tid < M) {
      float s = squares[tid];
#pragma unroll
      for (int f = 1; f < NF; ++f) s += squares[f * 16 + tid];
      g.ss_out[(size_t)tid * SY_STREAM_PARTS + blockIdx.x] = s;
    }
  }
}

// Blocks of 8 h rows.  One block runs per compute unit (the rings are its whole LDS): as many rows per block as 256 blocks need;
// where that is more than 128, rounds of equal blocks.  SwiGLU takes whole units.
static int half_units(int N, int epilogue) {
  const int halves = N / 8, rounds = (halves + 16 * 256 - 1) / (16 * 256);
  int h = (halves + rounds * 256 - 1) / (rounds * 256);
  if (epilogue == STREAM_SWIGLU) h = (h + 1) / 2 * 2;
  return h;
}
int stream_parts(int N) {
  const int h = half_units(N, STREAM_ADD);
  return (N / 8 + h - 1) / h;
}

template <int NF, int NA, bool ONCE>
static hipError_t launch_na(const StreamArgs& g, hipStream_t s) {
  const int grid = (g.N / 8 + g.half_units - 1) / g.half_units;
  switch (g.epilogue) {
    case STREAM_LOGITS: stream_kernel<NF, NA, STREAM_LOGITS, ONCE><<<grid, 64 * WAVES, 0, s>>>(g); break;
    case STREAM_ADD: stream_kernel<NF, NA, STREAM_ADD, ONCE><<<grid, 64 * WAVES, 0, s>>>(g); break;
    case STREAM_SWIGLU: stream_kernel<NF, NA, STREAM_SWIGLU, ONCE><<<grid, 64 * WAVES, 0, s>>>(g); break;
    case STREAM_QKV: stream_kernel<NF, NA, STREAM_QKV, ONCE><<<grid, 64 * WAVES, 0, s>>>(g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template <int NF>
static hipError_t launch_nf(const StreamArgs& g, hipStream_t s) {
  if (g.once) return g.M <= 8 ? launch_na<NF, 1, true>(g, s) : launch_na<NF, 2, true>(g, s);
  return g.M <= 8 ? launch_na<NF, 1, false>(g, s) : launch_na<NF, 2, false>(g, s);
}

hipError_t launch_stream(StreamArgs g, hipStream_t s) {
  if (g.M < 1 || g.M > SY_STREAM_ROWS || g.N % 16 != 0 || g.N < 16 || g.K % STAGE_K != 0 || g.K < STAGE_K) return hipErrorInvalidValue;
  if (g.epilogue != STREAM_ADD && (g.K > SY_STREAM_NORM_WIDTH || !g.ss || !g.gain || (g.epilogue == STREAM_LOGITS && !g.rows) || g.ss_parts < 1 || g.ss_parts > SY_STREAM_PARTS))
    return hipErrorInvalidValue;
  if (g.ss_out && stream_parts(g.N) > SY_STREAM_PARTS) return hipErrorInvalidValue;
  if (g.epilogue != STREAM_SWIGLU) {
    for (int i = 0; i < 3; ++i)
      if (g.w_rows[i] % 8 != 0) return hipErrorInvalidValue;
    if (g.w_rows[0] + g.w_rows[1] + g.w_rows[2] != g.N) return hipErrorInvalidValue;
  }
  g.half_units = half_units(g.N, g.epilogue);
  switch ((g.half_units + 1) / 2) {
    case 1: return launch_nf<1>(g, s);
    case 2: return launch_nf<2>(g, s);
    case 3: return launch_nf<3>(g, s);
    case 4: return launch_nf<4>(g, s);
    case 5: return launch_nf<5>(g, s);
    case 6: return launch_nf<6>(g, s);
    case 7: return launch_nf<7>(g, s);
    case 8: return launch_nf<8>(g, s);
    default: return hipErrorInvalidValue;
  }
}
