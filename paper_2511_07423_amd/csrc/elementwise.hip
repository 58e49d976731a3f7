// Small HBM-streaming kernels of the verify path: embedding gather, RMSNorm,
// rotary embedding fused with the paged KV append, the standalone KV append, the
// greedy accept-prefix scan, and a zero fill.  All are O(T*d) bytes and far from
// any roofline that matters; they are written for coalesced 16-byte accesses.
#include "common.h"

// ------------------------------------------------------------------ embedding, rotary table
// x[t][:] = float(E[token[t]][:]) and cs[t][i] = (cos, sin)(pos_t * base^(-2i/hd)), angle formed in double; ss (optional): the
// row's sum of squares as the first of its SY_STREAM_PARTS parts.  One block per token.  Token ids live on the device and
// cannot be validated by the host: an id outside [0, vocab) is clamped into the table instead of being followed out of
// bounds.  (Two kernels in one: each takes 4 us, nearly all of it latency, and their loads do not depend on each other.)
__global__ __launch_bounds__(256) void embed_kernel(const bf16_t* __restrict__ embed,
                                                    const int32_t* __restrict__ tokens, BatchMeta m,
                                                    float* __restrict__ x, float2* __restrict__ cs,
                                                    float* __restrict__ ss, int d, int vocab, int half, float base) {
  const int t = blockIdx.x;
  int tok = tokens[t];
  const int pos = m.tok_pos[t];
  tok = tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok);
  const bf16_t* src = embed + (size_t)tok * d;
  float* dst = x + (size_t)t * d;
  float sum = 0.f;
  for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
    uint4 v = *reinterpret_cast<const uint4*>(src + c);
    float4 lo = {bf2f(v.x & 0xFFFF), bf2f(v.x >> 16), bf2f(v.y & 0xFFFF), bf2f(v.y >> 16)};
    float4 hi = {bf2f(v.z & 0xFFFF), bf2f(v.z >> 16), bf2f(v.w & 0xFFFF), bf2f(v.w >> 16)};
    *reinterpret_cast<float4*>(dst + c) = lo;
    *reinterpret_cast<float4*>(dst + c + 4) = hi;
    sum += lo.x * lo.x + lo.y * lo.y + lo.z * lo.z + lo.w * lo.w + hi.x * hi.x + hi.y * hi.y + hi.z * hi.z + hi.w * hi.w;
  }
  for (int i = threadIdx.x; i < half; i += 256) {
    const double ang = (double)pos * pow((double)base, -(double)i / (double)half);
    double sn, cn;
    sincos(ang, &sn, &cn);
    cs[(size_t)t * half + i] = make_float2((float)cn, (float)sn);
  }
  if (!ss) return;
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  __shared__ float red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) ss[(size_t)t * SY_STREAM_PARTS] = red[0] + red[1] + red[2] + red[3];
}

hipError_t launch_embed(const bf16_t* embed, const int32_t* tokens, const BatchMeta& m, float* x, float2* cs, float* ss, int T,
                        int d, int vocab, int head_dim, float base, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  embed_kernel<<<T, 256, 0, s>>>(embed, tokens, m, x, cs, ss, d, vocab, head_dim / 2, base);
  return hipGetLastError();
}

// ------------------------------------------------------------------ RMSNorm
// y = x * rsqrt(mean(x^2) + eps) * g, fp32 in, fp16 (hi, lo) pair of SY_Y_SCALE y out (lo_off: lo = 0).  One block
// per output row; `rows` (optional) selects which input row feeds output row r.
// With n_parts > 0 the row first takes the pending K-split slices of the projection before it,
// x += sum_s parts[s], and the sum is written back to x (each thread re-reads only what it wrote).
__global__ __launch_bounds__(256) void rmsnorm_kernel(float* __restrict__ x, const float* __restrict__ parts,
                                                      int n_parts, size_t part_stride,
                                                      const bf16_t* __restrict__ gain,
                                                      const int32_t* __restrict__ rows,
                                                      uint16_t* __restrict__ y, uint16_t* __restrict__ y_lo, int d,
                                                      float eps, bool lo_off, bool paired) {
  const int r = blockIdx.x;
  const size_t row_at = (size_t)(rows ? rows[r] : r) * d;
  float* src = x + row_at;
  float ss = 0.f;
  for (int c = threadIdx.x * 4; c < d; c += 256 * 4) {
    float4 v = *reinterpret_cast<const float4*>(src + c);
    if (n_parts > 0) {
      for (int s = 0; s < n_parts; ++s) {
        const float4 pv = *reinterpret_cast<const float4*>(parts + (size_t)s * part_stride + row_at + c);
        v.x += pv.x; v.y += pv.y; v.z += pv.z; v.w += pv.w;
      }
      *reinterpret_cast<float4*>(src + c) = v;
    }
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  __shared__ float red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = rsqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps) * SY_Y_SCALE;
  // the pair as two arrays [rows][d], or (paired) as one array [rows][d / 32][hi 32 | lo 32]
  uint16_t* dst = y + (size_t)r * d * (paired ? 2 : 1);
  uint16_t* dst_lo = paired ? dst + 32 : y_lo + (size_t)r * d;
  for (int c = threadIdx.x * 4; c < d; c += 256 * 4) {
    float4 v = *reinterpret_cast<const float4*>(src + c);
    uint2 g = *reinterpret_cast<const uint2*>(gain + c);
    const float o0 = v.x * inv * bf2f(g.x & 0xFFFF), o1 = v.y * inv * bf2f(g.x >> 16);
    const float o2 = v.z * inv * bf2f(g.y & 0xFFFF), o3 = v.w * inv * bf2f(g.y >> 16);
    uint2 hi, lo;
    split_f16x2(o0, o1, hi.x, lo.x);
    split_f16x2(o2, o3, hi.y, lo.y);
    const size_t at = paired ? pair_col(c) : (size_t)c;
    *reinterpret_cast<uint2*>(dst + at) = hi;
    *reinterpret_cast<uint2*>(dst_lo + at) = lo_off ? make_uint2(0u, 0u) : lo;
  }
}

// The same for rows of at most 1024 IT values: the row stays in registers between the two passes (no re-read
// of x), and all loads of a pass are issued before anything is stored, so they are in flight together; the
// pending K slices are taken four at a time for the same reason (a slice per round trip is what a small batch,
// whose projections split K eight ways, otherwise spends its time on).
template <int IT>
__global__ __launch_bounds__(256) void rmsnorm_row_in_registers_kernel(
    float* __restrict__ x, const float* __restrict__ parts, int n_parts, size_t part_stride,
    const bf16_t* __restrict__ gain, const int32_t* __restrict__ rows, uint16_t* __restrict__ y,
    uint16_t* __restrict__ y_lo, int d, float eps, bool lo_off, bool paired) {
  const int r = blockIdx.x;
  const size_t row_at = (size_t)(rows ? rows[r] : r) * d;
  float* src = x + row_at;
  float4 v[IT];
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const int c = threadIdx.x * 4 + k * 1024;
    v[k] = c < d ? *reinterpret_cast<const float4*>(src + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  for (int s = 0; s < n_parts; s += 4) {
    float4 pv[4][IT];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = s + u < n_parts;
      const float* ps = parts + (size_t)(on ? s + u : s) * part_stride + row_at;
#pragma unroll
      for (int k = 0; k < IT; ++k) {
        const int c = threadIdx.x * 4 + k * 1024;
        pv[u][k] = on && c < d ? *reinterpret_cast<const float4*>(ps + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)               // slices are added in their order, as before
#pragma unroll
      for (int k = 0; k < IT; ++k) {
        v[k].x += pv[u][k].x; v[k].y += pv[u][k].y; v[k].z += pv[u][k].z; v[k].w += pv[u][k].w;
      }
  }
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const int c = threadIdx.x * 4 + k * 1024;
    if (n_parts > 0 && c < d) *reinterpret_cast<float4*>(src + c) = v[k];
    ss += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  __shared__ float red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = rsqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps) * SY_Y_SCALE;
  // the pair as two arrays [rows][d], or (paired) as one array [rows][d / 32][hi 32 | lo 32]
  uint16_t* dst = y + (size_t)r * d * (paired ? 2 : 1);
  uint16_t* dst_lo = paired ? dst + 32 : y_lo + (size_t)r * d;
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const int c = threadIdx.x * 4 + k * 1024;
    if (c >= d) continue;
    const uint2 g = *reinterpret_cast<const uint2*>(gain + c);
    const float o0 = v[k].x * inv * bf2f(g.x & 0xFFFF), o1 = v[k].y * inv * bf2f(g.x >> 16);
    const float o2 = v[k].z * inv * bf2f(g.y & 0xFFFF), o3 = v[k].w * inv * bf2f(g.y >> 16);
    uint2 hi, lo;
    split_f16x2(o0, o1, hi.x, lo.x);
    split_f16x2(o2, o3, hi.y, lo.y);
    const size_t at = paired ? pair_col(c) : (size_t)c;
    *reinterpret_cast<uint2*>(dst + at) = hi;
    *reinterpret_cast<uint2*>(dst_lo + at) = lo_off ? make_uint2(0u, 0u) : lo;
  }
}

hipError_t launch_rmsnorm(float* x, const float* parts, int n_parts, size_t part_stride, const bf16_t* gain,
                          const int32_t* rows, uint16_t* y_hi, uint16_t* y_lo, int n_rows, int d, float eps,
                          bool lo_off, bool paired, hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  if (d <= 4096)
    rmsnorm_row_in_registers_kernel<4><<<n_rows, 256, 0, s>>>(x, parts, n_parts, part_stride, gain, rows, y_hi, y_lo, d, eps, lo_off, paired);
  else if (d <= 8192)
    rmsnorm_row_in_registers_kernel<8><<<n_rows, 256, 0, s>>>(x, parts, n_parts, part_stride, gain, rows, y_hi, y_lo, d, eps, lo_off, paired);
  else
    rmsnorm_kernel<<<n_rows, 256, 0, s>>>(x, parts, n_parts, part_stride, gain, rows, y_hi, y_lo, d, eps, lo_off, paired);
  return hipGetLastError();
}

// ------------------------------------------------------------------ rotary + append
// Input row: fp32 [q heads | k heads | v heads] x hd, in NP K slices that are added in their order.
// q and k are rotated on adjacent pairs; q goes to a bf16 (hi, lo) pair [T][Hq][hd]; k and v go to
// the token's page and slot, which the host has looked up (through request, length and block table it is a chain of four
// loads for every block):
// K page [kv_head][slot][dim], V page [kv_head][dim][slot].
// A thread takes four values of one token, once: with NP known to the compiler all its slices are on their way together.
// Neighbouring tokens go to one XCD (blocks are dealt to the eight in turn), so that the 2-byte V stores of a page's tokens
// meet in one L2.  Bound by latency for small batches, by reading the slices for large ones.  8B shape, 5 slices: 128 tokens
// 8.7 us with three two-value rounds per thread and slices summed in a loop, 7.2 us with one round of four values,
// 6.0 us with neighbours on one XCD; 532 tokens (65 MB of slices) 19.4, 17.9 and 16.0 us.
#define SY_XCDS 8
template <int NP>
__global__ __launch_bounds__(256) void rope_append_kernel(const float* __restrict__ qkv, size_t part_stride,
                                                          const float2* __restrict__ cs, BatchMeta m,
                                                          bf16_t* __restrict__ q, bf16_t* __restrict__ q_lo,
                                                          bf16_t* __restrict__ k_layer, bf16_t* __restrict__ v_layer,
                                                          int T, int per_xcd, int Hq, int Hkv, int hd, bool lo_off) {
  const int width = (Hq + 2 * Hkv) * hd;
  const int t = blockIdx.x % SY_XCDS * per_xcd + blockIdx.y, e = (blockIdx.x / SY_XCDS * 256 + threadIdx.x) * 4;
  if (t >= T || e >= width) return;
  const int head = e / hd, dim = e % hd;
  const float* src = qkv + (size_t)t * width + e;
  f32x4 part[NP];
#pragma unroll
  for (int s = 0; s < NP; ++s) part[s] = *reinterpret_cast<const f32x4*>(src + (size_t)s * part_stride);
  const f32x4 c = *reinterpret_cast<const f32x4*>(cs + (size_t)t * (hd / 2) + dim / 2);   // (cos, sin) of two adjacent pairs
  const int page = m.tok_slot[t] / SY_PAGE, slot = m.tok_slot[t] % SY_PAGE;
  f32x4 v = part[0];
#pragma unroll
  for (int s = 1; s < NP; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] += part[s][r];
  if (head < Hq + Hkv) {
    float r0, r1, r2, r3;
    rotate_pair(v[0], v[1], c[0], c[1], r0, r1);
    rotate_pair(v[2], v[3], c[2], c[3], r2, r3);
    const uint32_t p0 = pack_bf2(r0, r1), p1 = pack_bf2(r2, r3);
    if (head < Hq) {
      const size_t at = ((size_t)t * Hq + head) * hd + dim;
      *reinterpret_cast<uint2*>(q + at) = make_uint2(p0, p1);
      *reinterpret_cast<uint2*>(q_lo + at) = lo_off ? make_uint2(0u, 0u)
                                                    : make_uint2(pack_bf2(r0 - bf2f(p0 & 0xFFFF), r1 - bf2f(p0 >> 16)),
                                                                 pack_bf2(r2 - bf2f(p1 & 0xFFFF), r3 - bf2f(p1 >> 16)));
    } else {
      *reinterpret_cast<uint2*>(k_layer + (((size_t)page * Hkv + head - Hq) * SY_PAGE + slot) * hd + dim) = make_uint2(p0, p1);
    }
  } else {
    bf16_t* dst = v_layer + (((size_t)page * Hkv + head - Hq - Hkv) * hd + dim) * SY_PAGE + slot;
#pragma unroll
    for (int r = 0; r < 4; ++r) dst[r * SY_PAGE] = (bf16_t)f2bf(v[r]);
  }
}

template <int NP>
static hipError_t launch_rope_np(const float* qkv, size_t part_stride, const float2* cs, const BatchMeta& m, bf16_t* q_hi,
                                 bf16_t* q_lo, bf16_t* k_layer, bf16_t* v_layer, int T, int Hq, int Hkv, int hd, bool lo_off,
                                 hipStream_t s) {
  const int quads = (Hq + 2 * Hkv) * hd / 4;
  const int per_xcd = (T + SY_XCDS - 1) / SY_XCDS;
  rope_append_kernel<NP><<<dim3(SY_XCDS * ((quads + 255) / 256), per_xcd), 256, 0, s>>>(
      qkv, part_stride, cs, m, q_hi, q_lo, k_layer, v_layer, T, per_xcd, Hq, Hkv, hd, lo_off);
  return hipGetLastError();
}

hipError_t launch_rope_append(const float* qkv, int n_parts, size_t part_stride, const float2* cs, const BatchMeta& m,
                              bf16_t* q_hi, bf16_t* q_lo, bf16_t* k_layer, bf16_t* v_layer, int T, int Hq, int Hkv,
                              int hd, bool lo_off, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  static_assert(SY_MAX_K_SLICES == 8, "one case per number of slices");
  switch (n_parts) {
#define SY_ROPE(NP) return launch_rope_np<NP>(qkv, part_stride, cs, m, q_hi, q_lo, k_layer, v_layer, T, Hq, Hkv, hd, lo_off, s)
    case 0: case 1: SY_ROPE(1);
    case 2: SY_ROPE(2);
    case 3: SY_ROPE(3);
    case 4: SY_ROPE(4);
    case 5: SY_ROPE(5);
    case 6: SY_ROPE(6);
    case 7: SY_ROPE(7);
    case 8: SY_ROPE(8);
#undef SY_ROPE
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------ standalone append
// Rows are bf16 already; a pure scatter, by one of two kernels.  The owner of a row (a page window) is found by binary
// search in prefix sums, so any number of rows per request is allowed.
//
// Small calls: a block per row, the shortest way from the lengths to the stores.
__global__ __launch_bounds__(128) void kv_append_rows_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                                             BatchMeta m, int B, bf16_t* __restrict__ k_layer,
                                                             bf16_t* __restrict__ v_layer, int n, int hd) {
  const int t = blockIdx.x;
  int lo = 0, hi = B;                       // find r with cu_tok[r] <= t < cu_tok[r+1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (m.cu_tok[mid] <= t) lo = mid; else hi = mid;
  }
  const int r = lo;
  const int pos = m.ctx_len[r] + (t - m.cu_tok[r]);
  const size_t page_at = (size_t)m.block_table[(size_t)r * m.max_pages + pos / SY_PAGE] * n * SY_PAGE;
  const int slot = pos % SY_PAGE;
  for (int e = threadIdx.x * 2; e < n; e += 128 * 2) {
    *reinterpret_cast<uint32_t*>(k_layer + page_at + ((size_t)(e / hd) * SY_PAGE + slot) * hd + e % hd) =
        *reinterpret_cast<const uint32_t*>(k + (size_t)t * n + e);
    const uint32_t vv = *reinterpret_cast<const uint32_t*>(v + (size_t)t * n + e);
    bf16_t* dst = v_layer + page_at + (size_t)e * SY_PAGE + slot;
    dst[0] = (bf16_t)(vv & 0xFFFF);
    dst[SY_PAGE] = (bf16_t)(vv >> 16);
  }
}

// Large calls: page tiles.  A wavefront owns 128 of a token's n = Hkv hd values for one page, i.e. up to
// 16 consecutive tokens: its K rows move in 16-byte pieces, its V values (two dims per lane, one load per token) are
// turned by LDS from token-major to the page's [dim][slot] order, so that both the K and the V tile of a whole page
// leave as contiguous 4 KB.  The first and the last page of a request may be shared with tokens that are not in this
// call: there only the covered slots are written, V by the pair where both slots of a word are covered.  n is a multiple of 128
// (synera_create).
// Bound by HBM: 24 requests, 28 K tokens, 231 MB read and written: 207 us with one block per row, 53 us a call, 36 us of it the kernel.  64 requests of
// 50 .. 100 rows, nearly half of whose pages are shared, the whole call with its wait: 55 us with a block per row, 43 with
// loads guarded by slot and 2-byte V stores in shared pages, 34.
__global__ __launch_bounds__(256) void kv_append_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                                        BatchMeta m, const int32_t* __restrict__ cu_win, int B,
                                                        bf16_t* __restrict__ k_layer, bf16_t* __restrict__ v_layer,
                                                        int n, int hd) {
  __shared__ __attribute__((aligned(16))) uint32_t turn[4][64 * 16];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e0 = (blockIdx.y * 4 + wave) * 128;
  if (e0 >= n) return;
  const int win = blockIdx.x;
  int lo = 0, hi = B;                       // find r with cu_win[r] <= win < cu_win[r+1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu_win[mid] <= win) lo = mid; else hi = mid;
  }
  const int r = lo;
  const int L = m.ctx_len[r], t0 = m.cu_tok[r], c = m.cu_tok[r + 1] - t0;
  const int page_pos = (L / SY_PAGE + win - cu_win[r]) * SY_PAGE;       // first position of the page
  const int s0 = max(L, page_pos) - page_pos, s1 = min(L + c, page_pos + SY_PAGE) - page_pos;   // covered slots, at least one
  const size_t page_at = (size_t)m.block_table[(size_t)r * m.max_pages + page_pos / SY_PAGE] * n * SY_PAGE;
  const size_t first = (size_t)(t0 + page_pos - L);                     // row of slot 0 (may lie before the call's rows)
  u32x4 kr[4];
  uint32_t vr[SY_PAGE];
  // (slots that are not covered load a covered one's row: without branches all loads are on their way together)
#pragma unroll
  for (int j = 0; j < 4; ++j)               // 4 tokens x 16 pieces per load
    kr[j] = *reinterpret_cast<const u32x4*>(k + (first + min(max(j * 4 + (lane >> 4), s0), s1 - 1)) * n + e0 + (lane & 15) * 8);
#pragma unroll
  for (int j = 0; j < SY_PAGE; ++j) vr[j] = *reinterpret_cast<const uint32_t*>(v + (first + min(max(j, s0), s1 - 1)) * n + e0 + 2 * lane);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int slot = j * 4 + (lane >> 4), e = e0 + (lane & 15) * 8;
    if (slot >= s0 && slot < s1)
      *reinterpret_cast<u32x4*>(k_layer + page_at + ((size_t)(e / hd) * SY_PAGE + slot) * hd + e % hd) = kr[j];
  }
  bf16_t* dst = v_layer + page_at + (size_t)e0 * SY_PAGE;               // 128 dims x 16 slots
  // lane's two rows of 16 slots = 16 words; the pieces of 4 words rotate with the lane so that the 16-byte LDS
  // accesses of neighbouring lanes fall on different banks
  uint32_t* mine = turn[wave] + lane * 16;
#pragma unroll
  for (int q = 0; q < 4; ++q) {             // piece q: slots (q & 1) * 8 .. + 7 of dim q >> 1
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t a = vr[(q & 1) * 8 + 2 * i], b = vr[(q & 1) * 8 + 2 * i + 1];
      w[i] = (q >> 1) ? (a >> 16) | (b & 0xFFFF0000u) : (a & 0xFFFFu) | (b << 16);
    }
    *reinterpret_cast<u32x4*>(mine + ((q + (lane >> 1)) & 3) * 4) = w;
  }
  __builtin_amdgcn_wave_barrier();
  const bool whole = s0 == 0 && s1 == SY_PAGE;                          // wavefront-uniform
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int piece = j * 64 + lane, from = piece >> 2;
    const u32x4 w = *reinterpret_cast<const u32x4*>(turn[wave] + from * 16 + (((piece & 3) + (from >> 1)) & 3) * 4);
    const int slot0 = (piece & 1) * 8;                                  // the piece's first slot
    bf16_t* to = dst + piece * 8;
    if (whole || (slot0 >= s0 && slot0 + 8 <= s1)) {
      *reinterpret_cast<u32x4*>(to) = w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool a = slot0 + 2 * i >= s0 && slot0 + 2 * i < s1, b = slot0 + 2 * i + 1 >= s0 && slot0 + 2 * i + 1 < s1;
        if (a && b) *reinterpret_cast<uint32_t*>(to + 2 * i) = w[i];
        else if (a) to[2 * i] = (bf16_t)(w[i] & 0xFFFF);
        else if (b) to[2 * i + 1] = (bf16_t)(w[i] >> 16);
      }
    }
  }
}

// The line between them (kv_append_by_rows): the call with its wait, 8B shape (n = 1024): 100 rows 25 us by rows, 27 by tiles; 300 rows 27.0, 27.5; 700
// rows 31, 30; 830 rows of 64 requests 33, 31.  n = 256: 1100 rows 26, 27; 1900 rows 31, 30; 3000 rows 30, 27.
bool kv_append_by_rows(int64_t T, int n) { return T * n <= 1 << 19; }

hipError_t launch_kv_append(const bf16_t* k, const bf16_t* v, const BatchMeta& m, const int32_t* cu_win, int n_win, int B,
                            bf16_t* k_layer, bf16_t* v_layer, int T, int Hkv, int hd, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const int n = Hkv * hd;
  if (!cu_win)
    kv_append_rows_kernel<<<T, 128, 0, s>>>(k, v, m, B, k_layer, v_layer, n, hd);
  else
    kv_append_kernel<<<dim3(n_win, (n + 511) / 512), 256, 0, s>>>(k, v, m, cu_win, B, k_layer, v_layer, n, hd);
  return hipGetLastError();
}

// ------------------------------------------------------------------ accept-prefix scan
// Thread i < B: a_0 = anchor (or the argmax of the last uncached token's row),
// a_j = argmax of draft j-1's row; n = longest prefix with d_j == a_j; correction
// = a_n.  Threads also copy the per-draft argmax rows to the caller's buffer.
__global__ void accept_kernel(const int32_t* __restrict__ tokens, const int32_t* __restrict__ anchor,
                              const int32_t* __restrict__ lm_argmax, BatchMeta m, int B, int R,
                              int32_t* __restrict__ out_argmax, int32_t* __restrict__ accept_len,
                              int32_t* __restrict__ correction) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < R) out_argmax[i] = lm_argmax[i];
  if (i >= B) return;
  const int u = m.n_unc[i];
  const int r0 = m.cu_draft[i], k = m.cu_draft[i + 1] - r0;
  const int32_t* d = tokens + m.cu_tok[i] + u;
  int32_t a = (u > 0) ? lm_argmax[m.first_row[i]] : anchor[i];
  int n = 0;
  while (n < k && d[n] == a) {
    a = lm_argmax[r0 + n];
    ++n;
  }
  accept_len[i] = n;
  correction[i] = a;
}

hipError_t launch_accept(const int32_t* tokens, const int32_t* anchor, const int32_t* lm_argmax, const BatchMeta& m,
                         int B, int R, int32_t* out_argmax, int32_t* accept_len, int32_t* correction,
                         hipStream_t s) {
  const int n = B > R ? B : R;
  if (n <= 0) return hipSuccess;
  accept_kernel<<<(n + 255) / 256, 256, 0, s>>>(tokens, anchor, lm_argmax, m, B, R, out_argmax, accept_len,
                                               correction);
  return hipGetLastError();
}

__global__ void fill_zero_kernel(float4* __restrict__ p, size_t n4) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n4; i += stride) p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t n4 = n / 4;   // callers pass multiples of 4
  int blocks = (int)((n4 + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  fill_zero_kernel<<<blocks, 256, 0, s>>>(reinterpret_cast<float4*>(p), n4);
  return hipGetLastError();
}
