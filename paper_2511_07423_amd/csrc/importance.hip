// Importance scores (Section 3.2): column-wise sums of the attention matrix softmax(Q K^T / sqrt(h)).
//
// For request i with chunk rows r = 0 .. c_i - 1 at positions L_i + r, key j in 0 .. L_i + c_i - 1:
//   I_j = (1 / Hq) sum over query heads hq, sum over rows r with L_i + r >= j of p_hq(r, j),
//   p_hq(r, j) = 2^(s scale log2e - m) / l,   s = q_hq(r) . k_kh(j),   (m, l) = the row's softmax
// statistics, which the attention kernel of the same layer has already formed and left in row_ml.  So
// one pass over the keys suffices: no second softmax reduction.
//
// The scores are a contraction, so they go through the matrix cores: S = K Q^T with
// v_mfma_f32_16x16x32_bf16, K (bf16 as it is in the cache) as the first operand, the query rows' bf16 (hi, lo)
// pairs as the second, both terms into one fp32 accumulator: the products are exact, as in fp32 arithmetic on
// hi + lo.  A lane then holds 4 keys of one query row: it forms the four probabilities and adds them to its own
// per-key sums; the 16 query rows of a fragment meet in one cross-lane sum at the very end.
//
// A unit of work is 256 consecutive keys of one request (one of the host's items) and one KV head; each of a block's
// four wavefronts takes 64 keys: four page tiles of 4 KB, loaded as they lie and turned to the MFMA's order by LDS.  The
// head's query rows pass through LDS in groups of 32, shared by the four wavefronts.  The heads' shares of a key are
// stored side by side in scratch and a second small kernel adds them in head order: no atomics, bit-reproducible.
// Blocks are persistent, two per compute unit, and while a unit's products run the next one's keys, first query rows
// and the record after that are already on their way: a block per unit spent most of its life in the chain item ->
// lengths -> page table -> keys, four latencies of a loaded memory system (129 us for the keys alone).  A small
// kernel folds that chain into one record per item beforehand.
// Bound by HBM (the K pages): 128 requests, 147 K keys, 302 MB: 429 us with one thread per key and scalar FMAs
// (5 GFLOP on the vector unit), 91 us.
#include "common.h"

#define SY_CONST_AS __attribute__((address_space(4)))
typedef __attribute__((ext_vector_type(8))) int imp_i32x8;
typedef __attribute__((ext_vector_type(4))) int imp_i32x4;

// Per item: {key0, n_keys, L, tok0, c, output index of key0, 0, 0} and the 16 pages of its keys (the last one repeated).

__global__ __launch_bounds__(256) void importance_items_kernel(ImportanceLaunch a) {
  const int i = (blockIdx.x * 256 + threadIdx.x) / 16, p = threadIdx.x % 16;
  if (i >= a.n_items) return;
  const int req = a.items[2 * i], key0 = a.items[2 * i + 1];
  const int L = a.ctx_len[req], tok0 = a.cu_tok[req], c = a.cu_tok[req + 1] - tok0;
  int32_t* rec = a.records + (size_t)i * SY_IMP_RECORD;
  rec[8 + p] = a.block_table[(size_t)req * a.max_pages + min(key0 / SY_PAGE + p, (L + c - 1) / SY_PAGE)];
  if (p == 0) {
    rec[0] = key0;
    rec[1] = L + c;
    rec[2] = L;
    rec[3] = tok0;
    rec[4] = c;
    rec[5] = a.cu_keys[req] + key0;
  }
}

// XOR of a staged row's 16-byte chunks, as for the attention kernel's K slots: a fragment read meets no bank twice.
template <int HD>
__device__ __forceinline__ int imp_swz(int row) {
  return HD == 128 ? (((row & 3) << 2) | (((row >> 2) & 1) << 1)) : ((((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1));
}

#define IMP_ROWS 32              // query rows staged at a time

// ONCE: the keys are marked as not wanted again (nt).
template <int HD, bool ONCE>
__global__ __launch_bounds__(256, 2) void importance_kernel(ImportanceLaunch a, int item0, int n_batch, float scale_log2) {
  constexpr int KS = HD / 32;                        // MFMA K steps over the head dimension
  constexpr int CPR = HD / 8;                        // 16-byte chunks of a row's high (or low) part
  constexpr int KL = SY_PAGE * CPR / 64;             // chunks per lane and page tile
  constexpr int QL = IMP_ROWS * 2 * CPR / 256;       // chunks per thread and group of query rows
  __shared__ __attribute__((aligned(16))) unsigned char lds[IMP_ROWS * 2 * HD * 2];
  __shared__ __attribute__((aligned(16))) unsigned char turn[4][SY_PAGE * HD * 2];
  __shared__ float2 lds_ml[IMP_ROWS];
  const int Hq = a.Hq, Hkv = a.Hkv, G = Hq / Hkv;
  const int tid = threadIdx.x, lane = tid & 63, n16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t g_inv = 65536u / (uint32_t)G + 1u;  // x g_inv >> 16 = x / G for rows below 32 x 16
  const int n_units = n_batch * Hkv;
  const SY_CONST_AS int32_t* records = reinterpret_cast<const SY_CONST_AS int32_t*>((uintptr_t)(a.records + (size_t)item0 * SY_IMP_RECORD));

  struct Unit { imp_i32x8 head; imp_i32x4 pages; };  // scalar registers
  auto record = [&](int u) {                         // heads of an item follow each other; past the end: the last unit
    const int item = min(u, n_units - 1) / Hkv;
    Unit r;
    r.head = *reinterpret_cast<const SY_CONST_AS imp_i32x8*>(records + (size_t)item * SY_IMP_RECORD);
    r.pages = *reinterpret_cast<const SY_CONST_AS imp_i32x4*>(records + (size_t)item * SY_IMP_RECORD + 8 + 4 * wave);
    return r;
  };
  auto load_k = [&](const Unit& r, int kh, u32x4 (&kr)[4][KL]) {
#pragma unroll
    for (int pg = 0; pg < 4; ++pg)
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        const auto* at = reinterpret_cast<const u32x4*>(a.k_layer + ((size_t)r.pages[pg] * Hkv + kh) * SY_PAGE * HD + (j * 64 + lane) * 8);
        kr[pg][j] = ONCE ? __builtin_nontemporal_load(at) : *at;
      }
  };
  auto load_q = [&](const Unit& r, int kh, int r0, u32x4 (&qr)[QL], float2& ml) {
    {
      const int row = min(r0 + (tid & (IMP_ROWS - 1)), r.head[4] * G - 1), tok = (int)((uint32_t)row * g_inv >> 16);
      ml = a.row_ml[(size_t)(r.head[3] + tok) * Hq + kh * G + row - tok * G];
    }
#pragma unroll
    for (int i = 0; i < QL; ++i) {
      const int p = i * 256 + tid, rw = p / (2 * CPR), ch = p % (2 * CPR);
      const int row = min(r0 + rw, r.head[4] * G - 1), tok = (int)((uint32_t)row * g_inv >> 16);
      const size_t at = ((size_t)(r.head[3] + tok) * Hq + kh * G + row - tok * G) * HD;
      qr[i] = *reinterpret_cast<const u32x4*>((ch < CPR ? a.q : a.q_lo) + at + (ch % CPR) * 8);
    }
  };

  int u = blockIdx.x;                                // the grid is no larger than n_units
  const int stride = gridDim.x;
  Unit cur = record(u), nxt = record(u + stride);
  // Loads return in order, so a wait for one is a wait for all before it: a unit's first two groups of query rows are
  // asked for before the next unit's keys, and nothing else is read from global memory while the products run.
  u32x4 kr[4][KL], qr[QL], qr1[QL];
  float2 ml, ml1;
  load_k(cur, u % Hkv, kr);
  load_q(cur, u % Hkv, 0, qr, ml);
  for (; u < n_units; u += stride) {
    const int kh = u % Hkv;
    const int key0 = cur.head[0] + 64 * wave, L = cur.head[2], n_rows = cur.head[4] * G;
    const bool cached = key0 + 63 < L;               // none of the wavefront's keys belongs to the chunk
    bf16x8 kf[4][KS];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        const int r = (j * 64 + lane) / CPR;
        *reinterpret_cast<u32x4*>(turn[wave] + r * (2 * HD) + ((lane % CPR ^ imp_swz<HD>(r)) << 4)) = kr[pg][j];
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int s = 0; s < KS; ++s)
        kf[pg][s] = *reinterpret_cast<const bf16x8*>(turn[wave] + n16 * (2 * HD) + (((4 * s + g4) ^ imp_swz<HD>(n16)) << 4));
      __builtin_amdgcn_wave_barrier();
    }
    const int un = min(u + stride, n_units - 1);     // past the end: loads that nobody uses
    load_q(cur, kh, IMP_ROWS, qr1, ml1);             // (past the chunk: its last row)
    load_k(nxt, un % Hkv, kr);
    float sum[4][4];                                 // [page][key 4 g4 + r]
#pragma unroll
    for (int pg = 0; pg < 4; ++pg)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[pg][r] = 0.f;
    for (int r0 = 0; r0 < n_rows; r0 += IMP_ROWS) {
      __syncthreads();                               // the group before is read
#pragma unroll
      for (int i = 0; i < QL; ++i) {
        const int p = i * 256 + tid, r = p / (2 * CPR), ch = p % (2 * CPR);
        *reinterpret_cast<u32x4*>(lds + r * (4 * HD) + (ch / CPR) * (2 * HD) + (((ch % CPR) ^ imp_swz<HD>(r)) << 4)) = qr[i];
        qr[i] = qr1[i];
      }
      if (tid < IMP_ROWS) lds_ml[tid] = ml;
      ml = ml1;
      __syncthreads();
      if (r0 + 2 * IMP_ROWS < n_rows) load_q(cur, kh, r0 + 2 * IMP_ROWS, qr1, ml1);
      const int most = min(IMP_ROWS, n_rows - r0);
      for (int rb = 0; rb < most; rb += 16) {
        const int rr = r0 + rb + n16, row = min(rr, n_rows - 1);       // chunk token row / G, query head row % G
        const int tok = (int)((uint32_t)row * g_inv >> 16);
        const float2 stat = lds_ml[rb + n16];
        f32x4 acc[4];
#pragma unroll
        for (int pg = 0; pg < 4; ++pg) acc[pg] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const unsigned char* from = lds + (rb + n16) * (4 * HD) + (((4 * s + g4) ^ imp_swz<HD>(n16)) << 4);
          const bf16x8 qh = *reinterpret_cast<const bf16x8*>(from);
          const bf16x8 ql = *reinterpret_cast<const bf16x8*>(from + 2 * HD);
#pragma unroll
          for (int pg = 0; pg < 4; ++pg) acc[pg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[pg][s], qh, acc[pg], 0, 0, 0);
#pragma unroll
          for (int pg = 0; pg < 4; ++pg) acc[pg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[pg][s], ql, acc[pg], 0, 0, 0);
        }
        const float inv = rr < n_rows ? 1.0f / stat.y : 0.f;
        if (cached) {                                                  // every row sees every key of the wavefront
#pragma unroll
          for (int pg = 0; pg < 4; ++pg)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              sum[pg][r] = fmaf(__builtin_amdgcn_exp2f(fmaf(acc[pg][r], scale_log2, -stat.x)), inv, sum[pg][r]);
        } else {
#pragma unroll
          for (int pg = 0; pg < 4; ++pg)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              // slots past the request's keys may hold anything: their p is dropped, not multiplied away
              const float p = __builtin_amdgcn_exp2f(fmaf(acc[pg][r], scale_log2, -stat.x)) * inv;
              sum[pg][r] += key0 + 16 * pg + 4 * g4 + r <= L + tok ? p : 0.f;
            }
        }
      }
    }
    load_q(nxt, un % Hkv, 0, qr, ml);
    float* share = a.parts + ((size_t)kh * n_batch + u / Hkv) * 256 + 64 * wave;
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
      float4 v = make_float4(sum[pg][0], sum[pg][1], sum[pg][2], sum[pg][3]);
      for (int o = 1; o < 16; o <<= 1) {
        v.x += __shfl_xor(v.x, o);
        v.y += __shfl_xor(v.y, o);
        v.z += __shfl_xor(v.z, o);
        v.w += __shfl_xor(v.w, o);
      }
      if (n16 == 0) *reinterpret_cast<float4*>(share + 16 * pg + 4 * g4) = v;
    }
    cur = nxt;
    nxt = record(u + 2 * stride);
  }
}

// Block = one item (256 keys of a request): score = sum of the Hkv shares, in head order.
__global__ __launch_bounds__(256) void importance_sum_kernel(ImportanceLaunch a, int item0, int n_batch) {
  const int32_t* rec = a.records + (size_t)(item0 + blockIdx.x) * SY_IMP_RECORD;
  if (rec[0] + (int)threadIdx.x >= rec[1]) return;
  float sum = 0.f;
#pragma unroll 8
  for (int kh = 0; kh < a.Hkv; ++kh) sum += a.parts[((size_t)kh * n_batch + blockIdx.x) * 256 + threadIdx.x];
  a.importance[rec[5] + threadIdx.x] = sum / (float)a.Hq;
}

hipError_t launch_importance(const ImportanceLaunch& a, hipStream_t s) {
  if (a.n_items <= 0) return hipSuccess;
  if (!a.parts || a.parts_cap < (size_t)a.Hkv * 256 || !a.records) return hipErrorInvalidValue;
  if (a.hd != 128 && a.hd != 64) return hipErrorInvalidValue;
  // Keys that the last-level cache would hardly hold beside what else a verify touches are read as not wanted again: 302 MB 93.3 ->
  // 91.2 us.  Below, a cache may hold them.
  const bool once = (size_t)a.n_items * 256 * a.Hkv * a.hd * 2 > ((size_t)128 << 20);
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)a.hd);
  importance_items_kernel<<<(a.n_items + 15) / 16, 256, 0, s>>>(a);
  // as many items per pass as the scratch holds shares for (one pass on every workload measured)
  const size_t fit = a.parts_cap / ((size_t)a.Hkv * 256);
  const int per_pass = (int)(fit < (size_t)a.n_items ? fit : (size_t)a.n_items);
  for (int item0 = 0; item0 < a.n_items; item0 += per_pass) {
    const int n_batch = a.n_items - item0 < per_pass ? a.n_items - item0 : per_pass;
    const int grid = (int)((long)n_batch * a.Hkv < a.blocks ? (long)n_batch * a.Hkv : a.blocks);
    auto* kernel = a.hd == 128 ? (once ? importance_kernel<128, true> : importance_kernel<128, false>)
                               : (once ? importance_kernel<64, true> : importance_kernel<64, false>);
    kernel<<<grid, 256, 0, s>>>(a, item0, n_batch, scale_log2);
    importance_sum_kernel<<<n_batch, 256, 0, s>>>(a, item0, n_batch);
  }
  return hipGetLastError();
}

// Thread i: mean score of request i's draft positions, and the probability of offloading by importance:
//   0 for i <= i_th / 2, 1 for i > i_th, else 1 / (1 + exp(theta ((i - i_th/2) / (i_th/2) - 1/2))).
__global__ void importance_dispatch_kernel(const float* __restrict__ importance, const int32_t* __restrict__ cu_keys,
                                           const int32_t* __restrict__ ctx_len, const int32_t* __restrict__ n_unc,
                                           const int32_t* __restrict__ cu_draft, int B, float i_th, float theta,
                                           float* __restrict__ mean_imp, float* __restrict__ p_imp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B) return;
  const int k = cu_draft[i + 1] - cu_draft[i];
  const float* at = importance + cu_keys[i] + ctx_len[i] + n_unc[i];
  float sum = 0.f;
  for (int j = 0; j < k; ++j) sum += at[j];
  const float m = k > 0 ? sum / (float)k : 0.f;
  if (mean_imp) mean_imp[i] = m;
  if (p_imp) {
    const float half = 0.5f * i_th;
    float p;
    if (m <= half) p = 0.f;
    else if (m > i_th) p = 1.f;
    else p = 1.0f / (1.0f + expf(theta * ((m - half) / half - 0.5f)));
    p_imp[i] = p;
  }
}

hipError_t launch_importance_dispatch(const float* importance, const int32_t* cu_keys, const int32_t* ctx_len,
                                      const int32_t* n_unc, const int32_t* cu_draft, int B, float i_th, float theta,
                                      float* mean_imp, float* p_imp, hipStream_t s) {
  if (B <= 0 || (!mean_imp && !p_imp)) return hipSuccess;
  importance_dispatch_kernel<<<(B + 127) / 128, 128, 0, s>>>(importance, cu_keys, ctx_len, n_unc, cu_draft, B, i_th,
                                                             theta, mean_imp, p_imp);
  return hipGetLastError();
}
