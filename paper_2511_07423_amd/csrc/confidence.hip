// Fused vocabulary-wide reduction: per logits row the argmax (lowest id on ties),
// its softmax probability (the confidence score, Section 3.2 of the paper) and the
// entropy in nats, in ONE pass over the row.
//
// Each thread keeps an online state (m, Z, S, id) over the elements it has seen:
//   m = running max, Z = sum e^(x-m), S = sum e^(x-m) (x-m), id = lowest index with x == m.
// A larger max rescales (Z, S) once per 16-byte chunk at most.  States combine
// associatively, first inside a wavefront by lane shuffles, then across the four
// wavefronts of the block through LDS.  At the end p_top1 = 1/Z and
// H = ln Z - S/Z.  HBM-bound: rows*vocab*sizeof(elem) bytes are read exactly once.
// Entries of -inf (tokens masked out by a top-k / top-p filter, Section 4.5) carry probability 0 and add
// nothing to the entropy; a row needs at least one finite entry.
#include "common.h"

#define LOG2E 1.4426950408889634f
#define LN2 0.6931471805599453f

struct ConfState {
  float m, Z, S;
  int id;
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Fold state b into a.
__device__ __forceinline__ void conf_merge(ConfState& a, const ConfState& b) {
  const float M = fmaxf(a.m, b.m);
  const float da = a.m - M, db = b.m - M;               // <= 0, finite (m starts at -1e30)
  const float ea = fast_exp2(da * LOG2E), eb = fast_exp2(db * LOG2E);
  const float S = ea * (a.S + a.Z * da) + eb * (b.S + b.Z * db);
  const float Z = ea * a.Z + eb * b.Z;
  int id = a.id;
  if (b.m > a.m || (b.m == a.m && b.id < a.id)) id = b.id;
  a.m = M; a.Z = Z; a.S = S; a.id = id;
}

template <int N>
__device__ __forceinline__ void conf_chunk(ConfState& st, const float (&v)[N], int base) {
  float cmax = v[0];
#pragma unroll
  for (int i = 1; i < N; ++i) cmax = fmaxf(cmax, v[i]);
  if (cmax > st.m) {                                       // rare after the first few chunks
    const float dm = st.m - cmax;
    const float sc = fast_exp2(dm * LOG2E);
    st.S = sc * (st.S + st.Z * dm);
    st.Z *= sc;
    st.m = cmax;
    int at = N - 1;
#pragma unroll
    for (int i = N - 2; i >= 0; --i) at = (v[i] == cmax) ? i : at;
    st.id = base + at;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    // bounded below: a masked logit (-inf) has weight e = 0 and must add 0 to S, not 0 * -inf
    const float t = fmaxf(v[i] - st.m, -1e30f);
    const float e = fast_exp2(t * LOG2E);
    st.Z += e;
    st.S = fmaf(e, t, st.S);
  }
}

template <bool BF16, bool ONCE>
__global__ __launch_bounds__(256) void confidence_kernel(const void* __restrict__ logits, int64_t vocab,
                                                         int64_t stride, int32_t* __restrict__ ids,
                                                         float* __restrict__ p1, float* __restrict__ H) {
  constexpr int VEC = BF16 ? 8 : 4;                        // elements per 16-byte load
  const int64_t row = blockIdx.x;
  const char* base = reinterpret_cast<const char*>(logits) + row * stride * (BF16 ? 2 : 4);
  const u32x4* src = reinterpret_cast<const u32x4*>(base);
  const int n_vec = (int)(vocab / VEC);
  // id starts at 0: a row without any finite entry (all NaN) then reports token 0, never an id
  // outside the vocabulary.
  ConfState st = {-1e30f, 0.f, 0.f, 0};

  auto consume = [&](const u32x4& raw, int c) {
    float v[VEC];
    if constexpr (BF16) {
      v[0] = bf2f(raw.x & 0xFFFF); v[1] = bf2f(raw.x >> 16);
      v[2] = bf2f(raw.y & 0xFFFF); v[3] = bf2f(raw.y >> 16);
      v[4] = bf2f(raw.z & 0xFFFF); v[5] = bf2f(raw.z >> 16);
      v[6] = bf2f(raw.w & 0xFFFF); v[7] = bf2f(raw.w >> 16);
    } else {
      v[0] = __uint_as_float(raw.x); v[1] = __uint_as_float(raw.y);
      v[2] = __uint_as_float(raw.z); v[3] = __uint_as_float(raw.w);
    }
    conf_chunk<VEC>(st, v, c * VEC);
  };

  // ONCE: marked as not wanted again (nt)
  auto load = [&](int at) { return ONCE ? __builtin_nontemporal_load(src + at) : src[at]; };
  int c = threadIdx.x;
  for (; c + 3 * 256 < n_vec; c += 4 * 256) {              // four 16-byte loads in flight per thread
    const u32x4 r0 = load(c), r1 = load(c + 256), r2 = load(c + 512), r3 = load(c + 768);
    consume(r0, c); consume(r1, c + 256); consume(r2, c + 512); consume(r3, c + 768);
  }
  for (; c < n_vec; c += 256) consume(load(c), c);
  // ragged tail (vocab not a multiple of the vector width): one element per thread
  for (int64_t e = (int64_t)n_vec * VEC + threadIdx.x; e < vocab; e += 256) {
    float v[1];
    v[0] = BF16 ? bf2f(reinterpret_cast<const bf16_t*>(base)[e]) : reinterpret_cast<const float*>(base)[e];
    conf_chunk<1>(st, v, (int)e);
  }

  for (int o = 1; o < 64; o <<= 1) {
    ConfState other;
    other.m = __shfl_xor(st.m, o);
    other.Z = __shfl_xor(st.Z, o);
    other.S = __shfl_xor(st.S, o);
    other.id = __shfl_xor(st.id, o);
    conf_merge(st, other);
  }
  __shared__ ConfState red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = st;
  __syncthreads();
  if (threadIdx.x == 0) {
    ConfState a = red[0];
    conf_merge(a, red[1]);
    conf_merge(a, red[2]);
    conf_merge(a, red[3]);
    ids[row] = a.id;
    if (p1) p1[row] = 1.0f / a.Z;
    if (H) H[row] = logf(a.Z) - a.S / a.Z;
  }
}

// ---------------------------------------------------------------------------------------------
// The same pass, keeping the k <= 256 most probable tokens of the row as well: the compressed form of a distribution
// that is transmitted instead of the full vector (Section 4.2, "Compression before transmission": a list that cuts
// 32000 entries by over 99.5 % has up to 160), and the margin score p_top1 - p_top2 of the layer-wise early exit
// (Section 4.3).  Equal logits: the lower id first.
//
// One block of 512 threads per row (four fit a compute unit: a few hundred rows run in one round); no list is kept
// while the row streams by.  Each thread remembers the maximum of each of its (up to NV) groups of 16-byte loads.
// Afterwards the k-th largest of the 512 thread maxima is a lower bound of the k-th largest logit, and a tight one:
// of independent logits about 1.4 k at k = 256, k + few for small k, are not below it.  Only the groups whose maximum reaches the bound are read again (from L2), their
// entries that reach it are collected in LDS, and each finds its rank by comparing with all others: ranks below k
// are the answer, in order.  Masked vocabularies (fewer finite thread maxima than the list is long) and plateaus of ties (more
// than TOPK_CAP entries at or above the bound) have few entries above one logit that very many hold: the list is filled up with its
// holders of the lowest ids, found by walking the row from its start.  Any other row with more than TOPK_CAP such entries takes an
// exact radix search over (logit, id), which ends with k entries.
// Bound by the one read of the row: 532 x 32000 f32, k = 160: 439 us with sorted lists kept across the lanes of
// each wavefront (an insertion per new entry), 26 us.  k = 64 with all but 50 entries of a row masked: 68 us with those lists, 230 us
// with the search for every such row, 23 us.
#define TOPK_WIDE_MAX 256
#define TOPK_THREADS 512
#define TOPK_CAP 1024

// Unsigned keys in the order of the logits; order_key's inverse is key_value.
__device__ __forceinline__ uint32_t order_key(float v) {
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}
// For the lists: 0 for NaN (never listed), -0 and +0 the same.
__device__ __forceinline__ uint32_t list_key(float v) { return v != v ? 0u : order_key(v + 0.0f); }

template <bool BF16>
struct RowReader {                                   // a row as 16-byte pieces plus a ragged tail
  static constexpr int VEC = BF16 ? 8 : 4;
  const char* base;
  int n_vec, n_tail;
  __device__ __forceinline__ RowReader(const void* logits, int64_t row, int64_t vocab, int64_t stride) {
    base = reinterpret_cast<const char*>(logits) + row * stride * (BF16 ? 2 : 4);
    n_vec = (int)(vocab / VEC);
    n_tail = (int)(vocab - (int64_t)n_vec * VEC);
  }
  __device__ __forceinline__ uint4 raw(int c) const { return reinterpret_cast<const uint4*>(base)[c]; }
  static __device__ __forceinline__ void unpack(const uint4& raw, float (&v)[VEC]) {
    if constexpr (BF16) {
      v[0] = bf2f(raw.x & 0xFFFF); v[1] = bf2f(raw.x >> 16);
      v[2] = bf2f(raw.y & 0xFFFF); v[3] = bf2f(raw.y >> 16);
      v[4] = bf2f(raw.z & 0xFFFF); v[5] = bf2f(raw.z >> 16);
      v[6] = bf2f(raw.w & 0xFFFF); v[7] = bf2f(raw.w >> 16);
    } else {
      v[0] = __uint_as_float(raw.x); v[1] = __uint_as_float(raw.y);
      v[2] = __uint_as_float(raw.z); v[3] = __uint_as_float(raw.w);
    }
  }
  __device__ __forceinline__ float at(int64_t e) const {
    return BF16 ? bf2f(reinterpret_cast<const bf16_t*>(base)[e]) : reinterpret_cast<const float*>(base)[e];
  }
  __device__ __forceinline__ float tail(int e) const { return at((int64_t)n_vec * VEC + e); }
};

// The row's statistics from every thread's own, left in *all (LDS); ends with a barrier.
template <int THREADS>
__device__ __forceinline__ void conf_block_merge(ConfState st, ConfState (&red)[THREADS / 64], ConfState* all) {
  for (int o = 1; o < 64; o <<= 1) {
    ConfState other;
    other.m = __shfl_xor(st.m, o);
    other.Z = __shfl_xor(st.Z, o);
    other.S = __shfl_xor(st.S, o);
    other.id = __shfl_xor(st.id, o);
    conf_merge(st, other);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = st;
  __syncthreads();
  if (threadIdx.x < 64) {
    ConfState a = red[threadIdx.x % (THREADS / 64)];
    for (int o = 1; o < THREADS / 64; o <<= 1) {
      ConfState other;
      other.m = __shfl_xor(a.m, o);
      other.Z = __shfl_xor(a.Z, o);
      other.S = __shfl_xor(a.S, o);
      other.id = __shfl_xor(a.id, o);
      conf_merge(a, other);
    }
    if (threadIdx.x == 0) *all = a;
  }
  __syncthreads();
}

template <bool BF16, int NV, bool MULTI>
__global__ __launch_bounds__(TOPK_THREADS) void confidence_topk_kernel(const void* __restrict__ logits, int64_t vocab,
                                                                       int64_t stride, int k, int32_t* __restrict__ ids,
                                                                       float* __restrict__ probs,
                                                                       float* __restrict__ margin, float* __restrict__ H) {
  constexpr int VEC = RowReader<BF16>::VEC;
  __shared__ ConfState red[TOPK_THREADS / 64], all;
  __shared__ __attribute__((aligned(16))) unsigned long long list[TOPK_CAP];   // (key, ~id): larger comes first
  __shared__ __attribute__((aligned(16))) uint32_t keys[TOPK_THREADS];
  __shared__ int cnts[2][TOPK_THREADS / 64];
  __shared__ int n_list;
  __shared__ float p_top[2];
  const int64_t row = blockIdx.x;
  const RowReader<BF16> rd(logits, row, vocab, stride);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int want = max(k, 2);                        // the margin needs the two best whatever k is
  // group j of this thread: loads (j per + g) TOPK_THREADS + tid, g < per
  const int per = MULTI ? (rd.n_vec + NV * TOPK_THREADS - 1) / (NV * TOPK_THREADS) : 1;

  // ---- the row streams by
  ConfState st = {-1e30f, 0.f, 0.f, 0};
  float gmax[NV];                                    // NaN: nothing comparable in the group
#pragma unroll
  for (int j = 0; j < NV; ++j) gmax[j] = __uint_as_float(0x7FC00000u);
  auto take = [&](const uint4& raw, int c, float& top) {
    float v[VEC];
    RowReader<BF16>::unpack(raw, v);
#pragma unroll
    for (int i = 0; i < VEC; ++i) top = fmaxf(top, v[i]);
    conf_chunk<VEC>(st, v, c * VEC);
  };
  if constexpr (MULTI) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      int c = j * per * TOPK_THREADS + tid;
#pragma unroll 4
      for (int g = 0; g < per; ++g, c += TOPK_THREADS) {
        const uint4 raw = rd.raw(min(c, rd.n_vec - 1));   // clamped, not skipped: the loads stay in flight together
        if (c < rd.n_vec) take(raw, c, gmax[j]);
      }
    }
  } else if (rd.n_vec > 0) {
    // four loads always in flight per thread (four at a time, of which the fifth waited for the fourth's arithmetic: 2000 x 32000 f32,
    // k = 160, 56.3 -> 53.8 us, 2048 x 128256 bf16 115 -> 110; bf16 rows of 33000 to 65000 entries, k = 160, 256 rows 20.3 -> 19.2, 1024
    // rows 47.6 -> 42.0 at 65000, 33.6 -> 33.3 at 33000; but 700 rows 32.7 -> 33.4 and 25.0 -> 25.5)
    constexpr int FLY = 4;
    const int last = rd.n_vec - 1;
    uint4 raw[FLY];
#pragma unroll
    for (int j = 0; j < FLY; ++j) raw[j] = rd.raw(min(j * TOPK_THREADS + tid, last));   // (past the end: never used)
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int c = j * TOPK_THREADS + tid;
      const uint4 now = raw[j % FLY];
      if (j + FLY < NV) raw[j % FLY] = rd.raw(min(c + FLY * TOPK_THREADS, last));
      if (c <= last) take(now, c, gmax[j]);
    }
  }
  uint32_t tail_key = 0;
  if (tid < rd.n_tail) {
    float v[1] = {rd.tail(tid)};
    tail_key = list_key(v[0]);
    conf_chunk<1>(st, v, rd.n_vec * VEC + tid);
  }
  float tmax = gmax[0];
#pragma unroll
  for (int j = 1; j < NV; ++j) tmax = fmaxf(tmax, gmax[j]);
  keys[tid] = max(list_key(tmax), tail_key);
  if (tid == 0) n_list = 0;
  if (tid < 2) p_top[tid] = 0.f;
  conf_block_merge<TOPK_THREADS>(st, red, &all);

  // ---- the want-th largest thread maximum, to its upper 24 bits: each wavefront counts for one of the 8 next digits
  uint32_t bound = 0;
  {
    uint4 q[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) q[i] = *reinterpret_cast<const uint4*>(keys + i * 256 + lane * 4);
    int buf = 0;
#pragma unroll
    for (int shift = 29; shift >= 8; shift -= 3) {
      const uint32_t t = bound | ((uint32_t)wave << shift);
      int n = 0;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(q[i].x >= t)) + __builtin_popcountll(__builtin_amdgcn_ballot_w64(q[i].y >= t)) +
             __builtin_popcountll(__builtin_amdgcn_ballot_w64(q[i].z >= t)) + __builtin_popcountll(__builtin_amdgcn_ballot_w64(q[i].w >= t));
      if (lane == 0) cnts[buf][wave] = n;
      __syncthreads();
      const unsigned long long ok = __builtin_amdgcn_ballot_w64(cnts[buf][lane & 7] >= want) & 0xFFull;   // bit 0 always
      bound |= (uint32_t)(31 - __builtin_clz((uint32_t)ok | 1u)) << shift;
      buf ^= 1;
    }
  }
  bound = max(bound, 1u);                            // fewer than want threads saw anything: every comparable entry

  // ---- collect what reaches the bound
  constexpr uint32_t MASKED = 0x007FFFFFu;           // list_key(-inf)
  uint32_t tie = bound <= MASKED ? MASKED : 0u;      // the logit whose holders fill the list up (block-uniform)
  auto composite = [](uint32_t key, int id) { return ((unsigned long long)key << 32) | (0xFFFFFFFFu - (uint32_t)id); };
  auto push = [&](unsigned long long c) {
    const int at = atomicAdd(&n_list, 1);
    if (at < TOPK_CAP) list[at] = c;
  };
  // Every entry of the groups that reach `from`, until the list is full.  (The maxima are compared as floats: four blocks to a
  // compute unit leave no registers for their keys as well.)
  auto collect = [&](float from, auto&& take) {
    uint32_t hit = 0;
#pragma unroll
    for (int j = 0; j < NV; ++j) hit |= gmax[j] >= from ? 1u << j : 0u;
    while (hit) {                                    // lanes take their groups side by side
      const int j = __builtin_ctz(hit);
      hit &= hit - 1;
      if (*(volatile int*)&n_list > TOPK_CAP) break;
      for (int g = 0; g < per; ++g) {
        const int c = (j * per + g) * TOPK_THREADS + tid;
        if (c >= rd.n_vec) break;
        float v[VEC];
        RowReader<BF16>::unpack(rd.raw(c), v);
#pragma unroll
        for (int i = 0; i < VEC; ++i) take(list_key(v[i]), c * VEC + i);
      }
    }
    if (tid < rd.n_tail) take(tail_key, rd.n_vec * VEC + tid);
  };
  {
    const uint32_t least = tie ? MASKED + 1u : bound;
    collect(key_value(least), [&](uint32_t key, int id) {
      if (key >= least) push(composite(key, id));
    });
  }
  __syncthreads();
  int n = n_list;
  if (n > TOPK_CAP && !tie) {                        // block-uniform
    // ---- a plateau at the bound?  The bound has 24 bits; groups above all logits that share them are few.  If the largest of those
    // logits is the maximum of enough groups, its holders fill the list up (nothing else is read again).
    __shared__ uint32_t sh_top;
    __shared__ int sh_groups;
    __syncthreads();                                 // n_list is read
    if (tid == 0) {
      n_list = 0;
      sh_top = 0;
      sh_groups = 0;
    }
    __syncthreads();
    const uint32_t last = bound | 0xFFu;
    const float least = key_value(bound), above = key_value(last + 1u);   // (beyond +inf: NaN, which nothing reaches)
    uint32_t top = tail_key >= bound && tail_key <= last ? tail_key : 0u;
    float gtop = __uint_as_float(0x7FC00000u);
#pragma unroll
    for (int j = 0; j < NV; ++j) gtop = fmaxf(gtop, gmax[j] >= least && !(gmax[j] >= above) ? gmax[j] : gtop);
    top = max(top, list_key(gtop));
    collect(above, [&](uint32_t key, int id) {
      if (key > last) push(composite(key, id));
      else if (key >= bound) top = max(top, key);
    });
    for (int o = 32; o > 0; o >>= 1) top = max(top, (uint32_t)__shfl_xor(top, o));
    if (lane == 0) atomicMax(&sh_top, top);
    __syncthreads();
    top = sh_top;
    gtop = key_value(top);
    int groups = tail_key == top ? 1 : 0;
#pragma unroll
    for (int j = 0; j < NV; ++j) groups += gmax[j] == gtop ? 1 : 0;
    for (int o = 32; o > 0; o >>= 1) groups += __shfl_xor(groups, o);
    if (lane == 0) atomicAdd(&sh_groups, groups);
    __syncthreads();
    if (n_list < want && n_list + sh_groups >= want) {   // block-uniform
      n = n_list;
      tie = top;
    }
  }
  if (tie && n < want) {                             // block-uniform
    // ---- the holders of `tie` with the lowest ids: VEC entries per thread and round, in id order
    const int need = want - n;
    int found = 0, buf = 0;
    for (int c0 = 0; c0 <= rd.n_vec && found < need; c0 += TOPK_THREADS) {
      const int c = c0 + tid;
      float v[VEC];
      RowReader<BF16>::unpack(rd.n_vec > 0 ? rd.raw(min(c, rd.n_vec - 1)) : make_uint4(0u, 0u, 0u, 0u), v);
      int before = 0, all = 0;                       // holders in the lanes below, in the wavefront
      unsigned long long mask[VEC];
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        const float x = c < rd.n_vec ? v[i] : (c == rd.n_vec && i < rd.n_tail ? rd.tail(i) : __uint_as_float(0x7FC00000u));
        mask[i] = __builtin_amdgcn_ballot_w64(list_key(x) == tie);
        before += __builtin_popcountll(mask[i] & ((1ull << lane) - 1));
        all += __builtin_popcountll(mask[i]);
      }
      if (lane == 0) cnts[buf][wave] = all;
      __syncthreads();
      int at = n + found + before;
#pragma unroll
      for (int w = 0; w < TOPK_THREADS / 64; ++w) {
        at += w < wave ? cnts[buf][w] : 0;
        found += cnts[buf][w];
      }
#pragma unroll
      for (int i = 0; i < VEC; ++i)
        if (mask[i] >> lane & 1) {
          if (at < want) list[at] = composite(tie, c * VEC + i);
          ++at;
        }
      buf ^= 1;
    }
    __syncthreads();
    n = min(n + found, want);
  }
  if (n > TOPK_CAP) {                                // block-uniform
    // ---- exact search: (key, ~id) digit by digit, 8 bits per pass over the row
    uint32_t* bins = keys;                           // 256 counters
    __shared__ unsigned long long sh_prefix;
    __shared__ int sh_above, sh_done;
    if (tid == 0) {
      sh_prefix = 0;
      sh_above = 0;
      sh_done = 0;
    }
    for (int shift = 56; shift >= 0; shift -= 8) {
      if (tid < 256) bins[tid] = 0;
      __syncthreads();
      if (sh_done) break;                            // block-uniform; nothing below is left out of step
      const unsigned long long prefix = sh_prefix;
      auto add = [&](float v, int id, bool on) {
        const uint32_t key = list_key(v);
        const unsigned long long c = composite(key, id);
        on = on && key != 0 && (shift == 56 || (c >> ((shift + 8) & 63)) == (prefix >> ((shift + 8) & 63)));
        const uint32_t bin = (uint32_t)(c >> shift) & 255u;
        // ties are why a row is here: the lanes that share the first lane's bin count as one
        const unsigned long long act = __builtin_amdgcn_ballot_w64(on);
        if (!act) return;
        const int l0 = __builtin_ctzll(act);
        const uint32_t b0 = __builtin_amdgcn_readlane(bin, l0);
        const unsigned long long same = __builtin_amdgcn_ballot_w64(on && bin == b0);
        if (lane == l0) atomicAdd(&bins[b0], (uint32_t)__builtin_popcountll(same));
        if (on && bin != b0) atomicAdd(&bins[bin], 1u);
      };
      for (int c0 = 0; c0 < rd.n_vec; c0 += TOPK_THREADS) {   // uniform trip count: whole wavefronts in `add`
        const int c = c0 + tid;
        float v[VEC];
        RowReader<BF16>::unpack(rd.raw(min(c, rd.n_vec - 1)), v);
#pragma unroll
        for (int i = 0; i < VEC; ++i) add(v[i], c * VEC + i, c < rd.n_vec);
      }
      if (rd.n_tail > 0) add(tid < rd.n_tail ? rd.tail(tid) : 0.f, rd.n_vec * VEC + tid, tid < rd.n_tail);
      __syncthreads();
      if (tid == 0) {
        int above = sh_above, b = 255;
        for (; b > 0 && above + (int)bins[b] < want; --b) above += (int)bins[b];
        sh_prefix = prefix | ((unsigned long long)b << shift);
        sh_above = above;
        if (above + (int)bins[b] <= want) sh_done = 1;  // the whole bin belongs to the list
        n_list = 0;
      }
      __syncthreads();
    }
    const unsigned long long least = sh_prefix;
    auto keep = [&](float v, int id) {
      const uint32_t key = list_key(v);
      const unsigned long long c = composite(key, id);
      if (key != 0 && c >= least) push(c);
    };
    for (int c = tid; c < rd.n_vec; c += TOPK_THREADS) {
      float v[VEC];
      RowReader<BF16>::unpack(rd.raw(c), v);
#pragma unroll
      for (int i = 0; i < VEC; ++i) keep(v[i], c * VEC + i);
    }
    if (tid < rd.n_tail) keep(rd.tail(tid), rd.n_vec * VEC + tid);
    __syncthreads();
    n = n_list;
  }

  // ---- ranks
  const float m = all.m, Z = all.Z;
  for (int at = tid; at < n; at += TOPK_THREADS) {
    const unsigned long long mine = list[at];
    int rank = 0, e = 0;
    for (; e + 1 < n; e += 2) {
      const ulonglong2 two = *reinterpret_cast<const ulonglong2*>(list + e);
      rank += (two.x > mine) + (two.y > mine);
    }
    if (e < n) rank += list[e] > mine;
    const float pr = fast_exp2((key_value((uint32_t)(mine >> 32)) - m) * LOG2E) / Z;   // (divided: one rounding)
    if (rank < k) {
      ids[row * k + rank] = (int32_t)(0xFFFFFFFFu - (uint32_t)mine);
      probs[row * k + rank] = pr;
    }
    if (rank < 2) p_top[rank] = pr;
  }
  for (int e = n + tid; e < k; e += TOPK_THREADS) {  // a row with fewer than k comparable entries
    ids[row * k + e] = 0;
    probs[row * k + e] = 0.f;
  }
  __syncthreads();
  if (tid == 0) {
    if (H) H[row] = logf(all.Z) - all.S / all.Z;
    if (margin) margin[row] = p_top[0] - p_top[1];
  }
}

hipError_t launch_confidence_topk(const void* logits, int dtype, int64_t rows, int64_t vocab, int64_t stride, int k,
                                  int32_t* ids, float* probs, float* margin, float* H, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (k > TOPK_WIDE_MAX) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)rows;
  const int64_t loads = (vocab / (dtype == 1 ? 8 : 4) + TOPK_THREADS - 1) / TOPK_THREADS;   // per thread
  // as many remembered maxima as a thread has loads, up to 32; then groups of loads share one
#define SY_TOPK(NV_, MULTI_)                                                                                          \
  if (dtype == 1)                                                                                                     \
    confidence_topk_kernel<true, NV_, MULTI_><<<grid, TOPK_THREADS, 0, s>>>(logits, vocab, stride, k, ids, probs, margin, H); \
  else                                                                                                                \
    confidence_topk_kernel<false, NV_, MULTI_><<<grid, TOPK_THREADS, 0, s>>>(logits, vocab, stride, k, ids, probs, margin, H);
  if (loads <= 8) { SY_TOPK(8, false) } else if (loads <= 16) { SY_TOPK(16, false) } else if (loads <= 32) { SY_TOPK(32, false) } else { SY_TOPK(32, true) }
#undef SY_TOPK
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Full-vocabulary top-p (nucleus): per row the smallest number of tokens, most probable first (equal logits by
// the lower id), whose probabilities sum to top_p, their mass, and the smallest logit kept.
//
// One block of 512 threads per row, four on a compute unit.  After the statistics pass (m, Z) the row is read twice
// more, from L2 or the last-level cache (kept in registers instead, half as many rows fit a compute unit: 50 against
// 46 us on 532 rows, 480 against 344 us on 2048 x 128256 bf16).  The cut is found by histogram: 1024 bins of 1/32 in the
// logit below the maximum, each with its entries' count and probability mass (one packed LDS atomic per entry; the bins are
// narrow so that the lanes of a wavefront rarely meet in one).  The bin where the running mass, from the largest
// logits down, reaches top_p holds a few dozen entries: they are listed and each sums the masses above itself.  A bin
// with more than NUC_CAP entries is first cut again by the order-preserving integer keys of its logits, down to a
// single key if need be (ties).  Masses are 40-bit fixed point: integer sums do not depend on the order in which
// threads arrive, so the result is reproducible.  A row without any mass (all -inf, or every logit below the running
// maximum's start of -1e30, as finfo.min masks are) has no cut: its nucleus is the holders of its largest logit, of mass 0.
// Bound by the one read of the row and, for few rows, by the chain of barriers: 532 x 32000 f32: 176 us with a
// four-pass radix search over the keys (every entry through two 64-bit LDS atomics on at most a handful of bins),
// 46 us.
#define NUC_THREADS 512
#define NUC_STAT_THREADS 256
#define NUC_BINS (2 * NUC_THREADS)
#define NUC_CAP 512
#define NUC_COUNT_SHIFT 42       // a bin packs (count << 42) + mass: masses of a row sum to 2^40 (1 + rounding)

template <bool BF16>
__global__ __launch_bounds__(NUC_THREADS, 8) void nucleus_kernel(const void* __restrict__ logits, int64_t vocab,
                                                              int64_t stride, float top_p, int32_t* __restrict__ count,
                                                              float* __restrict__ mass, float* __restrict__ cut_logit) {
  constexpr int VEC = RowReader<BF16>::VEC;
  __shared__ ConfState red[NUC_STAT_THREADS / 64];
  __shared__ float sh_m, sh_inv_z;
  __shared__ __attribute__((aligned(16))) unsigned long long bins[NUC_BINS];
  __shared__ uint32_t wide_count[NUC_BINS];          // counts of rows too long for the packed form
  __shared__ unsigned long long l_mass[NUC_CAP];
  __shared__ uint32_t l_key[NUC_CAP];
  __shared__ unsigned long long w_mass[NUC_THREADS / 64];
  __shared__ uint32_t w_count[NUC_THREADS / 64], w_last[NUC_THREADS / 64];
  __shared__ unsigned long long sh_above, sh_bin_mass;
  __shared__ uint32_t sh_count_above, sh_bin_count, sh_bin, sh_lo, sh_hi;
  __shared__ int n_list;
  const int64_t row = blockIdx.x;
  const RowReader<BF16> rd(logits, row, vocab, stride);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool wide = vocab >= (1ll << (64 - NUC_COUNT_SHIFT));
  auto each_value = [&](auto&& g) {                  // g(value) for every entry of the row
#pragma unroll 4
    for (int c = tid; c < rd.n_vec; c += NUC_THREADS) {
      float v[VEC];
      RowReader<BF16>::unpack(rd.raw(c), v);
#pragma unroll
      for (int i = 0; i < VEC; ++i) g(v[i]);
    }
    if (tid < rd.n_tail) g(rd.tail(tid));
  };

  // ---- statistics, by the first 256 threads: a count is an integer decided by sums over thousands of tokens, and one
  // in a hundred of them turns on the last bit of Z, so Z is summed in one fixed order whatever the block's size
  if (tid < NUC_STAT_THREADS) {                      // wavefront-uniform
    ConfState st = {-1e30f, 0.f, 0.f, 0};
    auto fold = [&](const uint4& raw, int c) {
      float v[VEC];
      RowReader<BF16>::unpack(raw, v);
      conf_chunk<VEC>(st, v, c * VEC);
    };
    int c = tid;
    for (; c + 3 * NUC_STAT_THREADS < rd.n_vec; c += 4 * NUC_STAT_THREADS) {   // four loads in flight per thread
      const uint4 r0 = rd.raw(c), r1 = rd.raw(c + NUC_STAT_THREADS), r2 = rd.raw(c + 2 * NUC_STAT_THREADS), r3 = rd.raw(c + 3 * NUC_STAT_THREADS);
      fold(r0, c);
      fold(r1, c + NUC_STAT_THREADS);
      fold(r2, c + 2 * NUC_STAT_THREADS);
      fold(r3, c + 3 * NUC_STAT_THREADS);
    }
    for (; c < rd.n_vec; c += NUC_STAT_THREADS) fold(rd.raw(c), c);
    if (tid < rd.n_tail) {
      const float v[1] = {rd.tail(tid)};
      conf_chunk<1>(st, v, rd.n_vec * VEC + tid);
    }
    for (int o = 1; o < 64; o <<= 1) {
      ConfState other;
      other.m = __shfl_xor(st.m, o);
      other.Z = __shfl_xor(st.Z, o);
      other.S = 0.f;
      other.id = 0;
      conf_merge(st, other);
    }
    if (lane == 0) red[wave] = st;
  } else {
    for (int i = tid - NUC_STAT_THREADS; i < NUC_BINS; i += NUC_THREADS - NUC_STAT_THREADS) {
      bins[i] = 0;
      wide_count[i] = 0;
    }
  }
  __syncthreads();
  if (tid == 0) {
    ConfState a = red[0];
#pragma unroll
    for (int w = 1; w < NUC_STAT_THREADS / 64; ++w) conf_merge(a, red[w]);
    sh_m = a.m;
    sh_inv_z = 1.0f / a.Z;
  }
  __syncthreads();
  const float m = sh_m, inv_z = sh_inv_z;
  const float fix = inv_z * 1099511627776.0f;
  auto fixed_mass = [&](float v) {                   // round(p 2^40), split exactly into its two words
    float x = fast_exp2((v - m) * LOG2E) * fix;
    x = x < 8388608.0f ? floorf(x + 0.5f) : x;       // from 2^23 on a float is whole
    if (__builtin_amdgcn_ballot_w64(x >= 4294967296.0f) == 0) return (unsigned long long)(uint32_t)x;   // p < 2^-8: most
    const float hi = floorf(x * 2.3283064365386963e-10f);
    return ((unsigned long long)(uint32_t)hi << 32) + (uint32_t)fmaf(hi, -4294967296.0f, x);
  };
  // top_p in the same fixed point; p sums to 1 within rounding, and where that leaves the whole row below the target
  // the cut is the smallest logit that still carries probability (masked tokens, -inf, are never part of a nucleus)
  // (a top_p below 2^-40 asks for one token, as the smallest target that a bin with mass can cross does)
  const unsigned long long asked = (unsigned long long)((double)top_p * 1099511627776.0), target = asked > 0 ? asked : 1;
  auto add = [&](int bin, float v) {
    const unsigned long long x = fixed_mass(v);
    atomicAdd(&bins[bin], wide ? x : x + (1ull << NUC_COUNT_SHIFT));
    if (wide) atomicAdd(&wide_count[bin], 1u);
  };
  auto first_bin = [&](float v) { return min((int)((m - v) * (NUC_BINS / 32.0f)), NUC_BINS - 1); };
  each_value([&](float v) { add(first_bin(v), v); });

  unsigned long long above = 0;                      // what lies above the bins: mass and count
  uint32_t count_above = 0;
  // Finds the bin the target falls into (the last one with any mass if none does, no bin if none has); leaves it in sh_*.
  // (The target is at least 1: the bin it falls into has mass.)
  auto find = [&]() {
    __syncthreads();
    static_assert(NUC_BINS == 2 * NUC_THREADS, "a lane sums two bins");
    const int b0 = wave * 128 + lane * 2;
    const ulonglong2 two = *reinterpret_cast<const ulonglong2*>(bins + b0);
    const unsigned long long mask = wide ? ~0ull : (1ull << NUC_COUNT_SHIFT) - 1;
    const unsigned long long m0 = two.x & mask, m1 = two.y & mask;
    const uint32_t c0 = wide ? wide_count[b0] : (uint32_t)(two.x >> NUC_COUNT_SHIFT);
    const uint32_t c1 = wide ? wide_count[b0 + 1] : (uint32_t)(two.y >> NUC_COUNT_SHIFT);
    unsigned long long sm = m0 + m1;                 // inclusive prefixes over the lanes
    uint32_t sc = c0 + c1;
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long tm = __shfl_up(sm, o);
      const uint32_t tc = __shfl_up(sc, o);
      if (lane >= o) {
        sm += tm;
        sc += tc;
      }
    }
    const unsigned long long pos = __builtin_amdgcn_ballot_w64(m0 + m1 > 0);
    if (lane == 63) {
      w_mass[wave] = sm;
      w_count[wave] = sc;
      w_last[wave] = pos ? 1u : 0u;
    }
    __syncthreads();
    unsigned long long before = above, total = above;
    uint32_t cbefore = count_above;
    int last_wave = 0;
#pragma unroll 1
    for (int w = 0; w < NUC_THREADS / 64; ++w) {     // (unrolled, its 64 registers of LDS reads push the row out)
      if (w < wave) {
        before += w_mass[w];
        cbefore += w_count[w];
      }
      total += w_mass[w];
      if (w_last[w]) last_wave = w;
    }
    const bool reached = total >= target;
    // exclusive values of this lane's two bins
    const unsigned long long e0 = before + sm - m0 - m1, e1 = e0 + m0;
    const uint32_t f0 = cbefore + sc - c0 - c1, f1 = f0 + c0;
    bool take0, take1;
    if (reached) {
      take0 = e0 < target && e0 + m0 >= target;
      take1 = e1 < target && e1 + m1 >= target;
    } else {
      const bool mine = wave == last_wave && pos && lane == 63 - __builtin_clzll(pos);
      take1 = mine && m1 > 0;
      take0 = mine && !take1;
    }
    if (take0 || take1) {
      sh_bin = b0 + (take1 ? 1 : 0);
      sh_above = take1 ? e1 : e0;
      sh_count_above = take1 ? f1 : f0;
      sh_bin_mass = take1 ? m1 : m0;
      sh_bin_count = take1 ? c1 : c0;
    }
    if (tid == 0) {
      if (total == above) {                          // no mass in any bin: nobody took one
        sh_bin = 0;
        sh_above = above;
        sh_count_above = count_above;
        sh_bin_mass = 0;
        sh_bin_count = 0xFFFFFFFFu;                  // more than the list holds: looked at where a crowded bin is
      }
      sh_lo = 0xFFFFFFFFu;
      sh_hi = 0;
      n_list = 0;
    }
    __syncthreads();
    above = sh_above;
    count_above = sh_count_above;
    return reached;
  };
  auto finish = [&](uint32_t key, unsigned long long group_mass, uint32_t holders, unsigned long long acc, uint32_t cnt) {
    const unsigned long long one = holders ? group_mass / holders : 0;
    uint32_t need = holders;
    if (one > 0 && acc < target) {
      const unsigned long long want = (target - acc + one - 1) / one;
      need = want < holders ? (uint32_t)want : holders;
    }
    if (need == 0) need = 1;
    count[row] = (int32_t)(cnt + need);
    if (mass) mass[row] = (float)((double)(acc + one * need) * (1.0 / 1099511627776.0));
    if (cut_logit) cut_logit[row] = key_value(key);
  };

  bool reached = find();
  uint32_t lo = 0, hi = 0xFFFFFFFFu;                 // keys of the bin's entries, once they have been asked for
  const int bin0 = (int)sh_bin;
  bool by_key = false;                               // membership: by first_bin == bin0, then by lo <= key <= hi
  while (sh_bin_count > NUC_CAP) {                   // block-uniform
    if (sh_bin_mass == 0) {                          // block-uniform: a row without mass
      uint32_t top = 0;                                // (one entry per thread and round: few registers, and rare)
#pragma unroll 1
      for (int64_t e = tid; e < vocab; e += NUC_THREADS) top = max(top, order_key(rd.at(e)));
      for (int o = 32; o > 0; o >>= 1) top = max(top, (uint32_t)__shfl_xor(top, o));
      if (lane == 0) atomicMax(&sh_hi, top);
      __syncthreads();
      top = sh_hi;
      int holders = 0;
#pragma unroll 1
      for (int64_t e = tid; e < vocab; e += NUC_THREADS) holders += order_key(rd.at(e)) == top ? 1 : 0;
      for (int o = 32; o > 0; o >>= 1) holders += __shfl_xor(holders, o);
      if (lane == 0) atomicAdd(&n_list, holders);
      __syncthreads();
      if (tid == 0) finish(top, 0, asked > 0 ? (uint32_t)n_list : 1u, 0, 0);
      return;
    }
    uint32_t mn = 0xFFFFFFFFu, mx = 0;
    each_value([&](float v) {
      const uint32_t key = order_key(v);
      if (by_key ? key >= lo && key <= hi : first_bin(v) == bin0) {
        mn = min(mn, key);
        mx = max(mx, key);
      }
    });
    for (int o = 32; o > 0; o >>= 1) {
      mn = min(mn, (uint32_t)__shfl_xor(mn, o));
      mx = max(mx, (uint32_t)__shfl_xor(mx, o));
    }
    if (lane == 0) {
      atomicMin(&sh_lo, mn);
      atomicMax(&sh_hi, mx);
    }
    for (int i = tid; i < NUC_BINS; i += NUC_THREADS) {
      bins[i] = 0;
      wide_count[i] = 0;
    }
    __syncthreads();
    lo = sh_lo;
    hi = sh_hi;
    by_key = true;
    if (lo == hi) {                                  // one logit, many holders
      if (tid == 0) finish(lo, sh_bin_mass, sh_bin_count, above, count_above);
      return;
    }
    int shift = 0;
    while (((hi - lo) >> shift) >= NUC_BINS) ++shift;
    each_value([&](float v) {
      const uint32_t key = order_key(v);
      if (key >= lo && key <= hi) add((int)((hi - key) >> shift), v);
    });
    reached = find();
    const uint32_t top = hi - (sh_bin << shift);
    if (shift == 0) {
      if (tid == 0) finish(top, sh_bin_mass, sh_bin_count, above, count_above);
      return;
    }
    const uint32_t width = (1u << shift) - 1u;
    lo = top - lo > width ? top - width : lo;
    hi = top;
  }
  each_value([&](float v) {
    const uint32_t key = order_key(v);
    if (by_key ? key >= lo && key <= hi : first_bin(v) == bin0) {
      const int at = atomicAdd(&n_list, 1);
      if (at < NUC_CAP) {                            // the bin's count says so
        l_key[at] = key;
        l_mass[at] = fixed_mass(v);
      }
    }
  });
  __syncthreads();
  const int n = min(n_list, NUC_CAP);
  if (tid >= n) return;
  const uint32_t key = l_key[tid];
  unsigned long long acc = above, group = 0;
  uint32_t cnt = count_above, holders = 0;
  bool lower = false;                                // an entry below this one carries probability
  for (int e = 0; e < n; ++e) {
    const uint32_t ke = l_key[e];
    const unsigned long long me = l_mass[e];
    if (ke > key) {
      acc += me;
      ++cnt;
    } else if (ke == key) {
      group += me;
      ++holders;
    } else {
      lower = lower || me > 0;
    }
  }
  if (reached ? acc < target && acc + group >= target : group > 0 && !lower)   // its holders agree: same values
    finish(key, group, holders, acc, cnt);
}

hipError_t launch_nucleus(const void* logits, int dtype, int64_t rows, int64_t vocab, int64_t stride, float top_p,
                          int32_t* count, float* mass, float* cut_logit, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const unsigned grid = (unsigned)rows;
  if (dtype == 1)
    nucleus_kernel<true><<<grid, NUC_THREADS, 0, s>>>(logits, vocab, stride, top_p, count, mass, cut_logit);
  else
    nucleus_kernel<false><<<grid, NUC_THREADS, 0, s>>>(logits, vocab, stride, top_p, count, mass, cut_logit);
  return hipGetLastError();
}

// Mean confidence of each chunk (rows cu_rows[b] .. cu_rows[b+1]) and its dispatch probability, the scaled
// sigmoid of Section 4.2: 1 for c <= c_th, else 1 / (1 + exp(k (c - c_th) / (1 - c_th) - k / 2)).
__global__ void chunk_dispatch_kernel(const float* __restrict__ p1, const int32_t* __restrict__ cu_rows, int B,
                                      float c_th, float k_slope, float* __restrict__ mean_conf,
                                      float* __restrict__ p_conf) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int r0 = cu_rows[b], r1 = cu_rows[b + 1];
  float sum = 0.f;
  for (int r = r0; r < r1; ++r) sum += p1[r];
  const float c = r1 > r0 ? sum / (float)(r1 - r0) : 0.f;
  mean_conf[b] = c;
  float pc = 1.0f;
  if (c > c_th) {
    const float norm = (c - c_th) / (1.0f - c_th) - 0.5f;
    pc = 1.0f / (1.0f + expf(k_slope * norm));
  }
  p_conf[b] = pc;
}

hipError_t launch_chunk_dispatch(const float* p1, const int32_t* cu_rows, int B, float c_th, float k_slope,
                                 float* mean_conf, float* p_conf, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  chunk_dispatch_kernel<<<(B + 127) / 128, 128, 0, s>>>(p1, cu_rows, B, c_th, k_slope, mean_conf, p_conf);
  return hipGetLastError();
}

// Top-p (nucleus) cut of compressed distributions: row r holds k probabilities, most probable first (the
// output of confidence_topk_kernel); n[r] = the smallest count whose float32 running sum, in list order,
// reaches top_p (all k if it never does), mass[r] = that sum.
// The running sum is serial by definition (its rounding decides the count), so the row comes in with coalesced loads,
// one entry per lane, and the lanes' entries are added one after the other from registers: a wavefront per row
// (a thread per row spent its time on a chain of uncoalesced loads: 532 lists of 160, 20 us, 4 us).
__global__ __launch_bounds__(256) void topp_count_kernel(const float* __restrict__ probs, int64_t rows, int k, float top_p,
                                                         int32_t* __restrict__ n, float* __restrict__ mass) {
  const int64_t r = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (r >= rows) return;
  const int lane = threadIdx.x & 63;
  float acc = 0.f;
  int kept = k;
  float next = lane < k ? probs[r * k + lane] : 0.f;
  for (int i0 = 0; i0 < k; i0 += 64) {
    const float cur = next;
    if (i0 + 64 < k) next = i0 + 64 + lane < k ? probs[r * k + i0 + 64 + lane] : 0.f;
    float upto = 0.f;                                // lane i: the running sum after entry i0 + i
#pragma unroll
    for (int i = 0; i < 64; ++i) {                   // past the end: adds 0
      acc += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur), i));
      upto = lane == i ? acc : upto;
    }
    const unsigned long long over = __builtin_amdgcn_ballot_w64(i0 + lane < k && upto >= top_p);
    if (over) {
      const int i = __builtin_ctzll(over);
      kept = i0 + i + 1;
      acc = __shfl(upto, i);
      break;
    }
  }
  if (lane == 0) {
    n[r] = kept;
    if (mass) mass[r] = acc;
  }
}

hipError_t launch_topp_count(const float* probs, int64_t rows, int k, float top_p, int32_t* n, float* mass,
                             hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  topp_count_kernel<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(probs, rows, k, top_p, n, mass);
  return hipGetLastError();
}

// ------------------------------------------------------------------ stochastic verification
// Speculative sampling of one request per block (the rule the paper cites for its "draft & verify" under
// top-k / top-p sampling): draft j is accepted with probability min(1, q_j(x_j) / p_j(x_j)); at the first
// rejection a token is drawn from norm(max(0, q_j - p_j)), after k acceptances from q_{k+1}.  q_j is the softmax
// of an LM-head row that the verify call left behind (row of the last uncached token for j = 0, of draft
// j-1 after that; its maximum and normaliser come from the confidence pass: q_v = exp(l_v - l_max) p_top1);
// p_j is the device's transmitted top-k list renormalised to 1.  The uniforms are inputs.
//
// One block of 16 wavefronts per request.  The tests of all drafts run side by side, a wavefront per draft (lanes
// over the list); the first that fails names the row to draw from.  The draw: each wavefront sums its own
// contiguous sixteenth of the vocabulary (16-byte loads, fp64 accumulators), corrected for the list's tokens that
// fall into it; the sixteenth that holds the target is walked again by its wavefront, 256 tokens at a time with a
// prefix scan, and the lane that crosses the target names the token.  Bound by one compute unit's read of one row
// of logits and the two dependent passes: 128 requests, lists of 160, vocabulary 32000: 1622 us with one thread
// walking the lists and each thread summing 125 neighbouring tokens, 39 us; 36.6 with the walk's logits asked for ahead.
#define SA_WAVES 16

__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__global__ __launch_bounds__(64 * SA_WAVES) void stochastic_accept_kernel(
    const float* __restrict__ logits, int vocab, const int32_t* __restrict__ lm_ids, const float* __restrict__ lm_p,
    const int32_t* __restrict__ tokens, BatchMeta m, int k_list, const int32_t* __restrict__ p_id,
    const float* __restrict__ p_prob, const float* __restrict__ u_accept, const float* __restrict__ u_sample,
    int32_t* __restrict__ accept_len, int32_t* __restrict__ out_token) {
  __shared__ int sh_ok[SA_WAVES * 2];                // draft j passes its test (chunks hold at most 32 drafts)
  __shared__ double sh_sum[SA_WAVES];
  __shared__ int l_id[TOPK_WIDE_MAX];                // the list to subtract at the rejected position
  __shared__ float l_p[TOPK_WIDE_MAX];               // its probabilities, renormalised to 1
  __shared__ double l_fix[TOPK_WIDE_MAX];            // what entry e changes in the sum of its sixteenth
  __shared__ int s_id[TOPK_WIDE_MAX];                // the entries inside the sixteenth that is walked, in list order
  __shared__ float s_p[TOPK_WIDE_MAX];
  const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = m.cu_draft[i], k = m.cu_draft[i + 1] - r0;
  const int32_t* d = tokens + m.cu_tok[i] + m.n_unc[i];
  for (int j = wave; j < k; j += SA_WAVES) {         // wavefront-uniform
    const int row = j == 0 ? m.first_row[i] : r0 + j - 1;
    const float* l = logits + (size_t)row * vocab;
    int x = d[j];
    x = x < 0 ? 0 : (x >= vocab ? vocab - 1 : x);
    const float q_x = __expf(l[x] - l[lm_ids[row]]) * lm_p[row];
    float sum = 0.f, p_x = 0.f;
    for (int e = lane; e < k_list; e += 64) {
      const float pe = p_prob[(size_t)(r0 + j) * k_list + e];
      sum += pe;
      p_x += p_id[(size_t)(r0 + j) * k_list + e] == x ? pe : 0.f;
    }
    sum = wave_sum(sum);
    p_x = wave_sum(p_x);
    const float ratio = p_x > 0.f ? fminf(1.0f, q_x * sum / p_x) : 0.f;
    if (lane == 0) sh_ok[j] = u_accept[r0 + j] < ratio;
  }
  __syncthreads();
  int n = 0;
  while (n < k && sh_ok[n]) ++n;
  const int row = (n == 0) ? m.first_row[i] : r0 + n - 1;      // n == k: the row after the last draft
  const float* l = logits + (size_t)row * vocab;
  const float l_max = l[lm_ids[row]], p_top = lm_p[row];
  const int n_list = n < k ? k_list : 0;                       // nothing to subtract after a full accept
  if (n_list > 0) {                                            // block-uniform
    float sum = 0.f;
    for (int e = lane; e < n_list; e += 64) sum += p_prob[(size_t)(r0 + n) * k_list + e];
    sum = wave_sum(sum);                                       // every wavefront forms the same sum
    const float list_inv = sum > 0.f ? 1.0f / sum : 0.f;       // an all-zero list subtracts nothing
    for (int e = tid; e < n_list; e += 64 * SA_WAVES) {
      l_id[e] = p_id[(size_t)(r0 + n) * k_list + e];
      l_p[e] = p_prob[(size_t)(r0 + n) * k_list + e] * list_inv;
    }
  }
  auto q_at = [&](float x) { return __expf(x - l_max) * p_top; };
  // sum of q over this wavefront's sixteenth; vocab is a multiple of 4 (of 128: synera_create)
  const int seg = (vocab + SA_WAVES * 256 - 1) / (SA_WAVES * 256) * 256;
  const int v0 = min(wave * seg, vocab), v1 = min(v0 + seg, vocab);
  double mine = 0.0;
#pragma unroll 4
  for (int v = v0 + lane * 4; v < v1; v += 256) {
    const float4 t = *reinterpret_cast<const float4*>(l + v);
    mine += (double)q_at(t.x) + (double)q_at(t.y) + (double)q_at(t.z) + (double)q_at(t.w);
  }
  __syncthreads();
  // entry e's correction, max(0, q - p) - q at its token; a token listed twice is corrected once, by its total
  for (int e = tid; e < n_list; e += 64 * SA_WAVES) {
    const int v = l_id[e];
    double fix = 0.0;
    if (v >= 0 && v < vocab) {
      const float q = q_at(l[v]);
      float w = q;
      int earlier = 0;
#pragma unroll 8
      for (int f = 0; f < n_list; ++f) {             // without branches: the LDS reads run ahead
        const bool same = l_id[f] == v;
        earlier |= same && f < e;
        w -= same ? l_p[f] : 0.f;
      }
      if (!earlier) fix = (double)(w > 0.f ? w : 0.f) - (double)q;
    }
    l_fix[e] = fix;
  }
  __syncthreads();
  for (int e = lane; e < n_list; e += 64)
    if (l_id[e] >= v0 && l_id[e] < v1) mine += l_fix[e];
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
  if (lane == 0) sh_sum[wave] = mine;
  __syncthreads();
  double total = 0.0;
  for (int t = 0; t < SA_WAVES; ++t) total += sh_sum[t];
  const double target = (double)u_sample[i] * total;
  double before = 0.0, at_last = 0.0, c = 0.0;
  int slice = -1, last = 0;                                    // last: the last sixteenth that holds any weight
  for (int t = 0; t < SA_WAVES; ++t) {
    if (slice < 0 && c + sh_sum[t] > target) {
      slice = t;
      before = c;
    }
    if (sh_sum[t] > 0.0) {
      last = t;
      at_last = c;
    }
    c += sh_sum[t];
  }
  if (slice < 0) {                                             // rounding put the target at the very end
    slice = last;
    before = at_last;
  }
  if (wave != slice) return;
  // ---- one wavefront from here on
  int n_sub = 0;
  for (int e0 = 0; e0 < n_list; e0 += 64) {
    const int e = e0 + lane;
    const bool in = e < n_list && l_id[e] >= v0 && l_id[e] < v1;
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(in);
    if (in) {
      const int at = n_sub + __builtin_popcountll(mask & ((1ull << lane) - 1));
      s_id[at] = l_id[e];
      s_p[at] = l_p[e];
    }
    n_sub += __builtin_popcountll(mask);
  }
  __builtin_amdgcn_wave_barrier();
  int token = -1, last_positive = -1;
  // pieces of 256 entries, asked for four to eight ahead: one at a time, each waited for its logits behind the prefix of the one before
  float4 now[4], next[4];
  auto ask = [&](int vb, float4 (&t)[4]) {                     // (past the sixteenth: its end again, never used; v1 >= 128)
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = *reinterpret_cast<const float4*>(l + min(vb + 256 * j + lane * 4, v1 - 4));
  };
  auto piece = [&](int vb, const float4& t) {
    const int v = vb + lane * 4;
    float w[4] = {0.f, 0.f, 0.f, 0.f};
    if (v < v1) {
      w[0] = q_at(t.x); w[1] = q_at(t.y); w[2] = q_at(t.z); w[3] = q_at(t.w);
      for (int e = 0; e < n_sub; ++e) {
        const int at = s_id[e] - v;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] -= at == r ? s_p[e] : 0.f;
      }
    }
    double own = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      w[r] = w[r] > 0.f ? w[r] : 0.f;
      if (w[r] > 0.f) last_positive = v + r;
      own += (double)w[r];
    }
    double upto = own;                                         // inclusive prefix over the lanes
    for (int o = 1; o < 64; o <<= 1) {
      const double left = __shfl_up(upto, o);
      if (lane >= o) upto += left;
    }
    const unsigned long long over = __builtin_amdgcn_ballot_w64(own > 0.0 && before + upto > target);
    if (over) {
      const int at = __builtin_ctzll(over);
      double left = __shfl_up(upto, 1);
      double cc = before + (lane > 0 ? left : 0.0);
      int pick = -1, pos = -1;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cc += (double)w[r];
        if (w[r] > 0.f) {
          pos = v + r;
          if (pick < 0 && cc > target) pick = v + r;
        }
      }
      token = __builtin_amdgcn_readlane(pick >= 0 ? pick : pos, at);
    }
    before += __shfl(upto, 63);
  };
  ask(v0, now);
  for (int vb = v0; vb < v1 && token < 0; vb += 1024) {
    ask(vb + 1024, next);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (vb + 256 * j < v1 && token < 0) piece(vb + 256 * j, now[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) now[j] = next[j];
  }
  if (token < 0) {
    for (int o = 32; o > 0; o >>= 1) last_positive = max(last_positive, __shfl_xor(last_positive, o));
    token = last_positive;
  }
  if (lane == 0) {
    accept_len[i] = n;
    out_token[i] = token >= 0 ? token : lm_ids[row];           // degenerate residual (p == q): the row's mode
  }
}

hipError_t launch_stochastic_accept(const float* logits, int vocab, const int32_t* lm_ids, const float* lm_p,
                                    const int32_t* tokens, const BatchMeta& m, int B, int k_list, const int32_t* p_id,
                                    const float* p_prob, const float* u_accept, const float* u_sample,
                                    int32_t* accept_len, int32_t* out_token, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  stochastic_accept_kernel<<<B, 64 * SA_WAVES, 0, s>>>(logits, vocab, lm_ids, lm_p, tokens, m, k_list, p_id, p_prob, u_accept,
                                             u_sample, accept_len, out_token);
  return hipGetLastError();
}

hipError_t launch_confidence(const void* logits, int dtype, int64_t rows, int64_t vocab, int64_t stride,
                             int32_t* ids, float* p1, float* H, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  // Matrices that no cache holds are read as not wanted again (nt).  2048 x 128256 bf16 (525 MB): 99.6 -> 89.8 us; 1131 x
  // 32000 f32 (145 MB, just written by the LM head): 28.7 -> 27 us; below, what a cache still holds counts: 589 x 32000 (75 MB)
  // 14.8 -> 15.1, 5 rows 9.6 -> 10.9 us.  Rows that do not start on a 128-byte line, and so share lines, gain as well: bf16 2048 x 50257
  // (pitch 50264) 42.2 -> 40.6, 2048 x 100277 78.7 -> 74.8, f32 1024 x 50257 38.0 -> 34.6; about 1000 rows of bf16 lose 1 to 2 %
  // (1024 x 128256 50.1 -> 51.0, 900 x 100001 38.8 -> 39.2).
  const bool once = rows * vocab * (dtype == 1 ? 2 : 4) > (128 << 20);
  auto* kernel = dtype == 1 ? (once ? confidence_kernel<true, true> : confidence_kernel<true, false>)
                            : (once ? confidence_kernel<false, true> : confidence_kernel<false, false>);
  kernel<<<(unsigned)rows, 256, 0, s>>>(logits, vocab, stride, ids, p1, H);
  return hipGetLastError();
}
