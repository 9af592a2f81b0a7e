// Children of the leaves a draft step expands (Sec. 3.1, maximum-likelihood
// tree expansion): per logits row, the k most probable tokens and their
// log-softmax values.
//
// Two kernels.  The first splits each row [V] fp16 into S contiguous ranges of
// 16-byte vectors, one 256-thread workgroup each (S = 1024 / n, at most 64:
// about one vector per thread at a 128256-entry vocabulary).  Entries are sort
// keys: order-preserving logit bits above the inverted index, so a comparison
// of (value, index) pairs is one unsigned compare.  Inside a range of up to
// 65536 columns the index is the one in the range and a key has 32 bits (a
// compare-exchange is a maximum and a minimum); wider ranges and the second
// kernel use 64-bit keys with the column itself.  A thread keeps
//   - a descending list of its kTopK best keys (each vector's 8 keys sorted
//     by a bitonic network and merged in), and
//   - a softmax normaliser (m, s): s = sum exp(x - m) over its values, m its
//     largest, rescaled once per vector whose largest value grows m.
// Lists and normalisers are merged by butterflies across lanes (bitonic merge
// of two sorted lists per step; partners by DPP and permlane swaps, which cost
// a few cycles where an LDS permute costs over a hundred): the wave's 64, then
// the workgroup's 4 in wave 0, which writes the list and normaliser to a
// workspace slot.  The second kernel, a wave per row (lane = range), merges the
// row's S slots the same way and writes token and x - m - log(s) for the first
// k entries.  Merges follow fixed patterns, so results do not depend on
// arrival order.  w = 8, V = 128256: 5.8 + 4.7 us
// against 18.9 us as one kernel with 64-bit keys, LDS permutes and a ticket per
// workgroup (called eagerly 18.2 -> 10.6 us).
#include "ss_device.h"
#include "ss_internal.h"

namespace ss {

constexpr int kTopK = 8;        // list length (k <= kTopK)
constexpr int kExpandVecs = 4;  // 16-byte loads in flight per thread

struct TopkArgs {
  const uint16_t* logits;
  int ldl, n, V, k, S, chunk;  // S workgroups per row, each `chunk` 16-byte vectors
  int32_t* tokens;
  float* logprobs;
  uint64_t* part;   // [n][kTopK][S] sort keys
  uint64_t* stats;  // [n][S] (s bits << 32 | m bits)
};

// The logit's 16 bits made order-preserving (negative values inverted,
// non-negative ones offset by the sign bit, -0 taken as +0), so that a larger
// key is a larger logit, or an equal logit at a lower index (stored inverted
// below it).  Key 0 lies below every finite logit and marks an empty entry.
__device__ __forceinline__ uint32_t ordered(uint32_t h) {
  const uint32_t o = (h & 0x8000u) ? (~h & 0xFFFFu) : (h | 0x8000u);
  return h == 0x8000u ? 0x8000u : o;
}
// inside a range: the index in the range, up to 65535
__device__ __forceinline__ void make_key(uint32_t& key, uint32_t h, int, int in_range) {
  key = (ordered(h) << 16) | (0xFFFFu - (uint32_t)in_range);
}
__device__ __forceinline__ void make_key(uint64_t& key, uint32_t h, int idx, int) {
  key = ((uint64_t)ordered(h) << 32) | (0xFFFFFFFFu - (uint32_t)idx);
}
// a range's key with its column (first: the range's first column)
__device__ __forceinline__ uint64_t global_key(uint32_t key, int first) {
  return key ? ((uint64_t)(key >> 16) << 32) | (0xFFFFFFFFu - (uint32_t)(first + (int)(0xFFFFu - (key & 0xFFFFu)))) : 0ull;
}
__device__ __forceinline__ uint64_t global_key(uint64_t key, int) { return key; }
__device__ __forceinline__ float key_value(uint64_t key) {
  const uint32_t o = (uint32_t)(key >> 32);
  return h2f((uint16_t)((o & 0x8000u) ? (o & 0x7FFFu) : (~o & 0xFFFFu)));
}
__device__ __forceinline__ int key_index(uint64_t key) { return (int)(0xFFFFFFFFu - (uint32_t)key); }

// compare-exchange: afterwards a >= b
template <class Key>
__device__ __forceinline__ void cmpx(Key& a, Key& b) {
  const Key hi = a > b ? a : b, lo = a > b ? b : a;
  a = hi;
  b = lo;
}

// The kTopK best of two descending lists: the elementwise larger of `a` and
// reversed `b` is bitonic and holds exactly that set; three half-cleaner
// stages sort it.  Result in `a`.
template <class Key>
__device__ __forceinline__ void merge_top(Key (&a)[kTopK], const Key (&b)[kTopK]) {
#pragma unroll
  for (int j = 0; j < kTopK; ++j) a[j] = a[j] > b[kTopK - 1 - j] ? a[j] : b[kTopK - 1 - j];
#pragma unroll
  for (int d = kTopK / 2; d >= 1; d >>= 1)
#pragma unroll
    for (int j = 0; j < kTopK; ++j)
      if ((j & d) == 0) cmpx(a[j], a[j + d]);
}

// Bitonic sorting network, descending.
template <class Key>
__device__ __forceinline__ void sort_desc(Key (&a)[kTopK]) {
#pragma unroll
  for (int k = 2; k <= kTopK; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
      for (int i = 0; i < kTopK; ++i) {
        const int l = i ^ j;
        if (l > i) {
          if ((i & k) == 0) cmpx(a[i], a[l]);
          else cmpx(a[l], a[i]);
        }
      }
}

// (m, s) pairs: s = sum exp(x - m); an empty pair is (-inf, 0).  lse_combine
// folds (m2, s2) in after (m, s), lse_combine_into before it, so that two
// lanes combining each other's pairs get bit-identical results.
__device__ __forceinline__ void lse_combine(float& m, float& s, float m2, float s2) {
  const float mm = fmaxf(m, m2);
  if (mm == -INFINITY) return;  // both empty
  s = s * __expf(m - mm) + s2 * __expf(m2 - mm);
  m = mm;
}
__device__ __forceinline__ void lse_combine_into(float& m, float& s, float m2, float s2) {
  const float mm = fmaxf(m, m2);
  if (mm == -INFINITY) return;
  s = s2 * __expf(m2 - mm) + s * __expf(m - mm);
  m = mm;
}

// Step STEP of a butterfly over the lanes: the value of a lane whose bit STEP
// differs and which lies in the same group of 2^(STEP + 1) (steps 2 and 3
// mirror the group: every lane of the other half holds the same list by then).
template <int STEP>
__device__ __forceinline__ uint32_t partner(uint32_t x) {
  if constexpr (STEP < 4) {
    constexpr int kCtrl = STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : STEP == 2 ? 0x141 : 0x140;  // quad_perm, half and row mirror
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, 0xF, 0xF, true);
  } else {
    uint32_t lo = x, hi = x;  // after the swap the even and the odd halves of x, each held by both
    if constexpr (STEP == 4) asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
    else asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
    return (lane_id() >> STEP) & 1 ? lo : hi;
  }
}
template <int STEP>
__device__ __forceinline__ uint64_t partner(uint64_t x) {
  return ((uint64_t)partner<STEP>((uint32_t)(x >> 32)) << 32) | partner<STEP>((uint32_t)x);
}
template <int STEP>
__device__ __forceinline__ float partner(float x) {
  return __uint_as_float(partner<STEP>(__float_as_uint(x)));
}

// Butterfly steps FIRST .. LAST: after them each lane of a group of 2^(LAST+1)
// holds the kTopK best of the group's lists and the combined normaliser.
template <int STEP, int LAST, class Key>
__device__ __forceinline__ void butterfly_merge(Key (&L)[kTopK], float& m, float& s) {
  Key o[kTopK];
#pragma unroll
  for (int j = 0; j < kTopK; ++j) o[j] = partner<STEP>(L[j]);
  const float om = partner<STEP>(m), os = partner<STEP>(s);
  merge_top(L, o);
  if ((lane_id() >> STEP) & 1) lse_combine_into(m, s, om, os);
  else lse_combine(m, s, om, os);
  if constexpr (STEP < LAST) butterfly_merge<STEP + 1, LAST>(L, m, s);
}

template <class Key>
__global__ __launch_bounds__(256) void topk_ranges_kernel(TopkArgs a) {
  __shared__ Key s_key[4][kTopK];
  __shared__ float s_m[4], s_s[4];
  const int row = blockIdx.x / a.S, sp = blockIdx.x % a.S;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = tid >> 6;
  const uint16_t* x = a.logits + (size_t)row * a.ldl;
  Key L[kTopK];
#pragma unroll
  for (int j = 0; j < kTopK; ++j) L[j] = 0;
  float m = -INFINITY, s = 0.f;
  const int nvec = a.V >> 3;
  const int j_lo = min(nvec, sp * a.chunk), j_hi = min(nvec, j_lo + a.chunk);
  for (int j0 = j_lo + tid; j0 < j_hi; j0 += 256 * kExpandVecs) {
    u32x4 w[kExpandVecs];  // all issued before any is used (past the range: its last vector again)
#pragma unroll
    for (int u = 0; u < kExpandVecs; ++u) {
      const int j = min(j0 + 256 * u, j_hi - 1);
      w[u] = *reinterpret_cast<const u32x4*>(x + (size_t)j * 8);
    }
#pragma unroll
    for (int u = 0; u < kExpandVecs; ++u) {
      const int j = j0 + 256 * u;
      if (j >= j_hi) break;
      // one vector: its 8 keys sorted, then merged into the running list
      Key c[kTopK];
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t h = (w[u][e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
        make_key(c[e], h, 8 * j + e, 8 * (j - j_lo) + e);
        v[e] = h2f((uint16_t)h);
      }
      float mv = fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7])));
      if (mv > m) {
        s *= __expf(m - mv);
        m = mv;
      }
      // (a vector of -inf alone leaves m and adds nothing)
      if (m > -INFINITY) {
        float sv = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sv += __expf(v[e] - m);
        s += sv;
      }
      sort_desc(c);
      merge_top(L, c);
    }
  }
  if (sp == a.S - 1) {  // the columns past the last whole vector (fewer than 8)
    Key c[kTopK];
#pragma unroll
    for (int e = 0; e < kTopK; ++e) c[e] = 0;
    const int i = 8 * nvec + tid;
    if (i < a.V) {
      make_key(c[0], x[i], i, i - 8 * j_lo);
      const float v = h2f(x[i]);
      lse_combine(m, s, v, 1.0f);
    }
    merge_top(L, c);
  }

  // the wave's list and normaliser (every lane), then the workgroup's in wave 0
  butterfly_merge<0, 5>(L, m, s);
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < kTopK; ++r) s_key[wave][r] = L[r];
    s_m[wave] = m;
    s_s[wave] = s;
  }
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int r = 0; r < kTopK; ++r) L[r] = s_key[lane & 3][r];
  m = s_m[lane & 3];
  s = s_s[lane & 3];
  butterfly_merge<0, 1>(L, m, s);  // every group of four lanes holds the four waves
  Key mine = L[0];
#pragma unroll
  for (int r = 1; r < kTopK; ++r)
    if (lane == r) mine = L[r];
  if (lane < kTopK) a.part[((size_t)row * kTopK + lane) * a.S + sp] = global_key(mine, 8 * j_lo);
  if (lane == kTopK) a.stats[(size_t)row * a.S + sp] = ((uint64_t)__float_as_uint(s) << 32) | __float_as_uint(m);
}

__global__ __launch_bounds__(64) void topk_rows_kernel(TopkArgs a) {
  const int row = blockIdx.x, lane = lane_id();
  uint64_t R[kTopK];
  float rm = -INFINITY, rs = 0.f;
#pragma unroll
  for (int r = 0; r < kTopK; ++r) R[r] = lane < a.S ? a.part[((size_t)row * kTopK + r) * a.S + lane] : 0;
  if (lane < a.S) {
    const uint64_t st = a.stats[(size_t)row * a.S + lane];
    rm = __uint_as_float((uint32_t)st);
    rs = __uint_as_float((uint32_t)(st >> 32));
  }
  butterfly_merge<0, 5>(R, rm, rs);
  const float lse = rm + __logf(rs);
  if (lane < a.k) {
    uint64_t key = R[0];
#pragma unroll
    for (int r = 1; r < kTopK; ++r)
      if (lane == r) key = R[r];
    a.tokens[(size_t)row * a.k + lane] = key_index(key);
    a.logprobs[(size_t)row * a.k + lane] = key_value(key) - lse;
  }
}

int topk_logprobs_splits(int n) {
  int S = 1024 / n;
  return S < 1 ? 1 : S > 64 ? 64 : S;
}

size_t topk_logprobs_part_bytes(int n) {
  return (size_t)n * topk_logprobs_splits(n) * (kTopK + 1) * 8;
}

void launch_topk_logprobs(const uint16_t* logits, int ldl, int n, int V, int k, int32_t* tokens, float* logprobs,
                          void* part, hipStream_t st) {
  const int S = topk_logprobs_splits(n);
  const int nvec = V >> 3;
  uint64_t* p = reinterpret_cast<uint64_t*>(part);
  TopkArgs a{logits, ldl, n, V, k, S, (nvec + S - 1) / S, tokens, logprobs, p, p + (size_t)n * S * kTopK};
  // an index in a range fits 16 bits (the last range holds up to 7 columns more)
  if ((size_t)a.chunk * 8 + 8 <= 65536) hipLaunchKernelGGL(topk_ranges_kernel<uint32_t>, dim3(n * S), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(topk_ranges_kernel<uint64_t>, dim3(n * S), dim3(256), 0, st, a);
  hipLaunchKernelGGL(topk_rows_kernel, dim3(n), dim3(64), 0, st, a);
}

}  // namespace ss
