// Greedy acceptance of a verified draft tree on the device, closing the
// verification step without a host round trip (target-side verification
// with the target's greedy choice: Sec. 3.1 and the Fig. 3 walk-through,
// where each iteration's output is the accepted root path followed by one
// token the target produced after it).
//
// Two kernels.  The first splits each logits row [V] fp16 into S contiguous
// ranges of 16-byte vectors, one 256-thread workgroup each (S = 1024 / T: about
// a thousand workgroups for any tree size; 8 loads in flight per thread).  A
// thread reduces each vector to its largest value by packed fp16 maxima, keeps
// the best vector over increasing indices and looks for the value's first place
// in it once at the end (comparing every value with the best pair so far made
// the kernel wait for the vector ALU: 7.7 -> 6.1 us); the wave and the
// workgroup combine pairs (larger value; on equal values the lower index), and
// the pair goes to a workspace slot.  The second, one workgroup, combines every
// row's S pairs (2^ceil(log2 S) lanes a row), which gives the first index of the
// row's largest value -- the target's choice after that node -- and then walks
// the tree in one wavefront (lane = node): from the root, the next node is the
// lowest-index child whose draft token equals the current node's choice (one
// ballot per step, at most T - 1 steps, each to a higher index), and the node
// where no child matches is accepted; its choice is the bonus token.
//
// The kernel boundary is what makes the pairs visible: one kernel whose last
// workgroup (tickets with acquire-release at agent scope) did the second part
// spent most of its time on the tickets' cache writebacks, one per workgroup.
// T = 64, V = 128256 (16.4 MB, from the Infinity Cache): 26.2 us as one kernel,
// 6.1 + 3.9 us as two.
#include <climits>

#include "ss_device.h"
#include "ss_internal.h"

namespace ss {

struct AcceptArgs {
  const uint16_t* logits;
  int ldl, T, V, S, chunk;  // S workgroups per row, each `chunk` 16-byte vectors
  const int32_t* tokens;
  const int32_t* parent;
  int32_t* argmax;
  int32_t* accepted;
  int32_t* bonus;
  int32_t* path_len;
  void* ws;
  uint64_t* part;  // [T][S] (index << 32 | value bits) per workgroup
  int lanes;       // lanes that combine a row in the second kernel: the power of two from S up
};

// (v, i) beats (bv, bi): larger value, or equal value at a lower index
__device__ __forceinline__ bool beats(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

constexpr int kAcceptVecs = 8;  // 16-byte loads in flight per thread

__global__ __launch_bounds__(256) void row_argmax_kernel(AcceptArgs a) {
  __shared__ float s_v[4];
  __shared__ int s_i[4];
  const int row = blockIdx.x / a.S, sp = blockIdx.x % a.S;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = tid >> 6;
  const uint16_t* x = a.logits + (size_t)row * a.ldl;
  // the best vector so far, its index and its largest value
  u32x4 bw = {0, 0, 0, 0};
  float bv = -INFINITY;
  int bj = INT_MAX;
  const int nvec = a.V >> 3;
  const int j_lo = min(nvec, sp * a.chunk), j_hi = min(nvec, j_lo + a.chunk);
  for (int j0 = j_lo + tid; j0 < j_hi; j0 += 256 * kAcceptVecs) {
    u32x4 w[kAcceptVecs];  // all issued before any is used (past the range: its last vector again)
#pragma unroll
    for (int u = 0; u < kAcceptVecs; ++u) {
      const int j = min(j0 + 256 * u, j_hi - 1);
      w[u] = *reinterpret_cast<const u32x4*>(x + (size_t)j * 8);
    }
#pragma unroll
    for (int u = 0; u < kAcceptVecs; ++u) {
      const int j = j0 + 256 * u;
      if (j >= j_hi) break;
      const half2v m0 = __builtin_elementwise_max(bitcast<half2v>(w[u][0]), bitcast<half2v>(w[u][1]));
      const half2v m1 = __builtin_elementwise_max(bitcast<half2v>(w[u][2]), bitcast<half2v>(w[u][3]));
      const half2v m2 = __builtin_elementwise_max(m0, m1);  // NaNs give way to numbers
      const float v = (float)__builtin_elementwise_max(m2[0], m2[1]);
      if (beats(v, j, bv, bj)) {
        bv = v;
        bj = j;
        bw = w[u];
      }
    }
  }
  int bi = a.V;
  if (bj != INT_MAX) {
#pragma unroll
    for (int e = 7; e >= 0; --e)
      if (h2f((uint16_t)(bw[e >> 1] >> (16 * (e & 1)))) == bv) bi = 8 * bj + e;
  }
  if (sp == a.S - 1) {  // the columns past the last whole vector
    for (int i = 8 * nvec + tid; i < a.V; i += 256) {
      const float v = h2f(x[i]);
      if (beats(v, i, bv, bi)) {
        bv = v;
        bi = i;
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float ov = __shfl_xor(bv, off, kWave);
    const int oi = __shfl_xor(bi, off, kWave);
    if (beats(ov, oi, bv, bi)) {
      bv = ov;
      bi = oi;
    }
  }
  if (lane == 0) {
    s_v[wave] = bv;
    s_i[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w)
      if (beats(s_v[w], s_i[w], bv, bi)) {
        bv = s_v[w];
        bi = s_i[w];
      }
    a.part[blockIdx.x] = ((uint64_t)(uint32_t)bi << 32) | __float_as_uint(bv);
  }
}

__global__ __launch_bounds__(1024) void greedy_accept_kernel(AcceptArgs a) {
  __shared__ int s_choice[64];
  const int tid = threadIdx.x;
  const int lane = lane_id();
  // the tree and its tokens, needed by wave 0 at the end, in flight first
  const bool in = tid < a.T;
  const int p = in ? a.parent[tid] : -1;
  const int tok = in ? a.tokens[tid] : 0;
  const int q = tid & (a.lanes - 1);
  for (int r0 = 0; r0 < a.T; r0 += 1024 / a.lanes) {
    const int row = r0 + tid / a.lanes;
    float cv = -INFINITY;
    int ci = a.V;
    if (row < a.T && q < a.S) {
      const uint64_t pq = a.part[(size_t)row * a.S + q];
      cv = __uint_as_float((uint32_t)pq);
      ci = (int)(pq >> 32);
    }
    for (int off = a.lanes >> 1; off >= 1; off >>= 1) {
      const float ov = __shfl_xor(cv, off, kWave);
      const int oi = __shfl_xor(ci, off, kWave);
      if (beats(ov, oi, cv, ci)) {
        cv = ov;
        ci = oi;
      }
    }
    if (row < a.T && q == 0) {
      const int c = ci < a.V ? ci : 0;  // a row of NaNs alone keeps the sentinel: report index 0
      a.argmax[row] = c;
      s_choice[row] = c;
    }
  }
  __syncthreads();
  if (tid >= kWave) return;

  // ---- one wavefront (lane = node): validate the tree and walk it ----
  const int choice = in ? s_choice[lane] : 0;
  const bool ok = !in || (lane == 0 ? p == -1 : (p >= 0 && p < lane));
  if (!__all(ok)) {
    if (lane == 0) report_error(a.ws, SWIFTSPEC_DEVERR_BAD_TREE);
    return;
  }
  int u = 0, L = 1;
  for (int step = 1; step < a.T; ++step) {  // each step moves to a higher index: at most T - 1
    const int want = __shfl(choice, u, kWave);
    const uint64_t cand = __ballot(in && lane > 0 && p == u && tok == want);
    if (cand == 0) break;
    u = (int)__builtin_ctzll(cand);
    ++L;
  }
  const int b = __shfl(choice, u, kWave);
  if (lane == 0) {
    *a.accepted = u;
    *a.bonus = b;
    if (a.path_len) *a.path_len = L;
  }
}

int greedy_accept_splits(int T) {
  int S = 1024 / T;
  return S < 1 ? 1 : S > 64 ? 64 : S;
}

void launch_greedy_accept(const uint16_t* logits, int ldl, int T, int V, const int32_t* tokens,
                          const int32_t* parent, int32_t* argmax, int32_t* accepted, int32_t* bonus,
                          int32_t* path_len, void* ws, void* part, hipStream_t st) {
  const int S = greedy_accept_splits(T);
  const int nvec = V >> 3;
  AcceptArgs a{logits, ldl, T, V, S, (nvec + S - 1) / S, tokens, parent, argmax, accepted, bonus, path_len, ws,
               reinterpret_cast<uint64_t*>(part), 1};
  while (a.lanes < S) a.lanes *= 2;
  hipLaunchKernelGGL(row_argmax_kernel, dim3(T * S), dim3(256), 0, st, a);
  hipLaunchKernelGGL(greedy_accept_kernel, dim3(1), dim3(1024), 0, st, a);
}

}  // namespace ss
