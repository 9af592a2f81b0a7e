// Dense fp16 LM head at small M for gfx950: logits[m][v] = fp16( xn[m] . W[v] ),
// xn = the final RMSNorm of the last hidden states (written by rmsnorm_kernel),
// W [V][H] fp16 row-major (the vocabulary projection of the 80-layer step).
//
// HBM-bound: the weight matrix (2.1 GB at V = 128256, H = 8192) is read once.
// Mapping (v_mfma_f32_16x16x32_f16, wave64): B operand = 16 vocabulary rows of
// W, A operand = 16 rows of xn.  A workgroup (4 waves x C tiles) owns 64 C
// vocabulary rows for the whole K: no split, no partials.  K advances in
// stages of 64, one 128-byte line of every row: weights and activations go
// straight into LDS with 16-byte loads (8 rows of 8 chunks per wave-wide load,
// so every memory request is a whole line), NS stages deep.  Chunk g of row r
// is stored at position g ^ (r / 2 mod 8), which makes the fragment reads (16
// rows, one chunk) hit every bank once.
//
// Rows lie 2 H bytes apart, for the usual H a multiple of the distance after
// which the memory channels repeat, so workgroups that all begin at k = 0 and
// advance together ask the same few channels for their lines.  Each workgroup
// therefore begins at a stage of its own (a hash of its index) and wraps
// around: V = 128256, H = 8192, 8 rows 446 -> 354 us, and nothing else in this
// kernel moved that time (deeper rings, more or fewer rows per workgroup).
// Measured (us, before -> now, and the rate): H 8192 at 64 rows 471 -> 366 (5.7
// TB/s), 32 rows 445 -> 353, 8 rows 443 -> 349 (6.0 TB/s, what a read-only
// kernel reaches); H 2048 at 8 rows 121 -> 93; V 8704, H 4736, 46 rows 53 -> 30.
#include "ss_device.h"
#include "ss_internal.h"

namespace ss {

constexpr int kLmWaves = 4;
constexpr int kLmK = 64;    // k of a stage: one 128-byte line per row

struct LmArgs {
  const uint16_t* xn;  // [M][H] fp16
  const uint16_t* W;   // [V][H] fp16
  uint16_t* logits;    // [M][ldl]
  int M, H, V, ldl;
};

// wait until at most `behind` stages (LPW loads each) of this wave remain in flight
template <int LPW, int K>
__device__ __forceinline__ void lm_wait(int behind) {
  if constexpr (K == 0) {
    vm_wait<0>();
  } else {
    if (behind >= K) vm_wait<LPW * K>();
    else lm_wait<LPW, K - 1>(behind);
  }
}

// kLong: rows of 64 MiB and more, 64 of which pass what a 32-bit buffer offset
// reaches: 64-bit addresses (rows past V or M repeat the last one).
template <int MT, int kLmCols, int NS, bool kLong>
__global__ __launch_bounds__(64 * kLmWaves) void lm_head_kernel(LmArgs a) {
  constexpr int kWBytes = kLmCols * 2048;                    // weights of a stage, per wave
  constexpr int kXBytes = MT * 2048;                         // activations of a stage
  constexpr int kStage = kXBytes + kLmWaves * kWBytes;
  constexpr int kXLoads = (MT * 2 + kLmWaves - 1) / kLmWaves;  // 1 KB loads per wave and stage
  constexpr int kLPW = kLmCols * 2 + kXLoads;
  __shared__ __attribute__((aligned(1024))) char smem[NS * kStage];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n16 = lane & 15, kq = lane >> 4;
  const int tile0 = blockIdx.x * (kLmWaves * kLmCols) + wave * kLmCols;
  const int ntiles = a.V >> 4;
  const int nst = a.H / kLmK;
  const uint32_t row_bytes = (uint32_t)a.H * 2u;
  const uint32_t lds0 = lds_address(smem);
  // this wave's rows of W; rows past V lie outside the buffer (zeros) and are
  // not stored
  const int first = min(tile0, ntiles - 1) * 16;
  const i32x4 rw = raw_rsrc(a.W + (size_t)first * a.H, (uint32_t)min(kLmCols * 16, a.V - first) * row_bytes);
  const i32x4 rx = raw_rsrc(a.xn, (uint32_t)a.M * row_bytes);
  // load l of a matrix: rows 8 l .. 8 l + 7, lane i takes row i / 8 and the
  // chunk that belongs at position i % 8 of it
  const int lr = lane >> 3, lp = lane & 7;
  uint32_t wv[kLmCols * 2], xv[kXLoads];
#pragma unroll
  for (int l = 0; l < kLmCols * 2; ++l) {
    const int row = 8 * l + lr;
    wv[l] = (uint32_t)row * row_bytes + (uint32_t)((lp ^ ((row >> 1) & 7)) * 16);
  }
#pragma unroll
  for (int j = 0; j < kXLoads; ++j) {
    const int l = (wave + kLmWaves * j) % (MT * 2);
    const int row = 8 * l + lr;
    // rows past M: row M - 1 again (their results are not stored)
    xv[j] = (uint32_t)min(row, a.M - 1) * row_bytes + (uint32_t)((lp ^ ((row >> 1) & 7)) * 16);
  }
  // the stage this workgroup begins at (multiplicative hash)
  const int rot = __builtin_amdgcn_readfirstlane((int)(((blockIdx.x * 2654435761u) >> 16) % (unsigned)nst));
  // LDS byte `at` of the ring from rows 8 l .. 8 l + 7 of m (n rows), k's from 64 k on
  auto load_long = [&](const uint16_t* m, int n, int l, int k, uint32_t at) {
    const int row = 8 * l + lr;
    const uint16_t* src = m + (size_t)min(row, n - 1) * a.H + (size_t)k * kLmK + (lp ^ ((row >> 1) & 7)) * 8;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(smem + at), 16, 0, 0);
  };
  auto issue = [&](int t) {
    const uint32_t slot = (uint32_t)((t % NS) * kStage), st = lds0 + slot;
    const int k = t + rot < nst ? t + rot : t + rot - nst;  // 64 k's from 64 k on
    const uint32_t off = (uint32_t)k * (kLmK * 2);
    if constexpr (kLong) {
#pragma unroll
      for (int l = 0; l < kLmCols * 2; ++l)
        load_long(a.W + (size_t)first * a.H, min(kLmCols * 16, a.V - first), l, k, slot + kXBytes + wave * kWBytes + l * 1024);
#pragma unroll
      for (int j = 0; j < kXLoads; ++j) {
        const int l = (wave + kLmWaves * j) % (MT * 2);
        load_long(a.xn, a.M, l, k, slot + l * 1024);
      }
      return;
    }
#pragma unroll
    for (int l = 0; l < kLmCols * 2; ++l) buffer_load_lds16(rw, wv[l], off, st + kXBytes + wave * kWBytes + l * 1024);
#pragma unroll
    for (int j = 0; j < kXLoads; ++j) buffer_load_lds16(rx, xv[j], off, st + ((wave + kLmWaves * j) % (MT * 2)) * 1024);
  };
  f32x4 acc[MT][kLmCols];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < kLmCols; ++ct) acc[mt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  // chunk g of row r lies at position g ^ ((r >> 1) & 7)
  uint32_t frag[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) frag[s] = (uint32_t)(n16 * 128 + (((4 * s + kq) ^ ((n16 >> 1) & 7)) * 16));
  auto compute = [&](int t) {
    const char* st = smem + (t % NS) * kStage;
    const char* sw = st + kXBytes + wave * kWBytes;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      half8 w[kLmCols];
#pragma unroll
      for (int ct = 0; ct < kLmCols; ++ct) w[ct] = *reinterpret_cast<const half8*>(sw + ct * 2048 + frag[s]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const half8 x = *reinterpret_cast<const half8*>(st + mt * 2048 + frag[s]);
#pragma unroll
        for (int ct = 0; ct < kLmCols; ++ct) acc[mt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, w[ct], acc[mt][ct], 0, 0, 0);
      }
    }
  };
#pragma unroll
  for (int j = 0; j < NS - 1; ++j)
    if (j < nst) issue(j);
  int t = 0;
  for (; t + NS - 1 < nst; ++t) {
    vm_wait<kLPW * (NS - 2)>();
    lds_barrier();
    issue(t + NS - 1);
    compute(t);
  }
  for (; t < nst; ++t) {
    lm_wait<kLPW, NS - 2>(nst - 1 - t);
    lds_barrier();
    compute(t);
  }

  // lane holds rows 4 kq + r of column n16 of each tile
#pragma unroll
  for (int ct = 0; ct < kLmCols; ++ct) {
    if (tile0 + ct >= ntiles) continue;
    const int col = (tile0 + ct) * 16 + n16;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = mt * 16 + kq * 4 + r;
        if (m < a.M) a.logits[(size_t)m * a.ldl + col] = f2h(acc[mt][ct][r]);
      }
  }
}

// kLmCols tiles per wave; NS stages: two workgroups per compute unit with one
// or two tiles, one with four (136 to 144 KB of LDS)
template <int C, bool kLong = false>
static void launch_cols(const LmArgs& a, hipStream_t st) {
  constexpr int kSmall = C == 1 ? 6 : 4, kLarge = C == 1 ? 4 : 3;
  const dim3 grid((a.V / 16 + kLmWaves * C - 1) / (kLmWaves * C)), wg(64 * kLmWaves);
  switch ((a.M + 15) / 16) {
    case 1: hipLaunchKernelGGL((lm_head_kernel<1, C, kSmall, kLong>), grid, wg, 0, st, a); break;
    case 2: hipLaunchKernelGGL((lm_head_kernel<2, C, kSmall, kLong>), grid, wg, 0, st, a); break;
    case 3: hipLaunchKernelGGL((lm_head_kernel<3, C, kLarge, kLong>), grid, wg, 0, st, a); break;
    default: hipLaunchKernelGGL((lm_head_kernel<4, C, kLarge, kLong>), grid, wg, 0, st, a); break;
  }
}

void launch_lm_head(const uint16_t* xn, int M, int H, const uint16_t* W, int V, uint16_t* logits, int ldl,
                    hipStream_t st) {
  const LmArgs a{xn, W, logits, M, H, V, ldl};
  // 256 rows per workgroup where those fill whole rounds of the compute units
  // (V 128256, 64 rows: 366 against 381 us with 128), 64 where 128 would leave
  // half of the units idle (V 8704: 30 against 41 us)
  const int n4 = (V + 255) / 256, rounds = (n4 + 255) / 256;
  if (H >= 1 << 25) launch_cols<1, true>(a, st);
  else if (V > 65536 && 10 * n4 >= 9 * 256 * rounds) launch_cols<4>(a, st);
  else if (V > 16384) launch_cols<2>(a, st);
  else launch_cols<1>(a, st);
}

}  // namespace ss
