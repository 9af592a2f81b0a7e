// W4A16 GEMMs at small M (the tree size) for gfx950.
//
// y[m][n] = sum_k x[m][k] * W'[n][k],  W'[n][k] = (q[n][k] - z[n][g]) * s[n][g],
// g = k / 128: the int4 AWQ-style projections of a decoder layer (SwiftSpec
// Sec. 3.3 and Sec. 5.1), plain (+ residual) or as the fused SwiGLU whose
// gate and up tiles share the activation fragments (Sec. 3.3).
//
// Matrix-core mapping (v_mfma_f32_16x16x32_f16, wave64):
//   * A operand = activations in the "prepared" layout (ss_device.h), 16
//     token rows per M-tile; B operand = weights, 16 output columns per
//     N-tile.  Rows >= M are zero.
//   * Lane (n = lane % 16, kq = lane / 16) loads 16 bytes = k in
//     [128 g + 32 kq, +32) of weight row n: one wave-wide load covers one
//     16-column x 128-k block, i.e. exactly one (scale, zero) group.
//   * Dequantisation to exact integers with fp16 "magic numbers": OR-ing the
//     low nibble field into 0x6400 (1024, unit 1) gives 1024 + q, OR-ing the
//     high nibble field (bits 4-7) into 0x5400 (64, unit 1/16) gives 64 + q,
//     and one packed fp16 subtraction of 1024 + z (64 + z) leaves q - z
//     exactly.  Activations are used as given (any fp16 value), each MFMA
//     sum of a group is C_g = sum_k x (q - z), and the accumulator takes
//     s C_g (one mixed-precision FMA per output element, fp16 s read in
//     place).
// Three forms share that mapping; plan_w4a16_gemm picks one by M, K and N:
//   * K-split workgroups (few rows, or a matrix small enough that reading
//     the activations once per few columns costs little);
//   * wide blocks (17 rows and more over a large matrix);
//   * stream-K, for the shapes between: a fixed grid of workgroups (4 waves
//     each) splits the (N-block, group) iteration space into equal
//     contiguous ranges; the 4 waves split an N-block's columns.  Per group,
//     every wave loads 1 KB contiguous blocks of its own weight tiles and a
//     quarter of the group's activation fragments into a register ring (3
//     groups deep), issued together so that the in-order vmcnt queue never
//     holds a weight prefetch behind an older activation load; the
//     activations pass through a 3-slot LDS ring shared by the 4 waves, with
//     one fence-free barrier per group.  An N-block split between
//     workgroups is published as fp32 partials; a fix-up kernel on the same
//     stream sums them in workgroup order (results are deterministic) and
//     runs the epilogue.  Consecutive ranges are placed on the same XCD
//     (blockIdx % 8 selects the XCD under round-robin dispatch).
#include "ss_device.h"
#include "ss_internal.h"

namespace ss {

enum { EPI_PLAIN = 0, EPI_SWIGLU = 1 };

// Kernel-native copy of an int4 matrix (written by prepack_w4_kernel):
//   q : [N/16 tiles][G groups][64 lanes] x 16 bytes -- lane kq*16 + c holds
//       the packed nibbles of k in [128 g + 32 kq, +32) of row 16 t + c, in
//       the original byte order; one wave-wide load is 1 KB contiguous and a
//       tile's groups follow each other;
//   sz: [N/16][G][16] x u32 -- scale (fp16 bits) | zero << 16 of row 16 t + c.
struct W4Ptr {
  const u32x4* q;
  const uint32_t* sz;
};

struct GemmArgs {
  W4Ptr w0, w1;
  int K, N, G;
  const uint16_t* a;  // prepared activations [MT][G][4][64][8]
  int M;
  const uint16_t* x;      // normalised in the kernel: plain rows [M][ldx], RMSNorm weight gamma [K]
  int ldx;
  const uint16_t* gamma;
  float eps;
  uint16_t* y;        // plain output [M][ldy] (nullable)
  int ldy;
  uint16_t* yp;       // prepared output for a following GEMM with K = N (nullable)
  const uint16_t* res;
  int ldr;
  int nblocks, nwg;
  uint32_t units;  // N-blocks x groups; units x nwg < 2^30 (K N / 2 < 2^32)
  float* part;
};

// first unit of workgroup v's range (32-bit: units x nwg stays below 2^30
// because a packed matrix fits a 32-bit buffer range)
__device__ __forceinline__ int range_begin(uint32_t units, int v, int nwg) {
  return (int)((units * (uint32_t)v) / (uint32_t)nwg);
}

template <int MT, int NWV>
struct BStage {
  u32x4 b[NWV];
  uint32_t sz[NWV];
};

// Kernel shapes.  R = register-ring depth (groups whose loads are in flight
// or waiting to be used), OCC = waves per SIMD the register budget is cut
// for, NWG = workgroup cap.  Measured on the Llama-3-70B layer: three
// groups deep at two waves per SIMD everywhere (fewer, deeper-ringed
// workgroups were slower); the SwiGLU stream takes one
// workgroup per N-block when there are enough N-blocks to fill the chip (no
// split, so no partials and no fix-up kernel).
struct GemmShape {
  int ring, occ, nwg;
};
constexpr GemmShape gemm_shape(int MT, bool swiglu) {
  return MT > 2 ? GemmShape{3, 2, 512} : swiglu ? GemmShape{3, 2, 768} : GemmShape{3, 2, 512};
}
constexpr int kRingL = 3;  // LDS ring of activation fragments

// The four MFMA B operands of one 16-column x 128-k weight block as a lane
// holds it (16 bytes w: k in [128 g + 32 kq, +32) of column lane % 16; the
// block's scale|zero word sz), dequantised to exact q - z (see the magic
// numbers above the loop of w4a16_gemm_kernel): low nibbles of the first
// and second 16 k, then high nibbles.  magic_lo / magic_hi hold 0x64006400
// and 0x54005400 in registers.
struct BFrag {
  half8 lo_a, lo_b, hi_a, hi_b;
};
__device__ __forceinline__ BFrag dequant_block(u32x4 w, uint32_t sz, uint32_t magic_lo, uint32_t magic_hi) {
  auto deq = [&](uint32_t x, uint32_t m, uint32_t magic, half2v zz) {
    return bitcast<uint32_t>(bitcast<half2v>((x & m) | (magic & ~m)) - zz);
  };
  const uint32_t s0 = w[0] >> 8, s1 = w[1] >> 8, s2 = w[2] >> 8, s3 = w[3] >> 8;
  constexpr uint32_t kLo = 0x000F000Fu, kHi = 0x00F000F0u;
  const uint32_t z = (sz >> 16) & 0xFFu;
  const half2v zlo = bitcast<half2v>((0x6400u + z) * 0x00010001u);
  const half2v zhi = bitcast<half2v>((0x5400u + 16u * z) * 0x00010001u);
  auto dl = [&](uint32_t x) { return deq(x, kLo, magic_lo, zlo); };
  auto dh = [&](uint32_t x) { return deq(x, kHi, magic_hi, zhi); };
  BFrag f;
  f.lo_a = bitcast<half8>(u32x4{dl(w[0]), dl(s0), dl(w[1]), dl(s1)});
  f.lo_b = bitcast<half8>(u32x4{dl(w[2]), dl(s2), dl(w[3]), dl(s3)});
  f.hi_a = bitcast<half8>(u32x4{dh(w[0]), dh(s0), dh(w[1]), dh(s1)});
  f.hi_b = bitcast<half8>(u32x4{dh(w[2]), dh(s2), dh(w[3]), dh(s3)});
  return f;
}

// Output epilogue of one N-block from the accumulators of wave `wave`
// (kColW column tiles, for SwiGLU followed by the matching up tiles): lane
// holds rows 4 * (lane / 16) + r of column lane % 16 of each tile.  The
// residual is read first (load_residual) so that its loads can overlap
// other loads of the caller.
template <int MT, int NWV, int EPI>
struct Epilogue {
  static constexpr int kColW = (EPI == EPI_SWIGLU) ? NWV / 2 : NWV;
  static constexpr int kColB = 4 * kColW;
  float rv[MT][kColW][4];

  // rows m0 + 16 mt + ... (m0: first row of the caller's M-tiles)
  __device__ __forceinline__ void load_residual(const GemmArgs& a, int nb, int wave, int lane, int m0 = 0) {
    const int ncol = lane & 15, kq = lane >> 4;
    const int col0 = (nb * kColB + wave * kColW) * 16;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int ct = 0; ct < kColW; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) rv[mt][ct][r] = 0.f;
    if (EPI == EPI_PLAIN && a.res) {
      // rows >= M read row 0 and are discarded
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int ct = 0; ct < kColW; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = m0 + mt * 16 + kq * 4 + r;
            rv[mt][ct][r] = h2f(a.res[(size_t)(m < a.M ? m : 0) * a.ldr + col0 + ct * 16 + ncol]);
          }
    }
  }

  __device__ __forceinline__ void write(const GemmArgs& a, int nb, int wave, int lane,
                                        const f32x4 (&acc)[MT][NWV], int m0 = 0) const {
    const int ncol = lane & 15, kq = lane >> 4;
    const int col0 = (nb * kColB + wave * kColW) * 16;
    const int G2 = a.N >> 7;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int ct = 0; ct < kColW; ++ct) {
        const int ncl = col0 + ct * 16 + ncol;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + mt * 16 + kq * 4 + r;
          if (m < a.M) {
            float val;
            if (EPI == EPI_SWIGLU) {
              const float gte = acc[mt][ct][r], up = acc[mt][ct + kColW][r];
              val = gte / (1.0f + __expf(-gte)) * up;
            } else {
              val = acc[mt][ct][r] + rv[mt][ct][r];
            }
            const uint16_t h = f2h(val);
            if (a.y) a.y[(size_t)m * a.ldy + ncl] = h;
            if (a.yp) store_prepared(a.yp, m, ncl, G2, h);
          }
        }
      }
  }
};

// Partial-sum slots: workgroup v publishes the accumulators of its range's
// first (slot 0) and last (slot 1) N-block when another range shares them;
// per slot, wave w's MT x kColW x kSrc fragments of 64 lanes x f32x4.  Plain
// stores and loads: the fix-up runs in the next kernel on the stream.
template <int MT, int NWV, int EPI>
__device__ __forceinline__ float* part_slot(const GemmArgs& a, int v, int slot, int wave) {
  constexpr int kColW = (EPI == EPI_SWIGLU) ? NWV / 2 : NWV;
  constexpr int kSrc = (EPI == EPI_SWIGLU) ? 2 : 1;
  constexpr int kWaveSlotFloats = MT * kColW * kSrc * kWave * 4;
  return a.part + (((size_t)v * 2 + slot) * 4 + wave) * kWaveSlotFloats;
}

template <int MT, int NWV, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(gemm_shape(MT, EPI == EPI_SWIGLU).occ)))
void w4a16_gemm_kernel(GemmArgs a) {
  constexpr int kColW = (EPI == EPI_SWIGLU) ? NWV / 2 : NWV;  // output column tiles per wave
  constexpr int kColB = 4 * kColW;                            // output column tiles per block
  constexpr int kSrc = (EPI == EPI_SWIGLU) ? 2 : 1;
  constexpr int kRing = gemm_shape(MT, EPI == EPI_SWIGLU).ring;
  __shared__ u32x4 abuf[kRingL][MT][4][kWave];  // activation fragments of 3 groups

  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar addressing
  const int ncol = lane & 15;
  const int kq = lane >> 4;
  const int G = a.G;
  const int b = blockIdx.x;
  const int v = (a.nwg % 8 == 0) ? (b % 8) * (a.nwg / 8) + b / 8 : b;
  const int u_lo = range_begin(a.units, v, a.nwg), u_hi = range_begin(a.units, v + 1, a.nwg);
  const int total = u_hi - u_lo;
  if (total <= 0) return;

  // Load cursor: unit u = (N-block u / G, group u % G), advanced once per
  // load step and held at the range's last unit (loads past the end repeat
  // it, so every step issues the same operations).
  int ld_i = 0, ld_nb = u_lo / G, ld_g = u_lo - (u_lo / G) * G;
  auto advance = [&]() {
    if (ld_i < total - 1) {
      ++ld_i;
      if (++ld_g == G) {
        ld_g = 0;
        ++ld_nb;
      }
    }
  };
  // Operand loads go through buffer resources: the wave-uniform part of an
  // address is a scalar offset and the lane's part a constant vector offset,
  // so a load costs no vector ALU work.
  const uint32_t q_bytes = (uint32_t)((size_t)a.K * a.N / 2), sz_bytes = (uint32_t)((size_t)a.N * G * 4);
  const auto rq0 = buffer_rsrc(a.w0.q, q_bytes), rs0 = buffer_rsrc(a.w0.sz, sz_bytes);
  const auto rq1 = buffer_rsrc(EPI == EPI_SWIGLU ? a.w1.q : a.w0.q, q_bytes);
  const auto rs1 = buffer_rsrc(EPI == EPI_SWIGLU ? a.w1.sz : a.w0.sz, sz_bytes);
  const auto ra = buffer_rsrc(a.a, (uint32_t)(MT * G * 4 * kWave * 16));
  const uint32_t lane16 = (uint32_t)lane * 16u, col4 = (uint32_t)ncol * 4u;
  auto load_b = [&](BStage<MT, NWV>& st) {
    const int tw = ld_nb * kColB + wave * kColW;  // first column tile of this wave
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt) {
      const bool up = EPI == EPI_SWIGLU && nt >= kColW;
      const uint32_t tg = (uint32_t)((tw + nt % kColW) * G + ld_g);
      st.b[nt] = buffer_load_x4(up ? rq1 : rq0, lane16, tg * 1024u);
      st.sz[nt] = buffer_load_x1(up ? rs1 : rs0, col4, tg * 64u);
    }
  };
  // wave w stages fragment w of every M-tile of the cursor's group; with
  // one M-tile, lanes of rows at or past M load nothing (those rows are
  // zeros in the prepared layout; whatever the register holds reaches only
  // output rows that are not written)
  auto load_a = [&](u32x4 (&r)[MT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (MT > 1 || ncol < a.M) r[mt] = buffer_load_x4(ra, lane16, (uint32_t)(((mt * G + ld_g) * 4 + wave) * 1024));
  };
  auto store_a = [&](int slot, const u32x4 (&r)[MT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) abuf[slot][mt][wave][lane] = r[mt];
  };

  f32x4 acc[MT][NWV];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Dequantisation to exact small integers: (w & 0x000F000F) | 0x64006400
  // is the fp16 pair (1024 + q, 1024 + q'), (w & 0x00F000F0) | 0x54005400 is
  // (64 + q, 64 + q') (the nibble sits at the 1/16 ... 1/2 mantissa bits of
  // 64, i.e. at units 1 ... 8); subtracting 1024 + z (resp. 64 + z) leaves
  // q - z exactly.  The MFMA sum of a group is C_g = sum_k x (q - z) and the
  // accumulator takes s C_g.  The magic constants are kept in registers
  // (opaque to the optimiser) so that mask-and-insert is one v_bfi_b32 with
  // the mask in a scalar register.
  uint32_t magic_lo = 0x64006400u, magic_hi = 0x54005400u;
  asm volatile("" : "+v"(magic_lo), "+v"(magic_hi));
  auto read_a = [&](int slot, half8 (&af)[MT][4]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int f = 0; f < 4; ++f) af[mt][f] = bitcast<half8>(abuf[slot][mt][f][lane]);
  };
  // group sums C_g of one unit (and the tiles' scale words); applied to the
  // accumulators one step later, so that no instruction waits on the MFMAs
  // just issued
  auto mfma_unit = [&](const half8 (&af)[MT][4], const BStage<MT, NWV>& st, f32x4 (&c)[MT][NWV],
                       uint32_t (&sw)[NWV]) {
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt) {
      const BFrag bf = dequant_block(st.b[nt], st.sz[nt], magic_lo, magic_hi);
      sw[nt] = st.sz[nt];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f32x4 cc = {0.f, 0.f, 0.f, 0.f};
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[mt][0], bf.lo_a, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[mt][1], bf.lo_b, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[mt][2], bf.hi_a, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[mt][3], bf.hi_b, cc, 0, 0, 0);
        c[mt][nt] = cc;
      }
    }
  };
  auto apply = [&](const f32x4 (&c)[MT][NWV], const uint32_t (&sw)[NWV]) {
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[mt][nt][r] = __builtin_fmaf(c[mt][nt][r], (float)bitcast<half2v>(sw[nt])[0], acc[mt][nt][r]);
  };

  auto emit = [&](int nb) {
    Epilogue<MT, NWV, EPI> ep;
    ep.load_residual(a, nb, wave, lane);
    ep.write(a, nb, wave, lane, acc);
  };
  auto zero_acc = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NWV; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // End of an N-block's share inside the range: write the outputs if the
  // range holds the whole N-block, else publish the partial (slot 0: the
  // range's first N-block, slot 1: its last) for the fix-up kernel.
  auto flush = [&](int nb) {
    const bool full = (long)nb * G >= u_lo && (long)(nb + 1) * G <= u_hi;
    if (full) {
      emit(nb);
    } else {
      float* mine = part_slot<MT, NWV, EPI>(a, v, nb == u_lo / G ? 0 : 1, wave);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int ct = 0; ct < kColW; ++ct) {
          const int t = mt * kColW + ct;
          *reinterpret_cast<f32x4*>(mine + ((size_t)(t * kSrc) * kWave + lane) * 4) = acc[mt][ct];
          if (EPI == EPI_SWIGLU)
            *reinterpret_cast<f32x4*>(mine + ((size_t)(t * kSrc + 1) * kWave + lane) * 4) = acc[mt][ct + kColW];
        }
    }
    zero_acc();
  };


  // ---- one continuous pipeline over the range's units ----
  // Step i (R = ring depth): issue the activation and weight loads of unit
  // i + R - 1 into register slot (i + R - 1) % R, write unit i + 1's
  // activation fragments (loaded R - 2 steps earlier; the compiler waits
  // for exactly that load) to LDS slot (i + 1) % 3 (last read at step
  // i - 2), barrier, compute unit i (whose fragments were written at step
  // i - 1) and flush when unit i ends its N-block's share.  Loads past the range's
  // end repeat its last unit (L2 hits), so every step issues the same
  // operations and the compiler's waits stay exact; the loop runs whole
  // rounds of R steps.
  BStage<MT, NWV> bs[kRing];
  u32x4 ar[kRing][MT];
#pragma unroll
  for (int j = 0; j < kRing - 1; ++j) {
    load_a(ar[j]);
    load_b(bs[j]);
    advance();
  }
  store_a(0, ar[0]);

  // a step past the range's end still retires its register slot, so that no
  // load into a ring register is pending where the compiler reuses it
  auto consume = [&](const BStage<MT, NWV>& st, const u32x4 (&r)[MT]) {
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt) asm volatile("" : : "v"(st.b[nt]), "v"(st.sz[nt]));
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) asm volatile("" : : "v"(r[mt]));
  };
  // Up to 32 rows the fragments and group sums are double-buffered: at step i
  // the wave reads unit i + 1's fragments (its LDS slot is complete once the
  // barrier of step i has passed) and applies unit i - 1's sums.  Above 32
  // rows the second buffers would cost the second wave per SIMD, so step i
  // reads, multiplies and applies its own unit.
  constexpr bool kPipe = MT <= 2;
  constexpr int kBuf = kPipe ? 2 : 1;
  half8 af[kBuf][MT][4];
  f32x4 cs[kBuf][MT][NWV];
  uint32_t sc[kBuf][NWV];
#pragma unroll
  for (int q = 0; q < kBuf; ++q)
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt) {
      sc[q][nt] = 0u;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) cs[q][mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  lds_barrier();
  if constexpr (kPipe) read_a(0, af[0]);
  // compute cursor: N-block and group of unit i
  int c_nb = u_lo / G, c_g = u_lo - (u_lo / G) * G;
  for (int i0 = 0; i0 < total; i0 += 2 * kRing) {
#pragma unroll
    for (int J = 0; J < 2 * kRing; ++J) {
      const int i = i0 + J;
      const int R = J % kRing, bq = kPipe ? (J & 1) : 0;
      load_a(ar[(R + kRing - 1) % kRing]);
      load_b(bs[(R + kRing - 1) % kRing]);
      advance();
      if (i < total) {
        if (i + 1 < total) store_a((i + 1) % kRingL, ar[(R + 1) % kRing]);
        lds_barrier();
        if constexpr (kPipe) {
          if (i + 1 < total) read_a((i + 1) % kRingL, af[bq ^ 1]);
          mfma_unit(af[bq], bs[R], cs[bq], sc[bq]);
          apply(cs[bq ^ 1], sc[bq ^ 1]);
        } else {
          read_a(i % kRingL, af[0]);
          mfma_unit(af[0], bs[R], cs[0], sc[0]);
        }
        if (i == total - 1 || c_g == G - 1) {
          apply(cs[bq], sc[bq]);
#pragma unroll
          for (int nt = 0; nt < NWV; ++nt) sc[bq][nt] = 0u;
          flush(c_nb);
        } else if constexpr (!kPipe) {
          apply(cs[0], sc[0]);
        }
        if (++c_g == G) {
          c_g = 0;
          ++c_nb;
        }
      } else {
        consume(bs[R], ar[(R + 1) % kRing]);
      }
    }
  }
}

// Split N-blocks: one workgroup per M-tile of an N-block (grid MT times the
// N-blocks) sums that tile's partials of the block's contributing ranges in
// workgroup order (deterministic) and writes its 16 rows; N-blocks inside
// one range were written by the GEMM kernel.  (One workgroup for all M-tiles
// of a block was slower: at 32 rows 20.4 -> 19.1 us for the 70B QKV, 35.3
// -> 34.1 us for the down projection; at 64 rows 51.4 -> 48.6 us for the
// down projection, whose one-workgroup form needs 256 VGPRs.)
template <int MT, int NWV, int EPI>
__global__ __launch_bounds__(256) void w4a16_fixup_kernel(GemmArgs a) {
  constexpr int MS = 1;  // M-tiles per workgroup
  constexpr int kBatch = 8;
  constexpr int kColW = (EPI == EPI_SWIGLU) ? NWV / 2 : NWV;
  constexpr int kSrc = (EPI == EPI_SWIGLU) ? 2 : 1;
  // the GEMM orders its ranges XCD-major (workgroup b on XCD b % 8 takes
  // range (b % 8) nwg/8 + b / 8), so the blocks of XCD x are the x-th eighth
  // of all blocks: fix-up workgroup (b, M-tile group) takes one of those of
  // its own XCD (b % 8, the grid holding MT copies of the blocks),
  // whose partials that XCD's L2 wrote
  const int b = blockIdx.x % a.nblocks;
  const int mt0 = blockIdx.x / a.nblocks;  // this workgroup's M-tile
  const int nb = (a.nwg % 8 == 0 && a.nblocks % 8 == 0) ? (b % 8) * (a.nblocks / 8) + b / 8 : b;
  const uint32_t U = a.units, lo = (uint32_t)(nb * a.G), nwg = (uint32_t)a.nwg;
  const int c_first = (int)(((lo + 1) * nwg - 1) / U);
  const int c_last = (int)(((lo + (uint32_t)a.G) * nwg - 1) / U);
  if (c_first == c_last) return;
  // every contributor after the first begins its range inside this block
  // (slot 0, its first block); the first one holds it in slot 1 (its last
  // block) unless its range begins exactly at the block
  const int slot_first = range_begin(U, c_first, a.nwg) < (int)lo ? 1 : 0;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  Epilogue<MS, NWV, EPI> ep;
  ep.load_residual(a, nb, wave, lane, mt0 * 16);  // in flight with the first partial loads
  f32x4 acc[MS][NWV];
#pragma unroll
  for (int mt = 0; mt < MS; ++mt)
#pragma unroll
    for (int nt = 0; nt < NWV; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = c_first; c0 <= c_last; c0 += kBatch) {
    // kBatch contributors' loads in flight at once, summed in order
    f32x4 pa[kBatch][MS][kColW], pb[kBatch][MS][kColW];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int c = c0 + j <= c_last ? c0 + j : c_last;
      const float* src = part_slot<MT, NWV, EPI>(a, c, c == c_first ? slot_first : 0, wave);
#pragma unroll
      for (int mt = 0; mt < MS; ++mt)
#pragma unroll
        for (int ct = 0; ct < kColW; ++ct) {
          const int t = (mt0 + mt) * kColW + ct;
          pa[j][mt][ct] = *reinterpret_cast<const f32x4*>(src + ((size_t)(t * kSrc) * kWave + lane) * 4);
          if (EPI == EPI_SWIGLU) pb[j][mt][ct] = *reinterpret_cast<const f32x4*>(src + ((size_t)(t * kSrc + 1) * kWave + lane) * 4);
        }
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      if (c0 + j > c_last) break;
#pragma unroll
      for (int mt = 0; mt < MS; ++mt)
#pragma unroll
        for (int ct = 0; ct < kColW; ++ct) {
          acc[mt][ct] += pa[j][mt][ct];
          if (EPI == EPI_SWIGLU) acc[mt][ct + kColW] += pb[j][mt][ct];
        }
    }
  }
  ep.write(a, nb, wave, lane, acc, mt0 * 16);
}

// ------------------------------------------------------------ wide blocks
// Many rows over a large matrix.  One workgroup of 8 waves owns 16
// weight tiles (plain: 256 columns; a fused SwiGLU: the gate and up tiles of
// 128) over one of S equal K ranges, two tiles per wave, and a step is one
// 128-k group.  The activation fragments of a group are read from L2 once
// per 16 weight tiles (4 or 8 in the stream-K kernel) and shared through a
// 3-slot LDS ring.  What bounds it is each SIMD's own work: per group its two
// waves have 8 MT MFMAs each and the dequantisation of two blocks, and with
// one workgroup per compute unit nothing hides a wave that does one after the
// other.  (K 8192, N 28672 SwiGLU by counters, 64 / 32 rows: matrix cores busy
// 45 / 28 % of the cycles, the vector ALUs 55 / 53 %, one or the other 83 / 70
// %; LDS reads 51 / 32 % of its bandwidth, waits for it 5 / 2 % of the waves'
// cycles; the weight stream 53 / 70 % of the read rate.)  So a step
// interleaves them: the products of each M-tile
// stand beside the LDS reads of the next M-tile's fragments, the previous
// M-tile's group sums times their scales, and a share of the next group's
// dequantisation; no instruction waits for the MFMA just issued.  Loads are
// four (weights) and five (activations) groups ahead in registers.
// Every element sums its groups in the order of the stream-K kernel.
// With S > 1 the ranges' partial sums go to memory and the fix-up kernel
// adds them in range order (deterministic).
// Measured against the stream-K kernel (us, weights rotated through HBM; 32
// / 45 / 64 rows): SwiGLU K 8192, N 28672 59.0 -> 58.3, 74.6 -> 69.1, 94.2
// -> 83.8 (3.0 TB/s of weights at 64 rows); K 28672, N 8192 39.0 -> 36.2,
// 44.4 -> 42.0, 53.6 -> 48.0.  (At 32 rows the SwiGLU is within 1 % of it by
// itself and 2 us faster in the 70B layer.)
constexpr int kWideW = 8;     // waves of a workgroup
constexpr int kWideStep = 4;  // K ranges are multiples of this many groups (the register ring's length)

template <int MT, bool SW>
__global__ __launch_bounds__(64 * kWideW) __attribute__((amdgpu_waves_per_eu(2))) void w4a16_wide_kernel(GemmArgs a) {
  constexpr int W = kWideW, NT = 2, kC = SW ? 1 : 2;  // weight and output column tiles per wave
  constexpr int kF = MT * 4;                          // activation fragments of a group
  constexpr int kLA = (kF + W - 1) / W;               // staged per wave
  constexpr int kR = kWideStep, kL = 3;
  __shared__ u32x4 abuf[kL][kF][kWave];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ncol = lane & 15, kq = lane >> 4;
  const int G = a.G, ntiles = a.N >> 4, S = a.nwg / a.nblocks, NS = G / kR;
  const int b = blockIdx.x;
  const int v = (a.nwg % 8 == 0) ? (b % 8) * (a.nwg / 8) + b / 8 : b;
  const int nb = __builtin_amdgcn_readfirstlane(v / S), sp = v - nb * S;  // block and K range
  const int s_lo = __builtin_amdgcn_readfirstlane(sp * NS / S);
  const int g_lo = s_lo * kR, total = (__builtin_amdgcn_readfirstlane((sp + 1) * NS / S) - s_lo) * kR;
  const uint32_t q_bytes = (uint32_t)((size_t)a.K * a.N / 2), sz_bytes = (uint32_t)((size_t)a.N * G * 4);
  const auto rq0 = buffer_rsrc(a.w0.q, q_bytes), rs0 = buffer_rsrc(a.w0.sz, sz_bytes);
  const auto rq1 = buffer_rsrc(SW ? a.w1.q : a.w0.q, q_bytes), rs1 = buffer_rsrc(SW ? a.w1.sz : a.w0.sz, sz_bytes);
  const auto ra = buffer_rsrc(a.a, (uint32_t)(MT * G * 4 * kWave * 16));
  const uint32_t lane16 = (uint32_t)lane * 16u, col4 = (uint32_t)ncol * 4u;
  const int t0 = nb * (W * kC) + wave * kC;  // first output column tile of the wave
  // tiles past the matrix (N / 16 not a multiple of a block's) repeat the last one and are not written
  auto clampt = [&](int t) { return t < ntiles ? t : ntiles - 1; };
  const uint32_t tq0 = (uint32_t)(clampt(t0) * G), tq1 = SW ? tq0 : (uint32_t)(clampt(t0 + 1) * G);

  struct Raw {
    u32x4 b[NT];
    uint32_t sz[NT];
  };
  Raw raw[kR];
  u32x4 ar[kR][kLA];
  auto load_a = [&](u32x4 (&r)[kLA], int i) {
    const int g = g_lo + (i < total ? i : total - 1);
#pragma unroll
    for (int j = 0; j < kLA; ++j) {
      int f = wave + W * j;
      f = f < kF ? f : wave % kF;
      r[j] = buffer_load_x4(ra, lane16, (uint32_t)((((f >> 2) * G + g) * 4 + (f & 3)) * 1024));
    }
  };
  auto load_b = [&](Raw& r, int i) {
    const int g = g_lo + (i < total ? i : total - 1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const uint32_t tg = (nt ? tq1 : tq0) + (uint32_t)g;
      r.b[nt] = buffer_load_x4(SW && nt ? rq1 : rq0, lane16, tg * 1024u);
      r.sz[nt] = buffer_load_x1(SW && nt ? rs1 : rs0, col4, tg * 64u);
    }
  };
  auto store_a = [&](int slot, const u32x4 (&r)[kLA]) {
#pragma unroll
    for (int j = 0; j < kLA; ++j) {
      int f = wave + W * j;
      f = f < kF ? f : wave % kF;
      abuf[slot][f][lane] = r[j];
    }
  };
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t magic_lo = 0x64006400u, magic_hi = 0x54005400u;
  asm volatile("" : "+v"(magic_lo), "+v"(magic_hi));
  {
    // prologue: groups 0 .. 3 in flight; groups 0 and 1 staged
#pragma unroll
    for (int j = 0; j < kR; ++j) {
      load_a(ar[j], j);
      load_b(raw[j], j);
    }
    BFrag bf[2][NT];
    float sc[2][NT];
    half8 af[2][4];
    f32x4 cs[2][NT];
    float sprev[NT];  // the previous group's scales
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      cs[0][nt] = cs[1][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      sprev[nt] = 0.f;
    }
    store_a(0, ar[0]);
    store_a(1, ar[1]);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      bf[0][nt] = dequant_block(raw[0].b[nt], raw[0].sz[nt], magic_lo, magic_hi);
      sc[0][nt] = (float)bitcast<half2v>(raw[0].sz[nt])[0];
    }
    load_a(ar[0], 4);
    load_a(ar[1], 5);
    load_b(raw[0], 4);
    lds_barrier();
#pragma unroll
    for (int f = 0; f < 4; ++f) af[0][f] = bitcast<half8>(abuf[0][f][lane]);
    int sl = 0;  // LDS slot of group i
    for (int i0 = 0; i0 < total; i0 += kR) {
#pragma unroll
      for (int J = 0; J < kR; ++J) {
        const int i = i0 + J;
        const int P = J & 1;
        const int sl1 = sl == 2 ? 0 : sl + 1, sl2 = sl1 == 2 ? 0 : sl1 + 1;
        // group i + 2 to LDS (slot read last at step i - 1), its registers refilled with group i + 6
        store_a(sl2, ar[(J + 2) % kR]);
        load_a(ar[(J + 2) % kR], i + 6);
        const Raw& rn = raw[(J + 1) % kR];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int pm = (J * MT + mt) & 1;
          // fragments of the next M-tile (of the next group after the last)
#pragma unroll
          for (int f = 0; f < 4; ++f)
            af[pm ^ 1][f] = bitcast<half8>(mt + 1 < MT ? abuf[sl][(mt + 1) * 4 + f][lane] : abuf[sl1][f][lane]);
#pragma unroll
          for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              const half8 bb = f == 0 ? bf[P][nt].lo_a : f == 1 ? bf[P][nt].lo_b : f == 2 ? bf[P][nt].hi_a : bf[P][nt].hi_b;
              const f32x4 z = {0.f, 0.f, 0.f, 0.f};
              cs[pm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[pm][f], bb, f == 0 ? z : cs[pm][nt], 0, 0, 0);
            }
          // previous M-tile's sums
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float s = mt ? sc[P][nt] : sprev[nt];
              acc[mt ? mt - 1 : MT - 1][nt][q] = __builtin_fmaf(cs[pm ^ 1][nt][q], s, acc[mt ? mt - 1 : MT - 1][nt][q]);
            }
          // a share of the next group's dequantisation: half h of tile nt
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              if ((nt * 2 + h) * MT / (2 * NT) == mt) {
                const BFrag d = dequant_block(rn.b[nt], rn.sz[nt], magic_lo, magic_hi);
                if (h == 0) {
                  bf[P ^ 1][nt].lo_a = d.lo_a;
                  bf[P ^ 1][nt].lo_b = d.lo_b;
                } else {
                  bf[P ^ 1][nt].hi_a = d.hi_a;
                  bf[P ^ 1][nt].hi_b = d.hi_b;
                  sc[P ^ 1][nt] = (float)bitcast<half2v>(rn.sz[nt])[0];
                  asm("" : "+v"(sc[P ^ 1][nt]));
                }
              }
          if (mt == MT - 1) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) sprev[nt] = sc[P][nt];
          }
        }
        load_b(raw[(J + 1) % kR], i + 5);
        lds_barrier();
        sl = sl1;
      }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[MT - 1][nt][q] = __builtin_fmaf(cs[(kR * MT - 1) & 1][nt][q], sprev[nt], acc[MT - 1][nt][q]);
    // retire the loads past the end
#pragma unroll
    for (int j = 0; j < kR; ++j) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) asm volatile("" : : "v"(raw[j].b[nt]), "v"(raw[j].sz[nt]));
#pragma unroll
      for (int f = 0; f < kLA; ++f) asm volatile("" : : "v"(ar[j][f]));
    }
  }
  if (S == 1) {
    const int G2 = a.N >> 7;
#pragma unroll
    for (int c = 0; c < kC; ++c) {
      const int t = t0 + c;
      if (t < ntiles) {
        const int col = t * 16 + ncol;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = mt * 16 + 4 * kq + r;
            if (m < a.M) {
              float val;
              if constexpr (SW) {
                const float gte = acc[mt][0][r];
                val = gte / (1.0f + __expf(-gte)) * acc[mt][1][r];
              } else {
                val = acc[mt][c][r] + (a.res ? h2f(a.res[(size_t)m * a.ldr + col]) : 0.f);
              }
              const uint16_t h = f2h(val);
              if (a.y) a.y[(size_t)m * a.ldy + col] = h;
              if (a.yp) store_prepared(a.yp, m, col, G2, h);
            }
          }
      }
    }
  } else {
    float* mine = a.part + (((size_t)v * W + wave) * MT * NT * kWave + lane) * 4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        *reinterpret_cast<f32x4*>(mine + (size_t)(mt * NT + nt) * kWave * 4) = acc[mt][nt];
  }
}

// The K ranges' partial sums of wide blocks, one wave per (block, M-tile,
// wave of the block), eight ranges' loads in flight.
template <int MT, bool SW>
__global__ __launch_bounds__(256) void w4a16_wide_fixup_kernel(GemmArgs a) {
  constexpr int WB = kWideW, kBatch = 8, NT = 2, kC = SW ? 1 : 2;
  const int S = a.nwg / a.nblocks;
  const int x = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wave = x % WB, mt = (x / WB) % MT, nb = x / (WB * MT);
  const int lane = lane_id();
  const int ncol = lane & 15, kq = lane >> 4, ntiles = a.N >> 4;
  const int t0 = nb * WB * kC + wave * kC;
  float rv[kC][4];
#pragma unroll
  for (int c = 0; c < kC; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mt * 16 + 4 * kq + r, t = t0 + c;
      rv[c][r] = (!SW && a.res && m < a.M && t < ntiles) ? h2f(a.res[(size_t)m * a.ldr + t * 16 + ncol]) : 0.f;
    }
  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < S; c0 += kBatch) {
    f32x4 pa[kBatch][NT];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int c = min(c0 + j, S - 1);
      const float* src = a.part + ((((size_t)(nb * S + c) * WB + wave) * MT + mt) * NT * kWave + lane) * 4;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) pa[j][nt] = *reinterpret_cast<const f32x4*>(src + nt * kWave * 4);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      if (c0 + j >= S) break;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] += pa[j][nt];
    }
  }
  const int G2 = a.N >> 7;
#pragma unroll
  for (int c = 0; c < kC; ++c) {
    const int t = t0 + c;
    if (t < ntiles) {
      const int col = t * 16 + ncol;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = mt * 16 + 4 * kq + r;
        if (m < a.M) {
          float val;
          if constexpr (SW) {
            const float gte = acc[0][r];
            val = gte / (1.0f + __expf(-gte)) * acc[1][r];
          } else {
            val = acc[c][r] + rv[c][r];
          }
          const uint16_t h = f2h(val);
          if (a.y) a.y[(size_t)m * a.ldy + col] = h;
          if (a.yp) store_prepared(a.yp, m, col, G2, h);
        }
      }
    }
  }
}

// ------------------------------------------------------- K-split workgroups
// One workgroup owns kC 16-column output tiles (a fused SwiGLU: their gate
// and up tiles) over the whole K range; its W waves take contiguous group
// ranges.  A wave streams its weight blocks (one group ahead) and its
// activation fragments (the prepared layout's, straight into the MFMA A
// operand, each M-tile's registers reloaded for the next group as soon as
// its last product has read them) and nothing is shared until the W partial
// sums are added in wave order through LDS: no barrier in the loop, no
// partials in memory, no second kernel, results deterministic.
//
// What bounds it: every workgroup reads the whole activation matrix from L2
// (about 11 TB/s over the chip), i.e. 4 MT / NT times its weight bytes, so
// NT (weight tiles per workgroup) is the smallest that leaves about one
// workgroup per compute unit, and shapes with both many rows and a long K
// stay on the stream-K kernel, which shares the activations through LDS.
// Up to 16 rows the rest is fixed cost (launch, first loads, the sum).
// Measured against the kernels used before (us, weights rotated through
// HBM, the plain ones with a residual; 8 / 32 / 64 rows): K 4096, N 4096 6.5
// -> 5.4, 10.2 -> 7.2, 12.6 -> 10.2; K 8192, N 8192 16.0 -> 13.3, 22.6 ->
// 15.5, 25.9 -> 22.0; K 8192, N 10240 18.5 -> 16.7, 23.9 -> 19.8, 28.4 ->
// 27.8; K 2048, N 8192 7.0 -> 5.1, 10.1 -> 5.9, 12.3 -> 7.8; SwiGLU K 8192, N
// 7168 17.1 -> 16.6, 30.6 -> 21.3, 34.6 -> 27.8; SwiGLU K 4096, N 14336 18.4
// -> 17.2, 24.5 -> 22.0, 34.1 -> 31.2.

// The W waves' partial sums of a K-split workgroup (red, after the barrier)
// added in wave order, and the workgroup's MT x kC output tiles written,
// dealt to the waves.
template <int W, int MT, int NT, bool SW>
__device__ __forceinline__ void ksplit_write(const GemmArgs& a, const f32x4 (&red)[W][MT * NT][kWave], int t0, int wave,
                                             int lane) {
  constexpr int kC = SW ? NT / 2 : NT;
  constexpr int kU = MT * kC;
  constexpr int kUW = (kU + W - 1) / W;
  const int ncol = lane & 15, kq = lane >> 4;
  const int G2 = a.N >> 7;
#pragma unroll
  for (int j = 0; j < kUW; ++j) {
    const int u = wave + j * W;
    if (u >= kU) break;
    const int mt = u / kC, c = u % kC;
    f32x4 sum = red[0][mt * NT + c][lane], up = {0.f, 0.f, 0.f, 0.f};
    if (SW) up = red[0][mt * NT + c + kC][lane];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      sum += red[w][mt * NT + c][lane];
      if (SW) up += red[w][mt * NT + c + kC][lane];
    }
    const int col = (t0 + c) * 16 + ncol;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mt * 16 + 4 * kq + r;
      if (m < a.M) {
        float val;
        if constexpr (SW) {
          const float gte = sum[r];
          val = gte / (1.0f + __expf(-gte)) * up[r];
        } else {
          val = sum[r] + (a.res ? h2f(a.res[(size_t)m * a.ldr + col]) : 0.f);
        }
        const uint16_t h = f2h(val);
        if (a.y) a.y[(size_t)m * a.ldy + col] = h;
        if (a.yp) store_prepared(a.yp, m, col, G2, h);
      }
    }
  }
}
template <int W, int MT, int NT, bool SW>
__global__ __launch_bounds__(64 * W) void w4a16_ksplit_kernel(GemmArgs a) {
  constexpr int kC = SW ? NT / 2 : NT;  // output column tiles of the workgroup
  __shared__ f32x4 red[W][MT * NT][kWave];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ncol = lane & 15, kq = lane >> 4;
  const int G = a.G;
  const int t0 = blockIdx.x * kC;
  const int g0 = wave * G / W, n = (wave + 1) * G / W - g0;
  const uint32_t q_bytes = (uint32_t)((size_t)a.K * a.N / 2), sz_bytes = (uint32_t)((size_t)a.N * G * 4);
  const auto rq0 = buffer_rsrc(a.w0.q, q_bytes), rs0 = buffer_rsrc(a.w0.sz, sz_bytes);
  const auto rq1 = buffer_rsrc(SW ? a.w1.q : a.w0.q, q_bytes);
  const auto rs1 = buffer_rsrc(SW ? a.w1.sz : a.w0.sz, sz_bytes);
  const auto ra = buffer_rsrc(a.a, (uint32_t)(MT * G * 4 * kWave * 16));
  const uint32_t lane16 = (uint32_t)lane * 16u, col4 = (uint32_t)ncol * 4u;
  struct Stage {
    u32x4 b[NT];
    uint32_t sz[NT];
  };
  Stage ring[2];
  u32x4 x[MT][4];
  auto load_b = [&](Stage& st, int i) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const uint32_t tg = (uint32_t)((t0 + nt % kC) * G + g0 + i);
      st.b[nt] = buffer_load_x4(SW && nt >= kC ? rq1 : rq0, lane16, tg * 1024u);
      st.sz[nt] = buffer_load_x1(SW && nt >= kC ? rs1 : rs0, col4, tg * 64u);
    }
  };
  auto load_x = [&](int mt, int i) {
    if (MT > 1 || ncol < a.M) {
#pragma unroll
      for (int f = 0; f < 4; ++f) x[mt][f] = buffer_load_x4(ra, lane16, (uint32_t)(((mt * G + g0 + i) * 4 + f) * 1024));
    }
  };
  uint32_t magic_lo = 0x64006400u, magic_hi = 0x54005400u;
  asm volatile("" : "+v"(magic_lo), "+v"(magic_hi));
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  load_b(ring[0], 0);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) load_x(mt, 0);
  auto step = [&](const Stage& st, Stage& nx, int i) {
    const bool more = i + 1 < n;
    if (more) load_b(nx, i + 1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const BFrag bf = dequant_block(st.b[nt], st.sz[nt], magic_lo, magic_hi);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f32x4 cc = {0.f, 0.f, 0.f, 0.f};
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(x[mt][0]), bf.lo_a, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(x[mt][1]), bf.lo_b, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(x[mt][2]), bf.hi_a, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(x[mt][3]), bf.hi_b, cc, 0, 0, 0);
        if (nt == NT - 1 && more) load_x(mt, i + 1);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[mt][nt][r] = __builtin_fmaf(cc[r], (float)bitcast<half2v>(st.sz[nt])[0], acc[mt][nt][r]);
      }
    }
  };
  for (int i = 0; i < n; i += 2) {
    step(ring[0], ring[1], i);
    if (i + 1 < n) step(ring[1], ring[0], i + 1);
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) red[wave][mt * NT + nt][lane] = acc[mt][nt];
  __syncthreads();
  ksplit_write<W, MT, NT, SW>(a, red, t0, wave, lane);
}

// ------------------------------------------- small M, RMSNorm in the GEMM
// The QKV projection and the fused SwiGLU read the RMSNorm of the residual
// stream (the decoder layer of Sec. 2).  Where K-split workgroups give each
// wave at most NG = 2 or 4 groups (norm_in_ksplit), the workgroup (which reads
// all of K anyway) normalises the plain rows x itself: every wave issues all its
// loads up front (the row chunks of its groups, gamma, then the weight
// blocks, so that the row sums wait for the row chunks only), sums x^2
// over its groups, the waves' sums meet in LDS,
// and each lane forms its operand values exactly as the norm kernel does,
// fp16((x * inv) * gamma) in fp32, inv = 1 / sqrt(sum_k x^2 / K + eps), so
// the operand is rounded where the unfused chain rounds it.  Rows at or
// past M lie outside the buffer range of x and load as zeros, without a
// branch.  The rows of one load sit at one stride (often a multiple of
// 4 KB), and lanes reading the same 16-byte position of their rows collide
// in the vector cache (a row stride of 4 KB + 16 B was 0.8 us faster on the
// 1B-shaped QKV, one of 4 KB + 128 B no faster): load f of row r takes the
// 16-byte chunk f ^ (r & 3) and two rounds of bitwise lane selects put the
// chunks back in order.
template <int W, int NT, bool SW, int NG>
__global__ __launch_bounds__(64 * W) void w4a16_ksplit_norm_kernel(GemmArgs a) {
  constexpr int kC = SW ? NT / 2 : NT;  // output column tiles of the workgroup
  static_assert(NG <= 4, "gam holds 16 chunks of 4 groups");
  __shared__ f32x4 red[W][NT][kWave];
  __shared__ float red_ss[W][16];
  __shared__ u32x4 gam[W][kWave];
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ncol = lane & 15, kq = lane >> 4;
  const int t0 = blockIdx.x * kC;
  const int G = a.G;
  const int g0 = wave * G / W, n = (wave + 1) * G / W - g0;  // 1 .. NG: the plan keeps W <= G <= NG W
  const uint32_t q_bytes = (uint32_t)((size_t)a.K * a.N / 2), sz_bytes = (uint32_t)((size_t)a.N * G * 4);
  const auto rq0 = buffer_rsrc(a.w0.q, q_bytes), rs0 = buffer_rsrc(a.w0.sz, sz_bytes);
  const auto rq1 = buffer_rsrc(SW ? a.w1.q : a.w0.q, q_bytes);
  const auto rs1 = buffer_rsrc(SW ? a.w1.sz : a.w0.sz, sz_bytes);
  const auto rx = buffer_rsrc(a.x, (uint32_t)((size_t)a.M * a.ldx * 2));
  // gamma over this wave's groups only (chunk c = 16 j + 4 kq + f of group
  // g0 + j); chunks past them load as zeros
  const auto rgm = buffer_rsrc(a.gamma + g0 * 128, (uint32_t)(n * 256));
  const uint32_t lane16 = (uint32_t)lane * 16u, col4 = (uint32_t)ncol * 4u;
  // this lane's 32 values k = 128 g + 32 kq + t of row ncol, at g = 0
  const uint32_t xrow = ((uint32_t)ncol * (uint32_t)a.ldx + 32u * (uint32_t)kq) * 2u;
  const int xsw = ncol & 3;  // load f takes chunk f ^ xsw
  const uint32_t xm1 = 0u - (uint32_t)(xsw & 1), xm2 = 0u - (uint32_t)(xsw >> 1);

  // the row chunks first, then gamma, then the weights: the row sums wait
  // for the first loads only, while the weight blocks are still in flight
  u32x4 b[NG][NT], x[NG][4];
  uint32_t sz[NG][NT];
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    const int g = g0 + (j < n ? j : n - 1);  // past the range: repeat the last group, unused
#pragma unroll
    for (int f = 0; f < 4; ++f) x[j][f] = buffer_load_x4(rx, xrow + (uint32_t)((f ^ xsw) * 16), (uint32_t)(g * 256));
  }
  const u32x4 gv = buffer_load_x4(rgm, lane16, 0);
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    const int g = g0 + (j < n ? j : n - 1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const uint32_t tg = (uint32_t)((t0 + nt % kC) * G + g);
      b[j][nt] = buffer_load_x4(nt >= kC ? rq1 : rq0, lane16, tg * 1024u);
      sz[j][nt] = buffer_load_x1(nt >= kC ? rs1 : rs0, col4, tg * 64u);
    }
  }
  gam[wave][lane] = gv;

  // chunk c is in load c ^ xsw: bitwise selects under the masks xm1, xm2 (a
  // conditional operator here becomes an indexed copy through scratch
  // memory); then this wave's part of each row's sum of squares
  float ssq = 0.f;
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    u32x4 t1[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) t1[c][e] = (x[j][c ^ 1][e] & xm1) | (x[j][c][e] & ~xm1);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[j][c][e] = (t1[c ^ 2][e] & xm2) | (t1[c][e] & ~xm2);
    if (j < n) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const half2v v = bitcast<half2v>(x[j][c][e]);
          ssq = __builtin_amdgcn_fdot2(v, v, ssq, false);
        }
    }
  }
  ssq += __shfl_xor(ssq, 16, kWave);
  ssq += __shfl_xor(ssq, 32, kWave);
  if (kq == 0) red_ss[wave][ncol] = ssq;
  __syncthreads();
  float tot = red_ss[0][ncol];
#pragma unroll
  for (int w = 1; w < W; ++w) tot += red_ss[w][ncol];
  const float inv = 1.0f / sqrtf(tot / (float)a.K + a.eps);

  uint32_t magic_lo = 0x64006400u, magic_hi = 0x54005400u;
  asm volatile("" : "+v"(magic_lo), "+v"(magic_hi));
  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    if (j < n) {
      uint32_t w[16];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const u32x4 gm = gam[wave][16 * j + 4 * kq + c];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // (x * inv) * gamma, each product rounded to fp32, then to fp16:
          // fused multiply-adds of +0 are those products (up to the sign
          // of an exact zero) and take the fp16 operands directly
          const half2v v = bitcast<half2v>(x[j][c][e]), gg = bitcast<half2v>(gm[e]);
          half2v o;
          o[0] = (_Float16)__builtin_fmaf(__builtin_fmaf((float)v[0], inv, 0.f), (float)gg[0], 0.f);
          o[1] = (_Float16)__builtin_fmaf(__builtin_fmaf((float)v[1], inv, 0.f), (float)gg[1], 0.f);
          w[4 * c + e] = bitcast<uint32_t>(o);
        }
      }
      u32x4 xa[4];
      pack_prepared(w, xa);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const BFrag bf = dequant_block(b[j][nt], sz[j][nt], magic_lo, magic_hi);
        f32x4 cc = {0.f, 0.f, 0.f, 0.f};
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(xa[0]), bf.lo_a, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(xa[1]), bf.lo_b, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(xa[2]), bf.hi_a, cc, 0, 0, 0);
        cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(bitcast<half8>(xa[3]), bf.hi_b, cc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[nt][r] = __builtin_fmaf(cc[r], (float)bitcast<half2v>(sz[j][nt])[0], acc[nt][r]);
      }
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) red[wave][nt][lane] = acc[nt];
  __syncthreads();
  ksplit_write<W, 1, NT, SW>(a, red, t0, wave, lane);
}

// ------------------------------------------------------- activation prep
// x [M][ldx] fp16 -> prepared layout; one thread per (M-tile, group, lane).
__global__ __launch_bounds__(256) void prepare_activations_kernel(const uint16_t* __restrict__ x, int M,
                                                                  int ldx, int G, int MT,
                                                                  uint16_t* __restrict__ out) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= MT * G * kWave) return;
  const int lane = idx % kWave;
  const int g = (idx / kWave) % G;
  const int mt = idx / (kWave * G);
  const int m = mt * 16 + (lane & 15);
  const int kq = lane >> 4;
  uint32_t a[16];
  if (m < M) {
    const u32x4* src = reinterpret_cast<const u32x4*>(x + (size_t)m * ldx + g * 128 + kq * 32);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4 v = src[i];
      a[4 * i] = v[0];
      a[4 * i + 1] = v[1];
      a[4 * i + 2] = v[2];
      a[4 * i + 3] = v[3];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0u;
  }
  u32x4 f[4];
  pack_prepared(a, f);
  uint16_t* base = out + (((size_t)mt * G + g) * 4) * kWave * 8;
#pragma unroll
  for (int fi = 0; fi < 4; ++fi) *reinterpret_cast<u32x4*>(base + ((size_t)fi * kWave + lane) * 8) = f[fi];
}

void launch_prepare_activations(const uint16_t* x, int M, int ldx, int K, uint16_t* out, hipStream_t st) {
  const int G = K / 128, MT = (M + 15) / 16;
  const int threads = MT * G * kWave;
  hipLaunchKernelGGL(prepare_activations_kernel, dim3((threads + 255) / 256), dim3(256), 0, st, x, M, ldx, G,
                     MT, out);
}

// ------------------------------------------------------------- prepack
// Canonical int4 matrix -> kernel-native copy (see W4Ptr).  A pure
// rearrangement of the same bits; one wave per (tile, group).
__global__ __launch_bounds__(256) void prepack_w4_kernel(const uint8_t* __restrict__ q,
                                                         const uint16_t* __restrict__ s,
                                                         const uint8_t* __restrict__ z, int K, int N,
                                                         u32x4* __restrict__ qp, uint32_t* __restrict__ szp) {
  const int G = K >> 7;
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);  // (tile, group)
  if (item >= (long)(N >> 4) * G) return;
  const int t = (int)(item / G), g = (int)(item % G);
  const int lane = lane_id();
  const int n = t * 16 + (lane & 15), kq = lane >> 4;
  qp[item * kWave + lane] = *reinterpret_cast<const u32x4*>(q + (size_t)n * (K >> 1) + (size_t)g * 64 + kq * 16);
  if (lane < 16) {
    const size_t si = (size_t)n * G + g;
    szp[item * 16 + lane] = (uint32_t)s[si] | ((uint32_t)z[si] << 16);
  }
}

void launch_prepack_w4(const uint8_t* q, const uint16_t* s, const uint8_t* z, int K, int N, void* packed,
                       hipStream_t st) {
  const long items = (long)(N / 16) * (K / 128);
  u32x4* qp = reinterpret_cast<u32x4*>(packed);
  uint32_t* szp = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(packed) + (size_t)K * N / 2);
  hipLaunchKernelGGL(prepack_w4_kernel, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, st, q, s, z, K, N, qp,
                     szp);
}

// ----------------------------------------------------------------- launch

static GemmArgs gemm_args(const GemmLaunch& L) {
  GemmArgs a = {};
  auto unpack = [&](const void* p) {
    return W4Ptr{reinterpret_cast<const u32x4*>(p),
                 reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(p) + (size_t)L.K * L.N / 2)};
  };
  a.w0 = unpack(L.w0);
  a.w1 = unpack(L.w1);
  a.K = L.K;
  a.N = L.N;
  a.G = L.K / 128;
  a.a = L.aprep;
  a.M = L.M;
  a.y = L.y;
  a.ldy = L.ldy;
  a.yp = L.yprep;
  a.res = L.res;
  a.ldr = L.ldr;
  a.nblocks = L.nblocks;
  a.nwg = L.nwg;
  a.units = (uint32_t)(L.nblocks * a.G);
  a.part = L.part;
  a.x = L.xnorm;
  a.ldx = L.ldx;
  a.gamma = L.gamma;
  a.eps = L.eps;
  return a;
}

template <int MT, int NW, int EPI>
static void launch_t(const GemmLaunch& L, hipStream_t st) {
  const GemmArgs a = gemm_args(L);
  hipLaunchKernelGGL((w4a16_gemm_kernel<MT, NW, EPI>), dim3(L.nwg), dim3(256), 0, st, a);
  // ranges split no N-block when every workgroup gets whole N-blocks
  if (L.nblocks % L.nwg != 0)
    hipLaunchKernelGGL((w4a16_fixup_kernel<MT, NW, EPI>), dim3(L.nblocks * MT), dim3(256), 0, st, a);
}

// instantiated shapes: SwiGLU one gate + one up tile per wave, plain one or
// two tiles per wave
template <int MT, int EPI>
static void launch_nw(const GemmLaunch& L, hipStream_t st) {
  if constexpr (EPI == EPI_SWIGLU) {
    launch_t<MT, 2, EPI>(L, st);
  } else {
    if (L.nw == 2) launch_t<MT, 2, EPI>(L, st);
    else launch_t<MT, 1, EPI>(L, st);
  }
}

template <int EPI>
static void launch_mt(const GemmLaunch& L, hipStream_t st) {
  switch ((L.M + 15) / 16) {
    case 1: launch_nw<1, EPI>(L, st); break;
    case 2: launch_nw<2, EPI>(L, st); break;
    case 3: launch_nw<3, EPI>(L, st); break;
    default: launch_nw<4, EPI>(L, st); break;
  }
}

template <int MT, bool SW>
static void launch_wide(const GemmLaunch& L, hipStream_t st) {
  const GemmArgs a = gemm_args(L);
  hipLaunchKernelGGL((w4a16_wide_kernel<MT, SW>), dim3(L.nwg), dim3(64 * kWideW), 0, st, a);
  if (L.nwg > L.nblocks)
    hipLaunchKernelGGL((w4a16_wide_fixup_kernel<MT, SW>), dim3(L.nblocks * MT * kWideW / 4), dim3(256), 0, st, a);
}
template <bool SW>
static void launch_wide_mt(const GemmLaunch& L, hipStream_t st) {
  switch ((L.M + 15) / 16) {
    case 2: launch_wide<2, SW>(L, st); break;
    case 3: launch_wide<3, SW>(L, st); break;
    default: launch_wide<4, SW>(L, st); break;
  }
}

template <int W, int MT, int NT, bool SW>
static void launch_ks(const GemmLaunch& L, hipStream_t st) {
  hipLaunchKernelGGL((w4a16_ksplit_kernel<W, MT, NT, SW>), dim3(L.N / 16 / (SW ? NT / 2 : NT)), dim3(64 * W), 0, st,
                     gemm_args(L));
}
// MTX: the most M-tiles that the plan gives this form
template <int W, int NT, bool SW, int MTX>
static void launch_ks_mt(const GemmLaunch& L, hipStream_t st) {
  const int mt = (L.M + 15) / 16;
  if constexpr (MTX >= 4) {
    if (mt == 4) return launch_ks<W, 4, NT, SW>(L, st);
  }
  if constexpr (MTX >= 3) {
    if (mt == 3) return launch_ks<W, 3, NT, SW>(L, st);
    if (mt == 2) return launch_ks<W, 2, NT, SW>(L, st);
  }
  launch_ks<W, 1, NT, SW>(L, st);
}
template <int W, int NT, bool SW, int NG = 2>
static void launch_ksn(const GemmLaunch& L, hipStream_t st) {
  hipLaunchKernelGGL((w4a16_ksplit_norm_kernel<W, NT, SW, NG>), dim3(L.N / 16 / (SW ? NT / 2 : NT)), dim3(64 * W), 0, st,
                     gemm_args(L));
}

void launch_w4a16_gemm(const GemmLaunch& L, hipStream_t st) {
  if (L.wide) {
    L.swiglu ? launch_wide_mt<true>(L, st) : launch_wide_mt<false>(L, st);
    return;
  }
  if (L.ksw && L.xnorm) {
    if (L.swiglu) {
      if (L.ksw == 8) launch_ksn<8, 4, true>(L, st);
      else if (L.K <= 1024) L.knt == 2 ? launch_ksn<4, 2, true>(L, st) : launch_ksn<4, 4, true>(L, st);
      else L.knt == 2 ? launch_ksn<4, 2, true, 4>(L, st) : launch_ksn<4, 4, true, 4>(L, st);
    } else if (L.K > 2048) {
      launch_ksn<8, 1, false, 4>(L, st);
    } else if (L.ksw == 8) {
      L.knt == 1 ? launch_ksn<8, 1, false>(L, st) : L.knt == 2 ? launch_ksn<8, 2, false>(L, st) : launch_ksn<8, 4, false>(L, st);
    } else {
      L.knt == 1 ? launch_ksn<4, 1, false>(L, st) : L.knt == 2 ? launch_ksn<4, 2, false>(L, st) : launch_ksn<4, 4, false>(L, st);
    }
    return;
  }
  if (L.ksw) {
    if (L.swiglu) {
      if (L.ksw == 4) launch_ks_mt<4, 4, true, 3>(L, st);
      else if (L.knt == 2) launch_ks_mt<8, 2, true, 4>(L, st);
      else launch_ks_mt<8, 4, true, 4>(L, st);
    } else if (L.ksw == 16) {
      L.knt == 1 ? launch_ks_mt<16, 1, false, 1>(L, st) : launch_ks_mt<16, 2, false, 1>(L, st);
    } else {
      if (L.knt == 1) launch_ks_mt<8, 1, false, 4>(L, st);
      else if (L.knt == 2) launch_ks_mt<8, 2, false, 4>(L, st);
      else launch_ks_mt<8, 4, false, 4>(L, st);
    }
    return;
  }
  if (L.swiglu) launch_mt<EPI_SWIGLU>(L, st);
  else launch_mt<EPI_PLAIN>(L, st);
}

// The longest K that one-tile K-split workgroups take above 16 rows.  nb: the
// stream-K form's column blocks.  Where nb is a multiple of 8 that form keeps
// a block's ranges and their fix-up on one XCD and wins from a shorter K on
// (40 rows, time of the K split over its: N 1024, nb 16, K 8192 1.01, K 10240
// 1.19; N 1280, nb 20, K 10240 0.85, K 14336 1.10).  Above 32 rows it cuts few
// blocks into slivers, and from K 16384 on it has half as many, of two tiles
// per wave (N 1024, nb 8: K 16384 0.81, K 20480 0.87).
static int ksplit_longest(int MT, int K, int tiles) {
  const int nb = K >= 16384 && tiles % 8 == 0 ? tiles / 8 : tiles / 4;
  if (tiles >= 224) return 24576 / MT;
  if (K >= 16384) return MT == 2 ? 0 : nb <= 6 ? K : nb <= 10 ? 20480 : nb <= 12 ? 16384 : 0;
  if (nb % 8 == 0) return (MT > 2 && nb == 8 ? 12288 : 10240) - 1024 * MT;
  return MT > 2 && nb <= 12 ? 14336 : 10240;
}

// K-split plan (ksw waves, knt weight tiles per workgroup) of a shape, or
// ksw = 0 for the stream-K kernel.  The lines come from both forms timed on
// 5000 shapes (N 256 .. 49152, K 1024 .. 28672, 1 to 62 rows, the plain ones
// with and without a residual, which favours stream-K by up to a tenth), the
// weights rotated through more memory than the Infinity Cache holds, as those
// of a model are; "times as fast" and ratios beside them are of that.  Weights
// read again from the Infinity Cache favour the K split by a further tenth to
// a fifth.
static void plan_ksplit(int MT, int M, int K, int tiles, bool swiglu, GemmPlan& p) {
  const int G = K / 128;
  if (swiglu) {
    // more column tiles: the stream-K form's shared activations win (N 28672:
    // 60 against 64 us at 32 rows), but not at up to 8 rows over a short K (1
    // row, N 17664: K 1536 0.79, K 3072 0.80, K 4096 0.82 of stream-K's time;
    // N 24576 0.95, 0.90, 0.93; N 28672 1.04, 0.98, 1.01)
    if (tiles > 1088 && (M > 8 || tiles > 1536 || K > 4096)) return;
    // few column tiles on a long K, as for the plain form below (K 27264, N
    // 1088, 59 rows 56.1 -> 33.0 us with stream-K; K 12288, N 2048 1.05 and
    // 1.12 times as fast at 40 and 60 rows; K 28672, N 5120 1.10 at 2 and 14
    // rows, K 20480 1.06 at 16)
    if (tiles < 448) {
      if (MT >= 3 && tiles > 16 && K > (tiles <= 32 ? 16384 : 10240)) return;
      if (K > 20480 && tiles > (M > 8 ? 48 : 256)) return;
    }
    // more than one workgroup per compute unit in two rounds that are not
    // full (17 to 32 rows, N 17408: K 6144 1.07, K 12288 1.05; 60 rows, K
    // 4096, N 9600 1.10)
    if (MT == 2 && tiles > 1024) return;
    if (MT == 4 && tiles > 512 && tiles < 832 && K > 3584) return;
    // above 32 rows at more than one workgroup per compute unit only for a
    // short K (K 5888, N 10816, 64 rows: 34.5 against 36.4 us, weights from the
    // Infinity Cache; from HBM K 6144 .. 20480, N 9216 1.1 .. 1.4 of stream-K)
    if (tiles > 512 && MT >= 3 && (K > 4096 || tiles > 1024)) return;
    // gate + up of one column tile up to one workgroup per compute unit, and
    // where the activations are short or few (weights from the Infinity Cache:
    // N 8640, K 3072, 4 rows: 10.2 against 11.7 us; 29 rows 14.6 against 14.9;
    // N 7808, K 4608, 1 and 8 rows: 12.2 and 12.7 against 12.8 and 13.2)
    p.knt = tiles <= 256 || (MT == 1 && K <= 2560) || (M <= 8 && (tiles > 512 || K <= 5120)) ? 2 : 4;
    // with about two workgroups per compute unit four waves each (K 4096, N
    // 14336, 16 rows: 15.7 against 17.7 us with eight, weights from the
    // Infinity Cache)
    p.ksw = p.knt == 4 && tiles > 512 && MT <= 3 ? 4 : 8;
    return;
  }
  const int wg4 = (tiles + 3) / 4, rounds = (wg4 + 255) / 256;
  if (tiles <= 256) {
    // one tile.  Above 16 rows few workgroups on a long K stream too little
    // at once, and the activation read of MT * K * 32 bytes per workgroup
    // grows: stream-K from there on (K 20992, N 1472, 36 rows 32.1 -> 20.3
    // us; K 8192, N 1536, 60 rows 1.16 times as fast)
    if (MT > 1 && K > ksplit_longest(MT, K, tiles)) return;
    p.knt = 1;
  } else if (tiles <= 512) {
    // N 8192, K 28672, 32 rows: 39.4 us with stream-K, 43.5 with the K split
    // (weights from the Infinity Cache); above 32 rows N 4608, K 10240 1.12
    // times as fast with stream-K
    if (MT > 1 && MT * K > 32768) return;
    // fewer columns a shorter K (24 rows, N 4352, K 12288 1.08)
    if (MT > 1 && tiles < 384 && K > (MT == 2 ? 10240 : 8192)) return;
    // up to 16 rows K 28672, N 4352 .. 7168 1.05 .. 1.10, K 20480 1.0
    if (K > 24576) return;
    p.knt = 2;
  } else if (tiles <= 1024) {
    // above 32 rows fewer than 192 workgroups do not pay on a long K (N
    // 11904, K 16896, 45 rows: 40.1 against 44.7 us; N 14144, K 25472: 75.3
    // against 64.8; weights from the Infinity Cache)
    // and fewer than 160 not on a shorter one (N 8448, K 8192 1.10 times as
    // fast with stream-K, K 6144 0.98)
    if (MT >= 3 && K > (tiles < 640 ? 6144 : 8192) && tiles < 768) return;
    // nor any number from 17 rows on a longer one (N 9216, K 16384, 24 rows
    // 1.12 times as fast with stream-K; N 12544, K 19456, 22 rows: 45.1
    // against 42.3 us, weights from the Infinity Cache)
    if (MT >= 2 && K > (tiles < 768 ? 14336 : 16384)) return;
    // nor up to 16 rows (16 rows: N 8448, K 14336 1.07 times as fast; N 12288,
    // K 20480 1.10; N 14336, K 28672 1.0)
    if (MT == 1 && K > (tiles < 704 ? 12288 : 16384) && tiles < 896) return;
    p.knt = K <= 2048 && MT <= 2 ? 2 : 4;
  } else {
    // beyond 256 workgroups only where they fill whole rounds of the chip (N
    // 28992, K 27008, 4 rows: 0.76 of stream-K's time; N 19328, K 24960:
    // 58 -> 66 us, weights from the Infinity Cache), or for a short K
    if (20 * wg4 < 17 * 256 * rounds && K > 2048 && !(MT == 1 && K <= 8192)) return;
    // not where K is a multiple of 8192, so that every tile begins at a
    // multiple of 64 KB (4 rows, K 8192: N 16640 1.29 and N 35200 1.19 times
    // as fast with stream-K; but N 28992, where stream-K has one tile per
    // wave, 0.85), nor from 17 rows on for N a multiple of 32768 (46
    // rows: K 2048 1.22, K 4096 1.16, K 7168 1.0)
    if (MT == 1 && K % 8192 == 0 && (tiles % 8 == 0 || tiles < 1600)) return;
    if (MT >= 2 && tiles % 2048 == 0) return;
    // nor from 17 rows on a very long K (K 27008, N 32768, 24 rows: 1.18; N 28992 0.92)
    if (MT >= 2 && K > 16384 && tiles % 8 == 0) return;
    p.knt = K <= 2048 && MT <= 2 ? 2 : 4;
  }
  // 16 waves where one M-tile leaves the registers and K the groups (K 14336,
  // N 4096, 8 rows: 10.9 against 14.0 us with 8, weights from the Infinity Cache)
  p.ksw = MT == 1 && G >= 32 && p.knt <= 2 ? 16 : 8;
}

// Wide blocks (p.wide): where the matrix is large enough that a workgroup per
// compute unit and K range has a long run of groups.  Lines from sweeps over 18
// SwiGLU and 26 plain shapes (K 1536 .. 28672, N 2112 .. 32384) at 29, 45 and
// 64 rows against the other two forms, weights from the Infinity Cache unless
// said otherwise; above 32 rows 350 shapes that they choose wide blocks for
// took 0.69 to 1.06 of stream-K's time with weights from HBM, one more than
// 1.03 (K 16384, N 6144).  S is the number of K ranges that fills one round of
// the 256 compute units (two rounds were slower at every shape: K 8192, N
// 26752, 64 rows 76 us at S = 1, 85 at 2), and shapes whose round would stay
// under 200 workgroups (144 with S = 1, which needs no partials) keep the
// other forms.
static void plan_wide(int MT, int K, int tiles, bool swiglu, GemmPlan& p) {
  if (MT < 2 || tiles < 1 || K % (128 * kWideStep)) return;
  const int nb = (tiles + (swiglu ? 8 : 16) - 1) / (swiglu ? 8 : 16);
  const int ranges = K / (128 * kWideStep), fill = 256 / nb;
  const int S = fill < ranges ? fill : ranges;
  if (S < 1 || nb * S < (S == 1 ? 144 : 200)) return;
  const double kn = 16.0 * tiles * K;
  if (swiglu) {
    // more column tiles than the K-split form takes: any K (K 1536, N 19776,
    // 45 rows 16.6 -> 16.1 us; K 4608, N 19136, 64 rows 45.2 -> 39.3); below
    // that, above 32 rows, a K long enough for two or three ranges (K 6144, N
    // 16256, 64 rows 44.2 -> 38.7; K 4608, N 13568 32.7 -> 31.1; K 3584, N
    // 14208 27.8 -> 28.3)
    if (tiles <= 1088 && (tiles <= 512 || MT < 3 || K < 4608)) return;
    // up to 32 rows only a long K (weights from HBM: K 1536 1.02 .. 1.06 of
    // stream-K's time, K 3072 0.98 .. 1.04, K 4608 .. 7168 0.9 .. 1.0, K 8192
    // 0.88 .. 0.98; from the Infinity Cache 1.04 .. 1.1 at any K: K 8192, N
    // 28672, 32 rows 57.9 -> 55.8 and 47.1 -> 51.5 us)
    if (MT == 2 && K < 8192) return;
  } else {
    // above 32 rows K 8192, N 21184 39.7 -> 36.7 us (45 rows); K 20480, N
    // 5952 36.3 -> 34.8 (64); K 28672, N 8192 54.8 -> 51.0 (64); not K 8192, N
    // 10240 (27.7 -> 27.4) or K 14336, N 4096 (25.3 -> 26.2) (weights from the
    // Infinity Cache).  Up to 32 rows, weights from HBM, where the K split
    // stops and the columns suffice: K 28672, N 8192, 32 rows 39.9 -> 36.1 us
    // (from the Infinity Cache 31.3 -> 32.8), K 18432, N 10240 0.83 of
    // stream-K's time (1.01), K 20480, N 6144 0.94 (0.98), K 20480, N 4608
    // 0.95 .. 1.0 (0.96 .. 1.04); K 16384, N 6144 1.04 (1.08)
    if (MT == 2 && tiles <= 1024 && (K < 16384 || tiles < (K >= 20480 ? 384 : 544))) return;
    // and only over two or more K ranges, as one leaves up to 112 units
    // idle (K 12288, 24 rows: N 36864 1.16, N 49152 1.15 times as fast with
    // stream-K, weights from HBM)
    if (MT == 2 && S < 2) return;
    if (K < 8192 || tiles <= 256 || kn < (K >= 16384 ? 1.0e8 : 1.4e8)) return;
  }
  p.wide = true;
  p.ksw = 0;
  p.nblocks = nb;
  p.nwg = nb * S;
  p.part_bytes = S > 1 ? (size_t)p.nwg * kWideW * MT * 2 * kWave * 16 : 0;
}

// The RMSNorm runs inside a K-split GEMM where a workgroup holds all of K in
// registers (1024 <= K <= 2048, one M-tile): every workgroup normalises all
// of K for itself, so it pays while that is short (K 2048, N 3072, 8 rows:
// 5.4 us against 6.6 with the norm kernel), and up to K 4096 for few rows and
// a column of one tile (K 3584, N 3712, 2 rows 7.6 against 8.3; 13 rows within
// 0.05 of it, N >= 10240 slower).  A SwiGLU has four waves of up
// to four groups where a workgroup's column is one tile or K at most 1536
// (8 rows, weights from HBM: K 1280, N 2048 1.09 times as fast as eight waves
// of two groups, N 8192 1.07; K 2048, N 8192 0.97), and one tile up to one
// workgroup per compute unit or where two would leave a second round nearly
// empty (N 10240: K 1280 1.17, K 2048 1.04 times as fast).
bool norm_in_ksplit(GemmPlan& p, int M, int K, int N, bool swiglu) {
  const int G = K / 128, tiles = N / 16;
  const int longest = !swiglu && tiles <= 256 && M <= 8 ? 32 : 16;
  if (!p.ksw || M > 16 || G < 8 || G > longest) return false;
  if (swiglu) {
    p.knt = tiles <= 256 || (tiles > 512 && tiles <= 832) ? 2 : 4;
    p.ksw = p.knt == 2 || G <= 12 ? 4 : 8;
  } else {
    p.knt = tiles <= 256 ? 1 : tiles <= 512 ? 2 : 4;
    p.ksw = G <= 8 ? 4 : 8;
  }
  return true;
}

GemmPlan plan_w4a16_gemm(int M, int K, int N, bool swiglu) {
  // nw = 16-column source tiles per wave (SwiGLU: half gate, half up); a
  // block (one workgroup's N-range) holds 4 waves' tiles
  GemmPlan p;
  const int tiles = N / 16;
  const int MT = (M + 15) / 16;
  plan_ksplit(MT, M, K, tiles, swiglu, p);
  if (swiglu) {
    p.nw = 2;  // one gate and one up tile per wave
    p.nblocks = tiles / 4;
  } else {
    // two tiles per wave halve the LDS fragment reads per weight byte: up
    // to 32 rows where that still leaves at least 64 blocks and K is long
    // (the 70B projections; at the 8B widths, 48 and 32 blocks, one tile per
    // wave is 10-26 % faster, and at K = 2048 15 %), above 32 rows where K
    // is long enough to keep the split-K partials small
    p.nw = (((MT <= 2 && tiles / 8 >= 64 && K >= 8192) || K >= 16384) && tiles % 8 == 0) ? 2 : 1;
    p.nblocks = tiles / (4 * p.nw);
  }
  const long units = (long)p.nblocks * (K / 128);
  int cap = gemm_shape(MT, swiglu).nwg;
  // whole N-blocks per workgroup when they alone fill the chip (the SwiGLU
  // at the 70B width: 448 blocks; at 48 and 64 rows 11 % faster than
  // stream-K, whose gate and up partials cost a 16 us fix-up at 64 rows)
  if (swiglu && p.nblocks >= 256 && p.nblocks <= 2 * cap) cap = p.nblocks;
  // up to 32 rows, about 8 ranges per N-block: more split the blocks into
  // slivers whose partials the fix-up must sum (1B-shaped projections with
  // 32 blocks: 12.0 -> 10.6 us at 256 workgroups instead of 512)
  if (!swiglu && MT <= 2 && 8 * p.nblocks < cap) cap = 8 * p.nblocks;
  p.nwg = (int)(units < cap ? units : cap);
  const int col_w = swiglu ? p.nw / 2 : p.nw;
  const int src = swiglu ? 2 : 1;
  // K-split workgroups and whole N-blocks write no partials
  p.part_bytes = p.ksw || p.nwg < 1 || p.nblocks % p.nwg == 0 ? 0 : (size_t)p.nwg * 2 * 4 * MT * col_w * src * kWave * 16;
  p.prep_bytes = (size_t)MT * (K / 128) * 4 * kWave * 16;
  plan_wide(MT, K, tiles, swiglu, p);
  return p;
}

}  // namespace ss
