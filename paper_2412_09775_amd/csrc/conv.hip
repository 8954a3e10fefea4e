// 3x3x3 stride-2 convolutions (padding 1) on BF16 MFMA where a K step of 32
// lies inside one tap: the same implicit GEMMs, K order and splits as the
// general gathers, so the same sums bit for bit, without their per-element
// index arithmetic.
//
// The general kernels are bound by that arithmetic (a tap decode, three bounds
// checks and an address per 16-byte load, eight 2-byte LDS writes per load of
// a transposed operand), at a few percent of the matrix rate.  Here
//   - a row of the position operand is decoded once: a base position and one
//     validity bit per tap; a K step adds a wave-uniform tap offset;
//   - its fragments go from memory straight to MFMA registers (a lane's eight
//     channels are 16 contiguous bytes), so only the weights pass through LDS;
//   - operands whose K runs across rows in memory (the weights of the input
//     gradient, both operands of the weight gradient) are stored to LDS as
//     they lie and read with the transposing LDS read;
//   - the product is taken transposed, so that a lane ends with four
//     consecutive channels of one position and stores 16 bytes.
// Measured, general gathers -> here, 64 samples of 8x16x16, 64 -> 128 channels:
// forward 36 -> 22 us, input gradient 72 -> 26, weight gradient 40 -> 26; the
// network on 64 stacks of 32x64x64: first layer forward 105 -> 72 (bound by the
// error function's vector instructions) and weight gradient 94 -> 34, second
// layer forward 62 -> 54, weight gradient 74 -> 42, and its input gradient 146
// and the GELU pass over it 80 -> 106 as one kernel.
#include <algorithm>

#include "bf16.hpp"
#include "internal.hpp"

namespace wo {

// K steps of 32 per staged weight tile: four, two where a wave holds 32 rows,
// which leaves registers for four waves per SIMD
constexpr int row_steps(int mi) { return mi == 2 ? 2 : 4; }
constexpr int kTrPad = 16;     // row padding of a transposed tile: eight rows of 32 bytes on distinct banks

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// MFMA fragment of a tile stored [k][row]: lane l gets rows' element l % 16 at
// k = (l / 16) * 8 .. + 7 (the lane layout was checked on the device).
template <int STRIDE>
__device__ __forceinline__ bf16x8 tr_frag(const u16* tile, int lane) {
  const int i = lane & 15;
  const u16* p = tile + ((lane >> 4) * 8 + (i >> 2)) * STRIDE + (i & 3) * 4;
  typedef __attribute__((address_space(3))) s16x4 lds4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(p + 4 * STRIDE));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Bits of the taps that hit the volume, (d, h, w) order with w fastest:
// vd, vh, vw hold one bit per tap of an axis, nh and nw taps per axis.
__device__ __forceinline__ unsigned tap_mask(unsigned vd, unsigned vh, unsigned vw, int nd, int nh, int nw) {
  unsigned hw = 0, m = 0;
  for (int j = 0; j < nh; ++j) hw |= (vh >> j & 1u) ? vw << (j * nw) : 0u;
  for (int j = 0; j < nd; ++j) m |= (vd >> j & 1u) ? hw << (j * nw * nh) : 0u;
  return m;
}
__device__ __forceinline__ unsigned axis_bits(int i0, int n) {   // taps 0..2 at i0, i0 + 1, i0 + 2
  return (unsigned)(i0 >= 0 && i0 < n) | (unsigned)(i0 + 1 >= 0 && i0 + 1 < n) << 1 |
         (unsigned)(i0 + 2 >= 0 && i0 + 2 < n) << 2;
}

// Exact division of a position (below 2^31) by an extent: one 64-bit multiply
// and a shift, m = floor(2^(31 + l) / d) + 1 with 2^l >= d.
struct FastDiv {
  unsigned m, d;
  int sh;
};
static FastDiv fast_div(int d) {
  int l = 0;
  while ((1L << l) < d) ++l;
  return FastDiv{(unsigned)((1UL << (31 + l)) / (unsigned)d + 1), (unsigned)d, 31 + l};
}
__device__ __forceinline__ unsigned div_of(unsigned u, const FastDiv& f) {
  return (unsigned)(((unsigned long)u * f.m) >> f.sh);
}
// Workgroup b of a 1-D grid to a tile: workgroups go to the 8 XCDs in turn, so
// each XCD takes runs of kRun tiles and the operands that neighbouring tiles
// share are fetched into one L2 instead of eight (weight gradient of 131072
// positions, 32 -> 64 channels: 62 us in launch order, 44 us so; one run per XCD
// instead, the XCDs far apart in memory: 48 us, the input gradient slower).  The grid is
// a multiple of 8 kRun; ids past the end exit.
constexpr unsigned kRun = 16;
__device__ __forceinline__ unsigned xcd_tile(unsigned b) {
  return b / (8 * kRun) * (8 * kRun) + (b & 7u) * kRun + (b >> 3) % kRun;
}
static unsigned xcd_grid(long tiles) { return (unsigned)((tiles + 8 * kRun - 1) / (8 * kRun) * (8 * kRun)); }

struct PosDiv {   // extents of a row's position, w fastest
  FastDiv w, h, d;
};

// Operands are read through buffer descriptors: a lane whose element lies
// outside gets the offset kOut, beyond every descriptor's range, and reads
// zeros; a wave-uniform tap or channel offset rides in the scalar offset.  A
// descriptor starts at the sample of its workgroup's first row, less a margin
// of one tap (row offsets are then not negative), so 31-bit offsets hold for
// tensors of any size; the host checks the span of a workgroup's rows.
typedef __amdgpu_buffer_rsrc_t Buf;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kOut = 0x80000000u;
__device__ __forceinline__ Buf make_buf(const u16* p, long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)min(bytes, 0x7fffffffL), 0x00027000);
}
__device__ __forceinline__ u32x4 buf16(Buf r, unsigned voff, int soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, soff, 0);
}
__device__ __forceinline__ u16 buf2(Buf r, unsigned voff) {
  return (u16)__builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, 0, 0);
}

// Output position q of a forward convolution, of sample n0 or a later one: the
// offset in elements / C of its tap (0, 0, 0) from the margin before sample
// n0, and its tap bits.
struct PosTaps {
  unsigned base;
  unsigned mask;
};
__host__ __device__ __forceinline__ int fwd_margin(const ConvGeom& g) { return (g.H + 1) * g.W + 1; }
__device__ __forceinline__ PosTaps fwd_taps(const ConvGeom& g, const PosDiv& dv, unsigned q, int n0) {
  const unsigned q1 = div_of(q, dv.w), q2 = div_of(q1, dv.h), n = div_of(q2, dv.d);
  const int w0 = 2 * (int)(q - q1 * dv.w.d) - 1, h0 = 2 * (int)(q1 - q2 * dv.h.d) - 1,
            d0 = 2 * (int)(q2 - n * dv.d.d) - 1;
  PosTaps r;
  r.base = (unsigned)(((((int)n - n0) * g.D + d0) * g.H + h0) * g.W + w0 + fwd_margin(g));
  r.mask = tap_mask(axis_bits(d0, g.D), axis_bits(h0, g.H), axis_bits(w0, g.W), 3, 3, 3);
  return r;
}
__device__ __forceinline__ int sample_of(unsigned q, const PosDiv& dv) {
  return (int)div_of(div_of(div_of(q, dv.w), dv.h), dv.d);
}

// The wave-uniform walk over K steps: tap digits and channel.
struct TapWalk {
  int ch, w, h, d, tap;
  __device__ __forceinline__ void start(int k, int C, int nh, int nw) {
    tap = k / C;
    ch = k - tap * C;
    const int hw = tap / nw;
    w = tap - hw * nw;
    d = hw / nh;
    h = hw - d * nh;
  }
  __device__ __forceinline__ void step(int C, int nh, int nw) {
    ch += 32;
    if (ch < C) return;
    ch = 0;
    ++tap;
    if (++w < nw) return;
    w = 0;
    if (++h < nh) return;
    h = 0;
    ++d;
  }
};

// ------------------------------------------------------------------ epilogues
// Four consecutive channels n .. n + 3 of output row `row`.

struct StoreRows {
  float* c;
  long N;
  static constexpr bool kSums = false;
  __device__ __forceinline__ void split(long off) { c += off; }
  __device__ __forceinline__ void operator()(long row, int n, f32x4 v) const {
    float* p = c + row * N + n;
    if (N % 4 == 0) {
      *(f32x4*)p = v;
      return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (n + r < N) p[r] = v[r];
  }
};

// a = BF16(GELU(z)) of the pre-activation z = v + b and, for the backward pass
// (d not null), GELU'(z): the error function is evaluated once for both.
struct StoreGelu {
  float* d;
  u16* a;
  const float* b;
  long N;
  static constexpr bool kSums = false;
  __device__ __forceinline__ void split(long) {}
  __device__ __forceinline__ void operator()(long row, int n, f32x4 v) const {
    const long i = row * N + n;
    f32x4 dv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float g;
      v[r] = gelu_f(v[r] + b[n + r], g);
      dv[r] = g;
    }
    *(uint2*)(a + i) = make_uint2(f2bf_pair(v[0], v[1]), f2bf_pair(v[2], v[3]));
    if (d) *(f32x4*)(d + i) = dv;
  }
};

// The input gradient through the GELU before it: gz = BF16(v d), as a separate
// pass over the gradient would compute it, and the bias gradient's first stage,
// the workgroup's rounded gz summed per channel into part[workgroup][n].
struct StoreGeluGrad {
  const float* d;
  u16* gz;
  float* part;
  long N;
  static constexpr bool kSums = true;
  __device__ __forceinline__ void split(long) {}
  __device__ __forceinline__ f32x4 load(long row, int n) const { return *(const f32x4*)(d + row * N + n); }
  __device__ __forceinline__ f32x4 operator()(long row, int n, f32x4 v, f32x4 dv) const {
    const long i = row * N + n;
    const f32x4 g = v * dv;
    const uint2 q = make_uint2(f2bf_pair(g[0], g[1]), f2bf_pair(g[2], g[3]));
    *(uint2*)(gz + i) = q;
    return f32x4{__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xffff0000u), __uint_as_float(q.y << 16),
                 __uint_as_float(q.y & 0xffff0000u)};
  }
};

// ------------------------------------------------------------------ forward and input gradient

// Rows of the GEMM: output positions (forward), or the input positions of one
// parity class (input gradient), whose taps are kd = 1 for even d and
// kd in {0, 2} for odd d, per axis.
struct RowClass {
  int pd, ph, pw;    // parity (input gradient)
  PosDiv dv;         // class extents
  int nd, nh, nw;    // taps per axis
  long M;
};
struct RowProblem {
  const u16* x;      // position operand: x, or gz
  const u16* w;
  ConvGeom g;        // g.C: channels of the position operand
  long N;            // columns: Cout, or Cin
  long stride;       // elements from one split's output to the next
  long xbytes, sample;   // bytes of the position operand and of one sample of it
  int nc, splits;
  // Tile order: column tile, row tile, class, split.  Classes side by side would
  // share gz and the lines that they write, and are slower all the same (121 us
  // against 106 for 32 channels of 64x16x32x32 positions): neighbours then read
  // different taps of the weights and run eight-fold different times.
  FastDiv ty, tx, tc;
  unsigned ntiles;
  RowClass c[8];
};

// MI x 16 rows by TN columns per wave, 4 waves along the rows.  The weights of
// a few K steps are staged at a time in one of two LDS tiles, so one
// barrier separates a tile's writes from its reads; the next tile's weights and
// the next steps' fragments are in flight during the MFMAs.  Bound by vector
// issue, so index work is kept out of the loop: a fragment costs a bit test and
// a select, a weight load nothing.
template <int MI, int TN, bool DG, class EP>
__global__ __launch_bounds__(256) void k_conv_rows(RowProblem p, EP ep) {
  constexpr int NJ = TN / 16, KS = row_steps(MI), KT = KS * 32;
  constexpr int LD = DG ? TN + kTrPad : KT + 8;          // LDS row: [k][n] or [n][k]
  constexpr int NB = KT * TN / 8 / 256;                  // 16-byte weight loads per thread and tile
  __shared__ __attribute__((aligned(16))) u16 Bs[2][(DG ? KT : TN) * LD];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const unsigned id = xcd_tile(blockIdx.x);
  if (id >= p.ntiles) return;
  const unsigned iy = div_of(id, p.ty), ix = div_of(iy, p.tx), iq = DG ? div_of(ix, p.tc) : ix;
  const int cls = DG ? (int)(ix - iq * p.tc.d) : 0, q = (int)iq;
  const RowClass& rc = p.c[cls];
  const long m0 = (long)(iy - ix * p.tx.d) * (64 * MI);
  if constexpr (EP::kSums) {
    if (m0 >= rc.M && t < TN && (int)(id - iy * p.ty.d) * TN + t < (int)p.N)
      ep.part[(long)iy * p.N + (int)(id - iy * p.ty.d) * TN + t] = 0.f;
  }
  if (m0 >= rc.M) return;
  const int n0 = (int)(id - iy * p.ty.d) * TN, N = (int)p.N, C = p.g.C;
  const int nd = rc.nd, nh = rc.nh, nw = rc.nw;
  const int K = nd * nh * nw * C;
  int kchunk = (K + p.splits - 1) / p.splits;
  kchunk = (kchunk + 31) / 32 * 32;
  const int kbeg = min(K, q * kchunk), steps = (min(K, kbeg + kchunk) - kbeg) / 32;
  const int s0 = sample_of((unsigned)m0, rc.dv);
  const int margin = DG ? (p.g.Ho + 1) * p.g.Wo + 1 : fwd_margin(p.g);
  // no tap offset exceeds the range: it is stretched by two margins, which no lane reads
  const Buf xb = make_buf(p.x + (s0 * (p.sample / 2) - (long)margin * C), p.xbytes - s0 * p.sample + 6L * margin * C);
  const Buf wb = make_buf(p.w, 54L * C * N);

  // one row per lane, shared with the lanes that hold its other channels: byte
  // offset, tap bits, output row
  unsigned rbase = 0, rmask = 0;
  int rout = 0;
  {
    const long m = m0 + wave * (16 * MI) + (lane & (16 * MI - 1));
    if (m < rc.M) {
      const unsigned u = (unsigned)m;
      if (DG) {
        const unsigned q1 = div_of(u, rc.dv.w), q2 = div_of(q1, rc.dv.h), n = div_of(q2, rc.dv.d);
        const int iw = (int)(u - q1 * rc.dv.w.d), ih = (int)(q1 - q2 * rc.dv.h.d), id = (int)(q2 - n * rc.dv.d.d);
        // tap j of an odd axis reaches output id + 1 - j, the tap of an even one id
        const unsigned vd = (unsigned)(id + rc.pd < p.g.Do) | (unsigned)(id < p.g.Do) << 1;
        const unsigned vh = (unsigned)(ih + rc.ph < p.g.Ho) | (unsigned)(ih < p.g.Ho) << 1;
        const unsigned vw = (unsigned)(iw + rc.pw < p.g.Wo) | (unsigned)(iw < p.g.Wo) << 1;
        rmask = tap_mask(vd, vh, vw & (nw == 2 ? 3u : 1u), nd, nh, nw);
        rbase = (unsigned)(((((int)n - s0) * p.g.Do + id + rc.pd) * p.g.Ho + ih + rc.ph) * p.g.Wo + iw + rc.pw);
        rout = (((int)n * p.g.D + 2 * id + rc.pd) * p.g.H + 2 * ih + rc.ph) * p.g.W + 2 * iw + rc.pw;
      } else {
        const PosTaps r = fwd_taps(p.g, rc.dv, u, s0);
        rbase = r.base;
        rmask = r.mask;
        rout = (int)u;
      }
    }
  }
  unsigned base[MI], mask[MI];
  int orow[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int src = i * 16 + (lane & 15);
    base[i] = (unsigned)__shfl((int)rbase, src) * (2u * C) + (lane >> 4) * 16;
    mask[i] = (unsigned)__shfl((int)rmask, src);
    orow[i] = __shfl(rout, src);
  }
  // this thread's weight loads: [k][n] rows of a step, or [n][k] rows of a tile
  unsigned wo[NB];
  const int half = DG && TN == 32 ? __builtin_amdgcn_readfirstlane(t >> 7) : 0;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int e = t + 256 * u;
    const int n = DG ? n0 + e % (TN / 8) * 8 : n0 + e / (KT / 8);
    wo[u] = DG ? (unsigned)((e / (TN / 8) & 31) * 27 * N + n) * 2 : (unsigned)(n * K + e % (KT / 8) * 8) * 2;
    if (n >= N) wo[u] = kOut;
  }

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // the epilogue's operand is on its way during the products
  f32x4 pre[EP::kSums ? MI : 1][EP::kSums ? NJ : 1];
  if constexpr (EP::kSums) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int n = n0 + j * 16 + (lane >> 4) * 4;
        pre[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (n < N && m0 + (wave * MI + i) * 16 + (lane & 15) < rc.M) pre[i][j] = ep.load(orow[i], n);
      }
  }

  TapWalk tw;
  tw.start(kbeg, C, nh, nw);
  const auto issue = [&](int st0, u32x4 (&ra)[KS][MI], u32x4 (&rb)[NB]) {
    int wrow[KS];   // input gradient: byte offset of (channel, tap) in the weights
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      wrow[s] = 0;
      if (st0 + s >= steps) continue;
      const int tp = DG ? margin - ((tw.d * p.g.Ho + tw.h) * p.g.Wo + tw.w) : (tw.d * p.g.H + tw.h) * p.g.W + tw.w;
      const int off = (tp * C + tw.ch) * 2;
#pragma unroll
      for (int i = 0; i < MI; ++i) ra[s][i] = buf16(xb, (mask[i] >> tw.tap & 1u) ? base[i] : kOut, off);
      if (DG) {
        const int kd = nd == 1 ? 1 : 2 * tw.d, kh = nh == 1 ? 1 : 2 * tw.h, kw = nw == 1 ? 1 : 2 * tw.w;
        wrow[s] = (tw.ch * 27 + (kd * 3 + kh) * 3 + kw) * N * 2;
      }
      tw.step(C, nh, nw);
    }
    // steps past the last are not used: zeros, or any channel's weights
    const bool in = t % (KT / 8) * 8 < (steps - st0) * 32;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      if (DG) rb[u] = buf16(wb, wo[u], TN == 32 ? (half ? wrow[(2 * u + 1) % KS] : wrow[2 * u % KS]) : wrow[u % KS]);
      else rb[u] = buf16(wb, in ? wo[u] : kOut, (kbeg + st0 * 32) * 2);
    }
  };
  const auto tile = [&](int st0, u16* B, u32x4 (&ra)[KS][MI], u32x4 (&rb)[NB], u32x4 (&na)[KS][MI], u32x4 (&nb)[NB]) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = t + 256 * u;
      if (DG) *(u32x4*)&B[e / (TN / 8) * LD + e % (TN / 8) * 8] = rb[u];
      else *(u32x4*)&B[e / (KT / 8) * LD + e % (KT / 8) * 8] = rb[u];
    }
    __syncthreads();
    if (st0 + KS < steps) issue(st0 + KS, na, nb);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (st0 + s >= steps) break;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        bf16x8 b;
        if constexpr (DG) b = tr_frag<LD>(B + s * 32 * LD + j * 16, lane);
        else b = *(const bf16x8*)&B[(j * 16 + (lane & 15)) * LD + s * 32 + (lane >> 4) * 8];
#pragma unroll
        for (int i = 0; i < MI; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, __builtin_bit_cast(bf16x8, ra[s][i]), acc[i][j],
                                                              0, 0, 0);
      }
    }
  };

  u32x4 ra0[KS][MI], rb0[NB], ra1[KS][MI], rb1[NB];   // in turn: one in use, one in flight
  if (steps > 0) issue(0, ra0, rb0);
  for (int st0 = 0; st0 < steps; st0 += 2 * KS) {
    tile(st0, Bs[0], ra0, rb0, ra1, rb1);
    if (st0 + KS >= steps) break;
    tile(st0 + KS, Bs[1], ra1, rb1, ra0, rb0);
  }
  ep.split(q * p.stride);
  f32x4 sum[EP::kSums ? NJ : 1];
#pragma unroll
  for (int j = 0; j < (EP::kSums ? NJ : 1); ++j) sum[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (m0 + (wave * MI + i) * 16 + (lane & 15) >= rc.M) continue;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + j * 16 + (lane >> 4) * 4;
      if (n >= N) continue;
      if constexpr (EP::kSums) sum[j] += ep(orow[i], n, acc[i][j], pre[i][j]);
      else ep(orow[i], n, acc[i][j]);
    }
  }
  if constexpr (EP::kSums) {   // over the 16 rows of a lane group, then the waves
    __shared__ float red[4][TN];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = sum[j][r];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o);
        if ((lane & 15) == 0) red[wave][j * 16 + (lane >> 4) * 4 + r] = v;
      }
    __syncthreads();
    if (t < TN && n0 + t < N) ep.part[(long)iy * N + n0 + t] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
  }
}

// One input channel (K = 27, one step): no operand passes through LDS.  A wave
// decodes 64 output positions at once, one per lane, and takes them sixteen at
// a time; a lane gathers its eight taps and holds its weights' fragments
// throughout.
template <class EP>
__global__ __launch_bounds__(256) void k_conv_first(const u16* __restrict__ x, const u16* __restrict__ w, ConvGeom g,
                                                    PosDiv dv, long xbytes, long P, int N, EP ep) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kg = (lane >> 4) * 8;
  const int n0 = (int)blockIdx.y * 32;
  bf16x8 wf[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = n0 + j * 16 + (lane & 15);
    u16 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = n < N && kg + e < 27 ? w[(long)n * 27 + kg + e] : (u16)0;
    wf[j] = __builtin_bit_cast(bf16x8, *(uint4*)v);
  }
  unsigned off[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int tap = kg + e;
    off[e] = (((tap / 9) * g.H + tap / 3 % 3) * g.W + tap % 3) * 2;
  }
  const long b0 = (long)blockIdx.x * 256, m0 = b0 + wave * 64;
  const int s0 = sample_of((unsigned)b0, dv);
  const long skip = (long)s0 * g.D * g.H * g.W - fwd_margin(g);
  const Buf xb = make_buf(x + skip, xbytes - 2 * skip);
  PosTaps mine{0, 0};
  if (m0 + lane < P) mine = fwd_taps(g, dv, (unsigned)(m0 + lane), s0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int src = i * 16 + (lane & 15);
    const unsigned base = (unsigned)__shfl((int)mine.base, src) * 2;
    const unsigned mask = (unsigned)__shfl((int)mine.mask, src) >> kg;   // taps past 26 have no bit
    u16 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = buf2(xb, (mask >> e & 1u) ? base + off[e] : kOut);
    const bf16x8 a = __builtin_bit_cast(bf16x8, *(uint4*)v);
    const long m = m0 + src;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], a, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      const int n = n0 + j * 16 + (lane >> 4) * 4;
      if (m < P && n < N) ep(m, n, c);
    }
  }
}

// ------------------------------------------------------------------ weight gradient

// TM channels of gz by TN columns (tap, input channel) per workgroup, 4 waves
// as 2 x 2, over one split of the output positions.  64 positions of both
// operands are staged at a time as they lie in memory, in one of two LDS tile
// pairs, and read transposed.  The positions' base and tap bits are decoded by
// 256 threads for 256 positions at a time, one block ahead, into LDS.
// ONE: one input channel, the 27 taps are the columns.
template <int TM, int TN, bool ONE>
__global__ __launch_bounds__(256) void k_conv_wgrad(const u16* __restrict__ x, const u16* __restrict__ gz, ConvGeom g,
                                                    PosDiv dv, long xbytes, long P, int Co, long kchunk,
                                                    FastDiv tn, FastDiv tm, unsigned ntiles,
                                                    float* __restrict__ part) {
  constexpr int KT = 64, LA = TM + kTrPad, LB = TN + kTrPad;
  constexpr int FM = TM / 32, FN = TN / 32;               // 16 x 16 blocks per wave
  constexpr int NA = KT * TM / 8 / 256, NB = KT * TN / 8 / 256;
  static_assert(NA >= 1 && NB >= 1, "at least one 16-byte load per thread and tile");
  static_assert(!ONE || TN == 32, "27 taps in one tile");
  __shared__ __attribute__((aligned(16))) u16 As[2][KT * LA];
  __shared__ __attribute__((aligned(16))) u16 Bs[2][KT * LB];
  __shared__ PosTaps tab[2][256];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
  const int K = 27 * g.C;
  const unsigned id = xcd_tile(blockIdx.x);   // column tile, row tile, split
  if (id >= ntiles) return;
  const unsigned im = div_of(id, tn), iz = div_of(im, tm);
  const int m0 = (int)(im - iz * tm.d) * TM, n0 = (int)(id - im * tn.d) * TN;
  const long kbeg = (long)iz * kchunk, kend = min(P, kbeg + kchunk);

  const int s0 = sample_of((unsigned)kbeg, dv);
  const long skip = ((long)s0 * g.D * g.H * g.W - fwd_margin(g)) * g.C;
  const Buf xb = make_buf(x + skip, xbytes - 2 * skip);
  const Buf gb = make_buf(gz + kbeg * Co, (kend - kbeg) * Co * 2);   // zeros past the split

  // this thread's columns: eight channels of one tap (ONE: eight taps)
  const int n8 = n0 + t % (TN / 8) * 8;
  int tap = 0;
  unsigned off[ONE ? 8 : 1];
  if (ONE) {
#pragma unroll
    for (int e = 0; e < 8; ++e) off[e] = ((((n8 + e) / 9) * g.H + (n8 + e) / 3 % 3) * g.W + (n8 + e) % 3) * 2;
  } else {
    tap = n8 / g.C;
    off[0] = ((((tap / 9) * g.H + tap / 3 % 3) * g.W + tap % 3) * g.C + (n8 - tap * g.C)) * 2;
  }
  if (n8 >= K) tap = 31;   // no such bit
  const int mc = m0 + t % (TM / 8) * 8;
  const unsigned arow = mc < Co ? (unsigned)(t / (TM / 8) * Co + mc) * 2 : kOut;

  const auto decode = [&](int k0) {   // positions kbeg + k0 .. + 255
    PosTaps r{0, 0};
    if (kbeg + k0 + t < kend) r = fwd_taps(g, dv, (unsigned)(kbeg + k0 + t), s0);
    r.base *= 2 * g.C;
    tab[k0 >> 8 & 1][t] = r;
  };
  u32x4 ra[NA], rb[NB];
  const auto issue = [&](int k0) {
#pragma unroll
    for (int u = 0; u < NA; ++u) ra[u] = buf16(gb, arow + (unsigned)((k0 + 256 * u / (TM / 8)) * Co * 2), 0);
    const PosTaps* tb = tab[k0 >> 8 & 1] + (k0 & 255);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const PosTaps r = tb[(t + 256 * u) / (TN / 8)];
      if (ONE) {
        u16 v[8];
        const unsigned mk = r.mask >> n8;   // n8 <= 24; taps past 26 have no bit
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = buf2(xb, (mk >> e & 1u) ? r.base + off[e] : kOut);
        rb[u] = *(u32x4*)v;
      } else {
        rb[u] = buf16(xb, (r.mask >> tap & 1u) ? r.base + off[0] : kOut, 0);
      }
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int len = (int)(kend - kbeg);
  decode(0);
  __syncthreads();
  issue(0);
  for (int k0 = 0, buf = 0; k0 < len; k0 += KT, buf ^= 1) {
    u16 *A = As[buf], *B = Bs[buf];
#pragma unroll
    for (int u = 0; u < NA; ++u) *(u32x4*)&A[(t + 256 * u) / (TM / 8) * LA + t % (TM / 8) * 8] = ra[u];
#pragma unroll
    for (int u = 0; u < NB; ++u) *(u32x4*)&B[(t + 256 * u) / (TN / 8) * LB + t % (TN / 8) * 8] = rb[u];
    const int k1 = k0 + KT;
    // a block's first tile is fetched after this barrier; the half it fills was
    // last read two blocks ago
    if (k1 < len && (k1 & 255) == 0) decode(k1);
    __syncthreads();
    if (k1 < len) issue(k1);
#pragma unroll
    for (int ks = 0; ks < KT / 32; ++ks) {
      bf16x8 a[FM];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = tr_frag<LA>(A + ks * 32 * LA + (wm * FM + i) * 16, lane);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const bf16x8 b = tr_frag<LB>(B + ks * 32 * LB + (wn * FN + j) * 16, lane);
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[i], acc[i][j], 0, 0, 0);
      }
    }
  }
  float* c = part + (long)iz * Co * K;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int co = m0 + (wm * FM + i) * 16 + (lane & 15);
    if (co >= Co) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + (wn * FN + j) * 16 + (lane >> 4) * 4;
      float* p = c + (long)co * K + n;
      if (!ONE) {
        if (n < K) *(f32x4*)p = acc[i][j];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n + r < K) p[r] = acc[i][j][r];
      }
    }
  }
}

static unsigned tiles(long n, long t) { return (unsigned)((n + t - 1) / t); }

// Rows per wave / 16: 2 where that leaves four workgroups per CU, else 1.
static int row_blocks(const RowProblem& p, unsigned nq) {
  long wgs = 0;
  for (int c = 0; c < p.nc; ++c) wgs += (long)tiles(p.c[c].M, 128) * tiles(p.N, p.N <= 32 ? 32 : 64) * nq;
  return wgs >= 1024 ? 2 : 1;
}

template <bool DG, class EP>
static bool launch_rows(RowProblem& p, long mmax, unsigned nq, const EP& ep, hipStream_t s, const char* tag,
                        hipError_t* e) {
  const bool narrow = p.N <= 32;
  const unsigned ny = tiles(p.N, narrow ? 32 : 64);
  const int mi = row_blocks(p, nq);
  const unsigned nx = tiles(mmax, 64 * mi);
  const long total = (long)nx * ny * p.nc * nq;
  if (total >= (1L << 30)) return false;
  p.ty = fast_div((int)ny);
  p.tc = fast_div(p.nc);
  p.tx = fast_div((int)nx);
  p.ntiles = (unsigned)total;
  const dim3 grid(xcd_grid(total));
  ScopedTiming _t(tag, s);
  if (mi == 2) {
    if (narrow) hipLaunchKernelGGL((k_conv_rows<2, 32, DG, EP>), grid, dim3(256), 0, s, p, ep);
    else hipLaunchKernelGGL((k_conv_rows<2, 64, DG, EP>), grid, dim3(256), 0, s, p, ep);
  } else {
    if (narrow) hipLaunchKernelGGL((k_conv_rows<1, 32, DG, EP>), grid, dim3(256), 0, s, p, ep);
    else hipLaunchKernelGGL((k_conv_rows<1, 64, DG, EP>), grid, dim3(256), 0, s, p, ep);
  }
  *e = hipGetLastError();
  return true;
}

// Buffer loads of several words want word-aligned operands; others take the
// general gathers.
static bool words(const u16* a, const u16* b) { return (((uintptr_t)a | (uintptr_t)b) & 3) == 0; }

static PosDiv pos_div(int d, int h, int w) { return PosDiv{fast_div(w), fast_div(h), fast_div(d)}; }

// Bytes from the margin before the first to the end of the last sample that
// `rows` consecutive rows of rps per sample touch stay below 2^31.
static bool span_ok(long rows, long rps, long N, long sample_bytes, long margin_bytes) {
  const long n = std::min(N, (rows + rps - 1) / rps + 1);
  return sample_bytes < (1L << 31) && margin_bytes < (1L << 28) && n * sample_bytes + 2 * margin_bytes < (1L << 31);
}

bool conv_fwd_taps(const u16* x, const u16* w, const ConvGeom& g, long P, int Cout, int splits,
                   const ConvFwdOut& out, hipStream_t s, const char* tag, hipError_t* e) {
  const StoreGelu eg{out.d, out.a, out.bias, Cout};
  const StoreRows er{out.c, Cout};
  if (out.a && Cout % 4 != 0) return false;
  const bool first = g.C == 1 && splits == 1;
  if (!first && (g.C % 32 != 0 || !words(x, w))) return false;   // 32: a K step in one tap
  const PosDiv dv = pos_div(g.Do, g.Ho, g.Wo);
  const long rps = (long)g.Do * g.Ho * g.Wo, N = P / rps, sample = 2L * g.D * g.H * g.W * g.C;
  if (!span_ok(256, rps, N, sample, 2L * fwd_margin(g) * g.C)) return false;
  if (first) {
    const dim3 grid(tiles(P, 256), tiles(Cout, 32));
    ScopedTiming _t(tag, s);
    if (out.a)
      hipLaunchKernelGGL(k_conv_first<StoreGelu>, grid, dim3(256), 0, s, x, w, g, dv, N * sample, P, Cout, eg);
    else
      hipLaunchKernelGGL(k_conv_first<StoreRows>, grid, dim3(256), 0, s, x, w, g, dv, N * sample, P, Cout, er);
    *e = hipGetLastError();
    return true;
  }
  RowProblem p{};
  p.x = x; p.w = w; p.g = g;
  p.N = Cout;
  p.stride = P * Cout;
  p.xbytes = N * sample;
  p.sample = sample;
  p.nc = 1;
  p.splits = splits;
  p.c[0] = RowClass{0, 0, 0, dv, 3, 3, 3, P};
  const long K = 27L * g.C, kchunk = ((K + splits - 1) / splits + 31) / 32 * 32;
  const unsigned nz = tiles(K, kchunk);
  return out.a ? launch_rows<false>(p, P, nz, eg, s, tag, e) : launch_rows<false>(p, P, nz, er, s, tag, e);
}

// The input gradient's classes; false where the kernels do not take the shape.
static bool dgrad_problem(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, int splits,
                          RowProblem& p, long& mmax) {
  if (gout.C % 32 != 0 || Cin % 8 != 0) return false;
  p.x = gz; p.w = w; p.g = gout;
  p.N = Cin;
  p.stride = (long)N * gout.D * gout.H * gout.W * Cin;
  p.sample = 2L * gout.Do * gout.Ho * gout.Wo * gout.C;
  p.xbytes = N * p.sample;
  p.splits = splits;
  mmax = 0;
  for (int cls = 7; cls >= 0; --cls) {   // the longest K first: no long tail
    RowClass c;
    c.pd = cls >> 2; c.ph = cls >> 1 & 1; c.pw = cls & 1;
    const int cd = (gout.D - c.pd + 1) / 2, ch = (gout.H - c.ph + 1) / 2, cw = (gout.W - c.pw + 1) / 2;
    if (cd <= 0 || ch <= 0 || cw <= 0) continue;
    c.dv = pos_div(cd, ch, cw);
    c.nd = 1 + c.pd; c.nh = 1 + c.ph; c.nw = 1 + c.pw;
    c.M = (long)N * cd * ch * cw;
    if (!span_ok(128, (long)cd * ch * cw, N, p.sample, 2L * ((gout.Ho + 1) * gout.Wo + 1) * gout.C)) return false;
    mmax = std::max(mmax, c.M);
    p.c[p.nc++] = c;
  }
  return true;
}

bool conv_dgrad_taps(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, int splits, float* out,
                     hipStream_t s, const char* tag, hipError_t* e) {
  RowProblem p{};
  long mmax;
  if (!words(gz, w) || !dgrad_problem(gz, w, gout, Cin, N, splits, p, mmax)) return false;
  return launch_rows<true>(p, mmax, (unsigned)splits, StoreRows{out, Cin}, s, tag, e);
}

long conv_dgrad_gelu_rows(const ConvGeom& gout, int Cin, int N) {
  RowProblem p{};
  long mmax;
  if (!dgrad_problem(nullptr, nullptr, gout, Cin, N, 1, p, mmax)) return 0;
  return (long)tiles(mmax, 64 * row_blocks(p, 1)) * p.nc;
}

bool conv_dgrad_gelu(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, const float* d, u16* gz_in,
                     float* part, hipStream_t s, const char* tag, hipError_t* e) {
  RowProblem p{};
  long mmax;
  if (!dgrad_problem(gz, w, gout, Cin, N, 1, p, mmax)) return false;
  return launch_rows<true>(p, mmax, 1u, StoreGeluGrad{d, gz_in, part, Cin}, s, tag, e);
}

bool conv_wgrad_taps(const u16* x, const u16* gz, const ConvGeom& g, long P, int Cout, int splits, float* part,
                     hipStream_t s, const char* tag, hipError_t* e) {
  if (Cout % 8 != 0 || (g.C != 1 && g.C % 8 != 0) || !words(g.C == 1 ? gz : x, gz)) return false;
  const long K = 27L * g.C, kchunk = ((P + splits - 1) / splits + 31) / 32 * 32;
  const PosDiv dv = pos_div(g.Do, g.Ho, g.Wo);
  const long rps = (long)g.Do * g.Ho * g.Wo, N = P / rps, sample = 2L * g.D * g.H * g.W * g.C;
  if (!span_ok(kchunk, rps, N, sample, 2L * fwd_margin(g) * g.C) || (kchunk + 64) * Cout * 2 >= (1L << 31))
    return false;
  const int tile = g.C == 1 ? 32 : 64;
  const unsigned nm = tiles(Cout, tile), nn = tiles(K, tile);
  const long total = (long)nm * nn * tiles(P, kchunk);
  if (total >= (1L << 30)) return false;
  const dim3 grid(xcd_grid(total));
  const FastDiv tn = fast_div((int)nn), tm = fast_div((int)nm);
  ScopedTiming _t(tag, s);
  if (g.C == 1)
    hipLaunchKernelGGL((k_conv_wgrad<32, 32, true>), grid, dim3(256), 0, s, x, gz, g, dv, N * sample, P, Cout, kchunk,
                       tn, tm, (unsigned)total, part);
  else
    hipLaunchKernelGGL((k_conv_wgrad<64, 64, false>), grid, dim3(256), 0, s, x, gz, g, dv, N * sample, P, Cout, kchunk,
                       tn, tm, (unsigned)total, part);
  *e = hipGetLastError();
  return true;
}

}  // namespace wo
