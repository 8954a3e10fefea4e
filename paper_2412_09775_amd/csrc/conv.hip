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
// forward 36 -> 23 us, input gradient 72 -> 33, weight gradient 40 -> 28; the
// network on 64 stacks of 32x64x64: first layer forward 105 -> 74 and weight
// gradient 94 -> 36, second layer's input gradient 146 -> 86.
#include <algorithm>

#include "bf16.hpp"
#include "internal.hpp"

namespace wo {

constexpr int kRowSteps = 4;   // K steps of 32 per staged weight tile
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

// Output position q of a forward convolution: the input position of its tap
// (0, 0, 0), which may lie outside (positions stay below 2^31, and the base
// above -2^31), and its tap bits.
struct PosTaps {
  int base;
  unsigned mask;
};
__device__ __forceinline__ PosTaps fwd_taps(const ConvGeom& g, unsigned q) {
  const unsigned q1 = q / (unsigned)g.Wo, q2 = q1 / (unsigned)g.Ho, n = q2 / (unsigned)g.Do;
  const int w0 = 2 * (int)(q - q1 * (unsigned)g.Wo) - 1, h0 = 2 * (int)(q1 - q2 * (unsigned)g.Ho) - 1,
            d0 = 2 * (int)(q2 - n * (unsigned)g.Do) - 1;
  PosTaps r;
  r.base = (((int)n * g.D + d0) * g.H + h0) * g.W + w0;
  r.mask = tap_mask(axis_bits(d0, g.D), axis_bits(h0, g.H), axis_bits(w0, g.W), 3, 3, 3);
  return r;
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

struct StoreGelu {
  float* z;
  u16* a;
  const float* b;
  long N;
  __device__ __forceinline__ void split(long) {}
  __device__ __forceinline__ void operator()(long row, int n, f32x4 v) const {
    const long i = row * N + n;
    u16 q[4];
    if (N % 4 == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[r] += b[n + r];
        q[r] = f2bf(gelu_f(v[r]));
      }
      *(f32x4*)(z + i) = v;
      *(uint2*)(a + i) = make_uint2(q[0] | (unsigned)q[1] << 16, q[2] | (unsigned)q[3] << 16);
      return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (n + r < N) {
        const float t = v[r] + b[n + r];
        z[i + r] = t;
        a[i + r] = f2bf(gelu_f(t));
      }
  }
};

// ------------------------------------------------------------------ forward and input gradient

// Rows of the GEMM: output positions (forward), or the input positions of one
// parity class (input gradient), whose taps are kd = 1 for even d and
// kd in {0, 2} for odd d, per axis.
struct RowClass {
  int pd, ph, pw;    // parity (input gradient)
  int cd, ch, cw;    // class extents
  int nd, nh, nw;    // taps per axis
  long M;
};
struct RowProblem {
  const u16* x;      // position operand: x, or gz
  const u16* w;
  ConvGeom g;        // g.C: channels of the position operand
  long N;            // columns: Cout, or Cin
  long stride;       // elements from one split's output to the next
  int nc, splits;
  RowClass c[8];
};

// MI x 16 rows by TN columns per wave, 4 waves along the rows.  The weights of
// kRowSteps K steps are staged at a time in one of two LDS tiles, so one
// barrier separates a tile's writes from its reads; the next tile's weights and
// the next steps' fragments are in flight during the MFMAs.
template <int MI, int TN, bool DG, class EP>
__global__ __launch_bounds__(256) void k_conv_rows(RowProblem p, EP ep) {
  constexpr int NJ = TN / 16, KS = kRowSteps, KT = KS * 32;
  constexpr int LD = DG ? TN + kTrPad : KT + 8;          // LDS row: [k][n] or [n][k]
  constexpr int NB = KT * TN / 8 / 256;                  // 16-byte weight loads per thread and tile
  __shared__ __attribute__((aligned(16))) u16 Bs[2][(DG ? KT : TN) * LD];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int cls = DG ? (int)(blockIdx.z % p.nc) : 0, q = DG ? (int)(blockIdx.z / p.nc) : (int)blockIdx.z;
  const RowClass& rc = p.c[cls];
  const long m0 = (long)blockIdx.x * (64 * MI);
  if (m0 >= rc.M) return;
  const int n0 = (int)blockIdx.y * TN, N = (int)p.N, C = p.g.C;
  const int nd = rc.nd, nh = rc.nh, nw = rc.nw;
  const int K = nd * nh * nw * C;
  int kchunk = (K + p.splits - 1) / p.splits;
  kchunk = (kchunk + 31) / 32 * 32;
  const int kbeg = min(K, q * kchunk), steps = (min(K, kbeg + kchunk) - kbeg) / 32;

  // this lane's rows: base address, tap bits, output row
  const u16* base[MI];
  unsigned mask[MI];
  long orow[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const long m = m0 + (wave * MI + i) * 16 + (lane & 15);
    const bool in = m < rc.M;
    const unsigned u = in ? (unsigned)m : 0u;
    long pos;
    if (DG) {
      const unsigned q1 = u / (unsigned)rc.cw, q2 = q1 / (unsigned)rc.ch, n = q2 / (unsigned)rc.cd;
      const int iw = (int)(u - q1 * (unsigned)rc.cw), ih = (int)(q1 - q2 * (unsigned)rc.ch),
                id = (int)(q2 - n * (unsigned)rc.cd);
      // tap j of an odd axis reaches output id + 1 - j, the tap of an even one id
      const unsigned vd = (unsigned)(id + rc.pd < p.g.Do) | (unsigned)(id < p.g.Do) << 1;
      const unsigned vh = (unsigned)(ih + rc.ph < p.g.Ho) | (unsigned)(ih < p.g.Ho) << 1;
      const unsigned vw = (unsigned)(iw + rc.pw < p.g.Wo) | (unsigned)(iw < p.g.Wo) << 1;
      mask[i] = tap_mask(vd, vh, vw & (nw == 2 ? 3u : 1u), nd, nh, nw);
      pos = (((long)n * p.g.Do + id + rc.pd) * p.g.Ho + ih + rc.ph) * p.g.Wo + iw + rc.pw;
      orow[i] = (((long)n * p.g.D + 2 * id + rc.pd) * p.g.H + 2 * ih + rc.ph) * p.g.W + 2 * iw + rc.pw;
    } else {
      const PosTaps r = fwd_taps(p.g, u);
      pos = r.base;
      mask[i] = r.mask;
      orow[i] = m;
    }
    if (!in) mask[i] = 0;
    base[i] = p.x + pos * C + (lane >> 4) * 8;
  }
  const u16* safe = p.x + (lane >> 4) * 8;   // in bounds: at least 32 channels

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  uint4 ra[KS][MI], rb[NB];
  unsigned ok[MI];   // bit s: step s of the loaded tile hits the volume
  TapWalk tw;
  tw.start(kbeg, C, nh, nw);
  const auto issue = [&](int st0) {
    long wrow[KS];   // input gradient: offset of (channel, tap) in the weights
#pragma unroll
    for (int i = 0; i < MI; ++i) ok[i] = 0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      wrow[s] = 0;
      if (st0 + s >= steps) continue;
      const int tp = DG ? -((tw.d * p.g.Ho + tw.h) * p.g.Wo + tw.w) : (tw.d * p.g.H + tw.h) * p.g.W + tw.w;
      const long off = (long)tp * C + tw.ch;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const bool v = mask[i] >> tw.tap & 1u;
        ok[i] |= (unsigned)v << s;
        ra[s][i] = *(const uint4*)(v ? base[i] + off : safe);
      }
      if (DG) {
        const int kd = nd == 1 ? 1 : 2 * tw.d, kh = nh == 1 ? 1 : 2 * tw.h, kw = nw == 1 ? 1 : 2 * tw.w;
        wrow[s] = ((long)tw.ch * 27 + (kd * 3 + kh) * 3 + kw) * N;
      }
      tw.step(C, nh, nw);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = t + 256 * u;
      rb[u] = make_uint4(0, 0, 0, 0);
      if (DG) {
        const int k = e / (TN / 8), n = n0 + e % (TN / 8) * 8, s = k >> 5;
        long o = wrow[0];
#pragma unroll
        for (int v = 1; v < KS; ++v) o = s == v ? wrow[v] : o;
        if (st0 + s < steps && n < N) rb[u] = *(const uint4*)(p.w + o + (long)(k & 31) * 27 * N + n);
      } else {
        const int n = n0 + e / (KT / 8), k = e % (KT / 8) * 8;
        if (st0 + (k >> 5) < steps && n < N)
          rb[u] = *(const uint4*)(p.w + (long)n * K + kbeg + st0 * 32 + k);
      }
    }
  };

  if (steps > 0) issue(0);
  for (int st0 = 0, buf = 0; st0 < steps; st0 += KS, buf ^= 1) {
    u16* B = Bs[buf];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = t + 256 * u;
      if (DG) *(uint4*)&B[e / (TN / 8) * LD + e % (TN / 8) * 8] = rb[u];
      else *(uint4*)&B[e / (KT / 8) * LD + e % (KT / 8) * 8] = rb[u];
    }
    uint4 fa[KS][MI];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[s][i] = (ok[i] >> s & 1u) ? ra[s][i] : make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (st0 + KS < steps) issue(st0 + KS);
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
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, __builtin_bit_cast(bf16x8, fa[s][i]), acc[i][j],
                                                              0, 0, 0);
      }
    }
  }
  ep.split(q * p.stride);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (m0 + (wave * MI + i) * 16 + (lane & 15) >= rc.M) continue;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + j * 16 + (lane >> 4) * 4;
      if (n < N) ep(orow[i], n, acc[i][j]);
    }
  }
}

// One input channel (K = 27, one step): no operand passes through LDS.  A wave
// decodes 64 output positions at once, one per lane, and takes them sixteen at
// a time; a lane gathers its eight taps and holds its weights' fragments
// throughout.
template <class EP>
__global__ __launch_bounds__(256) void k_conv_first(const u16* __restrict__ x, const u16* __restrict__ w, ConvGeom g,
                                                    long P, int N, EP ep) {
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
  int off[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int tap = kg + e;
    off[e] = ((tap / 9) * g.H + tap / 3 % 3) * g.W + tap % 3;
  }
  const long m0 = (long)blockIdx.x * 256 + wave * 64;
  PosTaps mine{0, 0};
  if (m0 + lane < P) mine = fwd_taps(g, (unsigned)(m0 + lane));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int src = i * 16 + (lane & 15);
    const int base = __shfl(mine.base, src);
    const unsigned mask = (unsigned)__shfl((int)mine.mask, src) >> kg;   // taps past 26 have no bit
    u16 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = mask >> e & 1u;
      const u16 r = x[in ? base + off[e] : 0];
      v[e] = in ? r : (u16)0;
    }
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
                                                    long P, int Co, long kchunk, float* __restrict__ part) {
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
  const int m0 = (int)blockIdx.x * TM, n0 = (int)blockIdx.y * TN;
  const long kbeg = (long)blockIdx.z * kchunk, kend = min(P, kbeg + kchunk);

  // this thread's columns: eight channels of one tap (ONE: eight taps)
  const int n8 = n0 + t % (TN / 8) * 8;
  int tap = 0, off[ONE ? 8 : 1];
  long ci = 0;
  if (ONE) {
#pragma unroll
    for (int e = 0; e < 8; ++e) off[e] = (((n8 + e) / 9) * g.H + (n8 + e) / 3 % 3) * g.W + (n8 + e) % 3;
  } else {
    tap = n8 / g.C;
    ci = n8 - tap * g.C;
    off[0] = ((tap / 9) * g.H + tap / 3 % 3) * g.W + tap % 3;
  }
  const bool col = ONE || n8 < K;
  const int mc = m0 + t % (TM / 8) * 8;
  const bool row = mc < Co;

  const auto decode = [&](long k0) {   // positions k0 .. k0 + 255
    const long k = k0 + t;
    PosTaps r{0, 0};
    if (k < kend) r = fwd_taps(g, (unsigned)k);
    tab[(k0 - kbeg) >> 8 & 1][t] = r;
  };
  uint4 ra[NA], rb[NB];
  const auto issue = [&](long k0) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const long k = k0 + (t + 256 * u) / (TM / 8);
      ra[u] = make_uint4(0, 0, 0, 0);
      if (row && k < kend) ra[u] = *(const uint4*)(gz + k * Co + mc);
    }
    const PosTaps* tb = tab[(k0 - kbeg) >> 8 & 1] + ((k0 - kbeg) & 255);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const PosTaps r = tb[(t + 256 * u) / (TN / 8)];
      rb[u] = make_uint4(0, 0, 0, 0);
      if (ONE) {
        u16 v[8];
        const unsigned mk = r.mask >> n8;   // n8 <= 24; taps past 26 have no bit
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool in = mk >> e & 1u;
          const u16 q = x[in ? r.base + off[e] : 0];
          v[e] = in ? q : (u16)0;
        }
        rb[u] = *(uint4*)v;
      } else if (col && (r.mask >> tap & 1u)) {
        rb[u] = *(const uint4*)(x + (long)(r.base + off[0]) * g.C + ci);
      }
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  decode(kbeg);
  __syncthreads();
  issue(kbeg);
  int buf = 0;
  for (long k0 = kbeg; k0 < kend; k0 += KT, buf ^= 1) {
    u16 *A = As[buf], *B = Bs[buf];
#pragma unroll
    for (int u = 0; u < NA; ++u) *(uint4*)&A[(t + 256 * u) / (TM / 8) * LA + t % (TM / 8) * 8] = ra[u];
#pragma unroll
    for (int u = 0; u < NB; ++u) *(uint4*)&B[(t + 256 * u) / (TN / 8) * LB + t % (TN / 8) * 8] = rb[u];
    const long k1 = k0 + KT;
    // a block's first tile is fetched after this barrier; the half it fills was
    // last read two blocks ago
    if (k1 < kend && ((k1 - kbeg) & 255) == 0) decode(k1);
    __syncthreads();
    if (k1 < kend) issue(k1);
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
  float* c = part + (long)blockIdx.z * Co * K;
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

template <bool DG, class EP>
static hipError_t launch_rows(const RowProblem& p, long mmax, unsigned nz, const EP& ep, hipStream_t s) {
  long wgs = 0;
  const bool narrow = p.N <= 32;
  for (int c = 0; c < p.nc; ++c) wgs += tiles(p.c[c].M, 128) * (long)tiles(p.N, narrow ? 32 : 64) * (nz / p.nc);
  // 32 rows per wave where that leaves four workgroups per CU; 16 below that
  const int mi = wgs >= 1024 ? 2 : 1;
  const dim3 grid(tiles(mmax, 64 * mi), tiles(p.N, narrow ? 32 : 64), nz);
  if (mi == 2) {
    if (narrow) hipLaunchKernelGGL((k_conv_rows<2, 32, DG, EP>), grid, dim3(256), 0, s, p, ep);
    else hipLaunchKernelGGL((k_conv_rows<2, 64, DG, EP>), grid, dim3(256), 0, s, p, ep);
  } else {
    if (narrow) hipLaunchKernelGGL((k_conv_rows<1, 32, DG, EP>), grid, dim3(256), 0, s, p, ep);
    else hipLaunchKernelGGL((k_conv_rows<1, 64, DG, EP>), grid, dim3(256), 0, s, p, ep);
  }
  return hipGetLastError();
}


bool conv_fwd_taps(const u16* x, const u16* w, const ConvGeom& g, long P, int Cout, int splits,
                   const ConvFwdOut& out, hipStream_t s, hipError_t* e) {
  const StoreGelu eg{out.z, out.a, out.bias, Cout};
  const StoreRows er{out.c, Cout};
  if (g.C == 1 && splits == 1) {
    const dim3 grid(tiles(P, 256), tiles(Cout, 32));
    if (out.a) hipLaunchKernelGGL(k_conv_first<StoreGelu>, grid, dim3(256), 0, s, x, w, g, P, Cout, eg);
    else hipLaunchKernelGGL(k_conv_first<StoreRows>, grid, dim3(256), 0, s, x, w, g, P, Cout, er);
    *e = hipGetLastError();
    return true;
  }
  if (g.C % 32 != 0) return false;   // a K step would straddle taps
  RowProblem p{};
  p.x = x; p.w = w; p.g = g;
  p.N = Cout;
  p.stride = P * Cout;
  p.nc = 1;
  p.splits = splits;
  p.c[0] = RowClass{0, 0, 0, 0, 0, 0, 3, 3, 3, P};
  const long K = 27L * g.C, kchunk = ((K + splits - 1) / splits + 31) / 32 * 32;
  const unsigned nz = tiles(K, kchunk);
  *e = out.a ? launch_rows<false>(p, P, nz, eg, s) : launch_rows<false>(p, P, nz, er, s);
  return true;
}

bool conv_dgrad_taps(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, int splits, float* out,
                     hipStream_t s, hipError_t* e) {
  if (gout.C % 32 != 0 || Cin % 8 != 0) return false;
  RowProblem p{};
  p.x = gz; p.w = w; p.g = gout;
  p.N = Cin;
  p.stride = (long)N * gout.D * gout.H * gout.W * Cin;
  p.splits = splits;
  long mmax = 0;
  for (int cls = 0; cls < 8; ++cls) {
    RowClass c;
    c.pd = cls >> 2; c.ph = cls >> 1 & 1; c.pw = cls & 1;
    c.cd = (gout.D - c.pd + 1) / 2; c.ch = (gout.H - c.ph + 1) / 2; c.cw = (gout.W - c.pw + 1) / 2;
    if (c.cd <= 0 || c.ch <= 0 || c.cw <= 0) continue;
    c.nd = 1 + c.pd; c.nh = 1 + c.ph; c.nw = 1 + c.pw;
    c.M = (long)N * c.cd * c.ch * c.cw;
    mmax = std::max(mmax, c.M);
    p.c[p.nc++] = c;
  }
  *e = launch_rows<true>(p, mmax, (unsigned)(p.nc * splits), StoreRows{out, Cin}, s);
  return true;
}

bool conv_wgrad_taps(const u16* x, const u16* gz, const ConvGeom& g, long P, int Cout, int splits, float* part,
                     hipStream_t s, hipError_t* e) {
  if (Cout % 8 != 0 || (g.C != 1 && g.C % 8 != 0)) return false;
  const long K = 27L * g.C, kchunk = ((P + splits - 1) / splits + 31) / 32 * 32;
  const unsigned nz = tiles(P, kchunk);
  if (g.C == 1)
    hipLaunchKernelGGL((k_conv_wgrad<32, 32, true>), dim3(tiles(Cout, 32), 1, nz), dim3(256), 0, s, x, gz, g, P, Cout,
                       kchunk, part);
  else
    hipLaunchKernelGGL((k_conv_wgrad<64, 64, false>), dim3(tiles(Cout, 64), tiles(K, 64), nz), dim3(256), 0, s, x, gz,
                       g, P, Cout, kchunk, part);
  *e = hipGetLastError();
  return true;
}

}  // namespace wo
