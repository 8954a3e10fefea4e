// The per-frequency operators of the linear model (forward H F, Tikhonov solve,
// adjoint H^H R) and the Z pass fused with them.
#include <algorithm>

#include "internal.hpp"

namespace wo {

// ------------------------------------------------------------------ per-frequency operators
//
// Channel values of one frequency sit at cell[ch * cs].  H(c, p) returns the
// transfer-function value of channel c and property p at this frequency.
// forward: y_c = sum_p H_cp x_p (+ N b_c at DC)
// solve:   F = (H^H H + eta I)^-1 H^H (x - N b delta)      (Eq. tls_solution)
// adjoint: y_p = sum_c conj(H_cp) x_c
// Outputs are scaled by inv_n (the 1/N of the inverse transform).

// CT > 0 fixes the channel count at compile time (static register indexing);
// CT == 0 takes it from Crt.
template <int P, int CT, typename HF>
__device__ __forceinline__ void freq_op(float2* cell, long cs, HF H, int Crt, int mode, float eta,
                                        const float* __restrict__ bg, bool dc, float n_full,
                                        float inv_n) {
  const int C = CT > 0 ? CT : Crt;
  if (mode == kModeForward) {
    float2 x[P];
#pragma unroll
    for (int p = 0; p < P; ++p) x[p] = cell[p * cs];
    for (int c = 0; c < C; ++c) {
      float2 y = make_float2(0.f, 0.f);
#pragma unroll
      for (int p = 0; p < P; ++p) y = cadd(y, cmul(H(c, p), x[p]));
      if (dc && bg) y.x += n_full * bg[c];
      cell[c * cs] = cscale(y, inv_n);
    }
    return;
  }
  if (mode == kModeAdjoint) {
    float2 y[P];
#pragma unroll
    for (int p = 0; p < P; ++p) y[p] = make_float2(0.f, 0.f);
    for (int c = 0; c < C; ++c) {
      const float2 xc = cell[c * cs];
#pragma unroll
      for (int p = 0; p < P; ++p) y[p] = cadd(y[p], cmul(cconj(H(c, p)), xc));
    }
#pragma unroll
    for (int p = 0; p < P; ++p) cell[p * cs] = cscale(y[p], inv_n);
    return;
  }
  if constexpr (CT == 1) {
    // one channel: H is a row h, and (h^H h + eta I)^-1 h^H = h^H / (h h^H + eta)
    // (Sherman-Morrison), so F_p = conj(h_p) x / (sum_q |h_q|^2 + eta)
    float2 xc = cell[0];
    if (dc && bg) xc.x -= n_full * bg[0];
    float2 h[P];
    float den = eta;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      h[p] = H(0, p);
      den += h[p].x * h[p].x + h[p].y * h[p].y;
    }
    const float sc = den > 0.f ? inv_n * __builtin_amdgcn_rcpf(den) : 0.f;   // hardware reciprocal
#pragma unroll
    for (int p = 0; p < P; ++p) cell[p * cs] = cscale(cmulconj(xc, h[p]), sc);
    return;
  }
  // solve: accumulate the lower triangle of M = H^H H, M_pq = sum_c conj(H_cp) H_cq,
  // and r = H^H x
  float2 m[P][P];
  float2 r[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    r[p] = make_float2(0.f, 0.f);
#pragma unroll
    for (int q = 0; q < P; ++q) m[p][q] = make_float2(0.f, 0.f);
  }
  for (int c = 0; c < C; ++c) {
    float2 xc = cell[c * cs];
    if (dc && bg) xc.x -= n_full * bg[c];
    float2 h[P];
#pragma unroll
    for (int p = 0; p < P; ++p) h[p] = H(c, p);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      r[p] = cadd(r[p], cmul(cconj(h[p]), xc));
#pragma unroll
      for (int q = 0; q <= p; ++q) m[p][q] = cadd(m[p][q], cmul(cconj(h[p]), h[q]));
    }
  }
  float2 F[P];
  if (P == 1) {
    const float den = m[0][0].x + eta;
    F[0] = den > 0.f ? cscale(r[0], __builtin_amdgcn_rcpf(den)) : make_float2(0.f, 0.f);
  } else {
    chol_solve<P>(m, r, eta, F);
  }
#pragma unroll
  for (int p = 0; p < P; ++p) cell[p * cs] = cscale(F[p], inv_n);
}

// The polarisation solve from the reduced bank at one frequency: with
// H_cp = Kr_cp u + Ki_cp v (u = H_phase, v = H_abs there), H^H H has the entries
// A |u|^2 + B |v|^2 + S Re(conj(u) v) + i D Im(conj(u) v) (constants of the
// coupling) and H^H x = conj(u) Kr^T x + conj(v) Ki^T x, so the 5 x 4 bank is
// never formed.  Algebraically the solve of freq_op with that bank.
__device__ __forceinline__ void pol5_solve(float2* cell, long cs, float2 u, float2 v,
                                           const Coupling* __restrict__ cp, float eta,
                                           const float* __restrict__ bg, bool dc, float n_full,
                                           float inv_n) {
  float2 yr[4], yi[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) yr[p] = yi[p] = make_float2(0.f, 0.f);
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    float2 xc = cell[c * cs];
    if (dc && bg) xc.x -= n_full * bg[c];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      yr[p] = cadd(yr[p], cscale(xc, cp->k[c][p][0]));
      yi[p] = cadd(yi[p], cscale(xc, cp->k[c][p][1]));
    }
  }
  const float uu = u.x * u.x + u.y * u.y, vv = v.x * v.x + v.y * v.y;
  const float2 w = cmulconj(v, u);   // conj(u) v
  float2 m[4][4], r[4], F[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    r[p] = cadd(cmulconj(yr[p], u), cmulconj(yi[p], v));
#pragma unroll
    for (int q = 0; q <= p; ++q) {
      const int e = p * (p + 1) / 2 + q;
      m[p][q] = make_float2(cp->a[e] * uu + cp->b[e] * vv + cp->s[e] * w.x, cp->d[e] * w.y);
    }
  }
  chol_solve<4>(m, r, eta, F);
#pragma unroll
  for (int p = 0; p < 4; ++p) cell[p * cs] = cscale(F[p], inv_n);
}

constexpr int kTfPrefetch = 8;   // transfer-function values a thread may hold in registers

// Geometry of the fused Z pass.  A plane of the spectrum holds R rows of row
// pitch Ls (plane pitch Ms), a plane of the bank R rows of pitch Lt (plane
// pitch Mt), or only the band rows in band order (bank_band); the pass covers
// the columns k < kt of the band rows (band_row: ky, nb) in tiles of W columns
// that do not cross a row.  The plain layout is one row: R = 1,
// Ls = Lt = kt = Ms = Mt = M, nb = 1.
struct ZopGeom {
  long Ms, Mt, Ls, Lt, kt;
  int R, ky, nb, tiles_row, bank_band;
};

// With compiled stages at most 72 VGPRs (7 waves per SIMD); no instance spills
// but the unreduced 5 x 4 bank's at 16, 18, 24, 27, 75, 96 and 128 planes (one or
// two registers each); the runtime-plan instances keep their allocation (they
// would spill).
// RED: tf holds the polarisation bank in reduced form, [2][Z][..] per patch
// (H_phase, H_abs), and the coupling cpl[patch] forms H_cp per frequency.
template <int P, int CT, int NS, bool RED>
__global__ __launch_bounds__(1024, NS > 0 ? 7 : 1) void k_zop(float2* __restrict__ spec,
                                              const float2* __restrict__ tf, int C, int Z, ZopGeom gm,
                                              int slots, int W, long tiles_m, FftPlan plan,
                                              int mode, float eta, const float* __restrict__ bg,
                                              float inv_n, float n_full,
                                              const Coupling* __restrict__ cpl) {
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + Z;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long bid = xcd_block();
  const long tile = bid % tiles_m;
  const long patch = bid / tiles_m;
  const int Zc = NS > 0 ? NS : Z;   // compile-time length for the index arithmetic
  const int wsh = pow2_shift(W);    // W is a power of two
  const int cin = mode == kModeForward ? P : C;
  const int cout = mode == kModeForward ? C : P;
  const int CH = cin > cout ? cin : cout;
  const long Ms = gm.Ms, Mt = gm.Mt;
  float2* sp = spec + patch * (long)slots * Z * Ms;
  const float2* tp = tf + patch * (long)(RED ? 2 : C * P) * Z * Mt;
  const float* bp = bg ? bg + patch * C : nullptr;
  const int brow = (int)(tile / gm.tiles_row);
  const long col0 = (tile - (long)brow * gm.tiles_row) * W;
  const int row = band_row(brow, gm.ky, gm.nb, gm.R);
  const long m0 = row * gm.Ls + col0;        // tile start in a spectrum plane
  const long mt0 = (gm.bank_band ? brow : row) * gm.Lt + col0;   // and in a bank plane
  const bool dc_tile = row == 0 && col0 == 0;
  const int weff = (int)min((long)W, gm.kt - col0);
  // Element (plane, w) of the tile: a plane pitch is below 2^32 (checked on
  // the host), so its offset is one 32 x 32 -> 64-bit multiply, not a 64-bit
  // product per element.
  float2* const st = sp + m0;
  const float2* const tt = tp + mt0;
  const unsigned ums = (unsigned)Ms, umt = (unsigned)Mt;
  auto soff = [&](int plane) { return (long)((unsigned long)(unsigned)plane * ums); };
  auto toff = [&](int plane) { return (long)((unsigned long)(unsigned)plane * umt); };
  // Issue this thread's transfer-function loads first: they complete while the
  // data tile is loaded and transformed.  Frequency f = tid + i * nthr.
  const int nfreq = Zc * W;
  const int fpt = (nfreq + nthr - 1) / nthr;
  // entries of the bank a frequency reads: P (one channel) or the pair (reduced)
  constexpr int NE = RED ? 2 : P;
  constexpr int NPF = RED ? 4 : kTfPrefetch;   // registers for the prefetched entries
  const bool prefetch = (RED || CT == 1) && NE * fpt <= NPF;
  float2 hreg[NPF];
  if (prefetch) {
#pragma unroll
    for (int j = 0; j < NPF; ++j) {
      const int i = j / NE, cp = j - i * NE;
      const int f = tid + i * nthr;
      if (i < fpt && f < nfreq) {
        const int z = f >> wsh, w = f & (W - 1);
        hreg[j] = w < weff ? tt[toff(cp * Zc + z) + w] : make_float2(0.f, 0.f);
      }
    }
  }
  TwFetch twf;   // as in the row passes
  tw_begin<NS>(twf, tw, Zc, tid, nthr);
  // LDS holds [z][ch][w]: line l = ch W + w, element z at z CH W
  if constexpr (NS > 0) {
    // first pass of the forward Z transform straight from memory
    first_pass_in<NS, 0, true, kEmax, false, false>(
        buf, cin * W, CH * W, 1, pow2_shift(cin * W), -1.f, tid, nthr,
        [&](int l, int z) {
          const int ch = l >> wsh, w = l & (W - 1);
          return w < weff ? st[soff(ch * Zc + z) + w] : make_float2(0.f, 0.f);
        },
        [&] { tw_end(twf, tw, Zc, tid, nthr); });
    static_passes<NS, 0, true, kEmax, false, false, 1, StaticPlan<NS>::passes()>(
        buf, cin * W, CH * W, 1, pow2_shift(cin * W), tw, -1.f, tid, nthr);
  } else {
    tw_end(twf, tw, Zc, tid, nthr);
    // element e = (ch, z, w) of the global tile goes to LDS [z][ch][w]
    float2 t[kEmax];
#pragma unroll
    for (int i = 0; i < kEmax; ++i) {
      const int e = tid + i * nthr;
      if (e < cin * Zc * W) {
        const int w = e & (W - 1), r = e >> wsh;
        const int z = r % Zc, ch = r / Zc;
        t[i] = w < weff ? st[soff(ch * Zc + z) + w] : make_float2(0.f, 0.f);
      }
    }
#pragma unroll
    for (int i = 0; i < kEmax; ++i) {
      const int e = tid + i * nthr;
      if (e < cin * Zc * W) {
        const int w = e & (W - 1), r = e >> wsh;
        const int z = r % Zc, ch = r / Zc;
        buf[(z * CH + ch) * W + w] = t[i];
      }
    }
    __syncthreads();
    fft_lines<NS, 0, true>(buf, LdsLines{cin * W, CH * W, 1, true, pow2_shift(cin * W)}, plan, tw, -1.f,
                           tid, nthr);
  }
  if (prefetch) {
#pragma unroll
    for (int i = 0; i < NPF / NE; ++i) {
      const int f = tid + i * nthr;
      if (i < fpt && f < nfreq) {
        const int z = f >> wsh, w = f & (W - 1);
        if (w < weff) {
          const bool dcf = z == 0 && dc_tile && w == 0;
          if constexpr (RED) {
            const float2 hph = hreg[i * 2], hab = hreg[i * 2 + 1];
            const float* kf = &cpl[patch].k[0][0][0];
            if (mode == kModeSolve)
              pol5_solve(buf + (long)z * CH * W + w, W, hph, hab, cpl + patch, eta, bp, dcf, n_full, inv_n);
            else
              freq_op<P, CT>(buf + (long)z * CH * W + w, W,
                             [&](int c, int p) {
                               return pol5_entry(kf[(c * P + p) * 2], kf[(c * P + p) * 2 + 1], hph, hab);
                             },
                             C, mode, eta, bp, dcf, n_full, inv_n);
          } else {
            freq_op<P, 1>(buf + (long)z * CH * W + w, W,
                          [&](int c, int p) { return hreg[i * P + p]; }, C, mode, eta, bp, dcf, n_full,
                          inv_n);
          }
        }
      }
    }
  } else {
    for (int f = tid; f < nfreq; f += nthr) {
      const int z = f >> wsh, w = f & (W - 1);
      if (w >= weff) continue;
      const float2* hp = tt + w;
      if constexpr (RED) {
        const float2 hph = hp[toff(z)], hab = hp[toff(Zc + z)];
        const float* kf = &cpl[patch].k[0][0][0];
        if (mode == kModeSolve)
          pol5_solve(buf + (long)z * CH * W + w, W, hph, hab, cpl + patch, eta, bp,
                     z == 0 && dc_tile && w == 0, n_full, inv_n);
        else
          freq_op<P, CT>(buf + (long)z * CH * W + w, W,
                         [&](int c, int p) {
                           return pol5_entry(kf[(c * P + p) * 2], kf[(c * P + p) * 2 + 1], hph, hab);
                         },
                         C, mode, eta, bp, z == 0 && dc_tile && w == 0, n_full, inv_n);
      } else {
        freq_op<P, CT>(buf + (long)z * CH * W + w, W,
                       [&](int c, int p) { return hp[toff((c * P + p) * Zc + z)]; }, C, mode, eta, bp,
                       z == 0 && dc_tile && w == 0, n_full, inv_n);
      }
    }
  }
  __syncthreads();
  if constexpr (NS > 0) {
    // last pass of the inverse Z transform straight to memory
    static_passes<NS, 0, true, kEmax, false, false, 0, StaticPlan<NS>::passes() - 1>(
        buf, cout * W, CH * W, 1, pow2_shift(cout * W), tw, 1.f, tid, nthr);
    last_pass_out<NS, 0, true, kEmax, false, false>(
        buf, cout * W, CH * W, 1, pow2_shift(cout * W), tw, 1.f, tid, nthr,
        [&](int l, int z, float2 v) {
          const int ch = l >> wsh, w = l & (W - 1);
          if (w < weff) st[soff(ch * Zc + z) + w] = v;
        });
  } else {
    fft_lines<NS, 0, true>(buf, LdsLines{cout * W, CH * W, 1, true, pow2_shift(cout * W)}, plan, tw, 1.f,
                           tid, nthr);
    float2 t[kEmax];
#pragma unroll
    for (int i = 0; i < kEmax; ++i) {
      const int e = tid + i * nthr;
      if (e < cout * Zc * W) {
        const int w = e & (W - 1), r = e >> wsh;
        const int z = r % Zc, ch = r / Zc;
        t[i] = buf[(z * CH + ch) * W + w];
      }
    }
#pragma unroll
    for (int i = 0; i < kEmax; ++i) {
      const int e = tid + i * nthr;
      if (e < cout * Zc * W) {
        const int w = e & (W - 1), r = e >> wsh;
        const int z = r % Zc, ch = r / Zc;
        if (w < weff) st[soff(ch * Zc + z) + w] = t[i];
      }
    }
  }
}

template <int P, int CT, bool RED = false>
static void zop_launch(bool use_static, long nwg, int thr, size_t lds, hipStream_t s, float2* spec,
                       const float2* tf, int C, int Z, const ZopGeom& gm, int slots, int W, long tiles,
                       FftPlan plan, int mode, float eta, const float* bg, float inv_n, float nf,
                       const Coupling* cpl) {
#define X_(NN)                                                                                   \
  case NN:                                                                                       \
    hipLaunchKernelGGL((k_zop<P, CT, NN, RED>), dim3((unsigned)nwg), dim3(thr), lds, s, spec, tf, C, Z, \
                       gm, slots, W, tiles, plan, mode, eta, bg, inv_n, nf, cpl);                \
    return;
  if (use_static) switch (Z) {
      WO_Z_SIZES(X_)
      default:
        break;
    }
#undef X_
  hipLaunchKernelGGL((k_zop<P, CT, 0, RED>), dim3((unsigned)nwg), dim3(thr), lds, s, spec, tf, C, Z, gm,
                     slots, W, tiles, plan, mode, eta, bg, inv_n, nf, cpl);
}

bool zop_choice_ok(int Z, int CH, const FftChoice& c) {
  const long elems = (long)c.w * Z * CH;
  return pow2_shift(c.w) >= 0 && c.w <= 64 && elems <= kMaxElems && threads_ok(c.threads, elems) &&
         (long)(Z + elems) * (long)sizeof(float2) <= lds_limit_bytes() && c.plan >= 0 && c.plan <= 3;
}

// At most 4096 elements per workgroup (8 per thread, 512 threads): the pass
// waits on its loads and stores between short bursts of arithmetic, and
// smaller workgroups let more of them share a CU (5 channels x 64 planes:
// 8 columns 249 us, 16 columns 282 us on the 64x1024x1024 volume).
FftChoice zop_default(int Z, int CH) {
  int W = tile_width(Z, CH);
  while (W > 1 && (long)W * Z * CH > 4096) W /= 2;
  return FftChoice{W, threads_for((long)CH * Z * W), 0};
}

bool zop_fits(int Z, int CH) { return zop_choice_ok(Z, CH, zop_default(Z, CH)); }

hipError_t launch_zop(float2* spec, const float2* tf, int C, int P, int Z, long M, int slots,
                      int npatch, int mode, float eta, const float* bg, float inv_n, double n_full,
                      hipStream_t s, const SpecBand* band, const Coupling* cpl) {
  if (cpl && (P != 4 || C != 5)) return hipErrorInvalidValue;
  if (band && (band->Y < 1 || M % band->Y != 0 || band->kt < 1 || band->kt > M / band->Y ||
               band->ky < 0))
    return hipErrorInvalidValue;
  const bool hb = band != nullptr;
  const SpecBand bc = hb ? *band : SpecBand{1, M, 0, 0};
  const int nbr = hb ? (2L * bc.ky + 1 >= bc.Y ? bc.Y : 2 * bc.ky + 1) : 1;
  const long mcov = hb ? (long)nbr * bc.kt : M;   // columns the pass covers per plane
  const FftKey key{kFftZop, Z, mcov, npatch,
                   P * 1000 + C * 10 + mode + (hb ? 100000 : 0) + (cpl ? 200000 : 0)};
  if (fft_recording())
    fft_record(key, [=] {
      return launch_zop(spec, tf, C, P, Z, M, slots, npatch, mode, eta, bg, inv_n, n_full, s,
                        hb ? &bc : nullptr, cpl);
    });
  const int cin = mode == kModeForward ? P : C;
  const int cout = mode == kModeForward ? C : P;
  const int CH = cin > cout ? cin : cout;
  FftChoice c;
  if (!fft_lookup(key, &c) || !zop_choice_ok(Z, CH, c)) c = zop_default(Z, CH);
  FftPlan plan;
  if (!make_plan_variant(Z, c.plan, &plan)) return hipErrorInvalidValue;
  const int W = c.w;
  ZopGeom gm;
  gm.R = bc.Y;
  gm.kt = bc.kt;
  gm.Ls = bc.kt;
  gm.bank_band = hb && bc.bank_band;
  gm.Lt = gm.bank_band ? bc.kt : M / bc.Y;
  gm.Ms = (long)bc.Y * bc.kt;
  gm.Mt = gm.bank_band ? (long)nbr * bc.kt : M;
  gm.nb = nbr;
  gm.ky = nbr == bc.Y ? bc.Y : bc.ky;
  if (gm.Ms >= (1L << 32) || gm.Mt >= (1L << 32)) return hipErrorInvalidValue;   // 32-bit plane offsets
  gm.tiles_row = (int)((bc.kt + W - 1) / W);
  const long tiles = (long)nbr * gm.tiles_row;
  const long nwg = tiles * npatch;
  const int thr = c.threads;
  const size_t lds = (size_t)(Z + CH * Z * W) * sizeof(float2);
  const float nf = (float)n_full;
  const bool st = c.plan == 0;
  ScopedTiming _t(P == 1 ? "k_zop<1>" : (P == 2 ? "k_zop<2>" : "k_zop<4>"), s);
#define WO_ZOP(PP, CC) \
  zop_launch<PP, CC>(st, nwg, thr, lds, s, spec, tf, C, Z, gm, slots, W, tiles, plan, mode, eta, bg, inv_n, nf, \
                     nullptr)
  if (cpl) zop_launch<4, 5, true>(st, nwg, thr, lds, s, spec, tf, C, Z, gm, slots, W, tiles, plan, mode, eta,
                                  bg, inv_n, nf, cpl);
  else if (P == 1) { if (C == 1) WO_ZOP(1, 1); else WO_ZOP(1, 0); }
  else if (P == 2) { if (C == 1) WO_ZOP(2, 1); else WO_ZOP(2, 0); }
  else if (P == 4) { if (C == 5) WO_ZOP(4, 5); else WO_ZOP(4, 0); }
  else return hipErrorInvalidValue;
#undef WO_ZOP
  return hipGetLastError();
}

template <int P>
__global__ __launch_bounds__(256) void k_op2d(float2* __restrict__ spec,
                                              const float2* __restrict__ tf, int C, long M,
                                              int slots, int mode, float eta,
                                              const float* __restrict__ bg, float inv_n,
                                              float n_full, long blocks_per_patch,
                                              const float* __restrict__ eta_pp) {
  const long patch = blockIdx.x / blocks_per_patch;
  const long m = (blockIdx.x - patch * blocks_per_patch) * (long)blockDim.x + threadIdx.x;
  if (m >= M) return;
  if (eta_pp) eta = eta_pp[patch];
  float2* sp = spec + patch * (long)slots * M;
  const float2* tp = tf + patch * (long)C * P * M;
  const float* bp = bg ? bg + patch * C : nullptr;
  const float2* hp = tp + m;
  freq_op<P, 0>(sp + m, M, [&](int c, int p) { return hp[(long)(c * P + p) * M]; }, C, mode, eta,
                bp, m == 0, n_full, inv_n);
}

hipError_t launch_op2d(float2* spec, const float2* tf, int C, int P, long M, int slots, int npatch,
                       int mode, float eta, const float* bg, float inv_n, double n_full,
                       hipStream_t s, const float* eta_pp) {
  const long bpp = (M + 255) / 256;
  const long nwg = bpp * npatch;
  const float nf = (float)n_full;
  switch (P) {
    case 1:
      { ScopedTiming _t("k_op2d<1>", s);
      hipLaunchKernelGGL(k_op2d<1>, dim3((unsigned)nwg), dim3(256), 0, s, spec, tf, C, M, slots,
                         mode, eta, bg, inv_n, nf, bpp, eta_pp); }
      break;
    case 2:
      { ScopedTiming _t("k_op2d<2>", s);
      hipLaunchKernelGGL(k_op2d<2>, dim3((unsigned)nwg), dim3(256), 0, s, spec, tf, C, M, slots,
                         mode, eta, bg, inv_n, nf, bpp, eta_pp); }
      break;
    case 4:
      { ScopedTiming _t("k_op2d<4>", s);
      hipLaunchKernelGGL(k_op2d<4>, dim3((unsigned)nwg), dim3(256), 0, s, spec, tf, C, M, slots,
                         mode, eta, bg, inv_n, nf, bpp, eta_pp); }
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace wo
