// Transfer-function synthesis (Table 1, scalar column) on the device.
//
// Label-free: per plane z, the direct field A_z = S P e^{i 2 pi kz (z - dz0)}
// and the scattered field B_z = P (i k_m / kz) e^{i 2 pi kz (z - dz0)} are
// generated on the lateral frequency grid (FP64 arithmetic, FP32 storage) and
// inverse-transformed along Y; a row kernel finishes the inverse transform
// along X, forms the point response c = b conj(a) / (X Y I_bg), transforms it
// forward along X and splits it into the half spectra of 2 Re c (phase) and
// -2 Im c (absorption).  The remaining Y (and, for 3D models, Z) transforms
// reuse the generic column passes.  Fluorescence does the same with the single
// field P e^{i 2 pi kz (z - dz0)} and the real PSF |h|^2 normalised to unit sum.
#include <algorithm>

#include "internal.hpp"

namespace wo {

// ------------------------------------------------------------------ parameters

// Per-patch optics travel as kernel arguments, so setting them needs no host
// staging buffer and stays asynchronous on the stream: 29 records of 120 bytes
// fill a launch's 4 KiB (256 patches of a tune: 9 launches of about 2 us, 32
// with the 8 records of before); a short argument block serves one or two.
template <int NB>
struct OpticsBatch {
  DevOptics o[NB];
};
constexpr int kOpticsBatch = 29;
static_assert(sizeof(OpticsBatch<kOpticsBatch>) <= 3584, "kernel arguments are limited to 4 KiB");

template <int NB>
__global__ void k_set_params(DevOptics* dst, OpticsBatch<NB> b, int count) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = b.o[i];
}

template <int NB>
static hipError_t set_params(DevOptics* dst, const DevOptics* host, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += NB) {
    OpticsBatch<NB> b;
    const int cnt = n - i0 < NB ? n - i0 : NB;
    for (int j = 0; j < cnt; ++j) b.o[j] = host[i0 + j];
    hipLaunchKernelGGL(k_set_params<NB>, dim3(1), dim3(64), 0, s, dst + i0, b, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_set_params(DevOptics* dst, const DevOptics* host, int n, hipStream_t s) {
  return n <= 2 ? set_params<2>(dst, host, n, s) : set_params<kOpticsBatch>(dst, host, n, s);
}

struct CouplingBatch {
  Coupling c[8];
};
static_assert(sizeof(CouplingBatch) <= 3584, "kernel arguments are limited to 4 KiB");

__global__ void k_set_coupling(Coupling* dst, CouplingBatch b, int count) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = b.c[i];
}

hipError_t launch_set_coupling(Coupling* dst, const Coupling* host, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += 8) {
    CouplingBatch b;
    const int cnt = n - i0 < 8 ? n - i0 : 8;
    for (int j = 0; j < cnt; ++j) b.c[j] = host[i0 + j];
    hipLaunchKernelGGL(k_set_coupling, dim3(1), dim3(64), 0, s, dst + i0, b, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The starting state of each virtual patch from what differs between patches
// (32 bytes, 96 patches a launch) and what they share.
constexpr int kTuneBatch = 96;
struct TuneBatch {
  TuneInit t[kTuneBatch];
};
static_assert(sizeof(TuneBatch) + sizeof(TuneShared) <= 3584, "kernel arguments are limited to 4 KiB");

__global__ __launch_bounds__(256) void k_set_tune(TuneState* dst, TuneBatch b, TuneShared c, int count,
                                                  int starts) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count * starts) return;
  const TuneInit t = b.t[i / starts];
  TuneState& d = dst[i];
  for (int k = 0; k < 4; ++k) {
    d.m[k] = d.v[k] = 0.0;
    d.lr[k] = c.lr[k];
    d.lo[k] = c.lo[k];
    d.hi[k] = k == 1 ? t.hi_na : c.hi[k];
  }
  d.eta = t.eta;
  d.nu_c = t.nu_c;
  d.band_count = t.band_count;
  d.loss = 0.0;
  for (int k = 0; k < 6; ++k) d.grad[k] = 0.0;
  for (int k = 0; k < 7; ++k) d.gab[k] = d.mab[k] = d.vab[k] = 0.0;
  d.lr_ab = c.lr_ab;
  d.bound_ab = c.bound_ab;
  d.t = 0;
  d.mask = c.mask;
  d.pad[0] = d.pad[1] = 0;
}

hipError_t launch_set_tune(TuneState* dst, const TuneInit* host, const TuneShared& shared, int np,
                           int starts, hipStream_t s) {
  for (int i0 = 0; i0 < np; i0 += kTuneBatch) {
    TuneBatch b;
    const int cnt = np - i0 < kTuneBatch ? np - i0 : kTuneBatch;
    for (int j = 0; j < cnt; ++j) b.t[j] = host[i0 + j];
    const long n = (long)cnt * starts;
    hipLaunchKernelGGL(k_set_tune, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       dst + (long)i0 * starts, b, shared, cnt, starts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------ reductions

// Deterministic workgroup sum of one double per thread (wave shuffles, then
// the wave partials in order).  Result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

// ------------------------------------------------------------------ fields, inverse Y

// ab layout per patch: field 0 (A, or the fluorescence field) [z][y][ca],
// then field 1 (B) [z][y][c]: c the compact column of the lateral frequency kx
// among B's XC kept columns (see field_column; c = kx when XC = X), ca among
// A's XA (last non-negative column KPA; XA = XC: the same columns), y one of
// the LY points of the inverse Y transform.  LY = Y is the grid's own transform; a shorter LY (still longer
// than twice the support's extent along y) samples the same band-limited
// fields more coarsely: frequency index i of the LY-point transform stands for
// the grid's frequency (i or i - LY) / (Y dy).  A workgroup owns one column tile of one patch and a
// chunk of ZC consecutive planes: the pupil values, which do not depend on z,
// are evaluated once into registers; each plane then only needs its phase.
// The workgroup of the first chunk also writes the tile's share of the pupil
// sum (sum S P^2 for label-free, sum P^2 for fluorescence) to
// partials[patch * tiles_x + tile].  ARM (NF = 1): one arm of the label-free pair
// alone (the nine-aperture model, whose apertures share B), B for opt.sector =
// kScatteredArm, else A; an instance of its own, because the choice at run time cost
// the fluorescence fields 2 us of 17 (96 x 128 x 160).
template <int NS, int NF, bool AB, bool CS, bool ARM>
__global__ __launch_bounds__(1024) void k_tf_fields_y(const DevOptics* __restrict__ opt,
                                                      Sampling sm, float2* __restrict__ ab,
                                                      double* __restrict__ partials, int W,
                                                      long tiles_x, int ZC, int XC, int KP, int LY,
                                                      int XA, int KPA, FftPlan plan) {
  __shared__ double red[kMaxThreads / 64];
  extern __shared__ float2 smem[];
  const int Y = NS > 0 ? NS : LY;   // transform length
  const int X = sm.nx, Z = sm.nz;
  // field f of this patch at plane z, row y, compact column c of B's layout;
  // nullptr where A keeps no column
  auto field_at = [&](long patch, int f, int z, int y, int c) -> float2* {
    float2* pa = ab + patch * (long)Z * Y * (NF == 2 ? XA + XC : XC);
    if (NF == 1 || f == 1) return pa + (NF == 2 ? (long)Z * Y * XA : 0) + ((long)z * Y + y) * XC + c;
    const int ca = XA == XC ? c : compact_column(field_column(c, KP, X, XC), KPA, X, XA);
    return ca < 0 ? nullptr : pa + ((long)z * Y + y) * XA + ca;
  };
  // frequency of transform index i: the grid's spacing 1 / (ny dy), wrapped at Y
  auto freq_y = [&](int i) { return (double)(i < (Y + 1) / 2 ? i : i - Y) / sm.Ly; };
  float2* tw = smem;
  float2* buf = smem + Y;
  const int tid = threadIdx.x, nthr = blockDim.x;
  fill_twiddles(tw, Y, tid, nthr);
  const long bid = xcd_block();
  const long tile = bid % tiles_x;
  const long rest = bid / tiles_x;
  const int zsplit = z_split(sm);
  const int nzc = z_chunk_count(Z, zsplit, ZC);
  const int zc = (int)(rest % nzc);
  const long patch = rest / nzc;
  int zbeg, zend;
  z_chunk_range(Z, zsplit, ZC, zc, &zbeg, &zend);
  const DevOptics o = opt[patch];
  // one field (fluorescence, or one label-free arm) or A and B
  constexpr bool fluor = NF == 1 && !ARM;
  const bool arm_b = ARM && o.sector == kScatteredArm;
  constexpr int nf = NF;
  constexpr int EPT = kEmax / NF;   // elements of a thread: Y * W * NF <= threads * kEmax
  const int x0 = (int)(tile * W);
  const int wsh = pow2_shift(W);     // W is a power of two
  const int nl = nf * W;              // lines of the tile: field f, column w (l = f W + w)
  const int lsh = pow2_shift(nl);
  if constexpr (NS > 0) {
    // The first pass of the inverse Y transform takes its inputs from registers
    // (the fields are computed where the butterfly needs them) and the last
    // pass writes to memory from registers: LDS carries only the passes
    // between.  Butterfly j of the first pass: line l = j mod nl, elements
    // ky = k + r NB0 (k = j / nl); of the last pass: outputs ky = k + r NSL.
    constexpr int NP = StaticPlan<NS>::passes();
    constexpr int R0 = StaticPlan<NS>::radix(0), NB0 = NS / R0;
    constexpr int RL = StaticPlan<NS>::radix(NP - 1), NSL = NS / RL;
    constexpr bool TB = CS || kTableTwiddles<NS>;   // the thin model's transforms (kTableTwiddles)
    constexpr int B0 = (kEmax + R0 - 1) / R0, BL = (kEmax + RL - 1) / RL;
    static_assert(NP >= 2, "compiled lateral lengths have at least two passes");
    double tkz[B0][R0];
    float fac[B0][R0];
    float ab2[AB ? B0 : 1][AB ? R0 : 1];   // 2 W(p): the aberration phase in units of pi
    {
      const double hw = soft_halfwidth(o, sm);
      const double km = o.n_medium / o.wavelength;
      const double ri = o.na_ill / o.wavelength;
      const DetAxis dax = det_axis(o);
      double cy, cx;
      source_centre(o, &cy, &cx);
      double psum = 0.0;
#pragma unroll
      for (int b = 0; b < B0; ++b) {
        const int j = tid + b * nthr;
        const int l = j & (nl - 1), k = j >> lsh;
        const int f = l >> wsh, c = x0 + (l & (W - 1));
        const int kx = field_column(c, KP, X, XC);
#pragma unroll
        for (int r = 0; r < R0; ++r) {
          tkz[b][r] = 0.0;
          fac[b][r] = 0.f;
          if constexpr (AB) ab2[b][r] = 0.f;
          if (j < nl * NB0 && c < XC) {
            const int ky = k + r * NB0;
            const double fy = freq_y(ky), fx = lateral_freq(kx, X, sm.Lx);
            const double P = det_pupil(o, dax, fy, fx, hw);
            if (P != 0.0) {
              const double kz = sqrt(fmax(km * km - (fy * fy + fx * fx), 0.0));
              tkz[b][r] = 2.0 * kz;
              if constexpr (AB) ab2[b][r] = (float)(2.0 * aberration_waves(o, fy, fx));
              if (fluor) {
                fac[b][r] = (float)P;
                psum += P * P;
              } else if (NF == 2 ? f == 0 : !arm_b) {
                double S = disc(fy - cy, fx - cx, ri, hw);
                if (o.sector >= 0 && octant(fy - cy, fx - cx) != o.sector) S = 0.0;
                fac[b][r] = (float)(S * P);
                psum += S * P * P;
              } else if (kz > 0.0) {
                fac[b][r] = (float)(P * km / kz);   // P * (i k_m / kz)
              }
            }
          }
        }
      }
      if (zc == 0) {
        const double tot = block_sum(psum, red);
        if (tid == 0) partials[patch * tiles_x + tile] = tot;
      }
    }
    // The phase pi arg(z), arg = 2 kz (z - dz0) (+ 2 W), is linear in the plane
    // position, which advances by dz within a chunk (chunks never cross the
    // jump of the wrapped axial order): each element carries its field value
    // of the current plane, the pupil factor times e^{i pi arg} (times i for
    // B), evaluated directly at the chunk's first plane (FP64 argument
    // reduction, FP32 sine and cosine) and then advanced plane by plane by
    // the step e^{i pi 2 kz dz}, one complex multiply.  Over at most ZC - 1
    // steps the products' rounding stays near 1e-6 relative.  CS (the thin
    // model, whose coarse grids average the rounding of fewer points): the step
    // is held as its rounded value and the remainder, as the rounded step alone
    // is off by up to 3e-8 rad in every plane (256 patches of 32 x 128 x 128:
    // gradient error against FP64 8.3e-7 without the remainder, 5.2e-7 with
    // it, both with twiddles as powers, 223 and 285 us; the 3D models keep the
    // plain step, 55 against 57 us).
    float2 ph[B0][R0], st[B0][R0], sl[CS ? B0 : 1][CS ? R0 : 1];
    {
      const double dzr = plane_z(zbeg, sm) - o.defocus;
#pragma unroll
      for (int b = 0; b < B0; ++b) {
        const int j = tid + b * nthr;
        const bool fa = !arm_b && ((j & (nl - 1)) >> wsh) == 0;   // A (or the fluorescence field), else B
#pragma unroll
        for (int r = 0; r < R0; ++r) {
          ph[b][r] = st[b][r] = make_float2(0.f, 0.f);
          if constexpr (CS) sl[b][r] = make_float2(0.f, 0.f);
          if (j < nl * NB0 && fac[b][r] != 0.f) {
            double arg = tkz[b][r] * dzr;
            if constexpr (AB) arg += (double)ab2[b][r];
            float sn, cs;
            sincospif((float)(arg - 2.0 * rint(0.5 * arg)), &sn, &cs);
            ph[b][r] = fa ? make_float2(fac[b][r] * cs, fac[b][r] * sn)
                          : make_float2(-fac[b][r] * sn, fac[b][r] * cs);   // e^{i phi} (i g)
            const double sa = tkz[b][r] * sm.dz;
            if constexpr (CS) {
              double sd, cd;
              sincospi(sa, &sd, &cd);
              st[b][r] = make_float2((float)cd, (float)sd);
              sl[b][r] = make_float2((float)(cd - st[b][r].x), (float)(sd - st[b][r].y));
            } else {
              sincospif((float)(sa - 2.0 * rint(0.5 * sa)), &sn, &cs);
              st[b][r] = make_float2(cs, sn);
            }
          }
        }
      }
    }
    for (int z = zbeg; z < zend; ++z) {
#pragma unroll
      for (int b = 0; b < B0; ++b) {
        const int j = tid + b * nthr;
        if (j < nl * NB0) {
          const int l = j & (nl - 1), k = j >> lsh;
          float2 v[R0];
#pragma unroll
          for (int r = 0; r < R0; ++r) {
            v[r] = ph[b][r];
            if (z + 1 < zend) {
              if constexpr (CS) ph[b][r] = cadd(cmul(ph[b][r], st[b][r]), cmul(ph[b][r], sl[b][r]));
              else ph[b][r] = cmul(ph[b][r], st[b][r]);
            }
          }
          dft_small<R0>(v, 1.f);   // span 1: no twiddles
#pragma unroll
          for (int r = 0; r < R0; ++r) buf[l + (k * R0 + r) * nl] = v[r];
        }
      }
      __syncthreads();
      static_passes<NS, 0, true, kEmax, false, false, 1, NP - 1, false, TB>(buf, nl, nl, 1, lsh, tw, 1.f, tid, nthr);
#pragma unroll
      for (int b = 0; b < BL; ++b) {
        const int j = tid + b * nthr;
        if (j < nl * NSL) {
          const int l = j & (nl - 1), k = j >> lsh;
          float2 w[RL];
          twiddles<RL, TB>(w, tw, k, true);   // span NSL = NS / RL: stride 1; the inverse
          float2 v[RL];
#pragma unroll
          for (int r = 0; r < RL; ++r) {
            v[r] = buf[l + (k + r * NSL) * nl];
            if (r > 0) v[r] = cmul(v[r], w[r]);
          }
          dft_small<RL>(v, 1.f);
          const int f = l >> wsh, c = x0 + (l & (W - 1));
          float2* dst = c < XC ? field_at(patch, f, z, 0, c) : nullptr;
          if (dst) {
            const int pitch = (NF == 2 && f == 0) ? XA : XC;
#pragma unroll
            for (int r = 0; r < RL; ++r) dst[(long)(k + r * NSL) * pitch] = v[r];
          }
        }
      }
      __syncthreads();   // the next plane's first pass writes the same LDS
    }
  } else {
    // z-independent factors of this thread's elements e = tid + i * nthr
    double tkz[EPT], sp[EPT], gg[NF == 1 ? 1 : EPT];
    float ab2[AB ? EPT : 1];   // 2 W(p): the aberration phase in units of pi
    {
      const double hw = soft_halfwidth(o, sm);
      const double km = o.n_medium / o.wavelength;
      const double ri = o.na_ill / o.wavelength;
      const DetAxis dax = det_axis(o);
      double cy, cx;
      source_centre(o, &cy, &cx);
      double psum = 0.0;
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        tkz[i] = 0.0;
        sp[i] = 0.0;
        if constexpr (AB) ab2[i] = 0.f;
        if (NF == 2) gg[i] = 0.0;
        const int e = tid + i * nthr;
        if (e < Y * W) {
          const int ky = e >> wsh, w = e & (W - 1);
          const int c = x0 + w;
          const int kx = field_column(c, KP, X, XC);
          if (c < XC) {
            const double fy = freq_y(ky), fx = lateral_freq(kx, X, sm.Lx);
            const double P = det_pupil(o, dax, fy, fx, hw);
            if (P != 0.0) {
              const double kz = sqrt(fmax(km * km - (fy * fy + fx * fx), 0.0));
              tkz[i] = 2.0 * kz;
              if constexpr (AB) ab2[i] = (float)(2.0 * aberration_waves(o, fy, fx));
              if (fluor) {
                sp[i] = P;
                psum += P * P;
              } else if (arm_b) {
                if (kz > 0.0) sp[i] = P * km / kz;
              } else {
                double S = disc(fy - cy, fx - cx, ri, hw);
                if (o.sector >= 0 && octant(fy - cy, fx - cx) != o.sector) S = 0.0;
                psum += S * P * P;
                sp[i] = S * P;
                if (NF == 2 && kz > 0.0) gg[i] = P * km / kz;   // P * (i k_m / kz)
              }
            }
          }
        }
      }
      if (zc == 0) {
        const double tot = block_sum(psum, red);
        if (tid == 0) partials[patch * tiles_x + tile] = tot;
      }
    }
    for (int z = zbeg; z < zend; ++z) {
      const double dzr = plane_z(z, sm) - o.defocus;
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const int e = tid + i * nthr;
        if (e < Y * W) {
          const int ky = e >> wsh, w = e & (W - 1);
          float2 A = make_float2(0.f, 0.f), B = make_float2(0.f, 0.f);
          if (sp[i] != 0.0 || (NF == 2 && gg[i] != 0.0)) {
            // phase 2 pi kz (z - dz0): reduce the argument (in units of pi) in FP64
            // to [-1, 1], then evaluate sin/cos in FP32
            double arg = tkz[i] * dzr;
            if constexpr (AB) arg += (double)ab2[i];
            const float rr = (float)(arg - 2.0 * rint(0.5 * arg));
            float snf, csf;
            sincospif(rr, &snf, &csf);
            const double sn = snf, cs = csf;
            A = arm_b ? make_float2((float)(-sp[i] * sn), (float)(sp[i] * cs))
                      : make_float2((float)(sp[i] * cs), (float)(sp[i] * sn));
            if (NF == 2) B = make_float2((float)(-gg[i] * sn), (float)(gg[i] * cs));   // e^{i phi} (i g)
          }
          buf[ky * nf * W + w] = A;
          if (NF == 2) buf[ky * nf * W + W + w] = B;
        }
      }
      __syncthreads();
      fft_lines<NS, 0, true>(buf, LdsLines{nf * W, nf * W, 1, true, pow2_shift(nf * W)}, plan, tw, 1.f,
                             tid, nthr);
      scatter_from_lds(buf, Y * nf * W, tid, nthr, [&](int e, float2 v) {
        const int ky = e >> (wsh + nf - 1);
        const int r = e & (nf * W - 1);
        const int f = r >> wsh, w = r & (W - 1);
        const int c = x0 + w;
        float2* dst = c < XC ? field_at(patch, f, z, ky, c) : nullptr;
        if (dst) *dst = v;
      });
      __syncthreads();
    }
  }
}

// Planes per workgroup of the z-chunked kernels: about `target` workgroups
// per launch, at most 16 planes.
int tf_z_chunk(const Sampling& sm, long tiles_x, long npatch, long target) {
  const long wg_per_plane = tiles_x * npatch;
  long zc = (long)sm.nz * wg_per_plane / target;
  if (zc < 1) zc = 1;
  if (zc > 16) zc = 16;
  if (zc > sm.nz) zc = sm.nz;
  return (int)zc;
}

bool tf_fields_choice_ok(int Z, const FftChoice& c) {
  return c.w >= 1 && c.w <= Z && c.threads == 0 && c.plan == 0;
}

// Each workgroup evaluates the z-independent pupil factors of its tile once
// (FP64 square roots and divisions) and its first plane in full, then
// advances the others by one complex multiply.  Few planes per workgroup
// repeat that set-up, many leave too few waves to hide the passes' waits, and
// a short last chunk of a half of the axis (the chunks do not cross its wrap)
// costs nearly as much as a full one.  Measured over 4..16 planes, 12 is best
// on 96x512x512 (60 tiles: 4 planes 80 us, 8 64 us, 12 55 us, 16 64 us) and on
// 64x1024x1024 (76 tiles: 6 planes 67 us, 8 64 us, 10 74 us, 12 58 us, 16 65
// us).  The default aims at about 480 workgroups and raises a chunk below 12
// planes to 12 while that still leaves 256 workgroups; the tuner picks the
// chunk by timing.
FftChoice tf_fields_default(int Z, long tiles, long npatch) {
  Sampling sm{};
  sm.nz = Z;
  const int zc = tf_z_chunk(sm, tiles, npatch, 480);
  if (zc < 12 && Z >= 12 && tiles * npatch * z_chunk_count(Z, (Z + 1) / 2, 12) >= 256)
    return FftChoice{12, 0, 0};
  return FftChoice{zc, 0, 0};
}

// Column-tile width of the field kernel: at most 4096 elements (512 threads)
// per workgroup.  The kernel synchronises its workgroup several times per
// plane, so several smaller workgroups per CU hide those waits better than
// one large one (measured: 96x512x512, 8 columns x 2 fields 169 us, 4 columns
// 135 us).
int tf_tile_width(const Sampling& sm, int ly, int fields) {
  const int nf = fields > 0 ? fields : (sm.model == kFluor3D ? 1 : 2);
  const long n = ly > 0 ? ly : sm.ny;
  const long lim = lds_limit_bytes() / (long)sizeof(float2);
  int W = 16;
  while (W > 1 && ((long)W * nf * n > 4096 || n + (long)W * nf * n > lim)) W /= 2;
  return W;
}

hipError_t launch_tf_fields_y(const DevOptics* opt, const Sampling& sm, int npatch, float2* ab,
                              double* partials, hipStream_t s, const LatSupport* sup, bool one_arm) {
  const LatSupport ls = sup ? *sup : full_support(sm);
  if (ls.xc < 1 || ls.xc > sm.nx || ls.kp < 0 || ls.kp >= ls.xc || ls.ly < 2 || ls.ly > sm.ny ||
      ls.xa < 1 || ls.xa > ls.xc || ls.kpa < 0 || ls.kpa > ls.kp ||
      ls.xa - ls.kpa > ls.xc - ls.kp)   // A's columns among B's
    return hipErrorInvalidValue;
  const int LY = ls.ly;
  const bool one_field = sm.model == kFluor3D || one_arm;
  const int xa = one_field ? ls.xc : ls.xa, kpa = one_field ? ls.kp : ls.kpa;
  FftPlan plan;
  if (!make_plan(LY, &plan)) return hipErrorInvalidValue;
  const int nf = one_field ? 1 : 2;
  const int W = tf_tile_width(sm, LY, nf);
  const long tiles = (ls.xc + W - 1) / W;
  const FftKey key{kFftTfFields, LY, tiles, (long)npatch, sm.nz * 10 + nf};
  if (fft_recording())
    fft_record(key, [=] { return launch_tf_fields_y(opt, sm, npatch, ab, partials, s, &ls, one_arm); });
  FftChoice fc;
  if (!fft_lookup(key, &fc) || !tf_fields_choice_ok(sm.nz, fc)) fc = tf_fields_default(sm.nz, tiles, npatch);
  const int ZC = fc.w;
  const long nwg = tiles * z_chunk_count(sm.nz, z_split(sm), ZC) * (long)npatch;
  const int thr = threads_for((long)LY * nf * W);
  const size_t lds = (size_t)(LY + LY * nf * W) * sizeof(float2);
  ScopedTiming _t("k_tf_fields_y", s);
#define WO_FIELDS_(NN, FF, AA, CC, RR)                                                           \
  hipLaunchKernelGGL((k_tf_fields_y<NN, FF, AA, CC, RR>), dim3((unsigned)nwg), dim3(thr), lds, s, opt, sm, \
                     ab, partials, W, tiles, ZC, ls.xc, ls.kp, LY, xa, kpa, plan)
  // compensated steps for the compiled lengths of the thin model
  const bool cs = sm.model == kLabelFreeThin;
#define WO_FIELDS(NN, AA)                                                                        \
  do {                                                                                           \
    if (one_arm) WO_FIELDS_(NN, 1, AA, false, true);                                             \
    else if (nf == 1) WO_FIELDS_(NN, 1, AA, false, false);                                       \
    else if (cs && NN > 0) WO_FIELDS_(NN, 2, AA, (NN > 0), false);                               \
    else WO_FIELDS_(NN, 2, AA, false, false);                                                    \
  } while (0)
#define X_(NN)                                                                                   \
  case NN:                                                                                       \
    if (sm.aberrated) WO_FIELDS(NN, true); else WO_FIELDS(NN, false);                            \
    return hipGetLastError();
  switch (LY) {
    WO_LATERAL_SIZES(X_)
    default:
      break;
  }
#undef X_
  if (sm.aberrated) WO_FIELDS(0, true); else WO_FIELDS(0, false);
#undef WO_FIELDS_
#undef WO_FIELDS
  return hipGetLastError();
}

// ------------------------------------------------------------------ rows: label-free

// out[patch * patch_stride + p * pstride + z * zstride + y * OP + k], k < KT,
// y < LY, p = 0 phase, 1 absorption (pstride < 0: phase only).  The fields are
// read in the compact column layout of the field kernel (XC columns, last
// non-negative column KP) and placed on an LX-point transform (frequency kx
// at index kx or LX + kx); the columns it does not store are zero.  TB: twiddles
// from the table (the thin model).
template <int NS, bool TB>
__global__ __launch_bounds__(1024) void k_tf_rows_lf(const double* __restrict__ partials,
                                                     long tiles_x, Sampling sm,
                                                     const float2* __restrict__ ab,
                                                     float2* __restrict__ out, long patch_stride,
                                                     long pstride, long zstride, int rows_per_wg,
                                                     long wg_per_patch, int XC, int KP, int KT,
                                                     int OP, int LY, int LX, int XA, int KPA,
                                                     FftPlan plan) {
  __shared__ double ibg_s;
  extern __shared__ float2 smem[];
  // transform lengths: LY rows per plane (the field kernel's), X = LX points
  // per row (compile-time for the index arithmetic)
  const int Y = LY, Z = sm.nz;
  const int X = NS > 0 ? NS : LX;
  float2* tw = smem;
  float2* buf = smem + X;
  const int tid = threadIdx.x, nthr = blockDim.x;
  fill_twiddles(tw, X, tid, nthr);
  const long patch = blockIdx.x / wg_per_patch;
  const long rpp = (long)Z * Y;
  const long row0 = (blockIdx.x - patch * wg_per_patch) * (long)rows_per_wg;
  const int nr = (int)min((long)rows_per_wg, rpp - row0);
  const int z0 = (int)(row0 / Y), y0 = (int)(row0 - (long)z0 * Y);
  const float2* a_src = ab + patch * rpp * (XA + XC);
  const float2* b_src = a_src + rpp * XA;
  const int PS = pad_shift(X);   // row padding
  const int LS = row_stride(X);      // padded line pitch in LDS
  // line 2r holds a (XA columns, last non-negative KPA), line 2r + 1 holds b
  // (XC, KP) of row r.  A column the field kernel does not store loads the
  // line's last non-negative column (a valid address, no branch, so the loads
  // of a thread stay in flight together) and is zeroed after the loads.
  auto load = [&](int t, int i) {
    const bool isb = t & 1;
    const int xc = isb ? XC : XA, kp = isb ? KP : KPA;
    const float2* src = (isb ? b_src : a_src) + (row0 + (t >> 1)) * xc;
    return src[i <= kp ? i : max(i - (X - xc), kp)];
  };
  auto kept = [&](int t, int i, float2 v) {
    const bool isb = t & 1;
    const int xc = isb ? XC : XA, kp = isb ? KP : KPA;
    return (i <= kp || i >= X - (xc - kp - 1)) ? v : make_float2(0.f, 0.f);
  };
  if constexpr (NS > 0) {
    // Inverse transforms of a and b in reversed radix order, the first pass
    // straight from memory; their last pass, the product c = b conj(a) /
    // (X Y I_bg) and the first pass of the forward transform of c run in
    // registers (the outputs of the one are the inputs of the other,
    // k + i NB); c goes to line 2r.
    constexpr int NP = StaticPlan<NS>::passes();
    constexpr int R0 = StaticPlan<NS>::radix(0);
    constexpr int NB = NS / R0;
    constexpr int BPF = (kEmax + 2 * R0 - 1) / (2 * R0);   // butterflies of a thread
    first_pass_in2<NS, 0, false, kEmax, true, true>(
        buf, 2 * nr, 1, LS, -1, 1.f, tid, nthr, load, kept,
        [&] { wave0_sum(partials + patch * tiles_x, tiles_x, &ibg_s); });   // sum S P^2
    const float cs = (float)(1.0 / ((double)X * (double)Y * ibg_s));
    static_passes<NS, 0, false, kEmax, true, true, 1, NP - 1, false, TB>(buf, 2 * nr, 1, LS, -1, tw, 1.f, tid,
                                                                         nthr);
    float2 cv[BPF][R0];
    int cr[BPF], ck[BPF];
#pragma unroll
    for (int b = 0; b < BPF; ++b) {
      const int j = tid + b * nthr;
      cr[b] = -1;
      if (j < nr * NB) {
        const int r = j / NB, k = j - r * NB;
        float2 w[R0];
        if constexpr (NP > 1) twiddles<R0, TB>(w, tw, k, true);   // span NB: stride 1; the inverse
        float2 va[R0], vb[R0];
#pragma unroll
        for (int i = 0; i < R0; ++i) {
          const int sl = RowPassSlots<NS, R0, 1>::load(k, i);
          va[i] = buf[2 * r * LS + sl];
          vb[i] = buf[(2 * r + 1) * LS + sl];
          if constexpr (NP > 1) {
            if (i > 0) {
              va[i] = cmul(va[i], w[i]);
              vb[i] = cmul(vb[i], w[i]);
            }
          }
        }
        dft_small<R0>(va, 1.f);
        dft_small<R0>(vb, 1.f);
#pragma unroll
        for (int i = 0; i < R0; ++i) cv[b][i] = cscale(cmulconj(vb[i], va[i]), cs);
        dft_small<R0>(cv[b], -1.f);
        cr[b] = r;
        ck[b] = k;
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < BPF; ++b) {
      if (cr[b] >= 0) {
#pragma unroll
        for (int i = 0; i < R0; ++i) 
          buf[2 * cr[b] * LS + RowPassSlots<NS, R0, 1>::store(ck[b] * R0, i)] = cv[b][i];
      }
    }
    __syncthreads();
    static_passes<NS, 0, false, kEmax, true, false, 1, NP, false, TB>(buf, nr, 1, 2 * LS, -1, tw, -1.f, tid, nthr);
  } else {
    gather_to_lds_map(buf, nr * 2 * X, tid, nthr, [&](int e) {
      const int t = e / X, i = e - t * X;
      return kept(t, i, load(t, i));
    }, [&](int e) {
      const int t = e / X;
      return t * LS + row_slot(e - t * X, PS);
    }, [&] { wave0_sum(partials + patch * tiles_x, tiles_x, &ibg_s); });   // sum S P^2
    __syncthreads();
    const float cs = (float)(1.0 / ((double)X * (double)Y * ibg_s));
    fft_lines<NS, 0, false, kEmax, true>(buf, LdsLines{2 * nr, 1, LS, false, -1, true}, plan, tw, 1.f,
                                         tid, nthr);
    for (int e = tid; e < nr * X; e += nthr) {
      const int r = e / X, i = row_slot(e - r * X, PS);
      const float2 a = buf[2 * r * LS + i], b = buf[(2 * r + 1) * LS + i];
      buf[2 * r * LS + i] = cscale(cmulconj(b, a), cs);
    }
    __syncthreads();
    fft_lines<NS, 0, false, kEmax, true>(buf, LdsLines{nr, 1, 2 * LS, false, -1, true}, plan, tw, -1.f,
                                         tid, nthr);
  }
  float2* op = out + patch * patch_stride;
  const float inv_kt = 1.0f / (float)KT;
  for (int e = tid; e < nr * KT; e += nthr) {
    const int r = div_small(e, inv_kt), k = e - r * KT;
    const float2 Ck = buf[2 * r * LS + row_slot(k, PS)];
    const float2 Cm = buf[2 * r * LS + row_slot(k == 0 ? 0 : X - k, PS)];
    int y = y0 + r, z = z0;
    while (y >= Y) { y -= Y; ++z; }
    const float2 U = make_float2(Ck.x + Cm.x, Ck.y - Cm.y);          // C + conj(C(-k))
    const float2 V = make_float2(-(Ck.y + Cm.y), Ck.x - Cm.x);       // i (C - conj(C(-k)))
    op[(long)z * zstride + (long)y * OP + k] = U;
    if (pstride >= 0) op[pstride + (long)z * zstride + (long)y * OP + k] = V;
  }
}

bool tf_rows_choice_ok(int X, const FftChoice& c) {
  const long elems = 2L * c.w * X;
  return c.w >= 1 && c.w <= 64 && elems <= kMaxElems && threads_ok(c.threads, elems) &&
         (long)(X + 2L * c.w * row_stride(X)) * (long)sizeof(float2) <= lds_limit_bytes() &&
         c.plan >= 0 && c.plan <= 3;
}

FftChoice tf_rows_default(int X) {
  int R = 2048 / X;                       // rows per workgroup (2 lines each)
  if (R < 1) R = 1;
  while (R > 1 && (2L * R * X > kMaxElems ||
                   (long)(X + 2L * R * row_stride(X)) * (long)sizeof(float2) > lds_limit_bytes()))
    --R;
  return FftChoice{R, threads_for(2L * R * X), 0};
}

hipError_t launch_tf_rows_labelfree(const double* partials, const Sampling& sm, int npatch,
                                    const float2* ab, float2* out, long patch_stride,
                                    long pstride, long zstride, hipStream_t s,
                                    const LatSupport* sup, int pitch) {
  const LatSupport ls = sup ? *sup : full_support(sm);
  const int LX = ls.lx, LY = ls.ly;
  if (ls.xc < 1 || ls.xc > LX || ls.kp < 0 || ls.kp >= ls.xc || ls.kt < 1 || 2 * (ls.kt - 1) > LX ||
      LX > sm.nx || LY < 2 || LY > sm.ny || ls.xa < 1 || ls.xa > ls.xc || ls.kpa < 0 ||
      ls.kpa > ls.kp || ls.xa - ls.kpa > ls.xc - ls.kp)
    return hipErrorInvalidValue;
  const int OP = pitch > 0 ? pitch : sm.nx / 2 + 1;
  if (OP < ls.kt) return hipErrorInvalidValue;
  const FftKey key{kFftTfRows, LX, LY, (long)npatch * sm.nz, pstride < 0 ? 1 : 0};
  if (fft_recording())
    fft_record(key, [=] {
      return launch_tf_rows_labelfree(partials, sm, npatch, ab, out, patch_stride, pstride, zstride, s,
                                      &ls, OP);
    });
  FftChoice c;
  if (!fft_lookup(key, &c) || !tf_rows_choice_ok(LX, c)) c = tf_rows_default(LX);
  const long tiles_x = (ls.xc + tf_tile_width(sm, LY) - 1) / tf_tile_width(sm, LY);
  FftPlan plan;
  if (!make_plan_variant(LX, c.plan, &plan)) return hipErrorInvalidValue;
  const int R = c.w;
  const long rpp = (long)sm.nz * LY;
  const long wpp = (rpp + R - 1) / R;
  const long nwg = wpp * npatch;
  const int thr = c.threads;
  const size_t lds = (size_t)(LX + 2L * R * row_stride(LX)) * sizeof(float2);
  ScopedTiming _t("k_tf_rows_lf", s);
#define WO_ROWS_LF(NN, TB)                                                                       \
  hipLaunchKernelGGL((k_tf_rows_lf<NN, TB>), dim3((unsigned)nwg), dim3(thr), lds, s, partials, tiles_x, \
                     sm, ab, out, patch_stride, pstride, zstride, R, wpp, ls.xc, ls.kp, ls.kt, OP, \
                     LY, LX, ls.xa, ls.kpa, plan)
#define X_(NN)                                                                                   \
  case NN:                                                                                       \
    if (sm.model == kLabelFreeThin) WO_ROWS_LF(NN, true);                                        \
    else WO_ROWS_LF(NN, kTableTwiddles<NN>);                                                     \
    return hipGetLastError();
  if (c.plan == 0) switch (LX) {
      WO_LATERAL_SIZES(X_)
      default:
        break;
    }
#undef X_
  WO_ROWS_LF(0, false);
#undef WO_ROWS_LF
  return hipGetLastError();
}

// ------------------------------------------------------------------ rows: nine apertures

// The phase responses of the eight sectors and the full disc, which share the
// scattered arm B and whose direct arms add up (A_8 = sum of the sectors').  a:
// [patch][8][z][y][XA], b: [patch][z][y][XC] (compact columns, last
// non-negative KPA, KP), partials: [patch][8][tiles_x].  Per row: the inverse X
// transforms of b and the eight a; at each x the nine responses 2 Re(b conj a_c)
// / (X Y I_c) (I_8 the sum of the sectors' I_c), which are real and go forward
// two to a complex line; out + (patch 9 + c) set_stride + z zstride + y OP + k,
// k < KT.  Nine inverse and five forward transforms a row, where the pairwise
// pass takes eighteen and nine and the fields' Y pass eighteen columns instead
// of nine: 48 x 512 x 512 (rows of 384) fields and rows 240 + 379 us, 76 + 321 us so;
// bound by VALU issue.  LDS line j nr + r: b (j = 0) or a_{j-1} of row r, then
// the packed responses 2j and 2j + 1.  72 VGPRs, seven waves a SIMD, in spite of up
// to 17 spills: a workgroup is five to nine waves, of which one or two more fit a CU
// (rows of 240, 12288 of them: 97 VGPRs 156 us, 72 98 us; 480: 313 and 244; 320: 159
// and 132); at 1024 points LDS holds one workgroup a CU whatever the registers.
template <int NS>
__global__ __launch_bounds__(1024, NS > 0 && NS < 1024 ? 7 : 1) void k_tf_rows_sectors(const double* __restrict__ partials, long tiles_x,
                                                          Sampling sm, const float2* __restrict__ a,
                                                          const float2* __restrict__ b,
                                                          float2* __restrict__ out, long set_stride,
                                                          long zstride, int rows_per_wg, long wg_per_patch,
                                                          LatSupport sup, int OP, FftPlan plan) {
  __shared__ double ibg_s[8];
  extern __shared__ float2 smem[];
  const int Y = sup.ly, Z = sm.nz;
  const int X = NS > 0 ? NS : sup.lx;
  float2* tw = smem;
  float2* buf = smem + X;
  const int tid = threadIdx.x, nthr = blockDim.x;
  TwFetch twf;   // as in the row passes of the linear model
  tw_begin<NS>(twf, tw, X, tid, nthr);
  const long patch = blockIdx.x / wg_per_patch;
  const long rpp = (long)Z * Y;
  const long row0 = (blockIdx.x - patch * wg_per_patch) * (long)rows_per_wg;
  const int nr = (int)min((long)rows_per_wg, rpp - row0);
  const float2* ap = a + patch * 8 * rpp * sup.xa;
  const float2* bp = b + patch * rpp * sup.xc;
  const int PS = pad_shift(X), LS = row_stride(X);
  const int z0 = (int)(row0 / Y), y0 = (int)(row0 - (long)z0 * Y);
  const float inv_nr = 1.0f / (float)nr;
  // as in k_tf_rows_lf: a column that is not stored loads a valid address and
  // is zeroed after the loads
  auto load = [&](int t, int i) {
    const int j = div_small(t, inv_nr), r = t - j * nr;
    const int xc = j == 0 ? sup.xc : sup.xa, kp = j == 0 ? sup.kp : sup.kpa;
    const float2* src = (j == 0 ? bp : ap + (long)(j - 1) * rpp * sup.xa) + (row0 + r) * xc;
    return src[i <= kp ? i : max(i - (X - xc), kp)];
  };
  auto kept = [&](int t, int i, float2 v) {
    const bool isb = t < nr;
    const int xc = isb ? sup.xc : sup.xa, kp = isb ? sup.kp : sup.kpa;
    return (i <= kp || i >= X - (xc - kp - 1)) ? v : make_float2(0.f, 0.f);
  };
  // forward and inverse transforms in batches of the lines a workgroup owns
  const int LB = nthr * kEmax / X;
  for (int l0 = 0; l0 < 9 * nr; l0 += LB) {
    const int nl = min(LB, 9 * nr - l0);
    float2* lb = buf + l0 * LS;
    if constexpr (NS > 0) {
      first_pass_in2<NS, 0, false, kEmax, true, false>(
          lb, nl, 1, LS, -1, 1.f, tid, nthr, [&](int l, int i) { return load(l0 + l, i); },
          [&](int l, int i, float2 v) { return kept(l0 + l, i, v); },
          [&] { if (l0 == 0) tw_end(twf, tw, X, tid, nthr); });
      static_passes<NS, 0, false, kEmax, true, false, 1, StaticPlan<NS>::passes()>(lb, nl, 1, LS, -1, tw, 1.f,
                                                                                   tid, nthr);
    } else {
      gather2_to_lds(lb, nl * X, tid, nthr, [&](int e) { const int l = e / X; return load(l0 + l, e - l * X); },
                     [&](int e, float2 v) { const int l = e / X; return kept(l0 + l, e - l * X, v); },
                     [&](int e) { const int l = e / X; return l * LS + row_slot(e - l * X, PS); },
                     [&] { if (l0 == 0) tw_end(twf, tw, X, tid, nthr); });
      __syncthreads();
      fft_lines<0, 0, false, kEmax, true>(lb, LdsLines{nl, 1, LS, false, -1, true}, plan, tw, 1.f, tid, nthr);
    }
  }
  {
    const int wave = tid >> 6, nw = nthr >> 6;
    for (int c = wave; c < 8; c += nw) {
      const double* p = partials + (patch * 8 + c) * tiles_x;
      double v = 0.0;
      for (long i = tid & 63; i < tiles_x; i += 64) v += p[i];
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      if ((tid & 63) == 0) ibg_s[c] = v;
    }
  }
  __syncthreads();
  float cs[9];
  {
    const double n2 = 2.0 / ((double)X * (double)Y);
    double tot = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      tot += ibg_s[c];
      cs[c] = (float)(n2 / ibg_s[c]);
    }
    cs[8] = (float)(n2 / tot);
  }
  for (int e = tid; e < nr * X; e += nthr) {
    const int r = e / X, sl = row_slot(e - r * X, PS);
    float2* p = buf + r * LS + sl;
    const float2 vb = p[0];
    float2 sum = make_float2(0.f, 0.f);
    float v[10];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float2 va = p[(long)(c + 1) * nr * LS];
      sum = cadd(sum, va);
      v[c] = cs[c] * (vb.x * va.x + vb.y * va.y);
    }
    v[8] = cs[8] * (vb.x * sum.x + vb.y * sum.y);
    v[9] = 0.f;
#pragma unroll
    for (int j = 0; j < 5; ++j) p[(long)j * nr * LS] = make_float2(v[2 * j], v[2 * j + 1]);
  }
  __syncthreads();
  for (int l0 = 0; l0 < 5 * nr; l0 += LB) {
    const int nl = min(LB, 5 * nr - l0);
    float2* lb = buf + l0 * LS;
    if constexpr (NS > 0)
      static_passes<NS, 0, false, kEmax, true, false, 0, StaticPlan<NS>::passes()>(lb, nl, 1, LS, -1, tw, -1.f,
                                                                                   tid, nthr);
    else
      fft_lines<0, 0, false, kEmax, true>(lb, LdsLines{nl, 1, LS, false, -1, true}, plan, tw, -1.f, tid, nthr);
  }
  const int KT = sup.kt;
  const float inv_kt = 1.0f / (float)KT;
  for (int e = tid; e < 5 * nr * KT; e += nthr) {
    const int l = div_small(e, inv_kt), k = e - l * KT;
    const int j = div_small(l, inv_nr), r = l - j * nr;
    const float2 zk = buf[l * LS + row_slot(k, PS)];
    const float2 zm = buf[l * LS + row_slot(k == 0 ? 0 : X - k, PS)];
    int y = y0 + r, z = z0;
    while (y >= Y) { y -= Y; ++z; }
    float2* op = out + (patch * 9 + 2 * j) * set_stride + (long)z * zstride + (long)y * OP + k;
    *op = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    if (j < 4) op[set_stride] = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
  }
}

// Rows per workgroup: about 2048 elements, and every line in LDS at once (rows up
// to some 1700 points on 160 KB); 0: longer rows, for the pairwise pass.
static int sectors_rows(int X) {
  int R = std::max(1, 2048 / (9 * X));
  return (long)(X + 9L * R * row_stride(X)) * (long)sizeof(float2) + 128 <= lds_limit_bytes() ? R : 0;
}
// Elements a workgroup owns at once, at most kMaxElems: every line, or five lines of
// longer rows and then the other four.
static long sectors_elems(int X, int R) {
  return 9L * R * X <= kMaxElems ? 9L * R * X : std::min<long>(5L * X, kMaxElems);
}

// Whether `rows` rows of X points take the shared arm.  Its second field launch and
// few, long workgroups cost a small bank more than the transforms saved (whole bank,
// shared and pairwise: 64 rows of 64 to 512 points 40-45 and 27-34 us, 512 rows of 160
// to 256 41-44 and 35-41, of 480 55 and 60; 1536 rows of 64 39 and 34, of 160 to 256
// 56-67 and 64-74, of 1024 149 and 142; 2048 rows of 64 to 512 40-107 and 40-106;
// 5120 to 6144 rows 57-280 and 64-293): from 2048 rows, or from 200000 points of rows
// up to 512.  Lengths on the runtime plan, whose 128 registers leave four waves a
// SIMD, take it where the workgroups that fit keep 85 % of those lanes busy (4096
// rows, shared to pairwise: 0.73 to 0.97 times at the eighteen such lengths, from 20
// to 900 points; of the others 1.26 at 250 points, 1.25 at 288, 1.22 at 500, but 0.73
// at 720), and beyond 1024 points, where the pairwise rows hold one pair a workgroup
// (1200 points 0.64, 1500 0.65 times).
bool tf_rows_sectors_fits(int X, long rows) {
  const int R = sectors_rows(X);
  if (R < 1) return false;
  if (X > 1024) return true;
  if (rows < 2048 && (X > 512 || rows * X < 200000)) return false;
  switch (X) {
#define X_(NN) case NN:
    WO_LATERAL_SIZES(X_)
#undef X_
    return true;
    default:
      break;
  }
  const long own = sectors_elems(X, R);
  const int waves = threads_for(own) / 64, groups = 4 / ((waves + 3) / 4);   // spread over four SIMDs
  return groups * own >= 85L * kMaxElems / 100;
}

hipError_t launch_tf_rows_sectors(const double* partials, const Sampling& sm, int npatch, const float2* a,
                                  const float2* b, float2* out, long set_stride, long zstride, int pitch,
                                  const LatSupport& ls, hipStream_t s) {
  const int LX = ls.lx, LY = ls.ly;
  const int R = sectors_rows(LX);
  if (R < 1 || ls.xc < 1 || ls.xc > LX || ls.kp < 0 || ls.kp >= ls.xc || ls.kt < 1 || 2 * (ls.kt - 1) > LX ||
      LX > sm.nx || LY < 2 || LY > sm.ny || ls.xa < 1 || ls.xa > ls.xc || ls.kpa < 0 || ls.kpa >= ls.xa ||
      pitch < ls.kt || npatch < 1)
    return hipErrorInvalidValue;
  FftPlan plan;
  if (!make_plan(LX, &plan)) return hipErrorInvalidValue;
  const long wpp = ((long)sm.nz * LY + R - 1) / R;
  const int W = tf_tile_width(sm, LY, 1);
  const long tiles = (ls.xa + W - 1) / W;
  const int thr = threads_for(sectors_elems(LX, R));
  const size_t lds = (size_t)(LX + 9L * R * row_stride(LX)) * sizeof(float2);
  ScopedTiming _t("k_tf_rows_sectors", s);
#define X_(NN)                                                                                      \
  case NN:                                                                                          \
    hipLaunchKernelGGL((k_tf_rows_sectors<NN>), dim3((unsigned)(wpp * npatch)), dim3(thr), lds, s,   \
                       partials, tiles, sm, a, b, out, set_stride, zstride, R, wpp, ls, pitch, plan); \
    return hipGetLastError();
  switch (LX) {
    WO_LATERAL_SIZES(X_)
    default:
      break;
  }
#undef X_
  hipLaunchKernelGGL((k_tf_rows_sectors<0>), dim3((unsigned)(wpp * npatch)), dim3(thr), lds, s, partials, tiles,
                     sm, a, b, out, set_stride, zstride, R, wpp, ls, pitch, plan);
  return hipGetLastError();
}

// ------------------------------------------------------------------ rows: fluorescence

// h: [patch][z][y][x] complex (after the inverse Y pass); out: [patch][z][y][Xh]
template <int NS>
__global__ __launch_bounds__(1024) void k_tf_rows_fl(const double* __restrict__ partials,
                                                     long tiles_x, Sampling sm,
                                                     const float2* __restrict__ h,
                                                     float2* __restrict__ out, int pairs_per_wg,
                                                     long wg_per_patch, FftPlan plan) {
  __shared__ double ibg_s;
  extern __shared__ float2 smem[];
  const int Y = sm.ny, X = sm.nx, Z = sm.nz, Xh = X / 2 + 1;
  float2* tw = smem;
  float2* buf = smem + X;
  const int tid = threadIdx.x, nthr = blockDim.x;
  fill_twiddles(tw, X, tid, nthr);
  const long patch = blockIdx.x / wg_per_patch;
  const long rpp = (long)Z * Y;
  const long row0 = (blockIdx.x - patch * wg_per_patch) * 2L * pairs_per_wg;
  const int nrows = (int)min(2L * pairs_per_wg, rpp - row0);
  const int np = (nrows + 1) / 2;
  const float2* src = h + patch * rpp * X;
  gather_to_lds(buf, 2 * np * X, tid, nthr, [&](int e) {
    const int l = e / X, i = e - l * X;
    return l < nrows ? src[(row0 + l) * X + i] : make_float2(0.f, 0.f);
  }, [&] { wave0_sum(partials + patch * tiles_x, tiles_x, &ibg_s); });   // sum P^2
  __syncthreads();
  fft_lines<NS, 0, false>(buf, LdsLines{2 * np, 1, X, false}, plan, tw, 1.f, tid, nthr);
  const double norm = 1.0 / ((double)Z * (double)X * (double)Y * ibg_s);
  const float nm = (float)norm;
  for (int e = tid; e < np * X; e += nthr) {
    const int q = e / X, i = e - q * X;
    const float2 u = buf[2 * q * X + i], v = buf[(2 * q + 1) * X + i];
    buf[2 * q * X + i] = make_float2((u.x * u.x + u.y * u.y) * nm, (v.x * v.x + v.y * v.y) * nm);
  }
  __syncthreads();
  fft_lines<NS, 0, false>(buf, LdsLines{np, 1, 2 * X, false}, plan, tw, -1.f, tid, nthr);
  float2* op = out + patch * rpp * Xh;
  for (int e = tid; e < np * Xh; e += nthr) {
    const int q = e / Xh, k = e - q * Xh;
    const float2 zk = buf[2 * q * X + k];
    const float2 zm = buf[2 * q * X + (k == 0 ? 0 : X - k)];
    const long r0 = row0 + 2 * q;
    op[r0 * Xh + k] = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    if (r0 + 1 < rpp && 2 * q + 1 < nrows)
      op[(r0 + 1) * Xh + k] = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
  }
}

hipError_t launch_tf_rows_fluor(const double* partials, const Sampling& sm, int npatch,
                                const float2* h, float2* out, hipStream_t s) {
  const long tiles_x = (sm.nx + tf_tile_width(sm) - 1) / tf_tile_width(sm);
  FftPlan plan;
  if (!make_plan(sm.nx, &plan)) return hipErrorInvalidValue;
  int Q = 2048 / sm.nx;                       // row pairs per workgroup
  if (Q < 1) Q = 1;
  while (Q > 1 && 2L * Q * sm.nx > kMaxElems) --Q;
  const long rpp = (long)sm.nz * sm.ny;
  const long wpp = (rpp + 2 * Q - 1) / (2 * Q);
  const long nwg = wpp * npatch;
  const int thr = threads_for(2L * Q * sm.nx);
  const size_t lds = (size_t)(sm.nx + 2 * Q * sm.nx) * sizeof(float2);
  ScopedTiming _t("k_tf_rows_fl", s);
#define X_(NN)                                                                                   \
  case NN:                                                                                       \
    hipLaunchKernelGGL((k_tf_rows_fl<NN>), dim3((unsigned)nwg), dim3(thr), lds, s, partials, tiles_x, \
                       sm, h, out, Q, wpp, plan);                                                \
    return hipGetLastError();
  switch (sm.nx) {
    WO_LATERAL_SIZES(X_)
    default:
      break;
  }
#undef X_
  hipLaunchKernelGGL((k_tf_rows_fl<0>), dim3((unsigned)nwg), dim3(thr), lds, s, partials, tiles_x, sm, h,
                     out, Q, wpp, plan);
  return hipGetLastError();
}

}  // namespace wo
