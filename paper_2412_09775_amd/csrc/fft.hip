// FFT passes and the per-frequency operators of the linear model.
//
// A 3D real transform is three passes over HBM: rows along X (real <-> half
// spectrum, two real rows packed into one complex line), columns along Y
// (strided, tiles of W contiguous half-spectrum columns staged through LDS),
// and columns along Z.  The Z pass is fused with the per-frequency operator
// (forward H F, Tikhonov solve, or adjoint H^H R) and the inverse Z transform,
// so the spectrum of every channel visits HBM once between the Y passes.
#include <algorithm>

#include "internal.hpp"

namespace wo {

// Column lengths with compiled stages, and those among them with the tile loop.
static bool loop_length(int n) {
  switch (n) {
#define X_(NN) case NN:
    WO_ALL_SIZES(X_)
#undef X_
    return true;
    default:
      return false;
  }
}
static bool compiled_length(int n) {
  switch (n) {
#define X_(NN) case NN:
    WO_EVEN_SIZES(X_)
    WO_Z_ONLY_SIZES(X_)
#undef X_
    return true;
    default:
      return loop_length(n);
  }
}

// ------------------------------------------------------------------ columns

// band: 0 every row; 1 stores only the band rows (ky, nb) of the transform;
// 2 loads only the band rows (the others are taken as zero).  At most 64
// VGPRs (8 waves per SIMD), so that two 1024-thread workgroups share a CU.
template <int NS, int WS, bool TB = kTableTwiddles<NS>>
__global__ __launch_bounds__(1024, 8) void k_cols(float2* __restrict__ data, int N, long M, int Wrt,
                                               long tiles_m, long planes_per_group,
                                               long group_stride, FftPlan plan, float sign,
                                               int band, int ky, int nb) {
  const int W = WS > 0 ? WS : Wrt;             // a power of two
  const int wsh = WS > 0 ? pow2_shift(WS) : pow2_shift(Wrt);
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + N;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long bid = xcd_block();
  const long tile = bid % tiles_m;
  const long plane = bid / tiles_m;
  const long pg = plane / planes_per_group, pi = plane - pg * planes_per_group;
  float2* base = data + (pg * group_stride + pi) * (long)N * M;
  const long m0 = tile * W;
  const int weff = (int)min((long)W, M - m0);
  const int Nc = NS > 0 ? NS : N;
  auto ld_ok = [&](int l, int n) { return l < weff && (band != 2 || in_band(n, ky, nb, Nc)); };
  auto st_ok = [&](int l, int n) { return l < weff && (band != 1 || in_band(n, ky, nb, Nc)); };
  TwFetch twf;   // as in the row passes
  tw_begin<NS>(twf, tw, Nc, tid, nthr);
  if constexpr (NS > 0) {
    // line l = column m0 + l; first pass straight from memory, last pass
    // straight to memory.  Element offsets within the plane in 32 bits (the
    // host launches the compiled lengths only for M < 2^24 and planes below
    // 2^32 elements): a 24-bit multiply-add per element instead of a 64-bit
    // product (about 9 VALU instructions per load or store before)
    const unsigned um = (unsigned)M, uc = (unsigned)m0;
    auto off = [&](int l, int n) { return __umul24((unsigned)n, um) + uc + (unsigned)l; };
    fft_direct<NS, WS, true, kEmax, false, TB>(
        buf, W, W, 1, wsh, tw, sign, tid, nthr,
        [&](int l, int n) { return ld_ok(l, n) ? base[off(l, n)] : make_float2(0.f, 0.f); },
        [&] { tw_end(twf, tw, Nc, tid, nthr); },
        [&](int l, int n, float2 v) {
          if (st_ok(l, n)) base[off(l, n)] = v;
        });
  } else {
    tw_end(twf, tw, Nc, tid, nthr);
    gather_to_lds(buf, Nc * W, tid, nthr, [&](int e) {
      const int n = e >> wsh, w = e & (W - 1);
      return ld_ok(w, n) ? base[(long)n * M + m0 + w] : make_float2(0.f, 0.f);
    }, [] {});
    __syncthreads();
    fft_lines<NS, WS, true>(buf, LdsLines{W, W, 1, true, wsh}, plan, tw, sign, tid, nthr);
    scatter_from_lds(buf, Nc * W, tid, nthr, [&](int e, float2 v) {
      const int n = e >> wsh, w = e & (W - 1);
      if (st_ok(w, n)) base[(long)n * M + m0 + w] = v;
    });
  }
}

// k_cols for a compiled length and tile width as a loop over tiles: workgroup
// g of G transforms tiles g, g + G, ... and issues the loads of its next tile
// right after the first pass of the current one, so that they are in flight
// during its remaining passes and stores.
template <int NS, int WS>
__global__ __launch_bounds__(1024) void k_cols_loop(float2* __restrict__ data, long M, long tiles_m,
                                                    long planes_per_group, long group_stride,
                                                    long total, float sign, int band, int ky,
                                                    int nb) {
  static_assert(NS > 0 && WS > 0, "compiled length and tile width");
  constexpr int W = WS;
  constexpr int NP = StaticPlan<NS>::passes();
  const int wsh = pow2_shift(WS);
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + NS;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long G = gridDim.x;
  auto tile_at = [&](long t, long& m0, int& weff) {
    const long tile = t % tiles_m, plane = t / tiles_m;
    const long pg = plane / planes_per_group, pi = plane - pg * planes_per_group;
    m0 = tile * W;
    weff = (int)min((long)W, M - m0);
    return data + (pg * group_stride + pi) * (long)NS * M;
  };
  auto issue = [&](FirstPassRaw<NS, kEmax, false>& raw, long t) {
    long m0;
    int weff;
    const float2* base = tile_at(t, m0, weff);
    first_pass_load<NS, WS, true, kEmax, false, false>(raw, W, wsh, tid, nthr, [&](int l, int n) {
      return l < weff && (band != 2 || in_band(n, ky, nb, NS)) ? base[(long)n * M + m0 + l]
                                                               : make_float2(0.f, 0.f);
    });
  };
  fill_twiddles(tw, NS, tid, nthr);   // before the loads, as in the row passes
  FirstPassRaw<NS, kEmax, false> raw;
  long t = xcd_block();   // G <= total: every workgroup has a first tile
  issue(raw, t);
  while (t < total) {
    long m0;
    int weff;
    float2* base = tile_at(t, m0, weff);
    first_pass_store<NS, WS, true, kEmax, false, false>(raw, buf, W, W, 1, wsh, sign, tid, nthr,
                                                        [](int, int, float2 v) { return v; });
    const long tn = t + G;
    if (tn < total) issue(raw, tn);
    static_passes<NS, WS, true, kEmax, false, false, 1, NP - 1>(buf, W, W, 1, wsh, tw, sign, tid, nthr);
    last_pass_out<NS, WS, true, kEmax, false, false>(buf, W, W, 1, wsh, tw, sign, tid, nthr,
                                                     [&](int l, int n, float2 v) {
                                                       if (l < weff && (band != 1 || in_band(n, ky, nb, NS)))
                                                         base[(long)n * M + m0 + l] = v;
                                                     });
    t = tn;
  }
}

// Column tile width: W contiguous complex values per row (W = 16 is one
// 128-byte segment), limited by the elements a workgroup may own and by the
// device's LDS per workgroup (twiddles + tile).
int tile_width(int n, int ch) {
  const long lim = lds_limit_bytes() / (long)sizeof(float2);
  int W = 16;
  while (W > 1 && ((long)W * n * ch > kMaxElems || n + (long)W * n * ch > lim)) W /= 2;
  return W;
}

// Static tile width for a compiled length: 16 columns when the tile fits the
// per-workgroup element budget, else the largest power of two that does.
constexpr int static_tile_width(int n) {
  int W = 16;
  while (W > 1 && W * n > kMaxElems) W /= 2;
  return W;
}

// Schedule plan 4: the compiled transform with the compiled tile width, as the
// tile loop k_cols_loop.
constexpr int kPlanColsLoop = 4;

static bool cols_choice_ok(int N, const FftChoice& c) {
  const long elems = (long)c.w * N;
  const bool loop_ok = c.plan == kPlanColsLoop && loop_length(N) && c.w == static_tile_width(N);
  return pow2_shift(c.w) >= 0 && c.w <= 64 && elems <= kMaxElems && threads_ok(c.threads, elems) &&
         (long)(N + elems) * (long)sizeof(float2) <= lds_limit_bytes() && c.plan >= 0 &&
         (c.plan <= 3 || loop_ok);
}

// Workgroups of a tile loop: as many as are resident on the device at once
// (all of them when the occupancy query fails), at most one per tile.
static long loop_grid(const void* fn, int thr, size_t lds, long total) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, thr, lds) != hipSuccess || per < 1 || cus < 1)
    return total;
  return std::min(total, (long)per * cus);
}

static FftChoice cols_default(int N) {
  const int W = compiled_length(N) && (long)(N + static_tile_width(N) * N) * (long)sizeof(float2) <=
                                          lds_limit_bytes()
                    ? static_tile_width(N)
                    : tile_width(N, 1);
  return FftChoice{W, threads_for((long)N * W), 0};
}

hipError_t launch_cols(float2* data, int N, long M, long planes_per_group, long group_stride,
                       long ngroups, float sign, hipStream_t s, const char* tag, int band, int ky, bool table) {
  if (band < 0 || band > 2 || (band != 0 && ky < 0)) return hipErrorInvalidValue;
  const int nb = band == 0 || 2L * ky + 1 >= N ? N : 2 * ky + 1;
  const FftKey key{kFftCols, N, M, planes_per_group * ngroups, band};
  if (fft_recording())
    fft_record(key, [=] {
      return launch_cols(data, N, M, planes_per_group, group_stride, ngroups, sign, s, tag, band, ky, table);
    });
  FftChoice c;
  if (!fft_lookup(key, &c) || !cols_choice_ok(N, c)) c = cols_default(N);
  FftPlan plan;
  if (!make_plan_variant(N, c.plan, &plan)) return hipErrorInvalidValue;
  const int W = c.w;
  const long tiles = (M + W - 1) / W;
  const long nwg = tiles * planes_per_group * ngroups;
  const int thr = c.threads;
  const size_t lds = (size_t)(N + N * W) * sizeof(float2);
  ScopedTiming _t(tag, s);
#define X_(NN)                                                                                  \
  case NN:                                                                                      \
    if (c.plan == kPlanColsLoop) {                                                              \
      const void* fn = reinterpret_cast<const void*>(&k_cols_loop<NN, static_tile_width(NN)>);  \
      const long g = loop_grid(fn, thr, lds, nwg);                                              \
      hipLaunchKernelGGL((k_cols_loop<NN, static_tile_width(NN)>), dim3((unsigned)g), dim3(thr), lds, \
                         s, data, M, tiles, planes_per_group, group_stride, nwg, sign, band, ky, nb); \
    } else if (W == static_tile_width(NN))                                                      \
      hipLaunchKernelGGL((k_cols<NN, static_tile_width(NN)>), dim3((unsigned)nwg), dim3(thr), lds, \
                         s, data, N, M, W, tiles, planes_per_group, group_stride, plan, sign, band, \
                         ky, nb);                                                               \
    else                                                                                        \
      hipLaunchKernelGGL((k_cols<NN, 0>), dim3((unsigned)nwg), dim3(thr), lds, s, data, N, M, W, \
                         tiles, planes_per_group, group_stride, plan, sign, band, ky, nb);      \
    return hipGetLastError();
  // the compiled kernels index a plane in 32 bits
  const bool small_plane = M < (1L << 24) && (long)N * M < (1L << 32);
#define T_(NN)                                                                                  \
  case NN:                                                                                      \
    hipLaunchKernelGGL((k_cols<NN, static_tile_width(NN), true>), dim3((unsigned)nwg), dim3(thr), lds, \
                       s, data, N, M, W, tiles, planes_per_group, group_stride, plan, sign, band, \
                       ky, nb);                                                                 \
    return hipGetLastError();
  if (table && c.plan == 0 && small_plane && W == static_tile_width(N)) switch (N) {
      WO_LATERAL_SIZES(T_)
      default:
        break;
    }
#undef T_
  if ((c.plan == 0 || c.plan == kPlanColsLoop) && small_plane) switch (N) {
      WO_ALL_SIZES(X_)
#undef X_
#define X_(NN)                                                                                  \
  case NN:                                                                                      \
    if (W != static_tile_width(NN)) break;                                                      \
    hipLaunchKernelGGL((k_cols<NN, static_tile_width(NN)>), dim3((unsigned)nwg), dim3(thr), lds, \
                       s, data, N, M, W, tiles, planes_per_group, group_stride, plan, sign, band, \
                       ky, nb);                                                                 \
    return hipGetLastError();
      WO_EVEN_SIZES(X_)
      WO_Z_ONLY_SIZES(X_)
      default:
        break;
    }
#undef X_
  hipLaunchKernelGGL((k_cols<0, 0>), dim3((unsigned)nwg), dim3(thr), lds, s, data, N, M, W, tiles,
                     planes_per_group, group_stride, plan, sign, band, ky, nb);
  return hipGetLastError();
}

// FFT along N of the columns kx < kt of the band rows, from compact planes
// src [g][N][Ys][kt] into full planes dst [g][N][Y][Xh] (band row b is row
// band_row(b, .., Ys) of a source plane and band_row(b, .., Y) of a
// destination plane).  Workgroup: W
// consecutive columns of one band row of one plane group.  While its loads
// are in flight a workgroup also writes the zeros of its share (zrows rows
// from bid * zrows) of the rest of dst: rows outside the band, columns kx >= kt.
template <int NS, int WS>
__global__ __launch_bounds__(1024) void k_cols_expand(const float2* __restrict__ src,
                                                      float2* __restrict__ dst, int N, int Ys, int Y,
                                                      int Xh, int kt, int ky, int nb, int Wrt,
                                                      int tiles_row, long tiles_g, long zrows,
                                                      long zrows_total, int band_out, FftPlan plan,
                                                      float sign) {
  const int W = WS > 0 ? WS : Wrt;   // a power of two
  const int wsh = WS > 0 ? pow2_shift(WS) : pow2_shift(Wrt);
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + N;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long bid = xcd_block();
  const long g = bid / tiles_g;
  const long t = bid - g * tiles_g;
  const int b = (int)(t / tiles_row), j = (int)(t - (long)b * tiles_row);
  const int ys = band_row(b, ky, nb, Ys), y = band_row(b, ky, nb, Y);
  const int kx0 = j * W;
  const int weff = min(W, kt - kx0);
  // plane pitches; a band-layout destination holds the band rows in order
  const long ms = (long)Ys * kt, md = band_out ? (long)nb * kt : (long)Y * Xh;
  const float2* sb = src + g * N * ms + (long)ys * kt + kx0;
  float2* db = dst + g * N * md + (band_out ? (long)b * kt : (long)y * Xh) + kx0;
  const int Nc = NS > 0 ? NS : N;
  fill_twiddles(tw, Nc, tid, nthr);   // before the loads, as in the row passes
  auto mid = [&] {
    const long r0 = bid * zrows, r1 = min(r0 + zrows, zrows_total);
    int yr = (int)(r0 % Y);
    for (long row = r0; row < r1; ++row) {
      float2* rp = dst + row * Xh;
      for (int k = (in_band(yr, ky, nb, Y) ? kt : 0) + tid; k < Xh; k += nthr) rp[k] = make_float2(0.f, 0.f);
      if (++yr == Y) yr = 0;
    }
  };
  if constexpr (NS > 0) {
    fft_direct<NS, WS, true, kEmax, false>(
        buf, W, W, 1, wsh, tw, sign, tid, nthr,
        [&](int l, int n) { return l < weff ? sb[(long)n * ms + l] : make_float2(0.f, 0.f); }, mid,
        [&](int l, int n, float2 v) {
          if (l < weff) db[(long)n * md + l] = v;
        });
  } else {
    gather_to_lds(buf, Nc * W, tid, nthr, [&](int e) {
      const int n = e >> wsh, w = e & (W - 1);
      return w < weff ? sb[(long)n * ms + w] : make_float2(0.f, 0.f);
    }, mid);
    __syncthreads();
    fft_lines<NS, WS, true>(buf, LdsLines{W, W, 1, true, wsh}, plan, tw, sign, tid, nthr);
    scatter_from_lds(buf, Nc * W, tid, nthr, [&](int e, float2 v) {
      const int n = e >> wsh, w = e & (W - 1);
      if (w < weff) db[(long)n * md + w] = v;
    });
  }
}

hipError_t launch_cols_expand(const float2* src, float2* dst, int N, int Ys, int Y, int Xh, int kt,
                              int ky, long ngroups, float sign, hipStream_t s, bool band_out) {
  if (kt < 1 || kt > Xh || ky < 0 || Ys < 1 || Ys > Y) return hipErrorInvalidValue;
  const int nb = 2L * ky + 1 < Y ? 2 * ky + 1 : Y;
  if (nb > Ys || (nb == Y && Ys != Y)) return hipErrorInvalidValue;   // the band fits both
  const int kyn = nb == Y ? Y : ky;
  const FftChoice c = cols_default(N);
  FftPlan plan;
  if (!make_plan_variant(N, c.plan, &plan)) return hipErrorInvalidValue;
  const int W = c.w;
  const int tiles_row = (kt + W - 1) / W;
  const long tiles_g = (long)nb * tiles_row;
  const long nwg = tiles_g * ngroups;
  const int thr = c.threads;
  const size_t lds = (size_t)(N + N * W) * sizeof(float2);
  const long zrows_total = band_out ? 0 : ngroups * N * (long)Y;   // rows with zeros to write
  const long zrows = (zrows_total + nwg - 1) / nwg;
  const int bo = band_out ? 1 : 0;
  ScopedTiming _t(band_out ? "k_cols_z_band" : "k_cols_expand", s);
#define X_(NN)                                                                                  \
  case NN:                                                                                      \
    if (W != static_tile_width(NN)) break;                                                      \
    hipLaunchKernelGGL((k_cols_expand<NN, static_tile_width(NN)>), dim3((unsigned)nwg), dim3(thr), \
                       lds, s, src, dst, N, Ys, Y, Xh, kt, kyn, nb, W, tiles_row, tiles_g,       \
                       zrows, zrows_total, bo, plan, sign);                                     \
    return hipGetLastError();
  if (c.plan == 0) switch (N) {
      WO_Z_SIZES(X_)
      default:
        break;
    }
#undef X_
  hipLaunchKernelGGL((k_cols_expand<0, 0>), dim3((unsigned)nwg), dim3(thr), lds, s, src, dst, N, Ys, Y,
                     Xh, kt, kyn, nb, W, tiles_row, tiles_g, zrows, zrows_total, bo, plan, sign);
  return hipGetLastError();
}

// ------------------------------------------------------------------ polarisation bank expansion

// One thread per (z, y, k) of a patch's half-spectrum plane stack: reads the
// label-free pair there (zero off the band rows and columns k >= kt) and writes
// the 20 entries of the 5 x 4 bank, contiguous in k for each entry.
__global__ __launch_bounds__(256) void k_pol5_mix(const Coupling* __restrict__ cpl,
                                                  const float2* __restrict__ red,
                                                  float2* __restrict__ tf, int Z, int Y, int Xh,
                                                  int kt, int ky, int nb, long per_patch) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long patch = blockIdx.y;
  if (gid >= per_patch) return;
  const int k = (int)(gid % Xh);
  const long zy = gid / Xh;
  const int y = (int)(zy % Y), z = (int)(zy / Y);
  const bool on = k < kt && in_band(y, ky, nb, Y);
  float2 u = make_float2(0.f, 0.f), v = u;
  if (on) {
    const int b = (nb == Y || y <= ky) ? y : y - (Y - nb);
    const long rp = (long)Z * nb * kt;          // one reduced volume
    const float2* src = red + patch * 2 * rp + ((long)z * nb + b) * kt + k;
    u = src[0];
    v = src[rp];
  }
  const float* kf = &cpl[patch].k[0][0][0];
  float2* dst = tf + patch * 20 * per_patch + gid;
#pragma unroll
  for (int j = 0; j < 20; ++j)
    dst[j * per_patch] = on ? pol5_entry(kf[2 * j], kf[2 * j + 1], u, v) : make_float2(0.f, 0.f);
}

hipError_t launch_pol5_mix(const Coupling* cpl, const float2* red, float2* tf, int Z, int Y, int Xh,
                           int kt, int ky, int npatch, hipStream_t s) {
  if (kt < 1 || kt > Xh || ky < 0 || npatch < 1 || npatch > 65535) return hipErrorInvalidValue;
  const int nb = 2L * ky + 1 < Y ? 2 * ky + 1 : Y;
  const int kyn = nb == Y ? Y : ky;
  const long per_patch = (long)Z * Y * Xh;
  const long blocks = (per_patch + 255) / 256;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  ScopedTiming _t("k_pol5_mix", s);
  hipLaunchKernelGGL(k_pol5_mix, dim3((unsigned)blocks, (unsigned)npatch), dim3(256), 0, s, cpl, red, tf,
                     Z, Y, Xh, kt, kyn, nb, per_patch);
  return hipGetLastError();
}

// ------------------------------------------------------------------ schedule candidates

static std::vector<int> thread_options(long elems) {
  std::vector<int> t;
  for (int per : {kEmax, kEmax / 2, kEmax / 4}) {
    long thr = (elems + per - 1) / per;
    thr = ((thr + 63) / 64) * 64;
    if (thr < 64) thr = 64;
    if (thr > kMaxThreads) continue;
    bool seen = false;
    for (int x : t) seen |= x == (int)thr;
    if (!seen) t.push_back((int)thr);
  }
  return t;
}

// Radix-plan variants of n whose pass sequences differ from each other (and,
// for compiled lengths, runtime plans other than the default order).
static std::vector<int> plan_options(int n) {
  std::vector<int> v{0};
  FftPlan p0, p;
  if (!make_plan_variant(n, 1, &p0)) return v;
  std::vector<unsigned long long> seen{p0.radices};
  for (int var : {2, 3}) {
    if (!make_plan_variant(n, var, &p)) continue;
    bool dup = false;
    for (auto r : seen) dup |= r == p.radices;
    if (!dup) {
      v.push_back(var);
      seen.push_back(p.radices);
    }
  }
  return v;
}

std::vector<FftChoice> fft_candidates(const FftKey& k) {
  std::vector<FftChoice> out;
  auto add = [&](const FftChoice& c) {
    for (auto& x : out)
      if (x.w == c.w && x.threads == c.threads && x.plan == c.plan) return;
    out.push_back(c);
  };
  std::vector<int> widths{1, 2, 4, 8, 16, 32, 64};
  const std::vector<int> plans = plan_options(k.n);
  if (k.kind == kFftRowsR2C || k.kind == kFftRowsC2R) {
    const FftChoice d = rows_default(k.n);
    add(d);
    widths.push_back(d.w);
    for (int pl : plans)
      for (int w : widths)
        for (int t : thread_options((long)w * k.n)) {
          const FftChoice c{w, t, pl};
          if (rows_choice_ok(k.n, c)) add(c);
        }
  } else if (k.kind == kFftCols) {
    const FftChoice d = cols_default(k.n);
    add(d);
    for (int pl : plans)
      for (int w : widths)
        for (int t : thread_options((long)w * k.n)) {
          const FftChoice c{w, t, pl};
          if (cols_choice_ok(k.n, c)) add(c);
        }
    for (int t : thread_options((long)static_tile_width(k.n) * k.n)) {
      const FftChoice c{static_tile_width(k.n), t, kPlanColsLoop};
      if (cols_choice_ok(k.n, c)) add(c);
    }
  } else if (k.kind == kFftTfRows) {
    const FftChoice d = tf_rows_default(k.n);
    add(d);
    for (int pl : plans)
      for (int w : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32})
        for (int t : thread_options(2L * w * k.n)) {
          const FftChoice c{w, t, pl};
          if (tf_rows_choice_ok(k.n, c)) add(c);
        }
  } else if (k.kind == kFftTfFields) {
    const int Z = k.extra / 10;
    add(tf_fields_default(Z, k.m, k.batch));
    for (int w : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96}) {
      const FftChoice c{w, 0, 0};
      if (tf_fields_choice_ok(Z, c)) add(c);
    }
  } else if (k.kind == kFftZop) {
    const int P = (k.extra % 100000) / 1000, C = (k.extra / 10) % 100, mode = k.extra % 10;
    const int cin = mode == kModeForward ? P : C;
    const int cout = mode == kModeForward ? C : P;
    const int CH = cin > cout ? cin : cout;
    const FftChoice d = zop_default(k.n, CH);
    add(d);
    for (int pl : plans)
      for (int w : widths)
        for (int t : thread_options((long)w * k.n * CH)) {
          const FftChoice c{w, t, pl};
          if (zop_choice_ok(k.n, CH, c)) add(c);
        }
  }
  return out;
}

}  // namespace wo
