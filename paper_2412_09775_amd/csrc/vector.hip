// Vector label-free transfer functions (Table 1, vector column, label-free row).
//
// The bank correlates two tensor-valued fields per plane z.  The detected
// scattered field of a unit dipole along n, u_i'n = IFFT2[P_i'j G_jn prop],
// and the detected direct field of the source times the conjugate incident
// field that drives the dipole, v_ik = IFFT2[S P_ik' e_k' conj(e_k) prop].
// The aplanatic pupil map Q(p) (3 x 2) gives both: the incident field of
// source point q is e = Q J, the detection tensor is P E Q^T, and its
// columns are transverse to the wave, so P E Q^T (I - k^ k^T) g = P E g Q^T.
// The direct light reaches the detector as P E J, so v_ik = J_i w_k with
// w_k = IFFT2[S P E conj(e_k) prop].  Q is real with five distinct entries q_a
// (Q_xy = Q_yx), so every field is one of, or a constant mix of, ten transforms:
//   U_a = IFFT2[i P E g q_a prop]     (u_i'n = U_a(n, i')),
//   W_a = IFFT2[S P E q_a prop]       (w_k = conj(J_x) W_a(k, 0) + conj(J_y) W_a(k, 1)),
// whatever the number of illumination states (a single state takes its three
// w_k instead of the five W_a).  A channel c (state s, analyser M_c) then responds to
// property p (tensor T_p) with
//   R_cp = 1 / (Y X I_bg) sum_n,k beta_n T_p^{nk} conj(w_k),
//   beta_n = sum_i' alpha_c,i' u_i'n,  alpha_c = J_s^H M_c,
// and H_cp = FFT3(2 Re R_cp).  The spectra vanish outside the detection
// pupil's columns: they are written on those columns only and inverse-
// transformed along Y there (column passes).  With a compiled row length one kernel per row
// (k_vec_rows) inverse-transforms the fields along X, forms every channel's real
// responses and transforms those forward, on the support's shortened lengths;
// otherwise a complex row pass writes the fields on the grid, k_vec_products
// multiplies them per voxel, and the row pass of the linear model transforms
// the responses.  The column passes of the linear model do the rest, on the
// bank's support.
#include <algorithm>

#include "internal.hpp"

namespace wo {

struct VecBatch {
  VecRec r[4];
};
static_assert(sizeof(VecBatch) <= 3584, "kernel arguments are limited to 4 KiB");

__global__ void k_set_vec(VecRec* dst, VecBatch b, int count) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = b.r[i];
}

hipError_t launch_set_vec(VecRec* dst, const VecRec* host, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += 4) {
    VecBatch b;
    const int cnt = n - i0 < 4 ? n - i0 : 4;
    for (int j = 0; j < cnt; ++j) b.r[j] = host[i0 + j];
    hipLaunchKernelGGL(k_set_vec, dim3(1), dim3(64), 0, s, dst + i0, b, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Entry a of the map Q read as Q_n,i' (n = x, y, z; i' = x, y).
constexpr int kQ[3][2] = {{0, 1}, {1, 2}, {3, 4}};
// Fields of a model with NS illumination states: five U, then the three w of a
// single state or the five W that every state mixes.
template <int NS>
struct VecFields {
  static constexpr int kW = NS == 1 ? 3 : 5;
  static constexpr int kF = 5 + kW;
};
int vec_fields(int NS) { return NS == 1 ? VecFields<1>::kF : VecFields<5>::kF; }

// w_k of channel state s at one point from the model's W fields there (W(a)).
template <int NS, typename WF>
__device__ __forceinline__ void vec_w(const VecRec& r, int s, WF W, float2 (&w)[3]) {
  if constexpr (NS == 1) {
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = W(k);
  } else {
    const float2 jx = make_float2(r.J[s][0][0], -r.J[s][0][1]), jy = make_float2(r.J[s][1][0], -r.J[s][1][1]);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = cadd(cmul(jx, W(kQ[k][0])), cmul(jy, W(kQ[k][1])));
  }
}

// One thread per lateral frequency (ky, kx) of one patch and chunk of planes:
// the pupil values and the map Q in FP64, then each plane's propagator phase.
// Q is written without angles: with w = 1 / (k_m (k_m + kz)),
//   Q = [[1 - px^2 w, -px py w], [-px py w, 1 - py^2 w], [-px / k_m, -py / k_m]].
// LY rows: row i of the LY-point transform stands for the grid's frequency
// (i or i - LY) / (ny dy); LY = ny is the grid's own transform, a shorter one
// (longer than twice the band) samples the same band-limited fields more
// coarsely along y.  Bound by its writes; one wave per 64 columns and 16 planes
// keeps the chip busy where a row's columns fill half of a 256-thread
// workgroup (5 states, 64 x 512 x 512: 21 fields in 65 us, 10 in 37).
constexpr int kVecPlanes = 16;
template <int NS>
__global__ __launch_bounds__(64) void k_vec_spectra(const DevOptics* __restrict__ opt,
                                                     const VecRec* __restrict__ rec, Sampling sm,
                                                     float2* __restrict__ fields, int XC, int KP, int LY) {
  constexpr int F = VecFields<NS>::kF;
  const int X = sm.nx, Z = sm.nz;
  const int nzc = (Z + kVecPlanes - 1) / kVecPlanes;
  const int zc = blockIdx.x % nzc;
  const int c = (blockIdx.x / nzc) * 64 + threadIdx.x;
  const int ky = blockIdx.y;
  const long patch = blockIdx.z;
  if (c >= XC) return;
  const int kx = field_column(c, KP, X, XC);
  const DevOptics o = opt[patch];
  const long plane = (long)LY * XC;
  float2* base = fields + patch * (long)F * Z * plane + (long)ky * XC + c;
  const double fy = (double)(ky < (LY + 1) / 2 ? ky : ky - LY) / sm.Ly;
  const double fx = lateral_freq(kx, X, sm.Lx);
  const double hw = soft_halfwidth(o, sm);
  const double km = o.n_medium / o.wavelength;
  const DetAxis dax = det_axis(o);
  const double P = det_pupil(o, dax, fy, fx, hw);
  double cy, cx;
  source_centre(o, &cy, &cx);
  const double S = disc(fy - cy, fx - cx, o.na_ill / o.wavelength, hw);
  const double kz = sqrt(fmax(km * km - (fy * fy + fx * fx), 0.0));
  float q[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
  float gp = 0.f, sp = 0.f;
  if (P != 0.0 && kz > 0.0) {
    const double w = 1.0 / (km * (km + kz));
    q[0] = (float)(1.0 - fx * fx * w);
    q[1] = (float)(-fx * fy * w);
    q[2] = (float)(1.0 - fy * fy * w);
    q[3] = (float)(-fx / km);
    q[4] = (float)(-fy / km);
    gp = (float)(P * km / kz);
    sp = (float)(S * P);
  }
  float2 ce[3];   // a single state: conj(e_k) = conj(Q_k0 Jx + Q_k1 Jy)
  if constexpr (NS == 1) vec_w<5>(rec[patch], 0, [&](int a) { return make_float2(q[a], 0.f); }, ce);   // J mixes the q_a
  const double ab2 = (gp != 0.f) ? 2.0 * aberration_waves(o, fy, fx) : 0.0;
  const int z1 = min(Z, (zc + 1) * kVecPlanes);
  for (int z = zc * kVecPlanes; z < z1; ++z) {
    float sn = 0.f, cs = 0.f;
    if (gp != 0.f) {
      const double arg = 2.0 * kz * (plane_z(z, sm) - o.defocus) + ab2;   // phase / pi
      sincospif((float)(arg - 2.0 * rint(0.5 * arg)), &sn, &cs);
    }
    float2* pz = base + (long)z * plane;
#pragma unroll
    for (int a = 0; a < 5; ++a) {
      const float g = gp * q[a];
      pz[(long)a * Z * plane] = make_float2(-g * sn, g * cs);   // i g e^{i phi}
    }
    const float2 e = make_float2(sp * cs, sp * sn);
#pragma unroll
    for (int a = 0; a < VecFields<NS>::kW; ++a) {
      float2 v;
      if constexpr (NS == 1) v = cmul(e, ce[a]);
      else v = cscale(e, q[a]);
      pz[(long)(5 + a) * Z * plane] = v;
    }
  }
}

hipError_t launch_vec_spectra(const DevOptics* opt, const VecRec* rec, const Sampling& sm, int npatch, int NS,
                              float2* fields, int XC, int KP, int LY, hipStream_t s) {
  if ((NS != 1 && NS != 5) || npatch < 1 || npatch > 65535 || LY < 2 || LY > sm.ny) return hipErrorInvalidValue;
  if (XC < 1 || XC > sm.nx || KP < 0 || KP >= XC) return hipErrorInvalidValue;
  const int nzc = (sm.nz + kVecPlanes - 1) / kVecPlanes;
  const dim3 grid((unsigned)(((XC + 63) / 64) * nzc), (unsigned)LY, (unsigned)npatch);
  ScopedTiming _t("k_vec_spectra", s);
  if (NS == 1)
    hipLaunchKernelGGL(k_vec_spectra<1>, grid, dim3(64), 0, s, opt, rec, sm, fields, XC, KP, LY);
  else
    hipLaunchKernelGGL(k_vec_spectra<5>, grid, dim3(64), 0, s, opt, rec, sm, fields, XC, KP, LY);
  return hipGetLastError();
}

// Complex FFT along X of L rows per workgroup (unnormalised; sign -1 forward,
// +1 inverse): row r of src holds the XC kept columns of the spectrum
// (field_column order, the others zero), row r of dst receives all X values.
// Compiled lengths (NS > 0) take the first pass from memory and write the
// last one to memory from registers, as the real row passes do; other
// lengths use the runtime plan.
template <int NS>
__global__ __launch_bounds__(1024) void k_rows_c2c(const float2* __restrict__ src, float2* __restrict__ dst,
                                                   int X, int XC, int KP, long nrows, FftPlan plan, int L,
                                                   float sign) {
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + X;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long row0 = (long)blockIdx.x * L;
  const int nl = (int)min((long)L, nrows - row0);
  const int Xc = NS > 0 ? NS : X;
  const int PS = pad_shift(Xc), LS = row_stride(Xc);
  const float2* in = src + row0 * XC;
  float2* out = dst + row0 * Xc;
  // the condition depends on the index only, so the loads stay in flight together
  auto load = [&](int l, int k) {
    const int c = compact_column(k, KP, Xc, XC);
    return c >= 0 ? in[(long)l * XC + c] : make_float2(0.f, 0.f);
  };
  fill_twiddles(tw, Xc, tid, nthr);
  if constexpr (NS > 0) {
    constexpr int NP = StaticPlan<NS>::passes();
    auto finish = [](int, int, float2 v) { return v; };
    auto store = [&](int l, int i, float2 v) { out[(long)l * NS + i] = v; };
    first_pass_in2<NS, 0, false, kEmax, true, false>(buf, nl, 1, LS, -1, sign, tid, nthr, load, finish,
                                                     [] {});
    static_passes<NS, 0, false, kEmax, true, false, 1, NP - 1>(buf, nl, 1, LS, -1, tw, sign, tid, nthr);
    last_pass_out<NS, 0, false, kEmax, true, false>(buf, nl, 1, LS, -1, tw, sign, tid, nthr, store);
  } else {
    auto slot = [&](int e) {
      const int l = e / Xc;
      return l * LS + row_slot(e - l * Xc, PS);
    };
    gather2_to_lds(buf, nl * Xc, tid, nthr, [&](int e) {
      const int l = e / Xc;
      return load(l, e - l * Xc);
    }, [](int, float2 v) { return v; }, slot, [] {});
    __syncthreads();
    fft_lines<0, 0, false, kEmax, true>(buf, LdsLines{nl, 1, LS, false, -1, true}, plan, tw, sign, tid,
                                        nthr);
    __syncthreads();
    scatter_from_lds_map(buf, nl * Xc, tid, nthr, slot, [&](int e, float2 v) { out[e] = v; });
  }
}

hipError_t launch_rows_c2c(const float2* src, float2* dst, int X, int XC, int KP, long nrows, float sign,
                           hipStream_t s) {
  if (X < 2 || nrows < 1 || XC < 1 || XC > X || KP < 0 || KP >= XC) return hipErrorInvalidValue;
  FftPlan plan;
  if (!make_plan(X, &plan)) return hipErrorInvalidValue;
  int L = 2048 / X;   // 2048 elements per workgroup, as the real row passes
  if (L < 1) L = 1;
  while (L > 1 && (long)L * X > kMaxElems) --L;
  if ((long)L * X > kMaxElems) return hipErrorInvalidValue;
  const size_t lds = (size_t)(X + (long)L * row_stride(X)) * sizeof(float2);
  if ((long)lds > lds_limit_bytes()) return hipErrorInvalidValue;
  const long nwg = (nrows + L - 1) / L;
  const int thr = threads_for((long)L * X);
  ScopedTiming _t("k_rows_c2c", s);
#define X_(NN)                                                                                       \
  case NN:                                                                                           \
    hipLaunchKernelGGL((k_rows_c2c<NN>), dim3((unsigned)nwg), dim3(thr), lds, s, src, dst, X, XC, KP, \
                       nrows, plan, L, sign);                                                        \
    return hipGetLastError();
  switch (X) {
    WO_LATERAL_SIZES(X_)
    default:
      break;
  }
#undef X_
  hipLaunchKernelGGL((k_rows_c2c<0>), dim3((unsigned)nwg), dim3(thr), lds, s, src, dst, X, XC, KP, nrows, plan,
                     L, sign);
  return hipGetLastError();
}

// The P responses of channel c (state s of w) at one point from the fields
// there: beta_n = sum_i' alpha_c,i' u_i'n, then sc Re(sum_n,k T_p^{nk} beta_n
// conj(w_k)) for every property p: put(p, value), p < P <= kVecProps.
constexpr int kVecProps = 8;
template <int NS, typename UF, typename WF, typename PUT>
__device__ __forceinline__ void vec_channel(const VecRec& r, int c, int P, float sc, UF U, WF W, PUT put) {
  const float2 a0 = make_float2(r.alpha[c][0][0], r.alpha[c][0][1]);
  const float2 a1 = make_float2(r.alpha[c][1][0], r.alpha[c][1][1]);
  float2 w[3], qm[3][3];
  vec_w<NS>(r, NS == 1 ? 0 : c, W, w);
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    const float2 b = cadd(cmul(a0, U(kQ[n][0])), cmul(a1, U(kQ[n][1])));
#pragma unroll
    for (int k = 0; k < 3; ++k) qm[n][k] = cmulconj(b, w[k]);
  }
#pragma unroll
  for (int p = 0; p < kVecProps; ++p) {
    if (p >= P) break;
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 9; ++e) acc += r.T[p][e][0] * qm[e / 3][e % 3].x - r.T[p][e][1] * qm[e / 3][e % 3].y;
    put(p, sc * acc);
  }
}

// Row lengths without compiled stages: one thread per voxel of one patch, from
// the fields on the grid.  NS is a template parameter so that the per-field
// arrays stay in registers.
template <int NS>
__global__ __launch_bounds__(256) void k_vec_products(const VecRec* __restrict__ rec,
                                                      const float2* __restrict__ fields,
                                                      float* __restrict__ out, long vox) {
  constexpr int C = NS == 1 ? 4 : 5, F = VecFields<NS>::kF;
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long patch = blockIdx.y;
  if (i >= vox) return;
  const VecRec& r = rec[patch];
  const int P = r.P;
  const float2* fp = fields + patch * (long)F * vox + i;
  float2 f[F];
#pragma unroll
  for (int a = 0; a < F; ++a) f[a] = fp[(long)a * vox];
  const float sc = 2.f * r.scale;
  float* op = out + patch * (long)C * P * vox + i;
#pragma unroll
  for (int c = 0; c < C; ++c)
    vec_channel<NS>(r, c, P, sc, [&](int a) { return f[a]; }, [&](int a) { return f[5 + a]; },
                    [&](int p, float v) { op[(long)(c * P + p) * vox] = v; });
}

hipError_t launch_vec_products(const VecRec* rec, const float2* fields, float* out, long vox, int NS, int npatch,
                               hipStream_t s) {
  if (vox < 1 || npatch < 1 || npatch > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((vox + 255) / 256), (unsigned)npatch);
  ScopedTiming _t("k_vec_products", s);
  if (NS == 1)
    hipLaunchKernelGGL(k_vec_products<1>, grid, dim3(256), 0, s, rec, fields, out, vox);
  else if (NS == 5)
    hipLaunchKernelGGL(k_vec_products<5>, grid, dim3(256), 0, s, rec, fields, out, vox);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// Compiled row lengths N (the grid's X or a shorter length that holds the
// responses' band without wrap-around): one workgroup per row (patch, z, y).
// The row's F fields are inverse-transformed along X from their XC kept columns
// in LDS, each x gets its C P responses, these
// replace the fields in LDS as real rows, two per complex line, and are
// transformed forward; the columns k < KT of each leave for the Y pass.  So
// neither the fields on the grid nor the responses visit HBM.  Bound by VALU
// issue (about 20 transforms and C N contractions of 160 instructions a row).
// 5 states x 4 properties, 64 x 512 x 512 (rows of 256): 21 fields, responses
// through HBM and a row pass 328 + 111 us, 308 us so.
// More lines than a workgroup owns at once go in batches.  BATCH: the responses
// of every channel do not fit LDS (five states, seven or eight properties, rows of
// 1024: 18 or 20 lines where 17 fit), so cb channels at a time are formed and
// transformed in the lines behind the fields, which stay; as many as fit, because
// a batch costs two barriers and a pass over the fields (8 x 512 x 1024, the bank:
// 7 properties 758 us, 8 849 us; per-channel rows and a row pass of their own
// took 808 and 879).
template <int NS, int N, bool BATCH = false>
__global__ __launch_bounds__(1024) void k_vec_rows(const VecRec* __restrict__ rec,
                                                   const float2* __restrict__ spec,
                                                   float2* __restrict__ out, int XC, int KP, int KT, long zy,
                                                   int cb) {
  constexpr int C = NS == 1 ? 4 : 5, F = VecFields<NS>::kF;
  constexpr bool SPLIT = F * N > kMaxElems;             // the fields in two batches
  constexpr int NB = SPLIT ? 5 : F;                      // lines of the first batch
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + N;
  const int LS = row_stride(N), PS = pad_shift(N);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long rowid = blockIdx.x;
  const long patch = rowid / zy, r = rowid - patch * zy;
  const VecRec& rv = rec[patch];
  const float2* sp = spec + patch * (long)F * zy * XC + r * XC;
  TwFetch twf;   // as in the row passes of the linear model
  tw_begin<N>(twf, tw, N, tid, nthr);
  constexpr int NP = StaticPlan<N>::passes();
#pragma unroll
  for (int l0 = 0; l0 < F; l0 += NB) {
    const int nl = F - l0 < NB ? F - l0 : NB;
    first_pass_in<N, 0, false, kEmax, true, false>(
        buf + l0 * LS, nl, 1, LS, -1, 1.f, tid, nthr,
        [&](int l, int k) {
          const int cc = compact_column(k, KP, N, XC);
          return cc >= 0 ? sp[(long)(l0 + l) * zy * XC + cc] : make_float2(0.f, 0.f);
        },
        [&] { if (l0 == 0) tw_end(twf, tw, N, tid, nthr); });
    static_passes<N, 0, false, kEmax, true, false, 1, NP>(buf + l0 * LS, nl, 1, LS, -1, tw, 1.f, tid, nthr);
  }
  // Response q = c P + p is the real (q even) or imaginary part of line q / 2
  // (BATCH: q counts from the batch's first response).
  // One thread owns point x of every line, so it may replace the fields there as
  // soon as it has read them; the channel index is uniform, so the constants of
  // a channel stay in scalar registers.
  const int P = rv.P, CB = BATCH ? cb : C;
  const float sc = 2.f * rv.scale_short;
  const int LB = nthr * kEmax / N;   // lines a workgroup owns at once
  const float inv_kt = 1.0f / (float)KT;
  float2* rb = BATCH ? buf + F * LS : buf;   // the responses' lines
  for (int c0 = 0; c0 < C; c0 += CB) {
    const int nq = min(CB, C - c0) * P, nlo = (nq + 1) / 2;
    for (int x = tid; x < N; x += nthr) {
      const int sl = row_slot(x, PS);
      float2 f[F];
#pragma unroll
      for (int a = 0; a < F; ++a) f[a] = buf[a * LS + sl];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        if (BATCH && (c < c0 || c >= c0 + CB)) continue;
        vec_channel<NS>(rv, c, P, sc, [&](int a) { return f[a]; }, [&](int a) { return f[5 + a]; },
                        [&](int p, float v) {
                          const int q = (BATCH ? c - c0 : c) * P + p;
                          ((float*)(rb + (q >> 1) * LS + sl))[q & 1] = v;
                        });
      }
      if (nq & 1) ((float*)(rb + (nlo - 1) * LS + sl))[1] = 0.f;
    }
    __syncthreads();
    for (int l0 = 0; l0 < nlo; l0 += LB)
      static_passes<N, 0, false, kEmax, true, false, 0, NP>(rb + l0 * LS, min(LB, nlo - l0), 1, LS, -1, tw, -1.f,
                                                            tid, nthr);
    float2* op = out + ((patch * C + c0) * (long)P * zy + r) * KT;
    for (int e = tid; e < nlo * KT; e += nthr) {
      const int l = div_small(e, inv_kt), k = e - l * KT;
      const float2 zk = rb[l * LS + row_slot(k, PS)];
      const float2 zm = rb[l * LS + row_slot(k == 0 ? 0 : N - k, PS)];
      op[(long)(2 * l) * zy * KT + k] = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
      if (2 * l + 1 < nq)
        op[(long)(2 * l + 1) * zy * KT + k] = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
    }
    if (BATCH) __syncthreads();   // the next batch writes the lines just read
  }
}

bool vec_rows_fused(int X) {
  switch (X) {
#define X_(NN) case NN:
    WO_LATERAL_SIZES(X_)
#undef X_
    return true;
    default:
      return false;
  }
}

hipError_t launch_vec_rows(const VecRec* rec, const float2* spec, float2* out, int X, int XC, int KP, int KT,
                           long zy, int NS, int P, int npatch, hipStream_t s) {
  if (!vec_rows_fused(X) || (NS != 1 && NS != 5) || zy < 1 || npatch < 1 || XC < 1 || XC > X || KP < 0 ||
      KP >= XC || KT < 1 || KT > X / 2 + 1 || P < 1 || P > kVecProps)
    return hipErrorInvalidValue;
  const int F = vec_fields(NS), C = NS == 1 ? 4 : 5;
  const long nwg = (long)npatch * zy;
  if (nwg > 0x7fffffffL) return hipErrorInvalidValue;
  const int thr = threads_for((long)((long)F * X > kMaxElems ? 5 : F) * X);
  // every channel's responses in place of the fields where they fit LDS, else as
  // many channels at a time as fit behind the fields (rows of 1024 only: the lines
  // of shorter rows always fit)
  const long most = (lds_limit_bytes() / (long)sizeof(float2) - X) / row_stride(X);   // lines
  const bool batch = (C * P + 1) / 2 > most;
  const int cb = batch ? (int)std::min<long>(C, std::max<long>(0, 2 * (most - F) / P)) : C;
  if (most < F || cb < 1 || (batch && (NS != 5 || X != 1024))) return hipErrorInvalidValue;
  const long lines = batch ? F + (cb * P + 1) / 2 : std::max(F, (C * P + 1) / 2);
  const size_t lds = (size_t)(X + lines * row_stride(X)) * sizeof(float2);
  ScopedTiming _t("k_vec_rows", s);
  if (batch) {
    hipLaunchKernelGGL((k_vec_rows<5, 1024, true>), dim3((unsigned)nwg), dim3(thr), lds, s, rec, spec, out, XC, KP,
                       KT, zy, cb);
    return hipGetLastError();
  }
#define X_(NN)                                                                                       \
  case NN:                                                                                           \
    if (NS == 1)                                                                                     \
      hipLaunchKernelGGL((k_vec_rows<1, NN>), dim3((unsigned)nwg), dim3(thr), lds, s, rec, spec, out, XC, KP, \
                         KT, zy, cb);                                                                \
    else                                                                                             \
      hipLaunchKernelGGL((k_vec_rows<5, NN>), dim3((unsigned)nwg), dim3(thr), lds, s, rec, spec, out, XC, KP, \
                         KT, zy, cb);                                                                \
    return hipGetLastError();
  switch (X) {
    WO_LATERAL_SIZES(X_)
    default:
      break;
  }
#undef X_
  return hipErrorInvalidValue;
}

}  // namespace wo
