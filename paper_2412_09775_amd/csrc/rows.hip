// Row passes of the linear model's transforms: real rows to half-spectrum rows and
// back, two real rows packed into one complex line.  Every even length of the
// factors 2, 3 and 5 from 32 to 1024 has compiled stages (constant radices, spans,
// addresses and twiddle tables); others take the runtime plan.  450-point rows, 75
// x 270 of them: R2C 48 -> 17 us, C2R of twice as many 103 -> 28 us compiled.
#include "internal.hpp"

namespace wo {

// ------------------------------------------------------------------ rows

__device__ __forceinline__ long group_row(long r, long rpg, long stride) {
  const long g = r / rpg;
  return g * stride + (r - g * rpg);
}

template <int NS, bool TB = kTableTwiddles<NS>>
__global__ __launch_bounds__(1024) void k_rows_r2c(const float* __restrict__ in,
                                                   float2* __restrict__ out, int X, RowGroups g,
                                                   FftPlan plan, int lines_per_wg, long nlines,
                                                   int KT, int OP) {
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + X;
  // element offsets of the line's rows (row index times the row pitch), -1
  // for a missing row: no 64-bit multiply per element
  __shared__ long rin[2 * 64], rout[2 * 64];
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long nrows = g.rows_per_group * g.ngroups;
  const long line0 = (long)blockIdx.x * lines_per_wg;
  const int nl = (int)min((long)lines_per_wg, nlines - line0);
  for (int t = tid; t < 2 * nl; t += nthr) {
    const long r = 2 * line0 + t;
    rin[t] = r < nrows ? group_row(r, g.rows_per_group, g.in_stride) * X : -1;
    rout[t] = r < nrows ? group_row(r, g.rows_per_group, g.out_stride) * OP : -1;
  }
  __syncthreads();
  const int Xc = NS > 0 ? NS : X;   // compile-time length for the index arithmetic
  const int PS = NS > 0 ? kStaticPad<NS> : pad_shift(Xc);   // row padding
  const int LS = row_stride(Xc);    // padded line pitch in LDS
  // a missing second row (odd row count) loads the first row again and is
  // zeroed after the loads
  auto load = [&](int l, int i) {
    const long ra = rin[2 * l], rb = rin[2 * l + 1];
    return make_float2(in[ra + i], in[(rb >= 0 ? rb : ra) + i]);
  };
  auto finish = [&](int l, int, float2 v) { return make_float2(v.x, rin[2 * l + 1] >= 0 ? v.y : 0.f); };
  // the twiddle-table loads are issued first and written to LDS once the data
  // loads are in flight
  TwFetch twf;
  tw_begin<NS>(twf, tw, Xc, tid, nthr);
  if constexpr (NS > 0) {
    // first pass straight from memory; radices 8 ... 8 16 where that saves a
    // pass (the first radix is the same)
    static_assert(OrderedPlan<NS, false, true>::radix(0) == OrderedPlan<NS, false>::radix(0), "first pass");
    first_pass_in2<NS, 0, false, kEmax, true, false>(buf, nl, 1, LS, -1, -1.f, tid, nthr, load, finish,
                                                     [&] { tw_end(twf, tw, Xc, tid, nthr); });
    static_passes<NS, 0, false, kEmax, true, false, 1, StaticPlan<NS, true>::passes(), true, TB>(
        buf, nl, 1, LS, -1, tw, -1.f, tid, nthr);
  } else {
    tw_end(twf, tw, Xc, tid, nthr);
    gather2_to_lds(buf, nl * Xc, tid, nthr, [&](int e) {
      const int l = e / Xc;
      return load(l, e - l * Xc);
    }, [&](int e, float2 v) { return finish(e / Xc, 0, v); }, [&](int e) {
      const int l = e / Xc;
      return l * LS + row_slot(e - l * Xc, PS);
    }, [] {});
    __syncthreads();
    fft_lines<NS, 0, false, kEmax, true>(buf, LdsLines{nl, 1, LS, false, -1, true}, plan, tw, -1.f, tid,
                                         nthr);
  }
  // half-spectrum columns k < KT (all Xh, or the band a caller keeps), row pitch OP
  const float inv_kt = 1.0f / (float)KT;
#pragma unroll
  for (int i = 0; i < kEmax; ++i) {
    const int e = tid + i * nthr;
    if (e < nl * KT) {
      const int l = div_small(e, inv_kt), k = e - l * KT;
      const float2 zk = buf[l * LS + row_slot(k, PS)];
      const float2 zm = buf[l * LS + row_slot(k == 0 ? 0 : Xc - k, PS)];
      const float2 A = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
      const float2 B = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
      out[rout[2 * l] + k] = A;
      if (rout[2 * l + 1] >= 0) out[rout[2 * l + 1] + k] = B;
    }
  }
}

template <int NS>
__global__ __launch_bounds__(1024) void k_rows_c2r(const float2* __restrict__ in,
                                                   float* __restrict__ out, int X, RowGroups g,
                                                   FftPlan plan, int lines_per_wg, long nlines,
                                                   float scale, int KT, int IP) {
  extern __shared__ float2 smem[];
  float2* tw = smem;
  float2* buf = smem + X;
  __shared__ long rin[2 * 64], rout[2 * 64];
  const int tid = threadIdx.x, nthr = blockDim.x;
  const long nrows = g.rows_per_group * g.ngroups;
  const long line0 = (long)blockIdx.x * lines_per_wg;
  const int nl = (int)min((long)lines_per_wg, nlines - line0);
  for (int t = tid; t < 2 * nl; t += nthr) {   // element offsets, as in k_rows_r2c
    const long r = 2 * line0 + t;
    rin[t] = r < nrows ? group_row(r, g.rows_per_group, g.in_stride) * IP : -1;
    rout[t] = r < nrows ? group_row(r, g.rows_per_group, g.out_stride) * X : -1;
  }
  __syncthreads();
  const int Xc = NS > 0 ? NS : X;   // compile-time length for the index arithmetic
  const int PS = NS > 0 ? kStaticPad<NS> : pad_shift(Xc);   // row padding
  const int LS = row_stride(Xc);    // padded line pitch in LDS
  auto slot = [&](int e) {
    const int l = e / Xc;
    return l * LS + row_slot(e - l * Xc, PS);
  };
  // input rows of pitch IP hold the half-spectrum columns k < KT; the
  // columns beyond are zero (the condition depends on the index only, so the
  // loads stay in flight together)
  auto load = [&](int l, int k) {
    const int kk = 2 * k > Xc ? Xc - k : k;
    const long ra = rin[2 * l], rb = rin[2 * l + 1];
    float2 A = make_float2(0.f, 0.f), B = A;
    if (kk < KT) {
      A = in[ra + kk];
      B = in[(rb >= 0 ? rb : ra) + kk];
    }
    return make_float4(A.x, A.y, B.x, B.y);
  };
  auto finish = [&](int l, int k, float4 v) {
    const bool mirror = 2 * k > Xc;
    const int kk = mirror ? Xc - k : k;
    float2 A = make_float2(v.x, v.y), B = make_float2(v.z, v.w);
    if (rin[2 * l + 1] < 0) B = make_float2(0.f, 0.f);
    if (kk == 0 || 2 * kk == Xc) { A.y = 0.f; B.y = 0.f; }   // Re of the inverse ignores them
    if (mirror) { A.y = -A.y; B.y = -B.y; }
    return make_float2(A.x - B.y, A.y + B.x);
  };
  // nontemporal stores: the real result is not read again by the call, so it
  // need not displace the spectra the next passes read from the caches
  // (label-free 96x512x512: 71 -> 58 us)
  auto store = [&](int l, int i, float2 v) {
    __builtin_nontemporal_store(v.x * scale, &out[rout[2 * l] + i]);
    if (rout[2 * l + 1] >= 0) __builtin_nontemporal_store(v.y * scale, &out[rout[2 * l + 1] + i]);
  };
  TwFetch twf;   // as in k_rows_r2c
  tw_begin<NS>(twf, tw, Xc, tid, nthr);
  if constexpr (NS > 0) {
    // first pass straight from memory, last pass straight to memory (the
    // 8 ... 8 16 plan of k_rows_r2c is slower here: its 16-point last pass
    // stores from half the threads, 320 -> 339 us on 4 x 64 x 1024 rows of 1024)
    constexpr int NP = StaticPlan<NS>::passes();
    first_pass_in2<NS, 0, false, kEmax, true, false>(buf, nl, 1, LS, -1, 1.f, tid, nthr, load, finish,
                                                     [&] { tw_end(twf, tw, Xc, tid, nthr); });
    static_passes<NS, 0, false, kEmax, true, false, 1, NP - 1>(buf, nl, 1, LS, -1, tw, 1.f, tid, nthr);
    last_pass_out<NS, 0, false, kEmax, true, false>(buf, nl, 1, LS, -1, tw, 1.f, tid, nthr, store);
  } else {
    tw_end(twf, tw, Xc, tid, nthr);
    gather2_to_lds(buf, nl * Xc, tid, nthr, [&](int e) {
      const int l = e / Xc;
      return load(l, e - l * Xc);
    }, [&](int e, float4 v) {
      const int l = e / Xc;
      return finish(l, e - l * Xc, v);
    }, slot, [] {});
    __syncthreads();
    fft_lines<NS, 0, false, kEmax, true>(buf, LdsLines{nl, 1, LS, false, -1, true}, plan, tw, 1.f, tid,
                                         nthr);
    scatter_from_lds_map(buf, nl * Xc, tid, nthr, slot, [&](int e, float2 v) {
      const int l = e / Xc;
      store(l, e - l * Xc, v);
    });
  }
}

// 2048 elements per workgroup (256 threads of 8): measured on the row passes
// of 1024- and 512-point rows against 1024 to 8192 elements and 2 to 8 per
// thread, the C2R pass is 3-4 % faster than with 4096 and the R2C pass equal
// within the run-to-run spread.
static int lines_per_wg_for(int X) {
  int L = 2048 / X;
  if (L < 1) L = 1;
  if (L > 64) L = 64;
  while (L > 1 && (long)L * X > kMaxElems) --L;
  return L;
}

bool rows_choice_ok(int X, const FftChoice& c) {
  const long elems = (long)c.w * X;
  return c.w >= 1 && c.w <= 64 && elems <= kMaxElems && threads_ok(c.threads, elems) &&
         (long)(X + (long)c.w * row_stride(X)) * (long)sizeof(float2) <= lds_limit_bytes() &&
         c.plan >= 0 && c.plan <= 3;
}

FftChoice rows_default(int X) {
  const int L = lines_per_wg_for(X);
  return FftChoice{L, threads_for((long)L * X), 0};
}

// Table entry for the launch, or the default; an entry the device cannot run
// falls back to the default.
static FftChoice rows_choice(const FftKey& k) {
  FftChoice c;
  if (fft_lookup(k, &c) && rows_choice_ok(k.n, c)) return c;
  return rows_default(k.n);
}

#define WO_CASE_ROWS(K, NN)                                                                      \
  case NN:                                                                                       \
    hipLaunchKernelGGL((K<NN>), dim3((unsigned)nwg), dim3(thr), lds, s, WO_ROWS_ARGS);          \
    return hipGetLastError();

hipError_t launch_rows_r2c(const float* in, float2* out, int X, const RowGroups& g, hipStream_t s,
                           int kt, int pitch, const char* tag, bool table) {
  const int Xh = X / 2 + 1;
  const int KT = kt > 0 ? kt : Xh, OP = pitch > 0 ? pitch : Xh;
  if (KT > Xh || OP < KT) return hipErrorInvalidValue;
  const long nrows = g.rows_per_group * g.ngroups;
  const FftKey key{kFftRowsR2C, X, 0, nrows, 0};
  if (fft_recording()) fft_record(key, [=] { return launch_rows_r2c(in, out, X, g, s, KT, OP, tag, table); });
  const FftChoice c = rows_choice(key);
  FftPlan plan;
  if (!make_plan_variant(X, c.plan, &plan)) return hipErrorInvalidValue;
  const long nlines = (nrows + 1) / 2;
  const int L = c.w;
  const long nwg = (nlines + L - 1) / L;
  const int thr = c.threads;
  const size_t lds = (size_t)(X + (long)L * row_stride(X)) * sizeof(float2);
  ScopedTiming _t(tag, s);
#define WO_ROWS_ARGS in, out, X, g, plan, L, nlines, KT, OP
#define X_(NN)                                                                                   \
  case NN:                                                                                       \
    hipLaunchKernelGGL((k_rows_r2c<NN, true>), dim3((unsigned)nwg), dim3(thr), lds, s, WO_ROWS_ARGS); \
    return hipGetLastError();
  if (table && c.plan == 0) switch (X) {
      WO_LATERAL_SIZES(X_)
      default:
        break;
    }
#undef X_
#define X_(NN) WO_CASE_ROWS(k_rows_r2c, NN)
  if (c.plan == 0) switch (X) {
      WO_LATERAL_SIZES(X_)
      WO_EVEN_SIZES(X_)
      X_(32) X_(48)
      default:
        break;
    }
  hipLaunchKernelGGL((k_rows_r2c<0>), dim3((unsigned)nwg), dim3(thr), lds, s, WO_ROWS_ARGS);
#undef X_
#undef WO_ROWS_ARGS
  return hipGetLastError();
}

hipError_t launch_rows_c2r(const float2* in, float* out, int X, const RowGroups& g, float scale,
                           hipStream_t s, int kt, int pitch) {
  const int Xh = X / 2 + 1;
  const int KT = kt > 0 ? kt : Xh, IP = pitch > 0 ? pitch : Xh;
  if (KT > Xh || IP < KT) return hipErrorInvalidValue;
  const long nrows = g.rows_per_group * g.ngroups;
  const FftKey key{kFftRowsC2R, X, 0, nrows, 0};
  if (fft_recording()) fft_record(key, [=] { return launch_rows_c2r(in, out, X, g, scale, s, KT, IP); });
  const FftChoice c = rows_choice(key);
  FftPlan plan;
  if (!make_plan_variant(X, c.plan, &plan)) return hipErrorInvalidValue;
  const long nlines = (nrows + 1) / 2;
  const int L = c.w;
  const long nwg = (nlines + L - 1) / L;
  const int thr = c.threads;
  const size_t lds = (size_t)(X + (long)L * row_stride(X)) * sizeof(float2);
  ScopedTiming _t("k_rows_c2r", s);
#define WO_ROWS_ARGS in, out, X, g, plan, L, nlines, scale, KT, IP
#define X_(NN) WO_CASE_ROWS(k_rows_c2r, NN)
  if (c.plan == 0) switch (X) {
      WO_LATERAL_SIZES(X_)
      WO_EVEN_SIZES(X_)
      X_(32) X_(48)
      default:
        break;
    }
  hipLaunchKernelGGL((k_rows_c2r<0>), dim3((unsigned)nwg), dim3(thr), lds, s, WO_ROWS_ARGS);
#undef X_
#undef WO_ROWS_ARGS
  return hipGetLastError();
}

}  // namespace wo
