// BF16 storage and the MFMA operand types shared by the convolution kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace wo {

typedef unsigned short u16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u16 f2bf(float f) {  // round to nearest even
  unsigned u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (u16)(u >> 16);  // inf / nan
  u += 0x7fffu + ((u >> 16) & 1u);
  return (u16)(u >> 16);
}
__device__ __forceinline__ float bf2f(u16 b) { return __uint_as_float(((unsigned)b) << 16); }

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

struct ConvGeom {
  int D, H, W, C;     // input volume and channels
  int Do, Ho, Wo;     // output volume
};

// The three convolution products on tap-sized K steps (conv.hip).  Each
// returns false where it does not take the shape; *e is the launch's status.
//   forward: C_q[p][co] partials of split q, or (z, a, b not null) the
//     pre-activation z = sum + b and a = BF16(GELU(z)) with one split
//   input gradient: out[q][position][ci] per split
//   weight gradient: part[q][co][tap * Cin + ci] per split of kchunk positions
struct ConvFwdOut {
  float* c;          // partials (a null)
  float* z;
  u16* a;
  const float* bias;
};
bool conv_fwd_taps(const u16* x, const u16* w, const ConvGeom& g, long P, int Cout, int splits,
                   const ConvFwdOut& out, hipStream_t s, hipError_t* e);
bool conv_dgrad_taps(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, int splits, float* out,
                     hipStream_t s, hipError_t* e);
bool conv_wgrad_taps(const u16* x, const u16* gz, const ConvGeom& g, long P, int Cout, int splits, float* part,
                     hipStream_t s, hipError_t* e);

}  // namespace wo
