// BF16 storage and the MFMA operand types shared by the convolution kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace wo {

typedef unsigned short u16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Rounded to nearest even by the conversion instruction.
__device__ __forceinline__ u16 f2bf(float f) { return __builtin_bit_cast(u16, (__bf16)f); }
__device__ __forceinline__ unsigned f2bf_pair(float lo, float hi) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}
__device__ __forceinline__ float bf2f(u16 b) { return __uint_as_float(((unsigned)b) << 16); }

// GELU(z) and GELU'(z), which share the error function.
__device__ __forceinline__ float gelu_f(float z, float& d) {
  const float e = erff(z * 0.70710678118654752f);
  d = 0.5f * (1.f + e) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
  return 0.5f * z * (1.f + e);
}

struct ConvGeom {
  int D, H, W, C;     // input volume and channels
  int Do, Ho, Wo;     // output volume
};

// The three convolution products on tap-sized K steps (conv.hip).  Each
// returns false where it does not take the shape; *e is the launch's status, tag
// its name in the timing report.
//   forward: C_q[p][co] partials of split q, or (a, bias not null) from the
//     pre-activation z = sum + bias the activation a = BF16(GELU(z)) and, d not
//     null, GELU'(z), with one split
//   input gradient: out[q][position][ci] per split
//   weight gradient: part[q][co][tap * Cin + ci] per split of kchunk positions
struct ConvFwdOut {
  float* c;          // partials (a null)
  float* d;
  u16* a;
  const float* bias;
};
bool conv_fwd_taps(const u16* x, const u16* w, const ConvGeom& g, long P, int Cout, int splits,
                   const ConvFwdOut& out, hipStream_t s, const char* tag, hipError_t* e);
bool conv_dgrad_taps(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, int splits, float* out,
                     hipStream_t s, const char* tag, hipError_t* e);
// The unsplit input gradient carried through the GELU of the layer before:
// gz_in = BF16(gradient * d), d = GELU'(z), and its sums per workgroup and channel, part
// (conv_dgrad_gelu_rows x Cin; 0 rows: shape not taken).
long conv_dgrad_gelu_rows(const ConvGeom& gout, int Cin, int N);
bool conv_dgrad_gelu(const u16* gz, const u16* w, const ConvGeom& gout, int Cin, int N, const float* d, u16* gz_in,
                     float* part, hipStream_t s, const char* tag, hipError_t* e);
bool conv_wgrad_taps(const u16* x, const u16* gz, const ConvGeom& g, long P, int Cout, int splits, float* part,
                     hipStream_t s, const char* tag, hipError_t* e);

}  // namespace wo
