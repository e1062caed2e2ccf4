// Declarations shared by the convolution kernels of the warm-start network
// (cnn.hip, conv.hip).  Not part of the public C ABI (include/lddmm_cnn.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lddmm_cnn.h"

namespace lddmm_cnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;

__device__ __forceinline__ float bf2f(u16 b) {
  return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// Round to nearest bf16, ties to even (NaN stays NaN).
__device__ __forceinline__ u16 f2bf(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (u16)(u >> 16);
}

enum { OP_FWD = 0, OP_DGRAD = 1, OP_WGRAD = 2 };

// One convolution's operands and geometry (see k_conv_gemm for the matrices).
struct ConvArgs {
  const u16* x;       // forward / wgrad input; dgrad: dy
  const u16* wb;      // forward: w; dgrad: wt; wgrad: dy
  const float* bias;
  const u16* mask;
  const u16* add;
  void* out;          // forward: y; dgrad: dx; wgrad: FP32 partial tiles
  int n, d, h, w, ci; // input geometry
  int od, oh, ow, co; // output geometry
  int s;
  int M, N, K, kchunk;
  int relu, out_f32, add_stride, add_off;
};

// conv.hip: forward and input-gradient convolutions with fragments loaded
// straight from global memory.  Returns false, launching nothing, for shapes it
// does not cover.
bool launch_conv_frag(int op, const ConvArgs& a, hipStream_t s);

// wgrad.hip: weight and bias (db may be null) gradients with part_floats floats of scratch.
// Returns false, launching nothing, for shapes it does not cover.
bool launch_wgrad(const ConvArgs& a, float* dw, float* db, float* part, size_t part_floats,
                  hipStream_t s);

}  // namespace lddmm_cnn
