// Operands of the warm-start network's convolutions, shared by the general
// kernels (pi_unet.hip) and those of the 3x3x3 and 1x1x1 layers (pi_conv.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace pu {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __host__ inline float bf2f(uint16_t b) {
  union {
    uint32_t u;
    float f;
  } v;
  v.u = (uint32_t)b << 16;
  return v.f;
}

// round to nearest even; NaN stays NaN
__device__ __host__ inline uint16_t f2bf(float f) {
  union {
    uint32_t u;
    float f;
  } v;
  v.f = f;
  if ((v.u & 0x7f800000u) == 0x7f800000u && (v.u & 0x007fffffu)) return (uint16_t)((v.u >> 16) | 0x40);
  const uint32_t r = v.u + 0x7fffu + ((v.u >> 16) & 1u);
  return (uint16_t)(r >> 16);
}

struct Tens {
  uint16_t *p;
  int n, d, h, w, c, ld, off;
};

struct ConvP {
  Tens x, y;
  const uint16_t *w;
  const float *bias;
  int taps, cin, cout;
  int md, mh, mw, sin, sout, ooz, ooy, oox;
  int relu, yfp32, acc;
  int64_t P;
  int8_t offs[27][3];
};

struct WgP {
  Tens x, g;
  int taps, cin, cout;
  int md, mh, mw, sin, sout, ooz, ooy, oox;
  int64_t P, chunk;
  float *part;   // [nsplit][taps][cin][cout]
  float *bpart;  // [nsplit][cout] or NULL
  int8_t offs[27][3];
};

// The kernels of pi_conv.hip; false where the operands are none of theirs
// (nothing is launched then).
bool conv_fast(const ConvP &a, hipStream_t s);
// Partial weight (and bias, if bpart) gradients over `nsplit` parts of the
// positions; parts may be empty (zeros).
bool wgrad_fast(const WgP &a, int nsplit, hipStream_t s);

}  // namespace pu
