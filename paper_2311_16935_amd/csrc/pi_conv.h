// Operands of the warm-start network's convolutions, shared by the general
// kernels (pi_unet.hip) and those of the 3x3x3 and 1x1x1 layers (pi_conv.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

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

// Whether a 3x3x3 weight gradient over `positions` in `nsplit` parts is faster
// from `boxes` boxes of 256 places (k_wgrad3) than tap by tap (k_wgrad).  A box
// takes 3.6 us of a workgroup (32 x 32 channels, one part, one per CU), however
// many of its places are positions of the grid; 32 positions take 1.44 us of a
// general workgroup (64 x 64 channels, one tap and part), and 2 ns for each
// of them once they fill the device.  32 channels, general kernel and boxes:
// 1 x 64^2 109 and 68 us, 64^2 x 1 110 and 257 us (boxes are eight long in x),
// 12^3 94 and 56, 16 of 4^3 58 and 66, 64 of 2^3 33 and 240, 4 x 64^3 (64
// channels in) 1900 and 170.
inline bool wgrad_boxes_pay(int64_t boxes, int64_t positions, int nsplit, int cin, int cout) {
  const double part = (double)((positions + nsplit - 1) / nsplit);
  const int64_t wg_box = (int64_t)nsplit * ((cin + 31) / 32) * ((cout + 31) / 32);
  const double wg_tap = (double)nsplit * ((cin + 63) / 64) * ((cout + 63) / 64) * 27;
  const double box_us = 3.6 * (double)((boxes + nsplit - 1) / nsplit * ((wg_box + 255) / 256));
  const double tap_us = std::max(1.44, 0.002 * wg_tap) * (double)(int64_t)((part + 31) / 32);
  return box_us < tap_us;
}

// The kernels of pi_conv.hip; false where the operands are none of theirs
// (nothing is launched then).
bool conv_fast(const ConvP &a, hipStream_t s);
// Partial weight (and bias, if bpart) gradients over `nsplit` parts of the
// positions; parts may be empty (zeros).
bool wgrad_fast(const WgP &a, int nsplit, hipStream_t s);

}  // namespace pu
