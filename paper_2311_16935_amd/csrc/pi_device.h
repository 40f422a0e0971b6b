// Device helpers shared by the streaming kernels (pi_kernels.hip) and the
// on-chip solve (pi_resident.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "pi_common.h"

namespace pi {

__device__ inline int dstate(uint32_t code, int d, int bits) {
  return (int)((code >> (bits * d)) & ((1u << bits) - 1u));
}

// ---------------------------------------------------------------------------
// lanes of a wave exchanging values in registers (v_mov with DPP, permlane
// swaps): a few cycles each, where __shfl goes through LDS (above 100)
// ---------------------------------------------------------------------------
struct D2 {
  double a, b;
};
// lanes 0-31 of a with lanes 0-31 of b, and lanes 32-63 of a with lanes 32-63 of b
__device__ inline D2 swap32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return D2{__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1])};
}
// the same between odd and even rows of 16 lanes
__device__ inline D2 swap16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return D2{__hiloint2double(hi[0], lo[0]), __hiloint2double(hi[1], lo[1])};
}
// value of the lane K places back inside the row of 16
template <int K>
__device__ inline double ror16(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + K, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + K, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Sum over the wave, in every lane.  Level by level the lanes i and i ^ 32,
// i ^ 16, ... i ^ 1 are added (once lanes 8 apart agree, the lane 4 back
// holds what lane i ^ 4 does, and so on down).
__device__ inline double wave_sum(double v) {
  const D2 a = swap32(v, v);
  v = a.a + a.b;
  const D2 b = swap16(v, v);
  v = b.a + b.b;
  v += ror16<8>(v);
  v += ror16<4>(v);
  v += ror16<2>(v);
  v += ror16<1>(v);
  return v;
}

// Value of the lane before (after); lane 0 (63) gets `end`.  Every lane of
// the wave must be active.
template <int CTRL>
__device__ inline float lane_shift(float v, float end) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(end), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ inline double lane_shift(double v, double end) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(end), __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(end), __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <typename T>
__device__ inline T lane_before(T v, T end) {
  return lane_shift<0x138>(v, end);  // wave_shr:1
}
template <typename T>
__device__ inline T lane_after(T v, T end) {
  return lane_shift<0x130>(v, end);  // wave_shl:1
}

// Code word of a cell whose face neighbours, their laterals and their far
// cells all hold data: every direction in its last state.
template <int ND>
__host__ __device__ constexpr uint32_t interior_code() {
  uint32_t c = kValidBit;
  for (int d = 0; d < 2 * ND; ++d) c |= (ND == 3 ? 18u : 6u) << ((ND == 3 ? 5 : 3) * d);
  return c;
}
template <int ND>
__host__ __device__ constexpr int interior_state() {
  return ND == 3 ? 18 : 6;
}

// From the sums of CG iteration j: alpha_j = r.r / p.q and, with
// |r_j - alpha_j q_j|^2 = r.r - 2 alpha_j r.q + alpha_j^2 q.q, beta_{j+1}.
// The fixed-point variant's inner solve stops once that residual is well
// below the tolerance (the FP64 outer step then confirms it), or once it is
// as small as the vector precision can resolve: beyond that only the
// residual's rounding-level constant part is left, which the singular
// operator cannot reduce (p.q -> 0 and alpha would blow up); the next outer
// step restarts from the FP64 residual.
struct CgScalars {
  double al, be;
  bool stop;
};
__device__ inline CgScalars cg_scalars(const Inst &in, const State *st, const double (&s)[4]) {
  const double pq = s[0], rq = s[1], qq = s[2], rr = s[3];
  const double al = pq != 0.0 ? rr / pq : 0.0;
  double rn = rr - 2.0 * al * rq + al * al * qq;
  if (!(rn > 0.0)) rn = 0.0;
  CgScalars c;
  c.al = al;
  c.be = rr != 0.0 ? rn / rr : 0.0;
  c.stop = in.inner_op != 0 && (rn <= 0.25 * in.tol * in.tol * st->normS2 || rn <= in.inner_floor * st->rr0);
  return c;
}

// Scalars of an outer step from its sums (r.r in FP64 and as the vectors
// hold it, delta.delta, P.P): residuals, the stopping tests of Algorithm 1,
// and the state the inner solve starts from.
__device__ inline void outer_scalars(const Inst &in, State *st, const double (&s)[4]) {
  const bool hd = st->have_delta != 0;
  // CG passes of the inner solve that just ended (BiCGStab counts its own)
  if (hd && !in.bicg) st->inner_total += min(st->stop_at, in.inner_iters);
  const double epsR = st->normS2 > 0.0 ? sqrt(s[0] / st->normS2) : 0.0;
  st->epsR = epsR;
  if (hd) st->epsP = s[3] > 0.0 ? sqrt(s[2] / s[3]) : 0.0;
  if (!isfinite(epsR)) {
    st->done = 1;
    st->status = 5;  // PI_ERR_DIVERGED
  } else if (epsR <= in.tol) {
    st->done = 1;
    st->status = 0;
  } else if (st->outer >= in.max_iter) {
    st->done = 1;
    st->status = 4;  // PI_ERR_NOT_CONVERGED
  } else {
    st->outer += 1;
    st->rr = s[1];
    st->rr0 = s[1];
    st->inner = 0;
    st->stop_at = kNoStop;
    st->dvalid = 0;
    st->first = 1;
    st->beta = 0.0;  // the first search direction is the residual itself
    st->have_delta = 1;
    // BiCGStab restarts with the new residual as its shadow vector
    st->rho = s[1];
    st->alpha = 1.0;
    st->omega = 1.0;
  }
}

}  // namespace pi
