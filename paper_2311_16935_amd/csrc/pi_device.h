// Device helpers shared by the streaming kernels (pi_kernels.hip) and the
// on-chip solve (pi_resident.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "pi_common.h"

namespace pi {

__device__ inline int dstate(uint32_t code, int d, int bits) {
  return (int)((code >> (bits * d)) & ((1u << bits) - 1u));
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
