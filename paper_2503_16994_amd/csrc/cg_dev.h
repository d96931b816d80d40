// Device-side steps of the CG recursion that more than one kernel performs.
#pragma once

#include "lqcd_kernels.h"

namespace lqcd {

__device__ inline bool finite(double v) { return v == v && fabs(v) <= 1.7976931348623157e308; }

// Fixed-order sum of at most 64 partials (n as in parts_count) by one wave,
// the result in every lane: the sum that a workgroup of several waves forms in
// its first wave (the others add zeros there), without a barrier.
__device__ inline double wave_psum(const double* p, int n) {
  const int l = threadIdx.x & 63;
  double v = l < parts_count(n) ? parts_at(p, n, l) : 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// r + beta p
template <typename A>
__device__ inline cpx<A> p_next(A beta, cpx<A> r, cpx<A> p) {
  return {fma(beta, p.re, r.re), fma(beta, p.im, r.im)};
}

// beta and the iteration control from the new |r|^2 = v; the denominator is
// rr_prev, the |r|^2 the alpha step of this iteration divided by (alpha sets
// it), so the fused beta/p kernel below can replace rr while its other
// workgroups still divide by the old value
__device__ inline void beta_step(CGState& c, double v) {
  c.iters += 1;
  if (!finite(v) || !finite(c.alpha)) {
    c.done = 1;
    c.status = CG_NONFINITE;
    c.skip_ru = 1;
    return;
  }
  const bool hit = v <= c.target2;
  const bool due = c.ru_every > 0 && c.iters - c.last_ru >= c.ru_every;
  const bool drop = v < c.delta2 * c.rr_max;
  if (hit || due || drop) {
    if (c.skip_ru) c.ru_drop = 0;  // a new request
    c.skip_ru = 0;
    if (hit) c.inner_hit = 1;
    if (hit || drop) c.ru_drop = 1;
  }
  c.beta = (c.rr_prev > 0.0) ? v / c.rr_prev : 0.0;
  c.rr = v;
  if (v > c.rr_max) c.rr_max = v;
  if (c.iters >= c.maxiter && c.skip_ru) {
    c.done = 1;
    c.status = CG_MAXITER;
  }
}

}  // namespace lqcd
