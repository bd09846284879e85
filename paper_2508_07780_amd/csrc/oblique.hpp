// Obliquely incident plane waves on the top face, shared by every kernel that updates its nodes.
#pragma once

#include "dd_common.hpp"

namespace dd {

// The time function of an obliquely incident plane wave at top-face node (x, y): the pulse of
// the source kind delayed by tau = pw_kx (x - pw_x0) + pw_ky (y - pw_y0).  Inside the pulse's
// support the sine's argument stays within 3 pi (the Gaussian-modulated sine: |omega u| <=
// omega t0 = 3 pi; one sine period: < 2 pi), where the hardware sine and exponential are
// accurate to about 1e-6, well inside the trace tolerance, and need no argument reduction.
// kind, tn: the step's source kind and time (t_n, or t_n - t0 for the Gaussian-modulated sine).
// A: a kernel's arguments with the wave's pw_* fields.
template <class A>
__device__ __forceinline__ float oblique_pulse_at(const A& a, int kind, float tn, int x, int y) {
  const float tau = __builtin_fmaf(a.pw_kx, (float)(x - a.pw_x0), a.pw_ky * (float)(y - a.pw_y0));
  const float u = tn - tau;
  if (kind == DD_SRC_GAUSS_SINE) {
    if (!(fabsf(u) <= a.pw_sup)) return 0.f;
    const float v = u * a.pw_iw;
    return __sinf(a.pw_omega * u) * __expf(-0.5f * v * v);
  }
  if (!(u > 0.f && u < a.pw_sup)) return 0.f;
  return __sinf(a.pw_omega * u);
}
}  // namespace dd
