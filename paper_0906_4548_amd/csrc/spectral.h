// Mode numbers and spectral multipliers shared by the axis-2 pass (passes.hip) and the plane kernels
// (plane.hip).
#pragma once
#include "dgp_internal.h"

namespace dgp {

struct Mode3 {
  int n0, n1, n2;        // signed mode numbers (n0 >= 0 on the half axis)
  bool q0, q1, q2;       // Nyquist flags
  int msq;               // |n|^2 (at most 3 x 256^2)
};

__device__ __forceinline__ Mode3 mode_of(int N, int k0, int k1, int k2) {
  Mode3 m;
  m.n0 = k0;
  m.n1 = (k1 < N / 2) ? k1 : k1 - N;
  m.n2 = (k2 < N / 2) ? k2 : k2 - N;
  m.q0 = (k0 == N / 2);
  m.q1 = (k1 == N / 2);
  m.q2 = (k2 == N / 2);
  m.msq = m.n0 * m.n0 + m.n1 * m.n1 + m.n2 * m.n2;
  return m;
}

// ic = 1/(N^3 |n|^2) and ib = -1/(N^3 kappa kf |n|), both 0 at n = 0; float32 fields form them in
// float32 (reciprocal and reciprocal-sqrt estimates, the reciprocal refined by one Newton step)
template <typename T>
__device__ __forceinline__ T inv_square(const SpecCoef& cf, const Mode3& m) {
  if constexpr (sizeof(T) == 4) {
    const float ms = float(m.msq);
    float r = __builtin_amdgcn_rcpf(ms);
    r = r * (2.0f - ms * r);
    return m.msq != 0 ? r * float(cf.inv_n3) : 0.0f;
  } else {
    const double ms = double(m.msq);   // reciprocal estimate and two Newton steps
    double r = __builtin_amdgcn_rcp(ms);
    r = fma(r, fma(-ms, r, 1.0), r);
    r = fma(r, fma(-ms, r, 1.0), r);
    return m.msq != 0 ? r * cf.inv_n3 : 0.0;
  }
}
template <typename T>
__device__ __forceinline__ T nonlocal_mult(const SpecCoef& cf, const Mode3& m) {
  if constexpr (sizeof(T) == 4) {
    return m.msq != 0 ? -__builtin_amdgcn_rsqf(float(m.msq)) * float(cf.nl_scale) : 0.0f;
  } else {
    const double ms = double(m.msq);   // reciprocal-sqrt estimate and two Newton steps
    double r = __builtin_amdgcn_rsq(ms);
    r = fma(0.5 * r, fma(-ms * r, r, 1.0), r);
    r = fma(0.5 * r, fma(-ms * r, r, 1.0), r);
    return m.msq != 0 ? -cf.nl_scale * r : 0.0;
  }
}

// multipliers (0 at k = 0) of S = A (1 - beta/kbar) delta, times 1/N^3, and of the linear solution
// S / (alpha - gamma/kbar), times 1/N^2: after the inverse transforms of axes 2 and 1 that is the
// linear solution's forward axis-0 spectrum
template <typename T>
__device__ __forceinline__ void source_mults(const SpecCoef& cf, const Mode3& m, T& ms, T& ml) {
  ms = T(0);
  ml = T(0);
  if (m.msq != 0) {
    const double ikb = 1.0 / (cf.kappa * cf.kf * sqrt(double(m.msq)));
    const double sv = cf.A * (1.0 - cf.beta * ikb);
    ms = T(sv * cf.inv_n3);
    ml = T(sv / (cf.alpha - cf.gamma * ikb) * cf.inv_n2);
  }
}

// phi(k), times 1/N^3 (0 at k = 0), from delta(k) (and u(k) under the nlDGP law): the modified Poisson
// equation or its linear and GR forms
template <typename T>
__device__ __forceinline__ cx<T> phi_of(const SpecCoef& cf, const Mode3& m, cx<T> d, cx<T> u) {
  if (m.msq == 0) return mk(T(0), T(0));
  const double ms = double(m.msq);
  const double kb = cf.kappa * cf.kf * sqrt(ms);
  const double ikb = 1.0 / kb;
  const double dr = double(d.x), di = double(d.y);
  double nr, ni, den;
  if (cf.force_mode == FORCE_GRH || cf.force_mode == FORCE_GR) {   // Eq. GRPoisson (kappa, om15 of the run's background)
    nr = cf.om15 * dr; ni = cf.om15 * di; den = kb * kb;
  } else {
    double ur, ui;
    if (cf.force_mode == FORCE_NLDGP) {
      ur = double(u.x); ui = double(u.y);
    } else {   // linear solution from delta
      const double sl = cf.A * (1.0 - cf.beta * ikb) / (cf.alpha - cf.gamma * ikb);
      ur = sl * dr; ui = sl * di;
    }
    const double cu = -cf.inv2eta + cf.c2 * ikb;
    nr = cf.om15 * dr + cu * ur;
    ni = cf.om15 * di + cu * ui;
    den = kb * kb + kb * cf.inv_eta_nl;
  }
  return mk(T(-nr / den * cf.inv_n3), T(-ni / den * cf.inv_n3));
}

}  // namespace dgp
