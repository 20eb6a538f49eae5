// Convergence decision of a relaxation pass (Eq. normres and the stopping rules), and the wavefront
// sums it and the kernels' reductions use.
#pragma once
#include "dgp_internal.h"

namespace dgp {

// sum over the W lanes of a wavefront segment (butterfly order, deterministic) in a workgroup of NT
// threads, all of which call it; a butterfly over lanes that the workgroup does not have would add
// what a shuffle from a missing lane returns, which is undefined
template <int W, int NT>
__device__ __forceinline__ double wave_sum(double x) {
  static_assert(W <= 64 && (W & (W - 1)) == 0 && NT % W == 0, "every segment must be whole");
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, W);
  return x;
}
template <int W, int NT>
__device__ __forceinline__ int wave_sum(int x) {
  static_assert(W <= 64 && (W & (W - 1)) == 0 && NT % W == 0, "every segment must be whole");
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, W);
  return x;
}

// A pass's sums of |R| and of the bad points from its partial sums, by a workgroup of NT threads (every
// thread returns them).  A pass is decided by the next pass's launch or, at the end of a chunk of
// passes, by a launch of its own, so on the meshes where both occur both must add in the same order:
// there each lane holds at most one partial sum (groups <= NT), consecutive 64 are added as a
// butterfly and the wavefronts in order, whatever NT is.  (Lanes with several partial sums in one of
// the two: the residuals of a 64^3 solve differed in the last place with the place of the host's looks.)
template <int NT>
__device__ __forceinline__ void pass_sums(const double* __restrict__ partial, int groups, double& sum_r, double& sum_bad) {
  constexpr int WW = NT < 64 ? NT : 64, NW = (NT + 63) / 64;
  __shared__ double wr[NW], wb[NW];
  double r = 0.0, bad = 0.0;
  const double2* p = reinterpret_cast<const double2*>(partial);
  for (int g = threadIdx.x; g < groups; g += NT) {
    const double2 v = p[g];
    r += v.x;
    bad += v.y;
  }
  r = wave_sum<WW, NT>(r);
  bad = wave_sum<WW, NT>(bad);
  if ((threadIdx.x & 63) == 0) {
    wr[threadIdx.x >> 6] = r;
    wb[threadIdx.x >> 6] = bad;
  }
  lds_barrier();
  sum_r = wr[0];
  sum_bad = wb[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) {
    sum_r += wr[i];
    sum_bad += wb[i];
  }
}

// normalised residual of the iterate that the pass evaluated; eps = 0 only for a uniform delta
// (S = 0), whose exact solution u = 0 has R = 0
__device__ __forceinline__ double ctl_residual(const SolveCtl& C, double sum_r, const SolveCfg& cfg) {
  const double n3 = double(cfg.n) * cfg.n * cfg.n;
  return C.eps > 0.0 ? sum_r / (n3 * C.eps) : (sum_r == 0.0 ? 0.0 : __builtin_huge_val());
}

// whether that residual decides the element (the cases of ctl_decide that set done)
__device__ __forceinline__ bool ctl_decides(const SolveCtl& C, double r, const SolveCfg& cfg) {
  if (r != r || r <= cfg.tol) return true;   // not a number: a non-finite iterate
  if (!(r < C.resid_min) && C.bad_seen && !cfg.fixed) return true;
  return C.iters + C.iters1 >= cfg.max_iter;
}

// The decision itself, by one thread: C is the element's block of the pass just run (sum_r, sum_bad: its
// sums of |R| and of the bad points).
__device__ __forceinline__ void ctl_decide(SolveCtl& C, SolveHist& H, double sum_r, double sum_bad,
                                           const SolveCfg& cfg) {
  const double n3 = double(cfg.n) * cfg.n * cfg.n;
  const double r = ctl_residual(C, sum_r, cfg);
  const int nbad = int(sum_bad);
  const int n = C.iters;
  if (n < kMaxHist) {
    H.resid[n] = r;
    H.bad[n] = double(nbad) / n3;
  }
  C.passes += 1;
  bool done = false;
  if (r != r) {   // a non-finite iterate (non-finite warm start, or divergence): nothing to return
    C.status = kStatusInvalid;
    C.result = C.cur;
    C.resid = r;
    done = true;
  } else if (r <= cfg.tol) {
    C.status = 0;
    C.result = C.cur;
    C.resid = r;
    C.final_bad = nbad;   // that pass's update sits in buffer C.out
    done = true;
  } else if (r < C.resid_min) {
    C.resid_min = r;
    C.best = C.cur;
  } else if (C.bad_seen && !cfg.fixed) {
    C.status = 2;
    C.result = C.best;
    C.resid = C.resid_min;
    done = true;
  }
  if (r < C.resid_min) C.resid_min = r;
  if (!done && n + C.iters1 >= cfg.max_iter) {
    if (cfg.fixed) {   // the requested number of updates: the last iterate
      C.status = 0;
      C.result = C.cur;
      C.resid = r;
    } else {
      C.status = 1;
      C.result = C.best;
      C.resid = C.resid_min;
    }
    done = true;
  }
  if (!done) {
    C.last_bad = nbad;
    C.bad_frac = double(nbad) / n3;
    if (nbad > 0) C.bad_seen = 1;
    C.iters = n + 1;
    const int nc = C.out;
    C.cur = nc;
    C.out = 3 - nc - C.best;
  }
  C.done = done ? 1 : 0;
}

}  // namespace dgp
