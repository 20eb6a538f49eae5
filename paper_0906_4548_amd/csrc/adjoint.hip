// Implicit adjoint of the converged field solve.
//
// The solve returns u* with G(u*, delta) = 0 for the discrete Eq. FullDGP2,
//   G(u) = lam [u^2 - sum_ij h_ij^2] + alpha u + gamma N u - S(delta).
// For a loss L(u*) the implicit-function theorem gives dL/ddelta = S^T mu with
// J^T mu = dL/du, J = dG/du.  The spectral operators H_ij (Hessian multipliers)
// and N (-1/kbar) are real and even, hence self-adjoint, so
//   J^T mu = D mu - M^T mu,   D = 2 (1-w) lam u + alpha,
//   M^T mu = 2 lam [ sum_ij H_ij (h_ij mu) - w u mu ] - gamma N mu,
// and the transposed relaxation mu <- D^{-1} (g + M^T mu) has the iteration
// spectrum of the forward relaxation linearised at u*, so it converges when the
// forward does.  With H_22 = I - <.> - H_00 - H_11 the six products collapse to
// five spectral ones plus a local term:
//   sum_ij H_ij(h_ij mu) = H_00((h00-h22) mu) + H_11((h11-h22) mu)
//                        + 2 [H_01(h01 mu) + H_02(h02 mu) + H_12(h12 mu)] + (h22 mu - <h22 mu>).
// One iteration runs four kernels: the axis-1 forward pass of the six product
// spectra, the axis-2 "combine" pass (six forward transforms in, the multipliers,
// one inverse out), the axis-1 inverse pass, and k_adj_step here, which takes the
// axis-0 inverse of the combined spectrum, applies the transposed update pointwise,
// forms the six products of the new multiplier and forward-transforms them along
// axis 0 for the next iteration.  k_adj_finalize decides convergence on the device
// (three multiplier buffers rotated like the forward solve's iterates), so the host
// only looks at the control blocks between chunks of iterations.
#include "dgp_internal.h"

namespace dgp {

template <typename T>
const cx<T>* twiddles(int n);   // device table exp(-2 pi i m / n), defined with the plan code

#define DGP_DISPATCH_N(n, CALL) \
  switch (n) {                  \
    case 8: CALL(8); break;     \
    case 16: CALL(16); break;   \
    case 32: CALL(32); break;   \
    case 64: CALL(64); break;   \
    case 128: CALL(128); break; \
    case 256: CALL(256); break; \
    case 512: CALL(512); break; \
    default: break;             \
  }

// mu = g / D; per workgroup, the number of points where D = 2 (1-w) lam u + alpha is at most
// dmin = 1e-12 alpha (the vertex value of a bad point gives D = 0 up to rounding: there the
// implicit adjoint does not exist) or not finite, and the number of non-finite g
// (part[b][group][0..1])
__global__ void __launch_bounds__(256)
k_adj_init(size_t n3, const double* __restrict__ g, const double* __restrict__ u, double* __restrict__ mu,
           double dscale, double alpha, double* __restrict__ part) {
  const int b = blockIdx.y;
  const size_t off = (size_t)b * n3;
  double nd = 0.0, ng = 0.0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256) {
    const double d = dscale * u[off + i] + alpha;
    const double gg = g[off + i];
    nd += (d > 1e-12 * alpha && isfinite(d)) ? 0.0 : 1.0;
    ng += isfinite(gg) ? 0.0 : 1.0;
    mu[off + i] = gg / d;
  }
  __shared__ double r0[256], r1[256];
  r0[threadIdx.x] = nd;
  r1[threadIdx.x] = ng;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      r0[threadIdx.x] += r0[threadIdx.x + st];
      r1[threadIdx.x] += r1[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[((size_t)b * gridDim.x + blockIdx.x) * 2] = r0[0];
    part[((size_t)b * gridDim.x + blockIdx.x) * 2 + 1] = r1[0];
  }
}

// Geometry of k_adj_step: radix-4 axis-0 transforms (the update holds five fields per element,
// the products two); registers planned for two waves per SIMD, i.e. 512 threads per CU, which are one
// workgroup from N = 128 on: as many column pairs as that allows make the longest row segments (8 x 128^3:
// 4 / 8 / 16 pairs 500 / 496 / 481 us, 256^3: 4 / 8 pairs 569 / 527 us).  Smaller meshes keep 128-byte
// rows: a single 64^3 mesh would be left with 64 workgroups.
template <int N>
struct AdjGeo {
  using P = typename PlanPick<N, 2>::type;
  static constexpr int R = P::R;
  using G = AxisTile<double, N, R>;
  static constexpr int kT = G::kT, kTP = N >= 128 ? 512 / kT : G::kTP, kThreads = kTP * kT;
};

// One transposed relaxation step fused with the axis-0 transforms around it, for a tile of
// axis-0 column pairs of batch element b (multiplier buffers indexed by the control block):
//   UPDATE: q = axis-0 inverse of the combined spectrum (the spectral part of M^T mu), then per
//     point M^T mu = q + 2 lam (h22 mu - <h22 mu>) - 2 lam w u mu, the residual
//     |D mu - M^T mu - g| and mu' = (g + M^T mu) / D, written to the next buffer;
//   !UPDATE: mu' = mu (the first products of an adjoint solve).
// Then the six products (h00-h22) mu', (h11-h22) mu', h01 mu', h02 mu', h12 mu', mu' are
// forward-transformed along axis 0 and written as half spectra [6][batch][N/2+1][N][N].
// Per workgroup: sum |res|, sum |g| and sum h22 mu' into part[b][group][0..2].
// Bound by HBM at two waves per SIMD, so every field is read once and ahead of the transform before
// its use (8 x 128^3, 2.16 GB a launch: h00 and h11 read again for their products 556 us, products
// formed with the update 519 us, loads ahead of the transforms 506 us, longer rows 481 us, 4.5 TB/s).
template <int N, bool UPDATE>
__global__ void __launch_bounds__(AdjGeo<N>::kThreads, 2)
k_adj_step(const cx<double>* __restrict__ qspec, double* __restrict__ mubuf, size_t mu_stride,
           const double* __restrict__ u, const double* __restrict__ h5, const double* __restrict__ g,
           const double* __restrict__ mean_u, const double* __restrict__ mean_h22mu,
           cx<double>* __restrict__ spec6, size_t spec_stride, double* __restrict__ part, AdjCoef k,
           const SolveCtl* __restrict__ ctl, const cx<double>* __restrict__ tw, int batch) {
  using T = double;
  using AG = AdjGeo<N>;
  using P = typename AG::P;
  constexpr int R = AG::R, TP = AG::kTP, TT = AG::kT, NT = AG::kThreads, H = N / 2 + 1;
  constexpr size_t NN = (size_t)N * N, N3 = NN * N;
  constexpr int LSZ = (H * 2 * TP > N * TP) ? H * 2 * TP : N * TP;
  const int b = blockIdx.z;
  if (ctl[b].done) return;
  int tile, i1;
  xcd_tile(tile, i1);
  const int c = threadIdx.x % TP, t = threadIdx.x / TP;
  const int i2 = (tile * TP + c) * 2;
  __shared__ cx<T> lds[LSZ];
  __shared__ double red[3][NT];
  LdsCol<T, TP> L{lds, c};
  const size_t fs = (size_t)batch * N3;
  const size_t off = (size_t)b * N3 + (size_t)i1 * N + i2;   // point (0, i1, i2) of a real field
  auto ld = [&](const double* f, int e) { return *reinterpret_cast<const cx<T>*>(f + off + (size_t)e * NN); };
  const double ub = mean_u[b];
  const double* mu = mubuf + (size_t)ctl[b].cur * mu_stride;
  double sr = 0.0, sg = 0.0, sh = 0.0;
  // the new multiplier and its first two products, formed where h00 and h11 are read
  cx<T> m[R], p0[R], p1[R], v[R];
  if constexpr (UPDATE) {
    const cx<T>* src = qspec + (size_t)b * H * NN + SpecRows<N>::col(i1) + i2;
    for (int kk = t; kk < H; kk += TT) {
      lds[kk * 2 * TP + 2 * c] = src[(size_t)kk * SpecRows<N>::kPlane];
      lds[kk * 2 * TP + 2 * c + 1] = src[(size_t)kk * SpecRows<N>::kPlane + 1];
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      cx<T> xa, xb;
      if (e <= N / 2) {
        xa = lds[e * 2 * TP + 2 * c];
        xb = lds[e * 2 * TP + 2 * c + 1];
        if (e == 0 || e == N / 2) { xa.y = T(0); xb.y = T(0); }
      } else {
        xa = conjg(lds[(N - e) * 2 * TP + 2 * c]);
        xb = conjg(lds[(N - e) * 2 * TP + 2 * c + 1]);
      }
      v[q] = mk(xa.x - xb.y, xa.y + xb.x);   // columns i2 (real part) and i2 + 1 (imaginary part)
    }
    // the point fields are fetched ahead of the transform (its barriers order the LDS only)
    cx<T> fm[R], fu[R], f0[R], f1[R], fg[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      fm[q] = ld(mu, e);
      fu[q] = ld(u, e);
      f0[q] = ld(h5, e);
      f1[q] = ld(h5 + fs, e);
      fg[q] = ld(g, e);
    }
    fft<T, N, P, +1>(v, tw, L, t);
    const double mh = mean_h22mu[b];
    double* mo = mubuf + (size_t)ctl[b].out * mu_stride;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      const cx<T> mm = fm[q], uu = fu[q], a0 = f0[q], a1 = f1[q], gg = fg[q];
      double mn[2], hh[2], q0[2], q1[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const double mj = j ? mm.y : mm.x, uj = j ? uu.y : uu.x, gj = j ? gg.y : gg.x;
        const double h22 = (uj - ub) - (j ? a0.y : a0.x) - (j ? a1.y : a1.x);
        const double mt = (j ? v[q].y : v[q].x) + k.lam2 * (h22 * mj - mh) - k.lam2 * k.w * uj * mj;
        const double d = k.dscale * uj + k.alpha;
        sr += fabs(d * mj - mt - gj);
        sg += fabs(gj);
        mn[j] = (gj + mt) / d;
        hh[j] = h22;
        q0[j] = ((j ? a0.y : a0.x) - h22) * mn[j];
        q1[j] = ((j ? a1.y : a1.x) - h22) * mn[j];
      }
      m[q] = mk(mn[0], mn[1]);
      p0[q] = mk(q0[0], q0[1]);
      p1[q] = mk(q1[0], q1[1]);
      sh += hh[0] * mn[0] + hh[1] * mn[1];
      *reinterpret_cast<cx<T>*>(mo + off + (size_t)e * NN) = m[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      const cx<T> uu = ld(u, e), a0 = ld(h5, e), a1 = ld(h5 + fs, e);
      m[q] = ld(mu, e);
      const double hx = (uu.x - ub) - a0.x - a1.x, hy = (uu.y - ub) - a0.y - a1.y;
      p0[q] = mk((a0.x - hx) * m[q].x, (a0.y - hy) * m[q].y);
      p1[q] = mk((a1.x - hx) * m[q].x, (a1.y - hy) * m[q].y);
      sh += hx * m[q].x + hy * m[q].y;
    }
  }
  cx<T>* dst0 = spec6 + (size_t)b * H * NN + SpecRows<N>::col(i1) + i2;
  cx<T> nx[R];   // the next product's Hessian entry, one field ahead
#pragma unroll 1
  for (int f = 0; f < 6; ++f) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      if (f < 2) {
        v[q] = f == 0 ? p0[q] : p1[q];
      } else if (f < 5) {
        v[q] = mk(nx[q].x * m[q].x, nx[q].y * m[q].y);
      } else {
        v[q] = m[q];
      }
      if (f >= 1 && f < 4) nx[q] = ld(h5 + (f + 1) * fs, e);
    }
    // (the first stage of the transform orders its LDS stores after every thread's previous reads)
    fft<T, N, P, -1>(v, tw, L, t);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) lds[(t + q * TT) * TP + c] = v[q];
    lds_barrier();
    cx<T>* dst = dst0 + f * spec_stride;
    for (int kk = t; kk < H; kk += TT) {
      const cx<T> zk = lds[kk * TP + c];
      const cx<T> zn = lds[((N - kk) & (N - 1)) * TP + c];
      store_stream(&dst[(size_t)kk * SpecRows<N>::kPlane], mk(T(0.5) * (zk.x + zn.x), T(0.5) * (zk.y - zn.y)));
      store_stream(&dst[(size_t)kk * SpecRows<N>::kPlane + 1], mk(T(0.5) * (zk.y + zn.y), T(0.5) * (zn.x - zk.x)));
    }
  }
  red[0][threadIdx.x] = sr;
  red[1][threadIdx.x] = sg;
  red[2][threadIdx.x] = sh;
  __syncthreads();
  for (int st = NT / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int j = 0; j < 3; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const size_t gi = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    const size_t groups = (size_t)gridDim.x * gridDim.y;
    for (int j = 0; j < 3; ++j) part[((size_t)b * groups + gi) * 3 + j] = red[j][0];
  }
}

// Convergence control of the adjoint iteration, one workgroup of 1024 threads per batch element (one
// workgroup walking the batch took 19.5 us at 8 x 128^3, now 5.8 us).  Per undecided element:
// <h22 mu'> for the next update; with EVAL, r = sum |res| / sum |g| of the multiplier that the
// step's update started from, and the stopping rules: r <= tol returns it; otherwise the
// minimum-residual multiplier is kept (buffer `best`), and at max_iter updates (or a non-finite r)
// that one is returned; else the buffers rotate.
template <bool EVAL>
__global__ void __launch_bounds__(1024)
k_adj_finalize(const double* __restrict__ part, int groups, SolveCtl* __restrict__ ctl, double* __restrict__ mean_h22mu,
               double inv_n3, double tol, int max_iter) {
  __shared__ double red[3][16];
  const int b = blockIdx.x;
  if (ctl[b].done) return;
  double a[3] = {0.0, 0.0, 0.0};
  const double* pb = part + (size_t)b * groups * 3;
  for (int gi = threadIdx.x; gi < groups; gi += 1024)
#pragma unroll
    for (int j = 0; j < 3; ++j) a[j] += pb[(size_t)gi * 3 + j];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) a[j] += __shfl_xor(a[j], o, 64);
    if ((threadIdx.x & 63) == 0) red[j][threadIdx.x >> 6] = a[j];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 1; i < 16; ++i)
    for (int j = 0; j < 3; ++j) red[j][0] += red[j][i];
  SolveCtl& C = ctl[b];
  mean_h22mu[b] = red[2][0] * inv_n3;
  if (EVAL) {
    const double r = red[1][0] > 0.0 ? red[0][0] / red[1][0] : 0.0;
    const int n = C.iters;
    C.passes += 1;
    bool done = false;
    if (r <= tol) {
      C.status = 0;
      C.result = C.cur;
      C.resid = r;
      done = true;
    } else if (r < C.resid_min) {
      C.resid_min = r;
      C.best = C.cur;
    }
    if (!done && (n >= max_iter || r != r)) {
      C.status = 1;
      C.result = C.best;
      C.resid = C.resid_min;
      done = true;
    }
    if (r < C.resid_min) C.resid_min = r;
    if (!done) {
      C.iters = n + 1;
      const int nc = C.out;
      C.cur = nc;
      C.out = 3 - nc - C.best;
    }
    C.done = done ? 1 : 0;
  }
}

// Ellipticity test (Appendix, Eq. EllipticMatrix): at every point the matrix of dF/d(h_ij),
// (2 lam u + alpha) I - 2 lam h, is definite (all eigenvalues of one sign) or not.  Sylvester's
// criterion on the leading principal minors decides definiteness; per-workgroup counts of the
// points that are not elliptic go to part[b][g][2] (second slot 0) for the mean reduction.
__global__ void __launch_bounds__(256)
k_nonelliptic(size_t n3, int batch, const double* __restrict__ u, const double* __restrict__ h5,
              const double* __restrict__ mean_u, double lam, double alpha, double* __restrict__ part) {
  const int b = blockIdx.y;
  const size_t off = (size_t)b * n3, fs = (size_t)batch * n3;
  const double ub = mean_u[b];
  double cnt = 0.0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256) {
    const size_t k = off + i;
    const double uu = u[k];
    const double h00 = h5[k], h11 = h5[fs + k], h01 = h5[2 * fs + k], h02 = h5[3 * fs + k], h12 = h5[4 * fs + k];
    const double h22 = (uu - ub) - h00 - h11;
    const double d = 2.0 * lam * uu + alpha, c = -2.0 * lam;
    const double m00 = d + c * h00, m11 = d + c * h11, m22 = d + c * h22;
    const double m01 = c * h01, m02 = c * h02, m12 = c * h12;
    const double d1 = m00;
    const double d2 = m00 * m11 - m01 * m01;
    const double d3 = m00 * (m11 * m22 - m12 * m12) - m01 * (m01 * m22 - m12 * m02) + m02 * (m01 * m12 - m11 * m02);
    const bool elliptic = (d1 > 0.0 && d2 > 0.0 && d3 > 0.0) || (d1 < 0.0 && d2 > 0.0 && d3 < 0.0);
    cnt += elliptic ? 0.0 : 1.0;
  }
  __shared__ double r[256];
  r[threadIdx.x] = cnt;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) r[threadIdx.x] += r[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[((size_t)b * gridDim.x + blockIdx.x) * 2] = r[0];
    part[((size_t)b * gridDim.x + blockIdx.x) * 2 + 1] = 0.0;
  }
}

static int adj_groups(size_t n3) {
  size_t g = (n3 + 255) / 256;
  return int(g > 1024 ? 1024 : g);
}

int adjoint_groups(size_t n3) { return adj_groups(n3); }

void launch_nonelliptic(size_t n3, int batch, const double* u, const double* h5, const double* mean_u, double lam,
                        double alpha, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_nonelliptic, dim3(adj_groups(n3), batch), dim3(256), 0, s, n3, batch, u, h5, mean_u, lam, alpha,
                     part);
}

void launch_adj_init(size_t n3, int batch, const double* g, const double* u, double* mu, double dscale, double alpha,
                     double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_init, dim3(adj_groups(n3), batch), dim3(256), 0, s, n3, g, u, mu, dscale, alpha, part);
}

int adj_step_groups(int n) {
  int g = 0;
#define C(NN) g = (NN / (2 * AdjGeo<NN>::kTP)) * NN;
  DGP_DISPATCH_N(n, C)
#undef C
  return g;
}

void launch_adj_step(int n, bool update, const cx<double>* qspec, double* mubuf, size_t mu_stride, const double* u,
                     const double* h5, const double* g, const double* mean_u, const double* mean_h22mu,
                     cx<double>* spec6, size_t spec_stride, double* part, const AdjCoef& k, const SolveCtl* ctl,
                     int batch, hipStream_t s) {
  const cx<double>* tw = twiddles<double>(n);
#define C(NN)                                                                                                   \
  {                                                                                                             \
    dim3 grid(NN / (2 * AdjGeo<NN>::kTP), NN, batch);                                                           \
    if (update)                                                                                                 \
      hipLaunchKernelGGL((k_adj_step<NN, true>), grid, dim3(AdjGeo<NN>::kThreads), 0, s, qspec, mubuf,         \
                         mu_stride, u, h5, g, mean_u, mean_h22mu, spec6, spec_stride, part, k, ctl, tw, batch); \
    else                                                                                                        \
      hipLaunchKernelGGL((k_adj_step<NN, false>), grid, dim3(AdjGeo<NN>::kThreads), 0, s, qspec, mubuf,        \
                         mu_stride, u, h5, g, mean_u, mean_h22mu, spec6, spec_stride, part, k, ctl, tw, batch); \
  }
  DGP_DISPATCH_N(n, C)
#undef C
}

void launch_adj_finalize(bool eval, const double* part, int groups, SolveCtl* ctl, double* mean_h22mu, size_t n3,
                         double tol, int max_iter, int batch, hipStream_t s) {
  if (eval)
    hipLaunchKernelGGL(k_adj_finalize<true>, dim3(batch), dim3(1024), 0, s, part, groups, ctl, mean_h22mu,
                       1.0 / double(n3), tol, max_iter);
  else
    hipLaunchKernelGGL(k_adj_finalize<false>, dim3(batch), dim3(1024), 0, s, part, groups, ctl, mean_h22mu,
                       1.0 / double(n3), tol, max_iter);
}

}  // namespace dgp
