// Plane kernels: axis-1 and axis-2 transforms of whole k0 planes in one launch.
//
// For a fixed k0 the axis-1 forward pass, the axis-2 pass with its spectral multipliers and the
// axis-1 inverse pass touch one N x N plane only.  Up to N = 64 that plane takes at most half of the
// LDS and one workgroup does all three on it (a 128^2 float32 plane fills it: 8 fields 193 us a
// launch against 183 for the three passes): the plane is read once and each output written once (7 instead of 15 spectra of memory traffic for the relaxation's six
// outputs), and a pass takes one launch instead of three.  On meshes this small a launch is bound
// by its latency chain (load, exchanges, store), so the outputs of a plane are spread over several
// workgroups, each repeating the forward transforms, while the device is not full.
#include "control.h"
#include "dgp_internal.h"
#include "spectral.h"

namespace dgp {

template <typename T>
const cx<T>* twiddles(int n);   // device table exp(-2 pi i m / n), defined with the plan code

template <typename T, int N>
struct PlaneGeo {
  using P = Plan8<N>;
  static constexpr int R = P::R, kT = N / R, kThreads = N * kT;
  // element e of row r at r * kLD + e + e / kPad: the padding spreads a first stage's stores (R elements
  // apart) over the banks and leaves the 16 consecutive columns of an access together
  static constexpr int kPad = 16, kLD = N + (N + kPad - 1) / kPad;
  static_assert(kThreads <= 1024 && kT <= 64 && 64 % kT == 0, "a row's threads sit in one wavefront");
  static_assert(sizeof(cx<T>) * N * (kLD + 1) <= 160 * 1024, "the plane and the twiddles must fit the LDS");
  static __device__ __forceinline__ int at(int r, int e) { return r * kLD + e + int(unsigned(e) / kPad); }
};

template <typename T, int N>
struct PlaneCol {   // exchanges of column c (any wavefronts)
  using G = PlaneGeo<T, N>;
  cx<T>* base;
  int c;
  template <int S>
  __device__ __forceinline__ cx<T> load_q(int j, int q) const { return base[G::at(j, c) + q * S * G::kLD]; }
  template <int Ns>
  __device__ __forceinline__ void store_q(int e, int q, cx<T> v) const { base[G::at(e, c) + q * Ns * G::kLD] = v; }
  __device__ __forceinline__ void sync() const { lds_barrier(); }
};
template <typename T, int N>
struct PlaneRow {   // exchanges of row r (inside one wavefront)
  using G = PlaneGeo<T, N>;
  cx<T>* base;
  int r;
  template <int S>
  __device__ __forceinline__ cx<T> load_q(int j, int q) const { return base[G::at(r, j) + q * S + q * S / G::kPad]; }
  template <int Ns>
  __device__ __forceinline__ void store_q(int e, int q, cx<T> v) const { base[G::at(r, e) + q * Ns + q * Ns / G::kPad] = v; }
  __device__ __forceinline__ void sync() const { wave_sync(); }
};

// Decision of the previous pass at the start of a relaxation plane launch, before the plane is loaded:
// every workgroup adds the partial sums of its element and so knows whether the element is done; the
// workgroup with `write` records the decision in the next control blocks.  A launch of its own for
// this takes 3.5 us and a gap, of a 26-31 us pass.  Returns whether the element is done.
template <int NT>
__device__ __forceinline__ bool decide_pass(const PassDecision& d, int b, bool write) {
  const SolveCtl& C = d.prev[b];
  if (C.done) {
    if (write && threadIdx.x == 0) d.next[b] = C;
    return true;
  }
  double sr, sb;
  pass_sums<NT>(d.partial + (size_t)b * d.groups * 2, d.groups, sr, sb);
  if (write && threadIdx.x == 0) {
    SolveCtl D = C;
    ctl_decide(D, d.hist[b], sr, sb, d.cfg);   // (no other workgroup touches the histories)
    d.next[b] = D;
  }
  return ctl_decides(C, ctl_residual(C, sr, d.cfg), d.cfg);
}

// `in`: axis-0 transformed spectra [batch][N/2+1][N][N] (SPEC_FORCES: delta, then u in_stride behind it);
// output o, inverse transformed along axes 2 and 1, to out + o * out_stride.  Workgroup
// (g, k0, b) forms the outputs g * per .. g * per + per - 1 (below nout).
//   SPEC_HSPLIT: the six relaxation fields h00, h11, h01, h02, h12 and the nonlocal term; mean_out[b] = <u>
//   SPEC_SOURCE: S and the linear solution;  SPEC_FORCES: g0, g1, g2 (and phi);  SPEC_CFIELD: C
template <typename T, int N, SpecMode MODE>
__global__ void __launch_bounds__((PlaneGeo<T, N>::kThreads))
k_plane(const cx<T>* __restrict__ in, size_t in_stride, cx<T>* __restrict__ out, size_t out_stride, int nout, int per,
        const cx<T>* __restrict__ tw, SpecCoef cf, double* __restrict__ mean_out, const SolveCtl* __restrict__ ctl,
        PassDecision dec) {
  using G = PlaneGeo<T, N>;
  using P = typename G::P;
  constexpr int R = G::R, TT = G::kT, H = N / 2 + 1;
  const int b = blockIdx.z, k0 = blockIdx.y;
  if constexpr (MODE == SPEC_HSPLIT) {
    if (dec.prev != nullptr) {
      if (decide_pass<G::kThreads>(dec, b, blockIdx.x == 0 && k0 == 0)) return;
    } else if (ctl != nullptr && ctl[b].done != 0) {
      return;
    }
  } else {
    if (ctl != nullptr && ctl[b].done != 0) return;
  }
  int tid = threadIdx.x;
  __shared__ cx<T> lds[N * G::kLD];
  __shared__ cx<T> twl[N];   // (the first twiddled stage would wait on a cold global load)
  for (int i = tid; i < N; i += G::kThreads) twl[i] = tw[i];   // ordered by the first exchange's barrier
  const size_t off = ((size_t)b * H + k0) * N * N;

  auto forward = [&](const cx<T>* src, cx<T> (&v)[R]) {
    const int c = tid % N, t = tid / N;      // column mapping
    const int r = tid / TT, tr = tid % TT;   // row mapping
    const PlaneCol<T, N> LC{lds, c};
    const PlaneRow<T, N> LR{lds, r};
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = src[off + c + (size_t)(t + q * TT) * N];
    fft<T, N, P, -1>(v, twl, LC, t);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) lds[G::at(t, c) + q * TT * G::kLD] = v[q];
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = lds[G::at(r, tr) + q * TT + q * TT / G::kPad];
    fft<T, N, P, -1>(v, twl, LR, tr);
  };
  cx<T> v[R];
  if constexpr (MODE == SPEC_FORCES) {
    cx<T> u[R];
    if (cf.force_mode == FORCE_NLDGP) {
      forward(in + in_stride, u);
      lds_barrier();   // the row exchanges before the next plane's column exchanges
    }
    forward(in, v);
#pragma unroll
    for (int q = 0; q < R; ++q)
      v[q] = phi_of(cf, mode_of(N, k0, tid / TT, tid % TT + q * TT), v[q], cf.force_mode == FORCE_NLDGP ? u[q] : v[q]);
  } else {
    forward(in, v);
  }
  if constexpr (MODE == SPEC_HSPLIT) {
    if (blockIdx.x == 0 && k0 == 0 && threadIdx.x == 0 && mean_out != nullptr) mean_out[b] = double(v[0].x) * cf.inv_n3;
  }
  const int o1 = min(nout, int(blockIdx.x) * per + per);
#pragma unroll 1
  for (int o = blockIdx.x * per; o < o1; ++o) {
    // opaque per output: addresses and multipliers are not held across the loop
    asm volatile("" : "+v"(tid));
    const int c = tid % N, t = tid / N, r = tid / TT, tr = tid % TT;
    const PlaneCol<T, N> LC{lds, c};
    const PlaneRow<T, N> LR{lds, r};
    // SPEC_HSPLIT: n_i n_j / |n|^2 (0 where an odd factor is at its Nyquist index); the part that is
    // constant along the row
    const Mode3 mr = mode_of(N, k0, r, 0);
    const T o0 = mr.q0 ? T(0) : T(mr.n0), o1f = mr.q1 ? T(0) : T(mr.n1);
    const T rowf = o == 0 ? T(mr.n0 * mr.n0) : o == 1 ? T(mr.n1 * mr.n1) : o == 2 ? o0 * o1f : o == 3 ? o0 : o1f;
    cx<T> w[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const Mode3 m = mode_of(N, k0, r, tr + q * TT);
      if constexpr (MODE == SPEC_HSPLIT) {   // row factor (n_i n_j or n_i) times the axis-2 factor / |n|^2
        T f = o == 5 ? nonlocal_mult<T>(cf, m) : rowf * inv_square<T>(cf, m);
        if (o == 3 || o == 4) f *= m.q2 ? T(0) : T(m.n2);
        w[q] = scale(v[q], f);
      } else if constexpr (MODE == SPEC_SOURCE) {
        T ms, ml;
        source_mults(cf, m, ms, ml);
        w[q] = scale(v[q], o ? ml : ms);
      } else if constexpr (MODE == SPEC_FORCES) {   // g_d = -(c/H0)^2 i k_d phi (k_d = 0 at its Nyquist index); phi
        const bool zero = (o == 0 && m.q0) || (o == 1 && m.q1) || (o == 2 && m.q2);
        const T f = zero ? T(0) : T(cf.force_scale * cf.kf * double(o == 0 ? m.n0 : o == 1 ? m.n1 : m.n2));
        w[q] = o == 3 ? v[q] : mk(f * v[q].y, -f * v[q].x);
      } else {   // SPEC_CFIELD
        const double ikb = m.msq != 0 ? 1.0 / (cf.kappa * cf.kf * sqrt(double(m.msq))) : 0.0;
        w[q] = scale(v[q], T(-ikb * ikb * cf.inv_n3));
      }
    }
    fft<T, N, P, +1>(w, twl, LR, tr);
    wave_sync();
#pragma unroll
    for (int q = 0; q < R; ++q) lds[G::at(r, tr) + q * TT + q * TT / G::kPad] = w[q];
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) w[q] = lds[G::at(t, c) + q * TT * G::kLD];
    fft<T, N, P, +1>(w, twl, LC, t);
    cx<T>* const dst = out + o * out_stride + off + c;
#pragma unroll
    for (int q = 0; q < R; ++q) dst[(size_t)(t + q * TT) * N] = w[q];
    lds_barrier();   // the column exchanges before the next output's row exchanges
  }
}

// Outputs per workgroup: one while all of a launch's workgroups fit the device at once, then as many
// as keep at most 512 workgroups (each repeats the forward transforms).
template <typename T, int N>
static void plane_n(SpecMode mode, const cx<T>* in, size_t is, cx<T>* out, size_t os, int nout, int batch,
                    const SpecCoef& cf, double* mean, const SolveCtl* ctl, hipStream_t s, const PassDecision& dec) {
  using G = PlaneGeo<T, N>;
  constexpr int H = N / 2 + 1;
  int per = 1;
  while (per < nout && batch * H * ((nout + per - 1) / per) > 512) ++per;
  const dim3 grid((nout + per - 1) / per, H, batch), blk(G::kThreads);
  const cx<T>* tw = twiddles<T>(N);
#define DGP_PLANE(M) hipLaunchKernelGGL((k_plane<T, N, M>), grid, blk, 0, s, in, is, out, os, nout, per, tw, cf, mean, ctl, dec)
  if (mode == SPEC_HSPLIT) DGP_PLANE(SPEC_HSPLIT);
  if (mode == SPEC_FORCES) DGP_PLANE(SPEC_FORCES);
  if constexpr (sizeof(T) == 8) {   // (the source and C are formed in float64)
    if (mode == SPEC_SOURCE) DGP_PLANE(SPEC_SOURCE);
    if (mode == SPEC_CFIELD) DGP_PLANE(SPEC_CFIELD);
  }
#undef DGP_PLANE
}

template <typename T>
bool plane_ok(int n) { return n <= kPlaneMax; }

template <typename T>
void launch_plane(int n, SpecMode mode, const cx<T>* in, size_t in_stride, cx<T>* out, size_t out_stride, int nout,
                  int batch, const SpecCoef& cf, double* mean_out, const SolveCtl* ctl, hipStream_t s,
                  const PassDecision* decision) {
  const PassDecision dec = decision ? *decision : PassDecision{};
#define C(NN) \
  case NN: plane_n<T, NN>(mode, in, in_stride, out, out_stride, nout, batch, cf, mean_out, ctl, s, dec); break;
  switch (n) {
    C(8) C(16) C(32) C(64)
    default: break;
  }
#undef C
}

template bool plane_ok<double>(int);
template bool plane_ok<float>(int);
template void launch_plane<double>(int, SpecMode, const cx<double>*, size_t, cx<double>*, size_t, int, int,
                                   const SpecCoef&, double*, const SolveCtl*, hipStream_t, const PassDecision*);
template void launch_plane<float>(int, SpecMode, const cx<float>*, size_t, cx<float>*, size_t, int, int,
                                  const SpecCoef&, double*, const SolveCtl*, hipStream_t, const PassDecision*);

}  // namespace dgp
