// Fused FFT-relaxation pass and its device-side convergence control.
//
// One relaxation pass (Sec. III B, Eq. FFTrelax with the w-split of Sec. III C)
// evaluates the residual of the current iterate u^(n) and produces u^(n+1).  The
// kernel here is its last stage: for a tile of axis-0 columns it
//   1. inverse-transforms along axis 0 the five Hessian spectra h00, h11, h01,
//      h02, h12 and the nonlocal spectrum Nf = -u(k)/kbar (the other two axes
//      were inverted by the preceding passes), accumulating in registers (float64;
//      float32 in the float32 form) sum_ij h_ij^2 and h22 = (u - <u>) - h00 - h11 (the trace identity:
//      h00 + h11 + h22 = u - <u>, exact on the mesh, saves a sixth transform);
//   2. evaluates, per point, the residual R of Eq. FullDGP2, B' of Eq. Bwpara,
//      the discriminant of Eq. nabla^2Cwpara and its + root in the stable form
//      2 B'/(alpha + sqrt(Delta)); a negative discriminant is a bad point and
//      takes the vertex -alpha/(2 (1-w) lam) (Sec. III C);
//   3. writes u^(n+1) and immediately forward-transforms it along axis 0, so
//      the next pass starts from its axis-0 spectrum;
//   4. reduces sum |R| (FP64) and the bad-point count per workgroup.
// k_finalize (one workgroup per batch element) or, up to 64^3, the next pass's plane
// launch then forms r = <|R|>/eps (Eq. normres) and runs the stopping rules; kernels of
// later passes read the per-element `done` flag and exit at once.
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "control.h"
#include "dgp_internal.h"

namespace dgp {

template <typename T>
const cx<T>* twiddles(int n);

// FFT plans of the axis-0 transforms in the relaxation pass (0: radix 8, 1: radix 16, 2: radix 4)
#ifndef DGP_PLAN_RELAX
#define DGP_PLAN_RELAX 2
#endif
#ifndef DGP_PLAN_RELAX_F32
#define DGP_PLAN_RELAX_F32 0
#endif
#ifndef DGP_RELAX_F32ACC
#define DGP_RELAX_F32ACC 1
#endif
#ifndef DGP_RELAX_TP_F32
#define DGP_RELAX_TP_F32 8
#endif
#ifndef DGP_RELAX_MINW_F32
#define DGP_RELAX_MINW_F32 1
#endif
// column pairs of the float32 kernel from N = 512 on
#ifndef DGP_RELAX_TP_WIDE_F32
#define DGP_RELAX_TP_WIDE_F32 16
#endif
// smallest N whose float32 relaxation kernel pairs its lanes: the two threads whose transform
// elements e and N - e share a spectral row sit in one wavefront and load that row in the same
// instruction (one request instead of two)
#ifndef DGP_RELAX_PAIRED_MIN
#define DGP_RELAX_PAIRED_MIN 256
#endif
// smallest N whose float32 relaxation kernel re-derives its lane indices at every field, so that
// the per-lane addresses built from them are not held across the field loop (at N = 512 the
// 1024-thread workgroup leaves 128 VGPRs per lane)
#ifndef DGP_RELAX_REMAT_MIN
#define DGP_RELAX_REMAT_MIN 256
#endif
// padding rows of the float32 kernel's transform exchanges (one after every DGP_RELAX_LDSPAD rows)
#ifndef DGP_RELAX_LDSPAD
#define DGP_RELAX_LDSPAD 8
#endif
// smallest N whose float32 relaxation kernel keeps the running h22 = -(h00 + h11) in LDS (each
// thread its own slots) instead of registers across the field loop
#ifndef DGP_RELAX_PARK_MIN
#define DGP_RELAX_PARK_MIN 256
#endif

// axis-0 tile of the relaxation kernel: AxisTile with an optional number of column pairs
template <typename T, int N, int R, int TPSET>
struct RelaxTile {
  static constexpr int kT = AxisTile<T, N, R>::kT;
  static constexpr int kTP = TPSET > 0 ? (TPSET < N / 2 ? TPSET : N / 2) : AxisTile<T, N, R>::kTP;
  static constexpr int kThreads = kTP * kT;
};

// geometry of the float32 relaxation kernel
template <typename T, int N>
struct RelaxGeo {
  static_assert(sizeof(T) == 4, "the block-synchronous relaxation kernel is the float32 one");
  // at N >= 512 the spectral planes are 2 MB apart and a 128-byte row segment per plane streams
  // poorly: radix 8 and 16 column pairs (256-byte segments)
  static constexpr bool kWide = N >= 512;
  using P = typename PlanPick<N, (kWide ? 0 : DGP_PLAN_RELAX_F32)>::type;
  static constexpr int R = P::R;
  using G = RelaxTile<T, N, R, (kWide ? DGP_RELAX_TP_WIDE_F32 : DGP_RELAX_TP_F32)>;
  // minimum wavefronts per SIMD the register allocation plans for (second launch bound)
  static constexpr int kMinWaves = DGP_RELAX_MINW_F32;
  // accumulators of the float32 form (sum h^2 and -(h00 + h11)): float32 or float64; the
  // residual, discriminant and root are float64 either way
  using Acc = typename std::conditional<DGP_RELAX_F32ACC, float, double>::type;
  // lane order of the paired loads (needs an even number of transform positions per wavefront)
  static constexpr bool kPaired = N >= DGP_RELAX_PAIRED_MIN && (64 / G::kTP) % 2 == 0;
  static constexpr bool kRemat = N >= DGP_RELAX_REMAT_MIN;
  static constexpr bool kPark = N >= DGP_RELAX_PARK_MIN;
};

// Per-point residual and update in float64 (Eqs. FullDGP2, Bwpara, nabla^2Cwpara).  The + root
// 2 B' / (alpha + sqrt(Delta)) is formed without branches: the hardware estimates of
// 1/sqrt(Delta) and of the reciprocal of the denominator (float64 instructions) are refined by
// one Newton step each, sqrt(Delta) = Delta / sqrt(Delta) gets one Heron correction and the
// quotient one residual correction (each correction squares the relative error).  Delta = 0 takes sqrt = 0, and a
// negative Delta (a bad point) takes the vertex -alpha / (2 (1-w) lam).  Straight-line code
// lets the compiler interleave the points of a thread.
struct PointCoef {
  double lam, w, alpha, gamma, omega, mu, vertex, c4;
};

__device__ __forceinline__ PointCoef point_coef(const SolveCfg& cfg, double mu) {
  PointCoef k;
  k.lam = cfg.lam;
  k.w = cfg.w;
  k.alpha = cfg.alpha;
  k.gamma = cfg.gamma;
  k.omega = cfg.omega;
  k.mu = mu;
  k.vertex = -cfg.alpha / (2.0 * (1.0 - cfg.w) * cfg.lam);
  k.c4 = 4.0 * (1.0 - cfg.w) * cfg.lam;
  return k;
}

// u: iterate, s: source, nf: nonlocal term, s2: sum of the squared Hessian entries other than
// h22, h22m: -(h00 + h11) (h22 = h22m + u - <u> by the trace identity)
__device__ __forceinline__ double relax_point(const PointCoef& k, double u, double s, double nf, double s2,
                                              double h22m, double& abs_r, int& nbad) {
  const double hz = h22m + (u - k.mu);
  const double sh2 = s2 + hz * hz;
  const double res = k.lam * (u * u - sh2) + k.alpha * u + k.gamma * nf - s;
  abs_r += fabs(res);
  const double bp = k.lam * (sh2 - k.w * u * u) - k.gamma * nf + s;
  const double disc = k.alpha * k.alpha + k.c4 * bp;
  nbad += disc < 0.0 ? 1 : 0;
  double y = __builtin_amdgcn_rsq(disc);
  y = y * (1.5 - (0.5 * disc) * (y * y));
  double sq = disc * y;
  sq = fma(0.5 * y, fma(-sq, sq, disc), sq);   // Heron correction of sqrt(Delta)
  sq = disc > 0.0 ? sq : 0.0;
  const double den = k.alpha + sq;
  double r = __builtin_amdgcn_rcp(den);
  r = r * (2.0 - den * r);
  const double num = 2.0 * bp;
  double x = num * r;
  x = fma(r, fma(-den, x, num), x);
  x = disc < 0.0 ? k.vertex : x;
  if (k.omega != 1.0) x = (1.0 - k.omega) * u + k.omega * x;
  return x;
}

template <int R, typename V, typename A>
__device__ __forceinline__ void relax_points(const PointCoef& k, const V (&up)[R], const V (&spv)[R], const V (&nfv)[R],
                                             const A (&s2)[R][2], const A (&h22)[R][2], double (&un)[R][2],
                                             double& abs_r, int& nbad) {
#pragma unroll
  for (int q = 0; q < R; ++q)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      un[q][j] = relax_point(k, double(j ? up[q].y : up[q].x), double(j ? spv[q].y : spv[q].x),
                             double(j ? nfv[q].y : nfv[q].x), double(s2[q][j]), double(h22[q][j]), abs_r, nbad);
}

// float32 kernel: block-synchronous transforms; each thread loads, one field ahead, exactly the
// spectral rows its transform elements need (row e, or row N - e conjugated), so the tile is not
// staged in LDS
template <typename T, int N>
__global__ void __launch_bounds__((RelaxGeo<T, N>::G::kThreads), (RelaxGeo<T, N>::kMinWaves))
k_relax(const cx<T>* __restrict__ spec6, size_t fstride, T* __restrict__ ubuf, const T* __restrict__ sfield,
        cx<T>* __restrict__ spec_u, double* __restrict__ partial, const double* __restrict__ mean_u, SolveCfg cfg,
        const SolveCtl* __restrict__ ctl, const cx<T>* __restrict__ tw) {
  using RG = RelaxGeo<T, N>;
  using P = typename RG::P;
  using Acc = typename RG::Acc;
  constexpr int R = P::R;
  using G = typename RG::G;
  constexpr int TP = G::kTP, TT = G::kT, H = N / 2 + 1;
  constexpr size_t N3 = (size_t)N * N * N;
  const int b = blockIdx.z;
  if (ctl[b].done) return;
  const int cur = ctl[b].cur, nxt = ctl[b].out;
  int tile, i1;
  xcd_tile(tile, i1);
  int c = threadIdx.x % TP;
  // transform element index t of this thread.  Paired order: positions g = 0, 1 take t = 0 and
  // TT/2 (their own partners), then g = 2k, 2k + 1 take t = k and TT - k, so a wavefront (64/TP
  // consecutive positions, an even count) holds both threads of every pair; elements e = t + q TT
  // and N - e = (TT - t) + (R - 1 - q) TT read the same spectral row
  const int g = threadIdx.x / TP;
  constexpr bool PAIRED = RG::kPaired;
  int t = !PAIRED ? g : g < 2 ? g * (TT / 2) : (g & 1) ? TT - (g >> 1) : (g >> 1);
  const int i2 = (tile * TP + c) * 2;
  // transform exchanges, then (kPark) R slots per thread for the running h22
  constexpr int PG = DGP_RELAX_LDSPAD, LROWS = PG > 0 ? N + N / PG : N;
  __shared__ cx<T> lds[LROWS * TP + (RG::kPark ? R * G::kThreads : 0)];
  cx<T>* const park = lds + LROWS * TP + threadIdx.x;   // slot q at park[q * kThreads]
  __shared__ double red[(G::kThreads + 63) / 64];
  __shared__ int redi[(G::kThreads + 63) / 64];
  // the twiddle table is read from LDS: the seven transforms of a pass would otherwise wait on
  // cached global loads at every stage
  __shared__ cx<T> twl[N];
  for (int i = threadIdx.x; i < N; i += G::kThreads) twl[i] = tw[i];

  const size_t col = (size_t)b * H * N * N + SpecRows<N>::col(i1) + i2;
  typedef float f4 __attribute__((ext_vector_type(4)));
  const size_t col0 = (size_t)b * H * N * N + SpecRows<N>::col(i1) + (size_t)tile * TP * 2;
  // element q of thread t is row e = t + q TT of the Hermitian-extended column pair; rows e > N/2
  // come from row N - e (conjugated when used); streaming loads (the last use of these spectra in
  // the pass).  With paired lanes, threads t > TT/2 load their elements in reverse slot order, so
  // that slot q of both threads of a pair addresses the same row.
  cx<T> pd[R][2];
  // (a workgroup-uniform base plus a 32-bit lane offset: one register per address)
  static_assert((size_t)(N / 2 + 1) * N * N * sizeof(cx<T>) < (size_t(1) << 32), "32-bit row offsets");
  auto fetch_direct = [&](int f) {
    const char* src = reinterpret_cast<const char*>(spec6 + f * fstride + col0);
#pragma unroll
    for (int q = 0; q < R; ++q) {   // slot q holds element R - 1 - q when rev
      const bool rev = PAIRED && t > TT / 2;
      const int e = t + (rev ? R - 1 - q : q) * TT;
      const unsigned r = e <= N / 2 ? e : N - e;
      const f4* a = reinterpret_cast<const f4*>(src + (r * SpecRows<N>::kPlane + 2u * c) * unsigned(sizeof(cx<T>)));
      const f4 x = __builtin_nontemporal_load(a);
      pd[q][0] = mk(T(x.x), T(x.y));
      pd[q][1] = mk(T(x.z), T(x.w));
    }
  };
  fetch_direct(0);

  Acc s2[R][2], h22[R][2];
  cx<T> v[R];
  cx<T> up[R], spv[R];
#pragma unroll 1
  for (int f = 0; f < 6; ++f) {
    if constexpr (RG::kRemat) asm volatile("" : "+v"(t), "+v"(c));   // opaque: recomputed per field
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      const bool rev = PAIRED && t > TT / 2;
      cx<T> xa = rev ? pd[R - 1 - q][0] : pd[q][0], xb = rev ? pd[R - 1 - q][1] : pd[q][1];
      if (e > N / 2) {
        xa = conjg(xa);
        xb = conjg(xb);
      }
      if (e == 0 || e == N / 2) { xa.y = T(0); xb.y = T(0); }
      v[q] = mk(xa.x - xb.y, xa.y + xb.x);   // x_a + i x_b
    }
    if (f < 5) fetch_direct(f + 1);
    {
      LdsCol<T, TP, PG> L{lds, c};
      fft<T, N, P, +1>(v, twl, L, t);
    }
    if (f < 5) {
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const Acc hx = Acc(v[q].x), hy = Acc(v[q].y);
        if (f == 0) {
          s2[q][0] = hx * hx;
          s2[q][1] = hy * hy;
          if constexpr (RG::kPark) {
            park[q * G::kThreads] = mk(T(-hx), T(-hy));
          } else {
            h22[q][0] = -hx;
            h22[q][1] = -hy;
          }
        } else if (f == 1) {
          s2[q][0] += hx * hx;
          s2[q][1] += hy * hy;
          if constexpr (RG::kPark) {
            const cx<T> hz = park[q * G::kThreads];
            park[q * G::kThreads] = mk(hz.x - T(hx), hz.y - T(hy));
          } else {
            h22[q][0] -= hx;
            h22[q][1] -= hy;
          }
        } else {
          s2[q][0] += Acc(2) * hx * hx;
          s2[q][1] += Acc(2) * hy * hy;
        }
      }
    }
  }
  // pointwise residual and update; v holds Nf (field addresses formed after the field loop)
  const T* uin = ubuf + ((size_t)cur * cfg.batch + b) * N3 + RealRows<T, N>::col(i1) + i2;
  const T* sp = sfield + (size_t)b * N3 + RealRows<T, N>::col(i1) + i2;
  const PointCoef pc = point_coef(cfg, mean_u[b]);
  T* uout = ubuf + ((size_t)nxt * cfg.batch + b) * N3 + RealRows<T, N>::col(i1) + i2;
  double abs_r = 0.0;
  int nbad = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const size_t off = (t + q * TT) * RealRows<T, N>::kPlane;
    up[q] = *reinterpret_cast<const cx<T>*>(uin + off);
    spv[q] = *reinterpret_cast<const cx<T>*>(sp + off);
  }
  if constexpr (RG::kPark) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const cx<T> hz = park[q * G::kThreads];
      h22[q][0] = Acc(hz.x);
      h22[q][1] = Acc(hz.y);
    }
  }
  double un[R][2];
  relax_points(pc, up, spv, v, s2, h22, un, abs_r, nbad);
  if constexpr (RG::kRemat) asm volatile("" : "+v"(t), "+v"(c));   // the epilogue's addresses from here
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const size_t off = (t + q * TT) * RealRows<T, N>::kPlane;
    const cx<T> o = mk(T(un[q][0]), T(un[q][1]));
    store_stream(reinterpret_cast<cx<T>*>(uout + off), o);   // read again next pass only
    v[q] = o;
  }
  // forward axis-0 transform of u^(n+1)
  {
    LdsCol<T, TP, PG> L{lds, c};
    fft<T, N, P, -1>(v, twl, L, t);
  }
  lds_barrier();
#pragma unroll
  for (int q = 0; q < R; ++q) lds[(t + q * TT) * TP + c] = v[q];
  constexpr int WW = G::kThreads < 64 ? G::kThreads : 64;
  abs_r = wave_sum<WW, G::kThreads>(abs_r);
  nbad = wave_sum<WW, G::kThreads>(nbad);
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = abs_r;
    redi[threadIdx.x >> 6] = nbad;
  }
  lds_barrier();
  cx<T>* dst = spec_u + col;
  for (int k = t; k < H; k += TT) {
    const cx<T> zk = lds[k * TP + c];
    const cx<T> zn = lds[((N - k) & (N - 1)) * TP + c];
    dst[(size_t)k * SpecRows<N>::kPlane] = mk(T(0.5) * (zk.x + zn.x), T(0.5) * (zk.y - zn.y));
    dst[(size_t)k * SpecRows<N>::kPlane + 1] = mk(T(0.5) * (zk.y + zn.y), T(0.5) * (zn.x - zk.x));
  }
  // per-wavefront sums added in wavefront order (deterministic)
  if (threadIdx.x == 0) {
    double sr = 0.0;
    int sb = 0;
#pragma unroll
    for (int i = 0; i < (G::kThreads + 63) / 64; ++i) {
      sr += red[i];
      sb += redi[i];
    }
    const size_t g = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    const size_t groups = (size_t)gridDim.x * gridDim.y;
    partial[((size_t)b * groups + g) * 2] = sr;
    partial[((size_t)b * groups + g) * 2 + 1] = double(sb);
  }
}


// ------------------------------------------------------------------ float64 kernel (wave-local)
// Same pass as k_relax, restructured so that each axis-0 transform is carried by the
// lanes of one wavefront: its Stockham exchanges then need wavefront ordering only,
// and the workgroup barriers drop from one pair per stage to one per field.  Global
// traffic stays coalesced: spectral tiles are fetched row-wise into a double-buffered,
// padded LDS tile; a transform reads its own two columns of the tile and reuses the
// same slots (only its wavefront touches them) for the exchanges.  Below N = 512, u and S are
// read row-wise too and redistributed to the transforms through the two tiles once the field
// loop is done.
#ifndef DGP_RELAXW_TP_F64
#define DGP_RELAXW_TP_F64 0
#endif
#ifndef DGP_RELAXW_MINW_F64
#define DGP_RELAXW_MINW_F64 3
#endif
// column pairs of the float64 kernel from N = 256 on
#ifndef DGP_RELAXW_TP_WIDE_F64
#define DGP_RELAXW_TP_WIDE_F64 8
#endif
// smallest N whose float64 relaxation kernel reads its twiddles from LDS
#ifndef DGP_RELAXW_TWLDS_MIN
#define DGP_RELAXW_TWLDS_MIN 256
#endif

// float64 kernel: u and S read row-wise (consecutive lanes on one row) and redistributed through
// LDS (1), instead of each lane reading its own transform's elements, 64 rows per instruction (0)
// (256^3 on gfx950: 345 vs 363 us per launch)
#ifndef DGP_RELAXW_US_LDS
#define DGP_RELAXW_US_LDS 1
#endif

template <typename T, int N>
struct RelaxWGeo {
  static_assert(sizeof(T) == 8, "the wave-local relaxation kernel is the float64 one");
  // at N >= 256: radix 8 (one 512-point transform per wavefront, two of 256) and 8 column pairs, whose
  // 256-byte spectral and 128-byte real row segments stream better than 4 pairs' half (256^3: 365 -> 348
  // us, with the twiddles in LDS and two waves per SIMD; radix 4 with 8 pairs 368-438 us, radix 8 with 4
  // pairs 370 us, 16 pairs 376 us).  At 128^3 radix 4 and 4 pairs are as fast (349 vs 350-365 us).
  static constexpr bool kWide = N >= 256;
  using P = typename PlanPick<N, (kWide ? 0 : DGP_PLAN_RELAX)>::type;
  static constexpr int R = P::R;
  using G = AxisTile<T, N, R>;
  static constexpr int kTPSet = kWide ? DGP_RELAXW_TP_WIDE_F64 : DGP_RELAXW_TP_F64;
  static constexpr int kTP = kTPSet > 0 ? (kTPSet < N / 2 ? kTPSet : N / 2) : G::kTP;
  static constexpr int kT = G::kT, kThreads = kTP * kT, H = N / 2 + 1;
  static constexpr int kMinWaves = kWide ? 2 : DGP_RELAXW_MINW_F64;   // the LDS tile allows two workgroups per CU at N = 256, one at 512
  // twiddles from an LDS copy: held in registers, the loop-invariant twiddles of the six
  // inverse transforms would need 56 VGPRs across the field loop at N = 512, where the kernel
  // already uses most of the 256 of a two-waves-per-SIMD allocation
  static constexpr bool kTwLds = N >= DGP_RELAXW_TWLDS_MIN;
  // u and S read row-wise and redistributed through LDS (below N = 512: the staging registers
  // would not fit the allocation there)
  static constexpr bool kUsLds = DGP_RELAXW_US_LDS && N < 512;
  static_assert(kT <= 64 && 64 % kT == 0, "a transform must stay inside one wavefront");
  static constexpr int kSP = 2 * kTP + 1;                            // padded tile row, complex
  static constexpr int kTile = H * kSP;
  static constexpr int kNPF = (H * kTP + kThreads - 1) / kThreads;   // column pairs fetched per thread
  static constexpr int kWaves = (kThreads + 63) / 64;
  static constexpr int kWidth = kThreads < 64 ? kThreads : 64;       // lanes of a wavefront sum
};

// Exchange slots of transform c inside its own two tile columns (2c, 2c+1).
template <typename T, int SP>
struct LdsPair {
  cx<T>* base;
  int c;
  __device__ __forceinline__ cx<T> load(int e) const { return base[(e >> 1) * SP + 2 * c + (e & 1)]; }
  __device__ __forceinline__ void store(int e, cx<T> v) const { base[(e >> 1) * SP + 2 * c + (e & 1)] = v; }
  // (S even; with Ns = 1 e is even, else Ns is)
  template <int S>
  __device__ __forceinline__ cx<T> load_q(int j, int q) const { return base[(j >> 1) * SP + 2 * c + (j & 1) + q * (S / 2) * SP]; }
  template <int Ns>
  __device__ __forceinline__ void store_q(int e, int q, cx<T> v) const {
    if constexpr (Ns == 1) base[(e >> 1) * SP + 2 * c + (q >> 1) * SP + (q & 1)] = v;
    else base[(e >> 1) * SP + 2 * c + (e & 1) + q * (Ns / 2) * SP] = v;
  }
  __device__ __forceinline__ void sync() const { wave_sync(); }
};


// (the second launch bound is the minimum number of wavefronts per SIMD to plan registers for)
template <typename T, int N>
__global__ void __launch_bounds__((RelaxWGeo<T, N>::kThreads), (RelaxWGeo<T, N>::kMinWaves))
k_relax_w(const cx<T>* __restrict__ spec6, size_t fstride, T* __restrict__ ubuf, const T* __restrict__ sfield,
          cx<T>* __restrict__ spec_u, double* __restrict__ partial, const double* __restrict__ mean_u, SolveCfg cfg,
          const SolveCtl* __restrict__ ctl, const cx<T>* __restrict__ tw) {
  using W = RelaxWGeo<T, N>;
  using P = typename W::P;
  constexpr int R = W::R, TP = W::kTP, TT = W::kT, NT = W::kThreads, H = N / 2 + 1, SP = W::kSP;
  constexpr int NPF = W::kNPF;
  constexpr size_t N3 = (size_t)N * N * N, NN = (size_t)N * N;
  const int b = blockIdx.z;
  if (ctl[b].done) return;
  const int cur = ctl[b].cur, nxt = ctl[b].out;
  int tile, i1;
  xcd_tile(tile, i1);
  const int i2 = tile * 2 * TP;
  const int c = threadIdx.x / TT, t = threadIdx.x % TT;   // transform mapping
  __shared__ cx<T> lds[2 * W::kTile];
  __shared__ double redd[W::kWaves];
  __shared__ int redi[W::kWaves];
  __shared__ cx<T> twl[W::kTwLds ? N : 1];
  const cx<T>* twp = tw;
  if constexpr (W::kTwLds) {
    for (int i = threadIdx.x; i < N; i += NT) twl[i] = tw[i];   // ordered by the first field's barrier
    twp = twl;
  }

  const size_t col0 = (size_t)b * H * NN + SpecRows<N>::col(i1) + i2;
  cx<T> pf[NPF][2];
  // every thread loads NPF pairs, indices past the tile clamped to its last pair, so the
  // staging registers are assigned unconditionally and stay in registers
  auto fetch = [&](int f) {
    const cx<T>* src = spec6 + f * fstride + col0;
#pragma unroll
    for (int r = 0; r < NPF; ++r) {
      const int idx = min(int(threadIdx.x) + r * NT, H * TP - 1);
      const int k = idx / TP, p = idx % TP;
      const cx<T>* q = src + (size_t)k * SpecRows<N>::kPlane + 2 * p;
      pf[r][0] = mk(q[0].x, q[0].y);   // member-wise: a 16-byte struct copy would stay in private memory
      pf[r][1] = mk(q[1].x, q[1].y);
    }
  };
  // (a clamped index rewrites the last pair with the value it already holds)
  auto stash = [&](cx<T>* buf) {
#pragma unroll
    for (int r = 0; r < NPF; ++r) {
      const int idx = min(int(threadIdx.x) + r * NT, H * TP - 1);
      const int k = idx / TP, p = idx % TP;
      buf[k * SP + 2 * p].x = pf[r][0].x;
      buf[k * SP + 2 * p].y = pf[r][0].y;
      buf[k * SP + 2 * p + 1].x = pf[r][1].x;
      buf[k * SP + 2 * p + 1].y = pf[r][1].y;
    }
  };
  fetch(0);

  double s2[R][2], h22[R][2];
  cx<T> v[R], up[R], spv[R];
#pragma unroll 1
  for (int f = 0; f < 6; ++f) {
    cx<T>* buf = lds + (f & 1) * W::kTile;
    stash(buf);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      cx<T> xa, xb;
      if (e <= N / 2) {
        xa = buf[e * SP + 2 * c];
        xb = buf[e * SP + 2 * c + 1];
        if (e == 0 || e == N / 2) { xa.y = T(0); xb.y = T(0); }
      } else {
        xa = conjg(buf[(N - e) * SP + 2 * c]);
        xb = conjg(buf[(N - e) * SP + 2 * c + 1]);
      }
      v[q] = mk(xa.x - xb.y, xa.y + xb.x);
    }
    if (f < 5) fetch(f + 1);
    LdsPair<T, SP> X{buf, c};
    fft<T, N, P, +1>(v, twp, X, t);
    if (f < 5) {
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const double hx = v[q].x, hy = v[q].y;
        if (f == 0) {
          s2[q][0] = hx * hx;
          s2[q][1] = hy * hy;
          h22[q][0] = -hx;
          h22[q][1] = -hy;
        } else if (f == 1) {
          s2[q][0] += hx * hx;
          s2[q][1] += hy * hy;
          h22[q][0] -= hx;
          h22[q][1] -= hy;
        } else {
          s2[q][0] += 2.0 * hx * hx;
          s2[q][1] += 2.0 * hy * hy;
        }
      }
    }
  }
  // pointwise residual and update (v holds Nf); u^(n+1) is staged in tile 0 (free since the last barrier).
  // The field addresses are formed here, after the field loop, so that they are not held in
  // registers across it.
  const PointCoef pc = point_coef(cfg, mean_u[b]);
  T* ust = reinterpret_cast<T*>(lds);
  double abs_r = 0.0;
  int nbad = 0;
  if constexpr (W::kUsLds) {
    // row-wise reads (TP lanes per row, one column pair each) into tile 0 (u) and tile 1 (S),
    // rows 2 TP + 1 values apart; tile 1 is free once every wavefront has finished its last
    // inverse transform (first barrier); the second barrier orders the reads before the forward
    // transform's exchanges in tile 1
    constexpr int NU = (N * TP + NT - 1) / NT;
    const T* ur = ubuf + ((size_t)cur * cfg.batch + b) * N3 + RealRows<T, N>::col(i1) + i2;
    const T* sr = sfield + (size_t)b * N3 + RealRows<T, N>::col(i1) + i2;
    cx<T> lu[NU], ls[NU];
#pragma unroll
    for (int r = 0; r < NU; ++r) {
      const int idx = min(int(threadIdx.x) + r * NT, N * TP - 1);
      const int e = idx / TP, p = idx % TP;
      lu[r] = *reinterpret_cast<const cx<T>*>(ur + e * RealRows<T, N>::kPlane + 2 * p);
      ls[r] = *reinterpret_cast<const cx<T>*>(sr + e * RealRows<T, N>::kPlane + 2 * p);
    }
    T* sst = reinterpret_cast<T*>(lds + W::kTile);
    lds_barrier();
#pragma unroll
    for (int r = 0; r < NU; ++r) {
      const int idx = min(int(threadIdx.x) + r * NT, N * TP - 1);
      const int e = idx / TP, p = idx % TP;
      ust[e * (2 * TP + 1) + 2 * p] = lu[r].x;
      ust[e * (2 * TP + 1) + 2 * p + 1] = lu[r].y;
      sst[e * (2 * TP + 1) + 2 * p] = ls[r].x;
      sst[e * (2 * TP + 1) + 2 * p + 1] = ls[r].y;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      up[q] = mk(ust[e * (2 * TP + 1) + 2 * c], ust[e * (2 * TP + 1) + 2 * c + 1]);
      spv[q] = mk(sst[e * (2 * TP + 1) + 2 * c], sst[e * (2 * TP + 1) + 2 * c + 1]);
    }
    lds_barrier();
  } else {
    const T* uin = ubuf + ((size_t)cur * cfg.batch + b) * N3 + RealRows<T, N>::col(i1) + i2 + 2 * c;
    const T* sp = sfield + (size_t)b * N3 + RealRows<T, N>::col(i1) + i2 + 2 * c;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      up[q] = *reinterpret_cast<const cx<T>*>(uin + e * RealRows<T, N>::kPlane);
      spv[q] = *reinterpret_cast<const cx<T>*>(sp + e * RealRows<T, N>::kPlane);
    }
  }
  double un[R][2];
  relax_points(pc, up, spv, v, s2, h22, un, abs_r, nbad);
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int e = t + q * TT;
    const cx<T> o = mk(T(un[q][0]), T(un[q][1]));
    ust[e * (2 * TP + 1) + 2 * c] = o.x;
    ust[e * (2 * TP + 1) + 2 * c + 1] = o.y;
    v[q] = o;
  }
  // forward axis-0 transform of u^(n+1), exchanges in the transform's own columns of tile 1
  {
    LdsPair<T, SP> X{lds + W::kTile, c};
    fft<T, N, P, -1>(v, twp, X, t);
  }
  abs_r = wave_sum<W::kWidth, NT>(abs_r);
  nbad = wave_sum<W::kWidth, NT>(nbad);
  if ((threadIdx.x & 63) == 0) {
    redd[threadIdx.x >> 6] = abs_r;
    redi[threadIdx.x >> 6] = nbad;
  }
  lds_barrier();
  // u^(n+1) out of tile 0 (coalesced); the spectrum into tile 1, column-major with one pad
  T* uout = ubuf + ((size_t)nxt * cfg.batch + b) * N3 + RealRows<T, N>::col(i1) + i2;
  for (int idx = threadIdx.x; idx < N * TP; idx += NT) {
    const int e = idx / TP, p = idx % TP;
    const cx<T> o = mk(ust[e * (2 * TP + 1) + 2 * p], ust[e * (2 * TP + 1) + 2 * p + 1]);
    *reinterpret_cast<cx<T>*>(uout + e * RealRows<T, N>::kPlane + 2 * p) = o;
  }
  cx<T>* zt = lds + W::kTile;
#pragma unroll
  for (int q = 0; q < R; ++q) zt[c * (N + 1) + t + q * TT] = v[q];
  lds_barrier();
  cx<T>* dst = spec_u + col0;
  for (int idx = threadIdx.x; idx < H * TP; idx += NT) {
    const int k = idx / TP, p = idx % TP;
    const cx<T> zk = zt[p * (N + 1) + k];
    const cx<T> zn = zt[p * (N + 1) + ((N - k) & (N - 1))];
    dst[(size_t)k * SpecRows<N>::kPlane + 2 * p] = mk(T(0.5) * (zk.x + zn.x), T(0.5) * (zk.y - zn.y));
    dst[(size_t)k * SpecRows<N>::kPlane + 2 * p + 1] = mk(T(0.5) * (zk.y + zn.y), T(0.5) * (zn.x - zk.x));
  }
  if (threadIdx.x == 0) {
    double sr = 0.0;
    int sb = 0;
    for (int i = 0; i < W::kWaves; ++i) {
      sr += redd[i];
      sb += redi[i];
    }
    const size_t g = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    const size_t groups = (size_t)gridDim.x * gridDim.y;
    partial[((size_t)b * groups + g) * 2] = sr;
    partial[((size_t)b * groups + g) * 2 + 1] = double(sb);
  }
}

// ------------------------------------------------------------------ small meshes (N <= 64)
// The same pass with one group of threads per field: a launch on a mesh this small does not fill the
// device, and its time is its latency chain, six transforms one after another in k_relax and
// k_relax_w.  Here the six fields are loaded and inverse-transformed at once by six groups, the
// transformed values meet in LDS, every thread takes pair-points of the update, and the first group
// forward-transforms u^(n+1).  A group's transforms (radix 8, one exchange up to N = 64) sit inside
// one wavefront.  One 32^3 float64 field: 10.8 -> 5.5 us, one 64^3: 13.6 -> 10.2 us; 5 x 64^3 float32
// 15.1 us either way.
constexpr int kRelaxSmallMax = 64;
template <typename T, int N>
struct RelaxSGeo {
  using P = Plan8<N>;
  static constexpr int R = P::R, kT = N / R;
  static constexpr int kBase = 128 / (4 * int(sizeof(T)));   // column pairs of a 128-byte row segment
  static constexpr int kTP = kBase < N / 2 ? kBase : N / 2;
  // whole wavefronts (the residual's sums shuffle over all lanes); threads past the six groups take
  // pair-points of the update only
  static constexpr int kGroup = kTP * kT, kWaves = (6 * kGroup + 63) / 64, kThreads = 64 * kWaves;
  static constexpr int kPts = N * kTP, kPPT = (kPts + kThreads - 1) / kThreads;   // pair-points, per thread
  // exchange rows padded by one after every 8, as in k_relax
  static constexpr int kField = (N + N / 8) * kTP;
  static_assert(64 % kGroup == 0, "a group's lanes sit in one wavefront");
};

template <typename T, int C>
struct LdsColWave : LdsCol<T, C, 8> {   // column exchanges inside one wavefront
  __device__ __forceinline__ void sync() const { wave_sync(); }
};

template <typename T, int N>
__global__ void __launch_bounds__((RelaxSGeo<T, N>::kThreads))
k_relax_small(const cx<T>* __restrict__ spec6, size_t fstride, T* __restrict__ ubuf, const T* __restrict__ sfield,
              cx<T>* __restrict__ spec_u, double* __restrict__ partial, const double* __restrict__ mean_u, SolveCfg cfg,
              const SolveCtl* __restrict__ ctl, const cx<T>* __restrict__ tw) {
  using G = RelaxSGeo<T, N>;
  using P = typename G::P;
  constexpr int R = G::R, TP = G::kTP, TT = G::kT, NT = G::kThreads, H = N / 2 + 1;
  constexpr size_t N3 = (size_t)N * N * N, NN = (size_t)N * N;
  const int b = blockIdx.z;
  if (ctl[b].done) return;
  int tile, i1;
  xcd_tile(tile, i1);
  const int i2 = tile * 2 * TP;
  const int f = threadIdx.x / G::kGroup, l = threadIdx.x % G::kGroup, c = l % TP, t = l / TP;
  __shared__ cx<T> lds[6 * G::kField];
  __shared__ cx<T> twl[N];
  __shared__ double red[G::kWaves];
  __shared__ int redi[G::kWaves];
  const size_t col0 = (size_t)b * H * NN + (size_t)i1 * N + i2;
  // the spectral rows of the thread's transform elements (row N - e conjugated), one column pair each
  const bool grouped = NT == 6 * G::kGroup || f < 6;
  cx<T> xa[R], xb[R];
  if (grouped) {
    const cx<T>* src = spec6 + f * fstride + col0 + 2 * c;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      const cx<T>* p = src + (size_t)(e <= N / 2 ? e : N - e) * NN;
      xa[q] = mk(p[0].x, p[0].y);
      xb[q] = mk(p[1].x, p[1].y);
    }
  }
  const size_t pt0 = (size_t)i1 * N + i2;
  const T* uin = ubuf + ((size_t)ctl[b].cur * cfg.batch + b) * N3 + pt0;
  const T* sp = sfield + (size_t)b * N3 + pt0;
  cx<T> up[G::kPPT], spv[G::kPPT];
#pragma unroll
  for (int k = 0; k < G::kPPT; ++k) {
    const int pt = min(int(threadIdx.x) + k * NT, G::kPts - 1);
    const size_t off = (size_t)(pt / TP) * NN + 2 * (pt % TP);
    up[k] = *reinterpret_cast<const cx<T>*>(uin + off);
    spv[k] = *reinterpret_cast<const cx<T>*>(sp + off);
  }
  for (int i = threadIdx.x; i < N; i += NT) twl[i] = tw[i];
  lds_barrier();
  cx<T> v[R];
  LdsColWave<T, TP> L;
  L.base = lds + f * G::kField;
  L.c = c;
  if (grouped) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int e = t + q * TT;
      if (e > N / 2) {
        xa[q] = conjg(xa[q]);
        xb[q] = conjg(xb[q]);
      }
      if (e == 0 || e == N / 2) { xa[q].y = T(0); xb[q].y = T(0); }
      v[q] = mk(xa[q].x - xb[q].y, xa[q].y + xb[q].x);   // x_a + i x_b
    }
    fft<T, N, P, +1>(v, twl, L, t);
    wave_sync();
#pragma unroll
    for (int q = 0; q < R; ++q) L.store(t + q * TT, v[q]);
  }
  lds_barrier();
  // pointwise residual and update; a pair-point's slots are read, and its first one rewritten, by
  // its own thread only
  const PointCoef pc = point_coef(cfg, mean_u[b]);
  T* uout = ubuf + ((size_t)ctl[b].out * cfg.batch + b) * N3 + pt0;
  double abs_r = 0.0;
  int nbad = 0;
#pragma unroll
  for (int k = 0; k < G::kPPT; ++k) {
    const int pt = int(threadIdx.x) + k * NT;
    if (pt >= G::kPts) break;
    const int e = pt / TP, pc2 = pt % TP;
    LdsCol<T, TP, 8> A{lds, pc2};
    cx<T> h[6];
#pragma unroll
    for (int g = 0; g < 6; ++g) {
      A.base = lds + g * G::kField;
      h[g] = A.load(e);
    }
    // sum of the squared entries other than h22 and -(h00 + h11), in the field's type
    T sx = h[0].x * h[0].x, sy = h[0].y * h[0].y;
    sx += h[1].x * h[1].x;
    sy += h[1].y * h[1].y;
#pragma unroll
    for (int g = 2; g < 5; ++g) {
      sx += T(2) * h[g].x * h[g].x;
      sy += T(2) * h[g].y * h[g].y;
    }
    const double ux = relax_point(pc, double(up[k].x), double(spv[k].x), double(h[5].x), double(sx),
                                  double(-h[0].x - h[1].x), abs_r, nbad);
    const double uy = relax_point(pc, double(up[k].y), double(spv[k].y), double(h[5].y), double(sy),
                                  double(-h[0].y - h[1].y), abs_r, nbad);
    const cx<T> o = mk(T(ux), T(uy));
    *reinterpret_cast<cx<T>*>(uout + (size_t)e * NN + 2 * pc2) = o;
    A.base = lds;
    A.store(e, o);
  }
  abs_r = wave_sum<64, NT>(abs_r);
  nbad = wave_sum<64, NT>(nbad);
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = abs_r;
    redi[threadIdx.x >> 6] = nbad;
  }
  lds_barrier();
  if (f == 0) {   // forward axis-0 transform of u^(n+1)
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = L.load(t + q * TT);
    fft<T, N, P, -1>(v, twl, L, t);
    wave_sync();
#pragma unroll
    for (int q = 0; q < R; ++q) L.store(t + q * TT, v[q]);
  }
  lds_barrier();
  cx<T>* dst = spec_u + col0;
  for (int idx = threadIdx.x; idx < H * TP; idx += NT) {
    const int k = idx / TP, p = idx % TP;
    const LdsCol<T, TP, 8> Z{lds, p};
    const cx<T> zk = Z.load(k), zn = Z.load((N - k) & (N - 1));
    dst[(size_t)k * NN + 2 * p] = mk(T(0.5) * (zk.x + zn.x), T(0.5) * (zk.y - zn.y));
    dst[(size_t)k * NN + 2 * p + 1] = mk(T(0.5) * (zk.y + zn.y), T(0.5) * (zn.x - zk.x));
  }
  if (threadIdx.x == 0) {
    double sr = 0.0;
    int sb = 0;
    for (int i = 0; i < G::kWaves; ++i) {
      sr += red[i];
      sb += redi[i];
    }
    const size_t g = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    const size_t groups = (size_t)gridDim.x * gridDim.y;
    partial[((size_t)b * groups + g) * 2] = sr;
    partial[((size_t)b * groups + g) * 2 + 1] = double(sb);
  }
}

// Convergence control: one workgroup of NT threads per batch element (pass_sums).  Latency bound: an
// element per workgroup, with no more threads than up to 512 partial sums need (5 x 64^3 float32
// passes, one workgroup walking the batch: 10.6 us, now 4.3 us; one 32^3 element 4.3 -> 3.7 us).
template <int NT>
__global__ void __launch_bounds__(NT)
k_finalize(const double* __restrict__ partial, int groups, SolveCtl* __restrict__ ctl, SolveHist* __restrict__ hist,
           SolveCfg cfg) {
  const int b = blockIdx.x;
  if (ctl[b].done) return;
  double sr, sb;
  pass_sums<NT>(partial + (size_t)b * groups * 2, groups, sr, sb);
  if (threadIdx.x == 0) ctl_decide(ctl[b], hist[b], sr, sb, cfg);
}

// Per-batch sums of |x| and of x per workgroup, the first level of a deterministic two-level reduction.
// A plain read: eight independent loads per thread are in flight (the mean of 256^3 counts: deposit 444 -> 433 us).
template <typename T>
__global__ void __launch_bounds__(256)
k_absmean_partial(const T* __restrict__ x, size_t n3, double* __restrict__ part) {
  const int b = blockIdx.y;
  const T* xb = x + (size_t)b * n3;
  constexpr int U = 8;
  const size_t step = (size_t)gridDim.x * 256;
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  double sa = 0.0, sm = 0.0;
  for (; i + (U - 1) * step < n3; i += U * step) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = xb[i + u * step];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sa += fabs(double(v[u]));
      sm += double(v[u]);
    }
  }
  for (; i < n3; i += step) {
    sa += fabs(double(xb[i]));
    sm += double(xb[i]);
  }
  sa = wave_sum<64, 256>(sa);
  sm = wave_sum<64, 256>(sm);
  __shared__ double ra[4], rm[4];
  if ((threadIdx.x & 63) == 0) {
    ra[threadIdx.x >> 6] = sa;
    rm[threadIdx.x >> 6] = sm;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[((size_t)b * gridDim.x + blockIdx.x) * 2] = ((ra[0] + ra[1]) + ra[2]) + ra[3];
    part[((size_t)b * gridDim.x + blockIdx.x) * 2 + 1] = ((rm[0] + rm[1]) + rm[2]) + rm[3];
  }
}

__global__ void __launch_bounds__(256)
k_absmean_final(const double* __restrict__ part, int groups, size_t n3, double* __restrict__ abs_mean,
                double* __restrict__ mean) {
  const int b = blockIdx.x;
  __shared__ double ra[256], rm[256];
  double sa = 0.0, sm = 0.0;
  for (int g = threadIdx.x; g < groups; g += 256) {
    sa += part[((size_t)b * groups + g) * 2];
    sm += part[((size_t)b * groups + g) * 2 + 1];
  }
  ra[threadIdx.x] = sa;
  rm[threadIdx.x] = sm;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      ra[threadIdx.x] += ra[threadIdx.x + s];
      rm[threadIdx.x] += rm[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (abs_mean) abs_mean[b] = ra[0] / double(n3);
    if (mean) mean[b] = rm[0] / double(n3);
  }
}

// ------------------------------------------------------------------ launchers
// (ev0, ev1: optional timing events recorded by the dispatch itself, at the kernel's start and
// end, without separate marker packets in the stream)
template <typename T, int N>
static void relax_n(const cx<T>* spec6, T* ubuf, const T* sfield, cx<T>* spec_u, double* partial,
                    const double* mean_u, int batch, const SolveCfg& cfg, const SolveCtl* ctl, hipStream_t s,
                    hipEvent_t ev0, hipEvent_t ev1) {
  constexpr size_t fstride = (size_t)(N / 2 + 1) * N * N;
  if constexpr (N <= kRelaxSmallMax) {
    using G = RelaxSGeo<T, N>;
    dim3 grid(N / (2 * G::kTP), N, batch);
    hipExtLaunchKernelGGL((k_relax_small<T, N>), grid, dim3(G::kThreads), 0, s, ev0, ev1, 0, spec6, fstride * batch,
                          ubuf, sfield, spec_u, partial, mean_u, cfg, ctl, twiddles<T>(N));
  } else if constexpr (sizeof(T) == 8) {
    using W = RelaxWGeo<T, N>;
    dim3 grid(N / (2 * W::kTP), N, batch);
    hipExtLaunchKernelGGL((k_relax_w<T, N>), grid, dim3(W::kThreads), 0, s, ev0, ev1, 0, spec6, fstride * batch,
                          ubuf, sfield, spec_u, partial, mean_u, cfg, ctl, twiddles<T>(N));
  } else {
    using G = typename RelaxGeo<T, N>::G;
    dim3 grid(N / (2 * G::kTP), N, batch);
    hipExtLaunchKernelGGL((k_relax<T, N>), grid, dim3(G::kThreads), 0, s, ev0, ev1, 0, spec6, fstride * batch,
                          ubuf, sfield, spec_u, partial, mean_u, cfg, ctl, twiddles<T>(N));
  }
}

template <typename T>
void launch_relax(int n, const cx<T>* spec6, T* ubuf, const T* sfield, cx<T>* spec_u, double* partial,
                  const double* mean_u, int batch, const SolveCfg& cfg, const SolveCtl* ctl, hipStream_t s,
                  hipEvent_t ev0, hipEvent_t ev1) {
#define C(NN) relax_n<T, NN>(spec6, ubuf, sfield, spec_u, partial, mean_u, batch, cfg, ctl, s, ev0, ev1)
  switch (n) {
    case 8: C(8); break;
    case 16: C(16); break;
    case 32: C(32); break;
    case 64: C(64); break;
    case 128: C(128); break;
    case 256: C(256); break;
    case 512: C(512); break;
    default: break;
  }
#undef C
}

// column pairs per workgroup of the relaxation kernel that launches for (T, N)
template <typename T, int N>
static constexpr int relax_tp() {
  if constexpr (N <= kRelaxSmallMax) return RelaxSGeo<T, N>::kTP;
  else if constexpr (sizeof(T) == 8) return RelaxWGeo<T, N>::kTP;
  else return RelaxGeo<T, N>::G::kTP;
}

// pass_sums adds in one order in both deciders of a pass on the meshes of the plane kernels: its partial
// sums take at most a lane each in the plane launch (N^2 / R threads) and in k_finalize (at most 512)
template <typename T, int N>
static constexpr bool one_partial_per_lane() {
  constexpr int groups = N / (2 * relax_tp<T, N>()) * N;
  return N > kPlaneMax || (groups <= N * N / Plan8<N>::R && groups <= 512);
}
static_assert(one_partial_per_lane<double, 8>() && one_partial_per_lane<double, 16>() && one_partial_per_lane<double, 32>() &&
              one_partial_per_lane<double, 64>() && one_partial_per_lane<float, 8>() && one_partial_per_lane<float, 16>() &&
              one_partial_per_lane<float, 32>() && one_partial_per_lane<float, 64>(), "the sums of a pass must not depend on the decider");

int relax_groups(int n, int elem_bytes) {
  int tp = 0;
#define C(NN)                                                                       \
  case NN:                                                                          \
    tp = (elem_bytes == 8) ? relax_tp<double, NN>() : relax_tp<float, NN>();       \
    break;
  switch (n) { C(8) C(16) C(32) C(64) C(128) C(256) C(512) default: return 0; }
#undef C
  return (n / (2 * tp)) * n;
}

void launch_finalize(const double* partial, int groups, SolveCtl* ctl, SolveHist* hist, const SolveCfg& cfg,
                     hipStream_t s) {
  if (groups <= 256) hipLaunchKernelGGL(k_finalize<256>, dim3(cfg.batch), dim3(256), 0, s, partial, groups, ctl, hist, cfg);
  else if (groups <= 512) hipLaunchKernelGGL(k_finalize<512>, dim3(cfg.batch), dim3(512), 0, s, partial, groups, ctl, hist, cfg);
  else hipLaunchKernelGGL(k_finalize<1024>, dim3(cfg.batch), dim3(1024), 0, s, partial, groups, ctl, hist, cfg);
}

// (by one wavefront)
__device__ __forceinline__ void reset_history(SolveHist& H) {
  for (int i = threadIdx.x; i < kMaxHist; i += 64) {
    H.resid[i] = -1.0;
    H.bad[i] = -1.0;
  }
}

__device__ void ctl_reset(SolveCtl& C) {
  C.done = 0;
  C.status = 0;
  C.iters = 0;
  C.cur = 0;
  C.out = 1;
  C.best = 2;
  C.result = 0;
  C.bad_seen = 0;
  C.passes = 0;
  C.last_bad = 0;
  C.final_bad = -1;
  C.resid = 0.0;
  C.resid_min = __builtin_huge_val();
  C.bad_frac = 0.0;
  C.mean_u = 0.0;
}

// a non-finite eps means a non-finite delta (or position): the element is decided at once as invalid
__device__ __forceinline__ void mark_invalid_input(SolveCtl& C) {
  if (!isfinite(C.eps)) {
    C.done = 1;
    C.status = kStatusInvalid;
  }
}

// eps of one element: sum of the |S| partial sums over n3, by a whole workgroup of NT threads (every
// thread returns it; fixed order)
template <int NT>
__device__ __forceinline__ double eps_of(const double* __restrict__ part, int groups, size_t n3) {
  __shared__ double w[NT / 64];
  double s = 0.0;
  for (int g = threadIdx.x; g < groups; g += NT) s += part[g];
  s = wave_sum<64, NT>(s);
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
  __syncthreads();
  s = w[0];
  for (int i = 1; i < NT / 64; ++i) s += w[i];
  return s / double(n3);
}

__global__ void __launch_bounds__(1024)
k_ctl_init(SolveCtl* __restrict__ ctl, SolveHist* __restrict__ hist, const double* __restrict__ part, int groups,
           size_t n3) {
  const int b = blockIdx.x;
  const double eps = eps_of<1024>(part + (size_t)b * groups, groups, n3);
  SolveCtl& C = ctl[b];
  if (threadIdx.x < 64) reset_history(hist[b]);
  if (threadIdx.x != 0) return;
  ctl_reset(C);
  C.eps = eps;
  C.iters1 = 0;
  C.passes1 = 0;
  C.phase1_done = 1;
  mark_invalid_input(C);
}

// -1: the float32 phase met its tolerance on the initial guess itself, whose float64 form
// already sits in the float64 phase's first buffer
__device__ __forceinline__ int handoff_buffer(const SolveCtl& C) {
  if (!C.done) return C.cur;
  if (C.status == 0 && C.iters == 0) return -1;
  return (C.status == 0 && C.final_bad == 0) ? C.out : C.result;
}

// log2 of the row group of a solve's own fields (RealRows) at mesh size 2^logn
template <typename T>
__host__ __device__ constexpr int own_group(int logn) {
  return sizeof(T) == 8 && (1 << logn) >= kRowGroupMin ? __builtin_ctz(kRowGroup) : logn;
}
// where the element i (C order) of such a field lies, for row groups of 2^lg
__device__ __forceinline__ size_t own_index(size_t i, int logn, int lg) {
  if (lg == logn) return i;
  const size_t n1 = (size_t(1) << logn) - 1, i2 = i & n1, i1 = (i >> logn) & n1, i0 = i >> (2 * logn);
  return (((((i1 >> lg) << logn) + i0) << lg) + (i1 & ((size_t(1) << lg) - 1))) << logn | i2;
}

// copies a field of the caller's into the solve's own row order
__global__ void __launch_bounds__(256)
k_take_field(const double* __restrict__ in, double* __restrict__ out, int logn) {
  const size_t n3 = size_t(1) << (3 * logn), b = (size_t)blockIdx.y * n3;
  const int lg = own_group<double>(logn);
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256)
    out[b + own_index(i, logn, lg)] = in[b + i];
}

// copies the selected buffer; with part != nullptr it also leaves per-workgroup sums of |x|
// and x (the layout k_absmean_final reads)
template <typename T>
__global__ void __launch_bounds__(256)
k_take_buffer(const SolveCtl* __restrict__ ctl, const T* __restrict__ U, int batch, int logn, double* __restrict__ dst,
              int handoff, double* __restrict__ part) {
  const size_t n3 = size_t(1) << (3 * logn);
  const int sg = own_group<T>(logn), dg = handoff ? own_group<double>(logn) : logn;
  const int b = blockIdx.y;
  const int src = handoff ? handoff_buffer(ctl[b]) : ctl[b].result;
  if (src < 0) return;   // (handoff only: no reduction is requested there)
  const T* in = U + ((size_t)src * batch + b) * n3;
  double* out = dst + (size_t)b * n3;
  double sa = 0.0, sm = 0.0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256) {
    const double v = double(in[own_index(i, logn, sg)]);
    out[own_index(i, logn, dg)] = v;
    sa += fabs(v);
    sm += v;
  }
  if (!part) return;
  sa = wave_sum<64, 256>(sa);
  sm = wave_sum<64, 256>(sm);
  __shared__ double ra[4], rm[4];
  if ((threadIdx.x & 63) == 0) {
    ra[threadIdx.x >> 6] = sa;
    rm[threadIdx.x >> 6] = sm;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[((size_t)b * gridDim.x + blockIdx.x) * 2] = ((ra[0] + ra[1]) + ra[2]) + ra[3];
    part[((size_t)b * gridDim.x + blockIdx.x) * 2 + 1] = ((rm[0] + rm[1]) + rm[2]) + rm[3];
  }
}

// keeps eps (the float64 source's) and records the float32 phase's counts
__global__ void __launch_bounds__(64) k_ctl_phase2(SolveCtl* __restrict__ ctl, SolveHist* __restrict__ hist) {
  SolveCtl& C = ctl[blockIdx.x];
  reset_history(hist[blockIdx.x]);
  if (threadIdx.x != 0) return;
  const int src = handoff_buffer(C);
  const bool invalid = C.status == kStatusInvalid;
  C.iters1 = C.iters + ((C.done && src == C.out) ? 1 : 0);
  C.passes1 = C.passes;
  C.phase1_done = C.done;
  ctl_reset(C);
  if (invalid) {
    C.done = 1;
    C.status = kStatusInvalid;
  }
}

static int absmean_groups(size_t n3) {
  size_t g = (n3 + 255) / 256;
  return int(g > 1024 ? 1024 : g);
}

static unsigned copy_groups(size_t n3) {
  const size_t g = (n3 + 255) / 256;
  return unsigned(g > 4096 ? 4096 : g);
}

void launch_handoff(SolveCtl* ctl, SolveHist* hist, const float* U32, int batch, int n, double* dst, hipStream_t s) {
  hipLaunchKernelGGL((k_take_buffer<float>), dim3(copy_groups((size_t)n * n * n), batch), dim3(256), 0, s, ctl, U32,
                     batch, __builtin_ctz(n), dst, 1, nullptr);
  hipLaunchKernelGGL(k_ctl_phase2, dim3(batch), dim3(64), 0, s, ctl, hist);
}

void launch_take_field(int n, const double* in, double* out, int batch, hipStream_t s) {
  hipLaunchKernelGGL(k_take_field, dim3(copy_groups((size_t)n * n * n), batch), dim3(256), 0, s, in, out,
                     __builtin_ctz(n));
}

// ------------------------------------------------------------------ spherical approximation
__global__ void __launch_bounds__(256)
k_spherical(size_t n3, const double* __restrict__ S, double* __restrict__ u, double alpha, double lam,
            double* __restrict__ partial) {
  const int b = blockIdx.y;
  const double c4 = 4.0 * (1.0 - 1.0 / 3.0) * lam;
  const double vertex = -alpha / (2.0 * (1.0 - 1.0 / 3.0) * lam);
  const double* sb = S + (size_t)b * n3;
  double* ub = u + (size_t)b * n3;
  int nbad = 0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256) {
    const double bp = sb[i];   // B' = S at u = 0 (Hessian and nonlocal terms vanish)
    const double disc = alpha * alpha + c4 * bp;
    if (disc < 0.0) {
      ub[i] = vertex;
      ++nbad;
    } else {
      ub[i] = 2.0 * bp / (alpha + sqrt(disc));
    }
  }
  nbad = wave_sum<64, 256>(nbad);
  __shared__ int rb[4];
  if ((threadIdx.x & 63) == 0) rb[threadIdx.x >> 6] = nbad;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[(size_t)b * gridDim.x + blockIdx.x] = double(((rb[0] + rb[1]) + rb[2]) + rb[3]);
}

__global__ void __launch_bounds__(256)
k_ctl_spherical(SolveCtl* __restrict__ ctl, SolveHist* __restrict__ hist, const double* __restrict__ eps_part,
                int eps_groups, const double* __restrict__ partial, int groups, size_t n3) {
  const int b = blockIdx.x;
  const double eps = eps_of<256>(eps_part + (size_t)b * eps_groups, eps_groups, n3);
  if (threadIdx.x < 64) reset_history(hist[b]);
  double nb = 0.0;
  for (int g = threadIdx.x; g < groups; g += 256) nb += partial[(size_t)b * groups + g];
  nb = wave_sum<64, 256>(nb);
  __shared__ double rb[4];
  if ((threadIdx.x & 63) == 0) rb[threadIdx.x >> 6] = nb;
  __syncthreads();
  if (threadIdx.x != 0) return;
  SolveCtl& C = ctl[b];
  ctl_reset(C);
  C.eps = eps;
  C.iters1 = 0;
  C.passes1 = 0;
  C.phase1_done = 1;
  C.done = 1;
  C.status = 0;
  C.iters = 1;
  C.result = 0;
  C.resid = -1.0;       // not evaluated: the approximation is not a root of Eq. FullDGP2
  C.resid_min = -1.0;
  C.bad_frac = (((rb[0] + rb[1]) + rb[2]) + rb[3]) / double(n3);
  hist[b].bad[0] = C.bad_frac;
  mark_invalid_input(C);
}

int spherical_groups(size_t n3) { return int(std::min<size_t>(4096, (n3 + 255) / 256)); }

void launch_spherical(size_t n3, int batch, const double* S, double* u, double alpha, double lam, double* partial,
                      SolveCtl* ctl, SolveHist* hist, const double* eps_part, int eps_groups, hipStream_t s) {
  const int g = spherical_groups(n3);
  hipLaunchKernelGGL(k_spherical, dim3(g, batch), dim3(256), 0, s, n3, S, u, alpha, lam, partial);
  hipLaunchKernelGGL(k_ctl_spherical, dim3(batch), dim3(256), 0, s, ctl, hist, eps_part, eps_groups, partial, g, n3);
}

template <typename T>
void launch_take_result(const SolveCtl* ctl, const T* U, int batch, int n, double* dst, double* scratch,
                        double* mean, hipStream_t s) {
  const size_t n3 = (size_t)n * n * n;
  const int g = absmean_groups(n3);
  hipLaunchKernelGGL((k_take_buffer<T>), dim3(g, batch), dim3(256), 0, s, ctl, U, batch, __builtin_ctz(n), dst, 0,
                     scratch);
  hipLaunchKernelGGL(k_absmean_final, dim3(batch), dim3(256), 0, s, scratch, g, n3, nullptr, mean);
}

template void launch_take_result<double>(const SolveCtl*, const double*, int, int, double*, double*, double*,
                                         hipStream_t);
template void launch_take_result<float>(const SolveCtl*, const float*, int, int, double*, double*, double*,
                                        hipStream_t);

void launch_ctl_init(SolveCtl* ctl, SolveHist* hist, const double* part, int groups, size_t n3, int batch,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_ctl_init, dim3(batch), dim3(1024), 0, s, ctl, hist, part, groups, n3);
}


size_t absmean_scratch_doubles(size_t n3, int batch) { return (size_t)absmean_groups(n3) * batch * 2; }

template <typename T>
void launch_absmean(size_t n3, const T* x, int batch, double* scratch, double* abs_mean, double* mean,
                    hipStream_t s) {
  const int g = absmean_groups(n3);
  hipLaunchKernelGGL((k_absmean_partial<T>), dim3(g, batch), dim3(256), 0, s, x, n3, scratch);
  hipLaunchKernelGGL(k_absmean_final, dim3(batch), dim3(256), 0, s, scratch, g, n3, abs_mean, mean);
}

void launch_pair_means(const double* part, int groups, size_t n3, int batch, double* out0, double* out1,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_absmean_final, dim3(batch), dim3(256), 0, s, part, groups, n3, out0, out1);
}

template void launch_relax<double>(int, const cx<double>*, double*, const double*, cx<double>*, double*,
                                   const double*, int, const SolveCfg&, const SolveCtl*, hipStream_t, hipEvent_t,
                                   hipEvent_t);
template void launch_relax<float>(int, const cx<float>*, float*, const float*, cx<float>*, double*,
                                  const double*, int, const SolveCfg&, const SolveCtl*, hipStream_t, hipEvent_t,
                                  hipEvent_t);
template void launch_absmean<long long>(size_t, const long long*, int, double*, double*, double*, hipStream_t);

}  // namespace dgp
