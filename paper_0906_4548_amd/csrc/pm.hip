// Particle-mesh kernels: deterministic CIC deposit, density contrast, CIC
// interpolation fused with the leapfrog kick-drift, and the CIC adjoint.
//
// CIC (Sec. III A, Eq. CIC): tent window W(x) = 1 - |x|/h per axis, 3D weight the
// product of the three; the same weights interpolate the force back (no
// self-force).  Mesh node j sits at x = j h.  The deposit is made bit-exact and
// order independent: per-axis weights (1 - f, f) in FP64 with no fused
// multiply-add, the 3D weight as (w_x w_y) w_z, quantised to Q = rint(W 2^40)
// and summed with 64-bit integer atomics.
#include <mutex>

#include "dgp_internal.h"

namespace dgp {

constexpr double kQScale = 1099511627776.0;  // 2^40

struct Cic {
  int i0[3], i1[3];
  double w0[3], w1[3];
};

// Integers out of float64 by adding a power of two that puts the unit in the last mantissa bit: the
// sum rounds to nearest even and its low bits are the integer.  (There is no float64 -> int64
// conversion instruction; the eight rint and conversion sequences of a particle were most of the
// deposit's vector instructions.)
// floor value fl modulo a power of two n <= 2^9; the conversion remains for |fl| >= 2^51
__device__ __forceinline__ int wrap_cell(double fl, int n) {
#pragma clang fp contract(off)
  long long b = __double_as_longlong(fl + 0x1.8p52);
  if (!(fabs(fl) < 0x1p51)) b = (long long)fl;
  return int(b) & (n - 1);
}
// rint(w 2^40) of a weight in [0, 1]
__device__ __forceinline__ unsigned long long quantise(double w) {
  return (unsigned long long)__double_as_longlong(fma(w, kQScale, 0x1p52)) & 0xfffffffffffffull;
}

// cell and weights of a particle at x (already in mesh units: x = pos * N / L)
__device__ __forceinline__ Cic cic_at(const double (&s3)[3], int n) {
#pragma clang fp contract(off)
  Cic c;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double s = s3[d];
    const double fl = floor(s);
    const double f = s - fl;
    const int i = wrap_cell(fl, n);   // periodic wrap (n is a power of two)
    c.i0[d] = i;
    c.i1[d] = (i + 1) & (n - 1);
    c.w0[d] = 1.0 - f;
    c.w1[d] = f;
  }
  return c;
}

template <typename P>
__device__ __forceinline__ Cic cic_of(const P* __restrict__ pos, long long np, long long p, int n, double scale) {
#pragma clang fp contract(off)
  double s3[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) s3[d] = double(pos[(size_t)d * np + p]) * scale;
  return cic_at(s3, n);
}

// Binned deposit.  A workgroup takes a chunk of consecutive particles, finds the
// periodic bounding box of their CIC cells and, when the box fits the LDS histogram,
// sums the chunk's quantised weights there with LDS atomics and then adds each
// non-zero box cell to the mesh with one global atomic.  Integer sums make the result
// identical to the direct deposit in any order; the gain needs spatially coherent
// chunks (particles stored in compact Lagrangian blocks).  A chunk whose box is too
// large takes the direct per-particle atomics.  Larger chunks mean fewer global atomics per
// particle (a box's surface grows slower than its volume) but more registers and LDS: the
// geometry is chosen by mesh size, from the measured deposit times of the Zel'dovich loads
// (256^3 float64 particles: 512 / 1024 / 2048 particles per chunk 357 / 299 / 322 us; 512^3
// float32 particles: 2.84 / 2.84 / 2.45 ms).  Each particle's cell and weights are computed again
// after the box instead of being held across its barriers (1024-particle chunks: 138 -> 58-68 VGPRs,
// occupancy 3 -> 4 waves per SIMD; the tile counts of 15.0M float32 particles in lattice order 118 ->
// 97 us), and the 2048-particle chunk sizes its histogram at three cells per particle (both: occupancy
// 2 -> 3, 512^3 2.43 -> 2.12 ms).  Three cells for the 1024-particle chunk make its counts faster still (81
// us) but send boxes of blocked loads to the direct path (256^3 step's deposit 231 -> 241 us).
template <int CH>
struct DepGeo {
  static constexpr int kChunk = CH;                         // particles per workgroup
  static constexpr int kPPT = CH / 256;                     // particles per thread
  static constexpr int kCap = (CH >= 2048 ? 3 : 4) * CH;    // cells of the LDS histogram (8 bytes each)
  static_assert(CH % 256 == 0, "chunk must be a multiple of the workgroup size");
};

// offset of cell i from the reference cell r on a periodic axis of n cells, in [-n/2, n/2)
__device__ __forceinline__ int periodic_offset(int i, int r, int n) {
  int o = i - r;
  if (o < -n / 2) o += n;
  if (o >= n / 2) o -= n;
  return o;
}

// Periodic bounding box of a chunk's CIC base cells, relative to the base cell cr of its
// first particle: offsets in [-n/2, n/2) per axis, box lo[d] .. lo[d] + ext[d] - 1 (the
// +1 corners included).  xs holds the positions of the thread's particles (p0 + threadIdx.x
// + 256 k), loaded by the caller.  Returns true when the box volume is at most `cap`.
// Every thread of the (256-thread) workgroup must call it.
template <int PPT, typename P>
__device__ __forceinline__ bool chunk_box(const P* __restrict__ pos, const P (&xs)[PPT][3], long long np, int n,
                                          double scale, long long p0, int cap, Cic& cr,
                                          int (&off)[PPT][3], int (&bx)[6]) {
  __shared__ int wlo[4][3], whi[4][3];
  __shared__ int sbox[7];
  cr = cic_of(pos, np, p0, n, scale);
  int lo[3] = {n, n, n}, hi[3] = {-n, -n, -n};
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const long long p = p0 + threadIdx.x + k * 256;
    if (p < np) {
      const double s3[3] = {double(xs[k][0]) * scale, double(xs[k][1]) * scale, double(xs[k][2]) * scale};
      const Cic c = cic_at(s3, n);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        off[k][d] = periodic_offset(c.i0[d], cr.i0[d], n);
        lo[d] = min(lo[d], off[k][d]);
        hi[d] = max(hi[d], off[k][d] + 1);
      }
    }
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo[d] = min(lo[d], __shfl_xor(lo[d], o, 64));
      hi[d] = max(hi[d], __shfl_xor(hi[d], o, 64));
    }
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      wlo[threadIdx.x >> 6][d] = lo[d];
      whi[threadIdx.x >> 6][d] = hi[d];
    }
  }
  lds_barrier();
  if (threadIdx.x == 0) {
    long long vol = 1;
    for (int d = 0; d < 3; ++d) {
      int l = wlo[0][d], h = whi[0][d];
      for (int w = 1; w < 4; ++w) {
        l = min(l, wlo[w][d]);
        h = max(h, whi[w][d]);
      }
      sbox[d] = l;
      sbox[3 + d] = h - l + 1;
      vol *= h - l + 1;
    }
    sbox[6] = vol <= cap ? 1 : 0;
  }
  lds_barrier();
#pragma unroll
  for (int d = 0; d < 6; ++d) bx[d] = sbox[d];
  return sbox[6] != 0;
}

// the positions of the thread's particles in a chunk (unused slots past np left at 0); streaming
// loads unless STREAM is false: a kernel reads each particle once
template <int PPT, bool STREAM = true, typename P>
__device__ __forceinline__ void load_chunk(const P* __restrict__ a, long long np, long long p0, P (&xs)[PPT][3]) {
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const long long p = p0 + threadIdx.x + k * 256;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const P* const x = &a[(size_t)d * np + p];
      if constexpr (STREAM) xs[k][d] = p < np ? __builtin_nontemporal_load(x) : P(0);
      else xs[k][d] = p < np ? *x : P(0);
    }
  }
}

// raise *bad when one of the thread's particles has a non-finite coordinate (the cell index of
// such a particle is still reduced into the mesh, so no access leaves it; the caller reports it)
template <int PPT, typename P>
__device__ __forceinline__ void flag_nonfinite(const P (&xs)[PPT][3], int* __restrict__ bad) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < PPT; ++k)
#pragma unroll
    for (int d = 0; d < 3; ++d) ok = ok && isfinite(double(xs[k][d]));
  if (!ok) atomicOr(bad, 1);
}

// mesh index of box cell i (row-major over the box extents), wrapped onto the periodic mesh
__device__ __forceinline__ size_t box_cell(int i, const Cic& cr, const int (&bx)[6], int n) {
  const int plane = bx[4] * bx[5];
  const int x = i / plane, r = i - x * plane;
  const int y = r / bx[5], z = r - y * bx[5];
  const size_t gx = (size_t)((cr.i0[0] + bx[0] + x) & (n - 1));   // periodic wrap (n is a power of two)
  const size_t gy = (size_t)((cr.i0[1] + bx[1] + y) & (n - 1));
  const size_t gz = (size_t)((cr.i0[2] + bx[2] + z) & (n - 1));
  return (gx * n + gy) * n + gz;
}

// Tile sort for chunks that are not compact (lattice-order loads: a chunk of 1024 spans the whole
// axis 2, so its box does not fit and every particle takes 8 global atomics, ~80 G/s: 15.0M float32
// particles in rows of 248 on 256^3, 1350 us).  Their particles are counted per tile of 8 x 8 x 64 cells
// (by the deposit kernel itself, which deposits the compact chunks as before), a prefix sum gives
// each tile its segment, k_tile_scatter copies the positions there, and k_tile_deposit sums a
// tile's particles in an LDS histogram of its 9 x 9 x 65 cells: the tile's own cells go to the mesh,
// the upper layer (cells of the next tiles) to a halo buffer that k_tile_halo adds, so neither needs
// atomics (boundary cells of 16^3 tiles added with global atomics: 223 us for k_tile_deposit where
// the rest of it takes 54 us).  Tiles are long in axis 2 for the mesh lines of the lower z layer,
// which the halo pass touches for one value each (16^3 tiles: 54 us, now 37 us), and for longer
// runs in the scatter.  A tile of several work items adds them with atomics.  The order inside a
// segment varies between runs; the integer sums do not.
constexpr int kTL[3] = {3, 3, 6};   // log2 of the tile's cells per axis
constexpr int kTX = 1 << kTL[0], kTY = 1 << kTL[1], kTZ = 1 << kTL[2];
constexpr int kTileCells = (kTX + 1) * (kTY + 1) * (kTZ + 1);
constexpr int kTileBoxCap = 4096;     // tiles of a chunk's bounding box (counters in LDS)
constexpr int kTileItem = 8192;       // particles per workgroup of k_tile_deposit
constexpr int kTileState = 4;         // words of TileSort::state
constexpr int kTileHalo = kTileCells - kTX * kTY * kTZ;
// device pointers into the caller's scratch
struct TileSort {
  unsigned* count;          // [tiles] particles per tile, then (after the scan) the scatter's cursors
  unsigned char* sorted;    // [chunks] 1: the chunk's particles go through the tiles
  uint4* items;             // (tile, first, count, single) per workgroup of k_tile_deposit
  unsigned* state;          // [0]: items, [1]: 1 when some chunk was deposited directly, [2]: 1 when some was sorted
  unsigned char* multi;     // [tiles] 1: the tile has several work items (or none: its halo is zeroed)
  unsigned long long* halo; // [tiles][kTileHalo] sums of a tile's upper layer
  void* pos;                // [3][np] positions by tile
};

// slot of cell (x, y, z) of a tile's upper layer in its halo: the face x = kTX, the rest of the face
// y = kTY, the rest of the face z = kTZ
__device__ __forceinline__ int halo_slot(int x, int y, int z) {
  if (x == kTX) return y * (kTZ + 1) + z;
  if (y == kTY) return (kTY + 1 + x) * (kTZ + 1) + z;
  return (kTY + 1 + kTX) * (kTZ + 1) + x * kTY + y;
}
// tile (x, y, z), wrapped, of an n^3 mesh and back
__device__ __forceinline__ int tile_index(int x, int y, int z, int n) {
  const int nx = n >> kTL[0], ny = n >> kTL[1], nz = n >> kTL[2];
  return ((x & (nx - 1)) * ny + (y & (ny - 1))) * nz + (z & (nz - 1));
}
__device__ __forceinline__ void tile_coords(int t, int n, int& x, int& y, int& z) {
  const int ny = n >> kTL[1], nz = n >> kTL[2];
  z = t % nz;
  y = (t / nz) % ny;
  x = t / (nz * ny);
}
static __host__ __device__ int tile_count(int n) { return (n >> kTL[0]) * (n >> kTL[1]) * (n >> kTL[2]); }

// the tiles of a chunk's bounding box: first tile (unwrapped) and extent per axis, at most the mesh's own
// (a chunk over the whole mesh that starts inside a tile meets that tile again at the other end: counted
// twice, the 4096 tiles of 256^3 came to 33 x 33 x 5 = 5445 and its chunks were not sorted)
__device__ __forceinline__ bool tile_box(const Cic& cr, const int (&bx)[6], int n, int (&t0)[3], int (&te)[3]) {
  int vol = 1;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    t0[d] = (cr.i0[d] + bx[d]) >> kTL[d];
    te[d] = min(((cr.i0[d] + bx[d] + bx[3 + d] - 2) >> kTL[d]) - t0[d] + 1, n >> kTL[d]);   // base cells only
    vol *= te[d];
  }
  return vol <= kTileBoxCap;
}
__device__ __forceinline__ int local_tile(const Cic& cr, const int (&off)[3], const int (&t0)[3], const int (&te)[3]) {
  int l = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int x = ((cr.i0[d] + off[d]) >> kTL[d]) - t0[d];
    l = l * te[d] + (x < te[d] ? x : x - te[d]);   // past the extent only where that is the whole axis
  }
  return l;
}
__device__ __forceinline__ int global_tile(int l, const int (&t0)[3], const int (&te)[3], int n) {
  return tile_index(t0[0] + l / (te[2] * te[1]), t0[1] + (l / te[2]) % te[1], t0[2] + l % te[2], n);
}

template <typename P, int CH, bool SORT>
__global__ void __launch_bounds__(256)
k_deposit_bin(const P* __restrict__ pos, long long np, int n, double scale, unsigned long long* __restrict__ grid,
              int* __restrict__ bad, TileSort ts) {
#pragma clang fp contract(off)
  using G = DepGeo<CH>;
  constexpr int kDepPPT = G::kPPT;
  __shared__ unsigned long long hist[G::kCap];
  const long long p0 = xcd_chunk() * G::kChunk;
  P xs[kDepPPT][3];
  load_chunk<kDepPPT>(pos, np, p0, xs);
  flag_nonfinite<kDepPPT>(xs, bad);
  Cic cr;
  int off[kDepPPT][3], bx[6];
  const bool binned = chunk_box<kDepPPT>(pos, xs, np, n, scale, p0, G::kCap, cr, off, bx);
  const int vol = bx[3] * bx[4] * bx[5];
  if constexpr (SORT) {
    static_assert(kTileBoxCap * sizeof(unsigned) <= sizeof(hist), "tile counters alias the histogram");
    int t0[3], te[3];
    const bool sorted = !binned && tile_box(cr, bx, n, t0, te);
    if (threadIdx.x == 0) {
      ts.sorted[p0 / CH] = sorted ? 1 : 0;
      // (all compact chunks of a blocked load set one word: read before it is written)
      if (sorted) ts.state[2] = 1u;
      else if (ts.state[1] == 0u) ts.state[1] = 1u;
    }
    if (sorted) {
      unsigned* const cnt = reinterpret_cast<unsigned*>(hist);
      const int tv = te[0] * te[1] * te[2];
      for (int i = threadIdx.x; i < tv; i += 256) cnt[i] = 0u;
      lds_barrier();
#pragma unroll
      for (int k = 0; k < kDepPPT; ++k)
        if (p0 + threadIdx.x + k * 256 < np) atomicAdd(&cnt[local_tile(cr, off[k], t0, te)], 1u);
      lds_barrier();
      for (int i = threadIdx.x; i < tv; i += 256)
        if (cnt[i] != 0u) atomicAdd(&ts.count[global_tile(i, t0, te, n)], cnt[i]);
      return;
    }
  }
  if (binned)
    for (int i = threadIdx.x; i < vol; i += 256) hist[i] = 0ull;
  lds_barrier();
#pragma unroll
  for (int k = 0; k < kDepPPT; ++k) {
    const long long p = p0 + threadIdx.x + k * 256;
    if (p >= np) continue;
    // the cell and weights again from the position (the chunk box's arithmetic)
    const double s3[3] = {double(xs[k][0]) * scale, double(xs[k][1]) * scale, double(xs[k][2]) * scale};
    const Cic c = cic_at(s3, n);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double wx = a ? c.w1[0] : c.w0[0];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const double wxy = wx * (b ? c.w1[1] : c.w0[1]);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          const double wgt = wxy * (cc ? c.w1[2] : c.w0[2]);
          const unsigned long long q = quantise(wgt);
          if (binned) {
            const int li = ((off[k][0] + a - bx[0]) * bx[4] + (off[k][1] + b - bx[1])) * bx[5] + (off[k][2] + cc - bx[2]);
            atomicAdd(&hist[li], q);
          } else {
            const size_t ix = (size_t)(a ? c.i1[0] : c.i0[0]);
            const size_t iy = (size_t)(b ? c.i1[1] : c.i0[1]);
            const size_t iz = (size_t)(cc ? c.i1[2] : c.i0[2]);
            atomicAdd(&grid[(ix * n + iy) * n + iz], q);
          }
        }
      }
    }
  }
  if (!binned) return;
  lds_barrier();
  for (int i = threadIdx.x; i < vol; i += 256) {
    const unsigned long long v = hist[i];
    if (v != 0ull) atomicAdd(&grid[box_cell(i, cr, bx, n)], v);
  }
}

// Exclusive prefix sum of the tile counts into segment starts (left in count, as the scatter's
// cursors) and the work items of k_tile_deposit; one workgroup, each thread a run of tiles.
__global__ void __launch_bounds__(1024)
k_tile_scan(TileSort ts, int tiles) {
  if (ts.state[2] == 0u) return;   // no sorted chunk (the item count stays 0)
  const int per = (tiles + 1023) / 1024, lo = min(int(threadIdx.x) * per, tiles), hi = min(lo + per, tiles);
  unsigned np = 0, ni = 0;
  for (int i = lo; i < hi; ++i) {
    np += ts.count[i];
    ni += (ts.count[i] + kTileItem - 1) / kTileItem;
  }
  // inclusive scan over the wavefront, then over the 16 wavefronts
  unsigned sp = np, si = ni;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned a = __shfl_up(sp, o, 64), b = __shfl_up(si, o, 64);
    if (int(threadIdx.x & 63) >= o) {
      sp += a;
      si += b;
    }
  }
  __shared__ unsigned wp[16], wi[16];
  if ((threadIdx.x & 63) == 63) {
    wp[threadIdx.x >> 6] = sp;
    wi[threadIdx.x >> 6] = si;
  }
  __syncthreads();
  for (int w = 0; w < int(threadIdx.x >> 6); ++w) {
    sp += wp[w];
    si += wi[w];
  }
  if (threadIdx.x == 1023) ts.state[0] = si;
  sp -= np;
  si -= ni;
  for (int i = lo; i < hi; ++i) {
    const unsigned c = ts.count[i];
    ts.count[i] = sp;
    ts.multi[i] = c == 0u || c > unsigned(kTileItem) ? 1 : 0;
    for (unsigned f = 0; f < c; f += kTileItem)
      ts.items[si++] = make_uint4(unsigned(i), sp + f, min(c - f, unsigned(kTileItem)), c <= unsigned(kTileItem) ? 1u : 0u);
    sp += c;
  }
}

// copies the positions of the sorted chunks to their tiles' segments
template <typename P, int CH>
__global__ void __launch_bounds__(256)
k_tile_scatter(const P* __restrict__ pos, long long np, int n, double scale, TileSort ts) {
  constexpr int PPT = CH / 256;
  __shared__ unsigned cnt[kTileBoxCap];
  if (ts.state[2] == 0u) return;
  const int tiles = tile_count(n);
  for (int i = blockIdx.x; i < tiles; i += gridDim.x)   // halos that k_tile_deposit adds to, or does not write
    if (ts.multi[i] != 0)
      for (int j = threadIdx.x; j < kTileHalo; j += 256) ts.halo[(size_t)i * kTileHalo + j] = 0ull;
  const long long p0 = xcd_chunk() * CH;
  if (ts.sorted[p0 / CH] == 0) return;
  P xs[PPT][3];
  load_chunk<PPT>(pos, np, p0, xs);
  Cic cr;
  int off[PPT][3], bx[6], t0[3], te[3];
  (void)chunk_box<PPT>(pos, xs, np, n, scale, p0, 0, cr, off, bx);
  (void)tile_box(cr, bx, n, t0, te);   // fits: the counting pass sorted this chunk
  const int tv = te[0] * te[1] * te[2];
  for (int i = threadIdx.x; i < tv; i += 256) cnt[i] = 0u;
  lds_barrier();
  int lt[PPT];
  unsigned rank[PPT];
#pragma unroll
  for (int k = 0; k < PPT; ++k)
    if (p0 + threadIdx.x + k * 256 < np) {
      lt[k] = local_tile(cr, off[k], t0, te);
      rank[k] = atomicAdd(&cnt[lt[k]], 1u);
    }
  lds_barrier();
  for (int i = threadIdx.x; i < tv; i += 256)
    if (cnt[i] != 0u) cnt[i] = atomicAdd(&ts.count[global_tile(i, t0, te, n)], cnt[i]);
  lds_barrier();
  P* const out = static_cast<P*>(ts.pos);
#pragma unroll
  for (int k = 0; k < PPT; ++k)
    if (p0 + threadIdx.x + k * 256 < np) {
      const size_t at = cnt[lt[k]] + rank[k];
#pragma unroll
      for (int d = 0; d < 3; ++d) out[(size_t)d * np + at] = xs[k][d];
    }
}

// deposits one item: up to kTileItem particles of one tile
template <typename P>
__global__ void __launch_bounds__(512)
k_tile_deposit(long long np, int n, double scale, TileSort ts, unsigned long long* __restrict__ grid) {
#pragma clang fp contract(off)
  __shared__ unsigned long long hist[kTileCells];
  if (blockIdx.x >= ts.state[0]) return;
  const uint4 it = ts.items[blockIdx.x];
  for (int i = threadIdx.x; i < kTileCells; i += 512) hist[i] = 0ull;
  lds_barrier();
  const P* const pos = static_cast<const P*>(ts.pos);
  for (unsigned i = threadIdx.x; i < it.z; i += 512) {
    const Cic c = cic_of(pos, np, (long long)(it.y + i), n, scale);
    const int l0 = ((c.i0[0] & (kTX - 1)) * (kTY + 1) + (c.i0[1] & (kTY - 1))) * (kTZ + 1) + (c.i0[2] & (kTZ - 1));
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double wx = a ? c.w1[0] : c.w0[0];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const double wxy = wx * (b ? c.w1[1] : c.w0[1]);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          const double wgt = wxy * (cc ? c.w1[2] : c.w0[2]);
          const unsigned long long q = quantise(wgt);
          atomicAdd(&hist[l0 + (a * (kTY + 1) + b) * (kTZ + 1) + cc], q);
        }
      }
    }
  }
  lds_barrier();
  int tx, ty, tz;
  tile_coords(int(it.x), n, tx, ty, tz);
  const bool single = it.w != 0u, direct = ts.state[1] != 0u;
  unsigned long long* const halo = ts.halo + (size_t)it.x * kTileHalo;
  for (int i = threadIdx.x; i < kTileCells; i += 512) {
    const unsigned long long v = hist[i];
    const int z = i % (kTZ + 1), y = (i / (kTZ + 1)) % (kTY + 1), x = i / ((kTZ + 1) * (kTY + 1));
    if (x == kTX || y == kTY || z == kTZ) {
      unsigned long long* const h = halo + halo_slot(x, y, z);
      if (single) *h = v;
      else if (v != 0ull) atomicAdd(h, v);
    } else if (v != 0ull) {
      unsigned long long* const g = grid + ((size_t)(tx * kTX + x) * n + (size_t)(ty * kTY + y)) * n + (size_t)(tz * kTZ + z);
      if (!single) atomicAdd(g, v);
      else *g = direct ? *g + v : v;   // this workgroup is the cell's only writer; the mesh was zero
    }
  }
}

// adds the halos to the lower-layer cells (some coordinate 0) of every tile: the cell's halo values
// are those of the tiles one step back along the axes where its coordinate is 0
__global__ void __launch_bounds__(256)
k_tile_halo(int n, TileSort ts, unsigned long long* __restrict__ grid) {
  if (ts.state[2] == 0u) return;
  int tx, ty, tz;
  tile_coords(blockIdx.x, n, tx, ty, tz);
  constexpr int kFaceX = kTY * kTZ, kFaceY = (kTX - 1) * kTZ, kFaces = kFaceX + kFaceY + (kTX - 1) * (kTY - 1);
  for (int i = threadIdx.x; i < kFaces; i += 256) {
    int x, y, z;
    if (i < kFaceX) {
      x = 0; y = i / kTZ; z = i % kTZ;
    } else if (i < kFaceX + kFaceY) {
      const int j = i - kFaceX;
      x = 1 + j / kTZ; y = 0; z = j % kTZ;
    } else {
      const int j = i - kFaceX - kFaceY;
      x = 1 + j / (kTY - 1); y = 1 + j % (kTY - 1); z = 0;
    }
    unsigned long long v = 0ull;
#pragma unroll
    for (int m = 1; m < 8; ++m) {   // bit d: one tile back along axis d
      const int a = m & 1, b = (m >> 1) & 1, c = m >> 2;
      if ((a && x != 0) || (b && y != 0) || (c && z != 0)) continue;
      v += ts.halo[(size_t)tile_index(tx - a, ty - b, tz - c, n) * kTileHalo + halo_slot(a ? kTX : x, b ? kTY : y, c ? kTZ : z)];
    }
    if (v != 0ull)
      grid[((size_t)(tx * kTX + x) * n + (size_t)(ty * kTY + y)) * n + (size_t)(tz * kTZ + z)] += v;
  }
}

// delta = counts * qscale - 1 minus its mean, qscale <q> - 1 (mean_q: the mean of the fixed-point counts,
// a deterministic reduction of the grid), in one pass
__global__ void __launch_bounds__(256)
k_counts_to_delta(const long long* __restrict__ grid, size_t n3, double qscale, double* __restrict__ delta,
                  const int* __restrict__ bad, const double* __restrict__ mean_q) {
#pragma clang fp contract(off)
  const bool nan_out = *bad != 0;   // a non-finite position: delta is undefined, mark it so
  const double m = *mean_q * qscale - 1.0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256) {
    const double d = double(grid[i]) * qscale;
    delta[i] = nan_out ? __builtin_nan("") : (d - 1.0) - m;
  }
}

// CIC interpolation of an NC-component field: f[k] = sum over the 8 corners of
// (w_x w_y) w_z times the corner value of component k; `at(a, b, c, k)` reads the value.
template <int NC, class At>
__device__ __forceinline__ void gather_corners(const Cic& c, const At& at, double (&f)[NC]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int k = 0; k < NC; ++k) f[k] = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const double wx = a ? c.w1[0] : c.w0[0];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const double wxy = wx * (b ? c.w1[1] : c.w0[1]);
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const double wgt = wxy * (cc ? c.w1[2] : c.w0[2]);
#pragma unroll
        for (int k = 0; k < NC; ++k) f[k] += wgt * at(a, b, cc, k);
      }
    }
  }
}

// flat mesh index of corner (a, b, cc) of a particle's CIC cell
__device__ __forceinline__ size_t corner_index(const Cic& c, int a, int b, int cc, int n) {
  const size_t ix = (size_t)(a ? c.i1[0] : c.i0[0]);
  const size_t iy = (size_t)(b ? c.i1[1] : c.i0[1]);
  const size_t iz = (size_t)(cc ? c.i1[2] : c.i0[2]);
  return (ix * n + iy) * n + iz;
}

// LDS staging of the particle gathers.  A workgroup takes a chunk of consecutive particles; when
// the periodic box of their cells fits, the box's mesh values are staged in LDS (coalesced rows,
// each cell read once) and the corners gathered from there, otherwise each corner is read from the
// mesh.  What bounds the direct gather of several components is the L2-to-L1 traffic of its rows (a
// wavefront of an 8^3 block touches ~24 lines of 128 bytes per component), which staging replaces by
// ~3.3 cells per particle (2.1M particles in 8^3 blocks on 128^3, three components: 70 -> 35 us).  The
// box search and its barriers cost what one component has to gain (19-20 us direct, 26-30 us staged),
// so single components are gathered directly.
#ifndef DGP_GATHER_CHUNK
#define DGP_GATHER_CHUNK 256
#endif
#ifndef DGP_GATHER_BIN_CAP
#define DGP_GATHER_BIN_CAP 1024
#endif
constexpr int kGatherChunk = DGP_GATHER_CHUNK;
constexpr int kGatherPPT = kGatherChunk / 256;
constexpr int kGatherCap = DGP_GATHER_BIN_CAP;
// how a gather is run (gather_how); template argument of the gather kernels
enum GatherHow : int {
  kGatherStage = 1,    // several components: compact chunks through LDS
  kGatherStream = 2,   // positions by streaming loads
  kGatherXcd = 4,      // chunks in XCD order
};
template <int HOW>
__device__ __forceinline__ long long gather_first() {   // the workgroup's first particle
  return ((HOW & kGatherXcd) ? xcd_chunk() : (long long)blockIdx.x) * kGatherChunk;
}
static_assert(kGatherChunk % 256 == 0, "chunk must be a multiple of the workgroup size");

// With kGatherStage, a chunk's box staged from the NC-component mesh [NC][N^3] into fl[NC][kGatherCap]; every
// thread of the workgroup calls it, and `apply(p, k, cell, at)` then runs for each of the thread's particles
// with at(a, b, c, component), the mesh value of a corner.
template <int NC, int HOW, typename P, typename M, class Apply>
__device__ __forceinline__ void gather_chunk(const M* __restrict__ mesh, const P* __restrict__ pos,
                                             const P (&xs)[kGatherPPT][3], long long np, long long p0, int n,
                                             double scale, M* fl, const Apply& apply) {
#pragma clang fp contract(off)
  const size_t n3 = (size_t)n * n * n;
  if constexpr (!(HOW & kGatherStage)) {
#pragma unroll
    for (int k = 0; k < kGatherPPT; ++k) {
      const long long p = p0 + threadIdx.x + k * 256;
      if (p >= np) continue;
      const double s3[3] = {double(xs[k][0]) * scale, double(xs[k][1]) * scale, double(xs[k][2]) * scale};
      const Cic c = cic_at(s3, n);
      apply(p, k, c, [&](int a, int b, int cc, int q) {
        return double(mesh[(size_t)q * n3 + corner_index(c, a, b, cc, n)]);
      });
    }
    return;
  }
  Cic cr;
  int off[kGatherPPT][3], bx[6];
  const bool binned = chunk_box<kGatherPPT>(pos, xs, np, n, scale, p0, kGatherCap, cr, off, bx);
  if (binned) {
    const int vol = bx[3] * bx[4] * bx[5];
    for (int i = threadIdx.x; i < vol; i += 256) {
      const size_t g = box_cell(i, cr, bx, n);
#pragma unroll
      for (int q = 0; q < NC; ++q) fl[q * kGatherCap + i] = mesh[(size_t)q * n3 + g];
    }
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < kGatherPPT; ++k) {
    const long long p = p0 + threadIdx.x + k * 256;
    if (p >= np) continue;
    // the cell and weights again from the position (the chunk box's arithmetic): not holding
    // them across the staging loop and its barrier leaves the kick-drift 65 instead of 75 VGPRs
    // (occupancy 6 -> 7-8; 512^3 float32 particles 2.71 -> 2.30 ms, 256^3 unchanged)
    const double s3[3] = {double(xs[k][0]) * scale, double(xs[k][1]) * scale, double(xs[k][2]) * scale};
    const Cic c = cic_at(s3, n);
    if (binned) {
      apply(p, k, c, [&](int a, int b, int cc, int q) {
        const int li = ((off[k][0] + a - bx[0]) * bx[4] + (off[k][1] + b - bx[1])) * bx[5] + (off[k][2] + cc - bx[2]);
        return double(fl[q * kGatherCap + li]);
      });
    } else {
      apply(p, k, c, [&](int a, int b, int cc, int q) {
        return double(mesh[(size_t)q * n3 + corner_index(c, a, b, cc, n)]);
      });
    }
  }
}

// out[k][p] = sum_c W_c(x_p) mesh[k][c]
template <typename P, typename M, int NC, int HOW>
__global__ void __launch_bounds__(256)
k_interp(const M* __restrict__ mesh, const P* __restrict__ pos, long long np, int n, double scale,
         double* __restrict__ out) {
  __shared__ M fl[(HOW & kGatherStage) ? NC * kGatherCap : 1];
  const long long p0 = gather_first<HOW>();
  P xs[kGatherPPT][3];
  load_chunk<kGatherPPT, (HOW & kGatherStream) != 0>(pos, np, p0, xs);
  gather_chunk<NC, HOW>(mesh, pos, xs, np, p0, n, scale, fl, [&](long long p, int, const Cic& c, const auto& at) {
    double f[NC];
    gather_corners<NC>(c, at, f);
#pragma unroll
    for (int q = 0; q < NC; ++q) __builtin_nontemporal_store(f[q], &out[(size_t)q * np + p]);
  });
}

// Leapfrog with momenta at half steps: p += kick * g(x_n); x += drift * p; wrap into [0, L), the force
// gathered through the staged box.
template <typename P, typename M>
__global__ void __launch_bounds__(256)
k_interp_kick_drift_bin(const M* __restrict__ mesh3, P* __restrict__ pos, P* __restrict__ vel, long long np,
                        int n, double scale, double box, double kick, double drift) {
#pragma clang fp contract(off)
  __shared__ M fl[3 * kGatherCap];
  const long long p0 = xcd_chunk() * kGatherChunk;
  // positions and velocities are loaded together up front and kept in registers
  P xs[kGatherPPT][3], vs[kGatherPPT][3];
  load_chunk<kGatherPPT>(pos, np, p0, xs);
  load_chunk<kGatherPPT>(vel, np, p0, vs);
  gather_chunk<3, kGatherStage>(mesh3, pos, xs, np, p0, n, scale, fl, [&](long long p, int k, const Cic& c, const auto& at) {
    double f[3];
    gather_corners<3>(c, at, f);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const size_t i = (size_t)d * np + p;
      const double v = double(vs[k][d]) + kick * f[d];
      double x = double(xs[k][d]) + drift * v;
      x = x - box * floor(x / box);
      P xo = P(x);
      if (xo >= P(box)) xo = xo - P(box);
      __builtin_nontemporal_store(P(v), &vel[i]);   // streaming: read again only by the next step
      __builtin_nontemporal_store(xo, &pos[i]);
    }
  });
}

// dL/dx_p of a loss whose derivative with respect to the weight of corner (a, b, cc) is
// val(a, b, cc): sum over the corners of val dW/dx (derivative of the unquantised weights)
template <class Val>
__device__ __forceinline__ void gather_weight_grad(const Cic& c, double scale, const Val& val, double (&g)[3]) {
  g[0] = g[1] = g[2] = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const double wx = a ? c.w1[0] : c.w0[0];
    const double dx = a ? scale : -scale;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const double wy = b ? c.w1[1] : c.w0[1];
      const double dy = b ? scale : -scale;
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const double wz = cc ? c.w1[2] : c.w0[2];
        const double dz = cc ? scale : -scale;
        const double v = val(a, b, cc);
        g[0] += v * dx * wy * wz;
        g[1] += v * wx * dy * wz;
        g[2] += v * wx * wy * dz;
      }
    }
  }
}

// dL/dx_p = (N^3/Np) sum_c g_c dW_c/dx_p  (derivative of the unquantised weights)
template <typename P, int HOW>
__global__ void __launch_bounds__(256)
k_deposit_backward(const P* __restrict__ pos, long long np, int n, double scale, const double* __restrict__ g,
                   double mass, double* __restrict__ grad) {
  const long long p0 = gather_first<HOW>();
  P xs[kGatherPPT][3];
  load_chunk<kGatherPPT, (HOW & kGatherStream) != 0>(pos, np, p0, xs);
  gather_chunk<1, HOW>(g, pos, xs, np, p0, n, scale, (double*)nullptr, [&](long long p, int, const Cic& c, const auto& at) {
    double gx[3];
    gather_weight_grad(c, scale, [&](int a, int b, int cc) { return at(a, b, cc, 0); }, gx);
#pragma unroll
    for (int d = 0; d < 3; ++d) __builtin_nontemporal_store(gx[d] * mass, &grad[(size_t)d * np + p]);
  });
}

// ------------------------------------------------------------------ CIC interpolation adjoint
// The interpolation out[m][p] = sum_c W_c(x_p) mesh[m][c] (Sec. III A: forces are interpolated
// with the deposit's assignment function, Eq. CIC; unquantised weights W_c = w_x w_y w_z) has,
// for g = dL/dout,
//   dL/dx_p        = sum_m g[m][p] sum_c mesh[m][c] dW_c/dx_p     (gather, k_interp_grad_pos)
//   dL/dmesh[m][c] = sum_p g[m][p] W_c(x_p)                       (scatter, k_interp_grad_mesh_bin)
// The scatter sums in 64-bit fixed point, so the result has the same bits in any particle order:
// every term is rounded to an integer multiple of 2^-e, e chosen per call so that no sum can
// reach 2^62 (a cell's sum is at most max|g| times its mass sum_p W_c, which the deposit of the
// same positions bounds).

// dL/dx_p: per particle, the 8 corners of its cell
template <typename P, int NC, int HOW>
__global__ void __launch_bounds__(256)
k_interp_grad_pos(const double* __restrict__ mesh, const P* __restrict__ pos, long long np, int n, double scale,
                  const double* __restrict__ g, double* __restrict__ grad) {
  __shared__ double fl[(HOW & kGatherStage) ? NC * kGatherCap : 1];
  const long long p0 = gather_first<HOW>();
  P xs[kGatherPPT][3];
  load_chunk<kGatherPPT, (HOW & kGatherStream) != 0>(pos, np, p0, xs);
  gather_chunk<NC, HOW>(mesh, pos, xs, np, p0, n, scale, fl, [&](long long p, int, const Cic& c, const auto& at) {
    double gm[NC], gx[3];
#pragma unroll
    for (int m = 0; m < NC; ++m) gm[m] = g[(size_t)m * np + p];
    gather_weight_grad(
        c, scale,
        [&](int a, int b, int cc) {
          double proj = 0.0;
#pragma unroll
          for (int m = 0; m < NC; ++m) proj += gm[m] * at(a, b, cc, m);
          return proj;
        },
        gx);
#pragma unroll
    for (int d = 0; d < 3; ++d) __builtin_nontemporal_store(gx[d], &grad[(size_t)d * np + p]);
  });
}

// part[block] = {bit pattern of the block's max |g| (non-negative doubles order like their bit
// patterns), its largest fixed-point mass of the grid}; *bad raised for a non-finite g.  Bound by
// reading g and the grid once (3 x 2.1M values on 128^3, 67 MB: 16 us); one atomicMax per wavefront
// on two shared words instead of the partials took 747 us, serialised on those words.
__global__ void __launch_bounds__(256)
k_max_abs_and_mass(const double* __restrict__ g, size_t count, const long long* __restrict__ grid, size_t n3,
                   ulonglong2* __restrict__ part, int* __restrict__ bad) {
  double m = 0.0;
  long long mm = 0;
  bool ok = true;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) {
    const double v = g[i];
    ok = ok && isfinite(v);
    m = fmax(m, fabs(v));
  }
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (size_t)gridDim.x * 256) mm = max(mm, grid[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    m = fmax(m, __shfl_xor(m, o, 64));
    mm = max(mm, __shfl_xor(mm, o, 64));
  }
  if (!ok) atomicOr(bad, 1);
  __shared__ double wm[4];
  __shared__ long long wmm[4];
  if ((threadIdx.x & 63) == 0) {
    wm[threadIdx.x >> 6] = m;
    wmm[threadIdx.x >> 6] = mm;
  }
  lds_barrier();
  if (threadIdx.x == 0) {
    m = fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
    mm = max(max(wmm[0], wmm[1]), max(wmm[2], wmm[3]));
    part[blockIdx.x] = make_ulonglong2((unsigned long long)__double_as_longlong(m), (unsigned long long)mm);
  }
}

// st[2] = e with (max|g|) (mass bound) 2^e < 2^62, from the partial maxima (one wavefront)
__global__ void __launch_bounds__(64)
k_interp_scale(const ulonglong2* __restrict__ part, int blocks, unsigned long long* __restrict__ st) {
  double gmax = 0.0;
  long long mm = 0;
  for (int i = threadIdx.x; i < blocks; i += 64) {
    const ulonglong2 v = part[i];
    gmax = fmax(gmax, __longlong_as_double((long long)v.x));
    mm = max(mm, (long long)v.y);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    gmax = fmax(gmax, __shfl_xor(gmax, o, 64));
    mm = max(mm, __shfl_xor(mm, o, 64));
  }
  if (threadIdx.x != 0) return;
  const double mass = double(mm) * 0x1p-40 * (1.0 + 0x1p-20) + 0x1p-20;
  const double bound = gmax * mass;
  int e = 0;
  if (bound > 0.0 && isfinite(bound)) {
    int ex = 0;
    (void)frexp(bound, &ex);   // bound < 2^ex
    e = 62 - ex;
    e = e > 960 ? 960 : (e < -960 ? -960 : e);
  }
  st[2] = (unsigned long long)(long long)e;
}

// Bound by the global atomics of the flush (one per touched box cell and component), the conversions and
// the LDS atomics together.  A chunk of 1024 particles with one component after another in a 24 KB
// histogram takes fewer of the first than one of 512 with all components at once (2.1M particles in
// 8^3 blocks, three components, 128^3: 113 -> 98 us; 2048 particles 104 us); 512 below 2^18 particles,
// where 1024 would leave the device idle, with a histogram of 2048 cells: boxes of small clustered loads
// fit it and not 1536 (32768 particles on 32^3, the whole adjoint: one component 73 and 29 us, three 132
// and 40 us).
template <typename P, int CH, int NC>
__global__ void __launch_bounds__(256)
k_interp_grad_mesh_bin(const P* __restrict__ pos, long long np, int n, double scale, const double* __restrict__ g,
                       const unsigned long long* __restrict__ st, unsigned long long* __restrict__ acc) {
#pragma clang fp contract(off)
  constexpr int PPT = CH / 256, CAP = (CH >= 1024 ? 3 : 4) * CH;
  __shared__ unsigned long long hist[CAP];
  const size_t n3 = (size_t)n * n * n;
  const int e = (int)(long long)st[2];
  const long long p0 = xcd_chunk() * CH;
  P xs[PPT][3];
  load_chunk<PPT>(pos, np, p0, xs);
  Cic cr;
  int off[PPT][3], bx[6];
  const bool binned = chunk_box<PPT>(pos, xs, np, n, scale, p0, CAP, cr, off, bx);
  const int vol = bx[3] * bx[4] * bx[5];
#pragma unroll 1
  for (int m = 0; m < NC; ++m) {
    const double* const gm = g + (size_t)m * np;
    unsigned long long* const am = acc + (size_t)m * n3;
    if (binned)
      for (int i = threadIdx.x; i < vol; i += 256) hist[i] = 0ull;
    lds_barrier();
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      const long long p = p0 + threadIdx.x + k * 256;
      if (p >= np) continue;
      const double gk = gm[p];
      // the cell and weights again from the position (the chunk box's arithmetic), opaque so that they
      // are not held across the components
      P x[3] = {xs[k][0], xs[k][1], xs[k][2]};
#pragma unroll
      for (int d = 0; d < 3; ++d) asm volatile("" : "+v"(x[d]));
      const double s3[3] = {double(x[0]) * scale, double(x[1]) * scale, double(x[2]) * scale};
      const Cic c = cic_at(s3, n);
      const int ox = periodic_offset(c.i0[0], cr.i0[0], n) - bx[0], oy = periodic_offset(c.i0[1], cr.i0[1], n) - bx[1],
                oz = periodic_offset(c.i0[2], cr.i0[2], n) - bx[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const double wx = a ? c.w1[0] : c.w0[0];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const double wxy = wx * (b ? c.w1[1] : c.w0[1]);
#pragma unroll
          for (int cc = 0; cc < 2; ++cc) {
            const double wgt = wxy * (cc ? c.w1[2] : c.w0[2]);
            const unsigned long long q = (unsigned long long)(long long)rint(ldexp(gk * wgt, e));
            if (binned) atomicAdd(&hist[((ox + a) * bx[4] + (oy + b)) * bx[5] + (oz + cc)], q);
            else atomicAdd(&am[corner_index(c, a, b, cc, n)], q);
          }
        }
      }
    }
    if (!binned) continue;
    lds_barrier();
    for (int i = threadIdx.x; i < vol; i += 256) {
      const unsigned long long v = hist[i];
      if (v != 0ull) atomicAdd(&am[box_cell(i, cr, bx, n)], v);
    }
    lds_barrier();   // before the next component clears the histogram
  }
}

// in place: the fixed-point sums (int64 bit patterns) become doubles q 2^-e (NaN when *bad)
__global__ void __launch_bounds__(256)
k_fixed_to_double(unsigned long long* __restrict__ x, size_t count, const unsigned long long* __restrict__ st,
                  const int* __restrict__ bad) {
  const int e = (int)(long long)st[2];
  const bool nan_out = *bad != 0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) {
    const double v = nan_out ? __builtin_nan("") : ldexp(double((long long)x[i]), -e);
    x[i] = (unsigned long long)__double_as_longlong(v);
  }
}

__global__ void __launch_bounds__(256) k_fill_zero(unsigned long long* __restrict__ x, size_t count) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) x[i] = 0ull;
}

// clears a deposit's grid, its non-finite flag and (words2 > 0) the tile sort's counters in one launch
__global__ void __launch_bounds__(256)
k_deposit_clear(unsigned long long* __restrict__ grid, size_t count, int* __restrict__ bad, unsigned* __restrict__ words,
                int words2) {
  const size_t i0 = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i0 == 0) *bad = 0;
  for (size_t i = i0; i < (size_t)words2; i += (size_t)gridDim.x * 256) words[i] = 0u;
  for (size_t i = i0; i < count; i += (size_t)gridDim.x * 256) grid[i] = 0ull;
}

template <typename T>
__global__ void __launch_bounds__(256) k_convert(size_t count, const void* __restrict__ in, int in_fp32, T* __restrict__ out) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256)
    out[i] = in_fp32 ? T(static_cast<const float*>(in)[i]) : T(static_cast<const double*>(in)[i]);
}

static unsigned gather_chunks(long long np) { return unsigned((np + kGatherChunk - 1) / kGatherChunk); }
static unsigned grid_strided(size_t count) {
  size_t g = (count + 255) / 256;
  return unsigned(g > 8192 ? 8192 : (g < 1 ? 1 : g));
}

// The tile sort is taken from 2^18 particles on meshes of at least 128^3 whose scratch holds the sorted
// positions; compact chunks keep the direct path inside it.  Lattice-order loads, whole deposit without
// and with it: 128^3 mesh, 64^3 / 96^3 / 128^3 particles 50 / 111 / 272 and 48 / 59 / 92 us; 256^3 mesh,
// 128^3 / 256^3 particles 326 / 1786 and 137 / 493 us; on 64^3 (64 tiles) 64^3 particles take 42 and
// 50 us.  In random order, 128^3 particles on 128^3 750 and 196 us, 4.2M / 16.8M on 256^3 1533 / 5805 and
// 500 / 1380 us; on 512^3 a random chunk spans more tiles than a workgroup counts (32768) and stays
// with direct atomics (33.6M: 13.3 and 13.2 ms).  A load in 8^3 blocks pays its four idle launches (and
// its chunks' marks): 128^3 particles on 128^3 46 and 49 us, 256^3 on 256^3 244 and 257 us, 512^3 float32
// on 512^3 1.66 and 1.71 ms.  (Fewer workgroups that walk their chunks, items or tiles make the idle
// launches cheaper, 512^3 1.67 ms, and the sorting ones slower: lattice order 2.95 -> 3.0-3.2 ms.)
static bool tile_sort(int n, size_t psize, long long np, int ch, void* scratch, size_t bytes, TileSort& ts) {
  if (!scratch || n < 128 || np < (1ll << 18) || np >= (1ll << 31)) return false;
  const size_t tiles = tile_count(n), chunks = (np + ch - 1) / ch;
  const size_t items = tiles + np / kTileItem;
  char* p = static_cast<char*>(scratch);
  auto take = [&](size_t sz) {
    char* q = p;
    p += (sz + 255) & ~size_t(255);
    return q;
  };
  ts.count = reinterpret_cast<unsigned*>(take((tiles + kTileState) * sizeof(unsigned)));   // state behind the counts
  ts.state = ts.count + tiles;
  ts.sorted = reinterpret_cast<unsigned char*>(take(chunks));
  ts.items = reinterpret_cast<uint4*>(take(items * sizeof(uint4)));
  ts.multi = reinterpret_cast<unsigned char*>(take(tiles));
  ts.halo = reinterpret_cast<unsigned long long*>(take(tiles * kTileHalo * sizeof(unsigned long long)));
  ts.pos = take(3 * (size_t)np * psize);
  return size_t(p - static_cast<char*>(scratch)) <= bytes;
}

template <typename P, int CH>
static void deposit_t(int n, double box, const P* pos, long long np, unsigned long long* grid, int* bad, void* scratch,
                      size_t bytes, hipStream_t s) {
  const double scale = double(n) / box;
  const unsigned g = unsigned((np + CH - 1) / CH);
  TileSort ts{};
  const bool sort = tile_sort(n, sizeof(P), np, CH, scratch, bytes, ts);
  const int tiles = sort ? tile_count(n) : 0;
  const size_t n3 = (size_t)n * n * n;
  hipLaunchKernelGGL(k_deposit_clear, dim3(grid_strided(n3)), dim3(256), 0, s, grid, n3, bad, ts.count,
                     sort ? tiles + kTileState : 0);
  if (!sort) {
    hipLaunchKernelGGL((k_deposit_bin<P, CH, false>), dim3(g), dim3(256), 0, s, pos, np, n, scale, grid, bad, ts);
    return;
  }
  hipLaunchKernelGGL((k_deposit_bin<P, CH, true>), dim3(g), dim3(256), 0, s, pos, np, n, scale, grid, bad, ts);
  hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, s, ts, tiles);
  hipLaunchKernelGGL((k_tile_scatter<P, CH>), dim3(g), dim3(256), 0, s, pos, np, n, scale, ts);
  hipLaunchKernelGGL((k_tile_deposit<P>), dim3(tiles + unsigned(np / kTileItem)), dim3(512), 0, s, np, n, scale, ts,
                     grid);
  hipLaunchKernelGGL(k_tile_halo, dim3(tiles), dim3(256), 0, s, n, ts, grid);
}

void launch_deposit(int n, double box, const void* pos, int pos_fp32, long long np, long long* grid, int* bad,
                    void* scratch, size_t scratch_bytes, hipStream_t s) {
  auto* out = reinterpret_cast<unsigned long long*>(grid);
  const float* p32 = static_cast<const float*>(pos);
  const double* p64 = static_cast<const double*>(pos);
  const bool big = n >= 512;   // chunk by mesh size (DepGeo)
  if (pos_fp32 && big) deposit_t<float, 2048>(n, box, p32, np, out, bad, scratch, scratch_bytes, s);
  else if (pos_fp32) deposit_t<float, 1024>(n, box, p32, np, out, bad, scratch, scratch_bytes, s);
  else if (big) deposit_t<double, 2048>(n, box, p64, np, out, bad, scratch, scratch_bytes, s);
  else deposit_t<double, 1024>(n, box, p64, np, out, bad, scratch, scratch_bytes, s);
}

double counts_scale(int n, long long np) { return ldexp(double((size_t)n * n * n) / double(np), -40); }

void launch_counts_to_delta(int n, const long long* grid, long long np, double* delta, const int* bad, hipStream_t s,
                            const double* mean_q) {
  const size_t n3 = (size_t)n * n * n;
  const double qscale = counts_scale(n, np);
  hipLaunchKernelGGL(k_counts_to_delta, dim3(grid_strided(n3)), dim3(256), 0, s, grid, n3, qscale, delta, bad, mean_q);
}

void launch_fill_zero(void* p, size_t words, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_strided(words)), dim3(256), 0, s, static_cast<unsigned long long*>(p),
                     words);
}


// How a gather is run.  A load of less than a particle per four cells (thin) cannot fill boxes of kGatherCap
// cells, and its chunks in dispatch order are as near to each other as in XCD order (2^18 particles on
// 256^3 in 8^3 blocks: one component 10.9 us against 12.1 in XCD order, three components 30.0 us direct
// against 33.8 staged).  Positions are streamed where what the kernel reads exceeds the 256 MB last-level
// cache, and read with plain loads below (one component: 2.1M float64 particles in blocks on 128^3 16.2 us
// plain, 19.1 us streamed; 4.2M on 256^3, 235 MB, 38 and 44 us; 16.8M float32, 335 MB, 129 and 104 us).
// LAUNCH(HOW) for the chosen HOW:
#define DGP_GATHER_LAUNCH(NC, thin, stream, LAUNCH)                                  \
  {                                                                                  \
    constexpr int dense = kGatherXcd | (NC > 1 ? kGatherStage : 0);                  \
    if (thin && stream) LAUNCH(kGatherStream);                                       \
    else if (thin) LAUNCH(0);                                                        \
    else if (stream) LAUNCH(dense | kGatherStream);                                  \
    else LAUNCH(dense);                                                              \
  }
static bool gather_thin(int n, long long np) { return 4 * np < (long long)n * n * n; }
static bool gather_streams(size_t bytes) { return bytes > (size_t(256) << 20); }

template <typename P, typename M, int NC>
static void interp_t(int n, double box, const M* mesh, const P* pos, long long np, double* out, hipStream_t s) {
  const double scale = double(n) / box;
  const bool thin = gather_thin(n, np), stream = gather_streams(NC * sizeof(M) * n * n * n + 3 * sizeof(P) * np);
#define L(HOW) \
  hipLaunchKernelGGL((k_interp<P, M, NC, (HOW)>), dim3(gather_chunks(np)), dim3(256), 0, s, mesh, pos, np, n, scale, out)
  DGP_GATHER_LAUNCH(NC, thin, stream, L)
#undef L
}
template <typename M, int NC>
static void interp_m(int n, double box, const M* mesh, const void* pos, int pos_fp32, long long np, double* out,
                     hipStream_t s) {
  if (pos_fp32) interp_t<float, M, NC>(n, box, mesh, static_cast<const float*>(pos), np, out, s);
  else interp_t<double, M, NC>(n, box, mesh, static_cast<const double*>(pos), np, out, s);
}

void launch_interp(int n, double box, const void* mesh, int mesh_fp32, int nc, const void* pos, int pos_fp32,
                   long long np, double* out, hipStream_t s) {
#define DGP_INTERP(NC)                                                                                        \
  if (mesh_fp32) interp_m<float, NC>(n, box, static_cast<const float*>(mesh), pos, pos_fp32, np, out, s);     \
  else interp_m<double, NC>(n, box, static_cast<const double*>(mesh), pos, pos_fp32, np, out, s);
  switch (nc) {
    case 1: DGP_INTERP(1) break;
    case 2: DGP_INTERP(2) break;
    default: DGP_INTERP(3) break;
  }
#undef DGP_INTERP
}

template <typename M>
static void kick_m(int n, double box, const M* mesh3, void* pos, void* vel, int fp32, long long np, double kick,
                   double drift, hipStream_t s) {
  const double scale = double(n) / box;
  const unsigned g = gather_chunks(np);
  if (fp32)
    hipLaunchKernelGGL((k_interp_kick_drift_bin<float, M>), dim3(g), dim3(256), 0, s, mesh3, static_cast<float*>(pos),
                       static_cast<float*>(vel), np, n, scale, box, kick, drift);
  else
    hipLaunchKernelGGL((k_interp_kick_drift_bin<double, M>), dim3(g), dim3(256), 0, s, mesh3,
                       static_cast<double*>(pos), static_cast<double*>(vel), np, n, scale, box, kick, drift);
}

void launch_interp_kick_drift(int n, double box, const void* mesh3, int mesh_fp32, void* pos, void* vel, int fp32,
                              long long np, double kick, double drift, hipStream_t s) {
  if (mesh_fp32)
    kick_m(n, box, static_cast<const float*>(mesh3), pos, vel, fp32, np, kick, drift, s);
  else
    kick_m(n, box, static_cast<const double*>(mesh3), pos, vel, fp32, np, kick, drift, s);
}

template <typename P>
static void deposit_backward_t(int n, double box, const P* pos, long long np, const double* grad_delta, double* grad_pos,
                               hipStream_t s) {
  const double scale = double(n) / box;
  const double mass = double(n) * n * n / double(np);
  const bool thin = gather_thin(n, np), stream = gather_streams(sizeof(double) * n * n * n + 3 * sizeof(P) * np);
#define L(HOW)                                                                                                          \
  hipLaunchKernelGGL((k_deposit_backward<P, (HOW)>), dim3(gather_chunks(np)), dim3(256), 0, s, pos, np, n, scale, grad_delta, \
                     mass, grad_pos)
  DGP_GATHER_LAUNCH(1, thin, stream, L)
#undef L
}
void launch_deposit_backward(int n, double box, const void* pos, int pos_fp32, long long np, const double* grad_delta,
                             double* grad_pos, hipStream_t s) {
  if (pos_fp32) deposit_backward_t(n, box, static_cast<const float*>(pos), np, grad_delta, grad_pos, s);
  else deposit_backward_t(n, box, static_cast<const double*>(pos), np, grad_delta, grad_pos, s);
}

template <typename P, int NC>
static void interp_bwd_t(int n, double box, const double* mesh, const P* pos, long long np, const double* g,
                         double* grad_pos, double* grad_mesh, long long* grid, unsigned long long* st, double* red,
                         int* bad, void* scratch, size_t scratch_bytes, hipStream_t s) {
  const double scale = double(n) / box;
  const size_t n3 = (size_t)n * n * n;
  if (grad_pos) {
    const bool thin = gather_thin(n, np), stream = gather_streams(8 * NC * n3 + (3 * sizeof(P) + 8 * NC) * np);
#define L(HOW)                                                                                                           \
  hipLaunchKernelGGL((k_interp_grad_pos<P, NC, (HOW)>), dim3(gather_chunks(np)), dim3(256), 0, s, mesh, pos, np, n, scale, \
                     g, grad_pos)
    DGP_GATHER_LAUNCH(NC, thin, stream, L)
#undef L
  }
  if (!grad_mesh) return;
  auto* acc = reinterpret_cast<unsigned long long*>(grad_mesh);
  launch_fill_zero(acc, NC * n3, s);
  launch_deposit(n, box, pos, sizeof(P) == 4, np, grid, bad, scratch, scratch_bytes, s);
  const int blocks = int(absmean_scratch_doubles(n3, 1) / 2);   // one pair of words per block
  hipLaunchKernelGGL(k_max_abs_and_mass, dim3(blocks), dim3(256), 0, s, g, (size_t)NC * np, grid, n3,
                     reinterpret_cast<ulonglong2*>(red), bad);
  hipLaunchKernelGGL(k_interp_scale, dim3(1), dim3(64), 0, s, reinterpret_cast<const ulonglong2*>(red), blocks, st);
  if (np >= (1ll << 18))
    hipLaunchKernelGGL((k_interp_grad_mesh_bin<P, 1024, NC>), dim3(unsigned((np + 1023) / 1024)), dim3(256), 0, s, pos, np,
                       n, scale, g, st, acc);
  else
    hipLaunchKernelGGL((k_interp_grad_mesh_bin<P, 512, NC>), dim3(unsigned((np + 511) / 512)), dim3(256), 0, s, pos, np, n,
                       scale, g, st, acc);
  hipLaunchKernelGGL(k_fixed_to_double, dim3(grid_strided(NC * n3)), dim3(256), 0, s, acc, NC * n3, st, bad);
}

void launch_interp_backward(int n, double box, const double* mesh, int nc, const void* pos, int pos_fp32, long long np,
                            const double* g, double* grad_pos, double* grad_mesh, long long* grid,
                            unsigned long long* st, double* red, int* bad, void* scratch, size_t scratch_bytes,
                            hipStream_t s) {
#define DGP_IB(P, NC) \
  interp_bwd_t<P, NC>(n, box, mesh, static_cast<const P*>(pos), np, g, grad_pos, grad_mesh, grid, st, red, bad, scratch, \
                     scratch_bytes, s)
  if (pos_fp32) {
    if (nc == 1) DGP_IB(float, 1);
    else if (nc == 2) DGP_IB(float, 2);
    else DGP_IB(float, 3);
  } else {
    if (nc == 1) DGP_IB(double, 1);
    else if (nc == 2) DGP_IB(double, 2);
    else DGP_IB(double, 3);
  }
#undef DGP_IB
}

// ------------------------------------------------------------------ allocation-free deposit scratch
// Device scratch of the allocation-free deposit entry point: the per-workgroup partial sums of the
// mean removal, the mean and the non-finite flag.  One copy per device, held until the process
// ends; every call on a device shares it, so calls that overlap on one device race.  Host code
// uses the per-device address from hipGetSymbolAddress, never the array's name.
constexpr size_t kNoallocScratchDoubles = 4096;   // 32 KiB
static __device__ __align__(256) double scratch[kNoallocScratchDoubles];

static void* g_noalloc_ptr[64];
static std::mutex g_noalloc_mu;

int noalloc_scratch(double** ptr, size_t* capacity) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -1;
  if (dev < 0 || dev >= 64) return -2;
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (g_noalloc_ptr[dev] == nullptr) {   // once per device, with that device current
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return -1;
    g_noalloc_ptr[dev] = p;
  }
  *ptr = static_cast<double*>(g_noalloc_ptr[dev]);
  *capacity = kNoallocScratchDoubles;
  return 0;
}

template <typename T>
void launch_convert(size_t count, const void* in, int in_fp32, T* out, hipStream_t s) {
  hipLaunchKernelGGL((k_convert<T>), dim3(grid_strided(count)), dim3(256), 0, s, count, in, in_fp32, out);
}
template void launch_convert<double>(size_t, const void*, int, double*, hipStream_t);
template void launch_convert<float>(size_t, const void*, int, float*, hipStream_t);

}  // namespace dgp
