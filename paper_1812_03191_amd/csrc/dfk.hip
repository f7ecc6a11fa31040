// dfk.hip -- gfx950 kernels of libdfmesh.
//
// The update of one level over a step dt follows the staging list of Velasco
// Romero & Masset (2018), Sect. 3.3, with the split source step of eq. 15:
//   kick(dt/2) -> compression, diffusion, heat release (dt) -> transport (dt)
//   -> kick(dt/2)
//
// Storage and arithmetic.  Every field is stored as its departure from the
// uniform background (rho0, e0, wind (-V, 0, 0), momenta rho0 (-V, 0, 0)) in
// the run's storage type T: double (FP64 runs) or float (FP32 runs).  The
// stencils are written for departures: the uniform background transfer is the
// same through every face and cancels from every flux difference, so it is
// never formed, and the potential difference across a face is taken in a form
// free of cancellation.  Forces, totals and the time step are reduced in FP64.
//
// Launch shape.  Box kernels launch a 1-D grid of 64 x 4 tiles times one plane;
// level 0 reads its outer boundary conditions on the fly (clamped indices, a
// zero departure beyond the inflow face), so it stores no ghost data; finer
// levels advance their whole ghost shell, filled once per parent step.
#include "dfk.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>

namespace dfk {

namespace {

constexpr int BX = 64, BY = 4;

struct Box {
  int lo[3], hi[3];
};

inline bool empty_grid(const dim3 &g) { return g.x == 0; }

// The hardware hands workgroups to the 8 XCDs round-robin (workgroup h runs
// on XCD h % 8).  thread_cell gives each XCD one contiguous range of tiles: a
// band of rows through all planes, walked plane by plane (x-tile fastest, then
// y-tile within the band, then plane), so the neighbour planes a stencil
// reads are in its own L2 (a few planes of one band fit there) and neighbour
// rows are too except at band edges.
inline dim3 grid_of(const Box &b) {
  int ex = b.hi[0] - b.lo[0], ey = b.hi[1] - b.lo[1], ez = b.hi[2] - b.lo[2];
  if (ex <= 0 || ey <= 0 || ez <= 0) return dim3(0, 1, 1);
  long n = (long)((ex + BX - 1) / BX) * ((ey + BY - 1) / BY) * ez;
  return dim3((unsigned)n, 1, 1);
}

// A block's place in its launch: the hardware's, or, in a launch that
// carries the blocks of several runs (the engine's batched stages), its place
// among its own run's blocks.
struct Blk {
  unsigned id, n;
};
__device__ __forceinline__ Blk grid_blk() { return Blk{blockIdx.x, gridDim.x}; }

__device__ __forceinline__ bool thread_cell(const Box &b, int &i, int &j, int &k, Blk bk = grid_blk()) {
  const unsigned nbx = (unsigned)(b.hi[0] - b.lo[0] + BX - 1) / BX;
  const unsigned nby = (unsigned)(b.hi[1] - b.lo[1] + BY - 1) / BY;
  const unsigned N = bk.n, h = bk.id;
  const unsigned nbz = N / (nbx * nby);
  const unsigned q = N / 8, r = N % 8, x = h % 8, s = h / 8;
  unsigned L = (x < r) ? x * (q + 1) + s : r * (q + 1) + (x - r) * q + s;
  const unsigned hq = nby / 8, hr = nby % 8;
  unsigned y0 = 0, hb = hq + (hr > 0);
  for (unsigned bb = 0; bb < 8; ++bb) {
    hb = hq + (bb < hr ? 1u : 0u);
    unsigned nt = nbx * hb * nbz;
    if (L < nt || bb == 7) break;
    L -= nt;
    y0 += hb;
  }
  const unsigned bx = L % nbx, t = L / nbx;
  const unsigned by = y0 + t % hb, bz = t / hb;
  i = b.lo[0] + (int)(bx * BX + threadIdx.x);
  j = b.lo[1] + (int)(by * BY + threadIdx.y);
  k = b.lo[2] + (int)bz;
  return i < b.hi[0] && j < b.hi[1];
}

// Flat tiles, for the box kernels whose lanes do not exchange values along x
// (and for the level-0 pair kernels, whose lanes check for it): the (x, row)
// entries of a plane are numbered row by row and each wave takes 64
// consecutive ones, so that rows whose length is not a multiple of 64 share
// waves (a row of 64 entries is one wave, and the tiles are those of
// thread_cell); blocks of four waves go to the XCDs in bands through all
// planes as there.  A lane's previous lane then holds the previous entry of
// its row unless the lane is the first of its wave or its entry the first of
// its row.  With WS = BX - 1 entries per wave, the waves overlap by one entry:
// the last lane holds the entry after the wave's own (the next wave's first).
template <int WS = BX>
inline dim3 grid_of_flat(const Box &b) {
  const long ex = b.hi[0] - b.lo[0], ey = b.hi[1] - b.lo[1], ez = b.hi[2] - b.lo[2];
  if (ex <= 0 || ey <= 0 || ez <= 0) return dim3(0, 1, 1);
  return dim3((unsigned)((ex * ey + WS * BY - 1) / (WS * BY) * ez), 1, 1);
}

template <int WS = BX>
__device__ __forceinline__ bool thread_cell_flat(const Box &b, int &i, int &j, int &k, Blk bk = grid_blk()) {
  const unsigned ex = (unsigned)(b.hi[0] - b.lo[0]), ey = (unsigned)(b.hi[1] - b.lo[1]);
  const unsigned nby = (ex * ey + WS * BY - 1) / (WS * BY);  // blocks per plane
  const unsigned N = bk.n, h = bk.id;
  const unsigned nbz = N / nby;
  const unsigned q = N / 8, r = N % 8, x = h % 8, s = h / 8;
  unsigned L = (x < r) ? x * (q + 1) + s : r * (q + 1) + (x - r) * q + s;
  const unsigned hq = nby / 8, hr = nby % 8;
  unsigned y0 = 0, hb = hq + (hr > 0);
  for (unsigned bb = 0; bb < 8; ++bb) {
    hb = hq + (bb < hr ? 1u : 0u);
    unsigned nt = hb * nbz;
    if (L < nt || bb == 7) break;
    L -= nt;
    y0 += hb;
  }
  const unsigned by = y0 + L % hb, bz = L / hb;
  const unsigned f = by * (WS * BY) + threadIdx.y * WS + threadIdx.x;
  i = b.lo[0] + (int)(f % ex);
  j = b.lo[1] + (int)(f / ex);
  k = b.lo[2] + (int)bz;
  return f < ex * ey;
}

// Element indices are 32-bit (a field holds fewer than 2^31 entries and at most
// 4 GiB, checked when a mesh is created): with a uniform 64-bit base in scalar registers the
// loads and stores then take a 32-bit per-lane offset, with no 64-bit address
// arithmetic per lane.
using idx_t = int;

__device__ __forceinline__ idx_t lin(const Geo &G, int i, int j, int k) {
  return (idx_t)G.off + i + j * (idx_t)G.sy + k * (idx_t)G.sz;
}

__device__ __forceinline__ idx_t dstride(const Geo &G, int d) {
  return d == 0 ? 1 : (d == 1 ? (idx_t)G.sy : (idx_t)G.sz);
}

// Load and store at a non-negative element index whose byte offset fits 32
// bits (no field exceeds 4 GiB): the address is a uniform base plus
// an unsigned 32-bit lane offset, which the hardware adds itself.
template <typename T>
__device__ __forceinline__ T gld(const T *p, idx_t i) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) +
                                      (unsigned)i * (unsigned)sizeof(T));
}

template <typename T>
__device__ __forceinline__ void gst(T *p, idx_t i, T v) {
  *reinterpret_cast<T *>(reinterpret_cast<char *>(p) + (unsigned)i * (unsigned)sizeof(T)) = v;
}

// W adjacent cells of a row in one lane: T itself, or a two-element vector
// whose loads and stores are single 8- or 16-byte accesses (the first cell's
// index is even and rows start 128-byte aligned)
template <typename T, int W>
struct lanes_of {
  using type = T;
};
template <>
struct lanes_of<double, 2> {
  using type = double __attribute__((ext_vector_type(2)));
};
template <>
struct lanes_of<float, 2> {
  using type = float __attribute__((ext_vector_type(2)));
};

// a * b + c with one rounding, per element of a lane vector
template <typename V>
__device__ __forceinline__ V fmav(V a, V b, V c) {
  return __builtin_elementwise_fma(a, b, c);
}

template <typename V, typename T>
__device__ __forceinline__ V gldv(const T *p, idx_t i) {
  return *reinterpret_cast<const V *>(reinterpret_cast<const char *>(p) + (unsigned)i * (unsigned)sizeof(T));
}
template <typename V, typename T>
__device__ __forceinline__ void gstv(T *p, idx_t i, V v) {
  *reinterpret_cast<V *>(reinterpret_cast<char *>(p) + (unsigned)i * (unsigned)sizeof(T)) = v;
}

// Loads and stores through a buffer descriptor, for accesses that a few lanes of
// a wave make: a lane whose byte offset lies past the buffer's end (BUF_NONE and
// a little more) reads zero and stores nothing, so the others' accesses need no
// branch.  Buffers are smaller than 3 GiB (the frontier's: 16 faces of at most
// 4096^2 values, 2 GiB).
constexpr unsigned BUF_NONE = 0xC0000000u;
using Buf = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Buf make_buf(const void *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ void buf_load(Buf b, unsigned off, unsigned soff, float &v) {
  v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, off, soff, 0));
}
__device__ __forceinline__ void buf_load(Buf b, unsigned off, unsigned soff, double &v) {
  v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, off, soff, 0));
}
__device__ __forceinline__ void buf_store(Buf b, unsigned off, unsigned soff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, off, soff, 0);
}
__device__ __forceinline__ void buf_store(Buf b, unsigned off, unsigned soff, double v) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), b, off, soff, 0);
}

// W per-cell values of a lane as its lanes_of vector
template <typename V, typename T, int W>
__device__ __forceinline__ V to_lanes(const T (&a)[W]) {
  if constexpr (W == 1) {
    return a[0];
  } else {
    V v;
    v.x = a[0];
    v.y = a[1];
    return v;
  }
}

template <typename V, typename T, int W>
__device__ __forceinline__ void from_lanes(V v, T (&a)[W]) {
  if constexpr (W == 1) {
    a[0] = v;
  } else {
    a[0] = v.x;
    a[1] = v.y;
  }
}

// cell-centre coordinate: the perturber is the central vertex of the level
template <typename T>
__device__ __forceinline__ T xcen(const Geo &G, int d, int i) {
  return (T)(((double)i - G.org[d] + 0.5) * G.dx);
}

// Quotient and square root in the storage type, from the hardware reciprocal
// and reciprocal square root instead of the correctly rounded expansions: in
// FP64 the hardware reciprocal (relative error up to 4.6e-8, measured on
// gfx950) takes one Newton step and the quotient is the dividend times it
// (within 2.2e-15 of the quotient, measured over 4 M divisors; a second step
// would reach about an ulp), the square root one Goldschmidt step and one
// residual correction (within an ulp); in FP32 both are the single hardware
// instructions (about 1 ulp each).  Every use has a normal
// positive operand or divisor (densities and energies near their background,
// squared distances of at least a quarter cell, sums of two slopes of one
// sign; a van Leer quotient of slopes of opposite signs is selected away).
__device__ __forceinline__ double qdiv(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(r, fma(-b, r, 1.0), r);
  return a * r;
}
__device__ __forceinline__ float qdiv(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
template <typename V>
__device__ __forceinline__ V qdiv(V a, V b) {
  return V{qdiv(a.x, b.x), qdiv(a.y, b.y)};  // two-element vectors, per element
}
__device__ __forceinline__ double qsqrt(double x) {
  // hardware reciprocal square root, one of Goldschmidt's steps towards
  // g = sqrt(x), h = 1/(2 sqrt(x)), one residual correction (within an ulp,
  // as with two steps: measured over 4 M arguments on gfx950)
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  return fma(fma(-g, g, x), h, g);
}
__device__ __forceinline__ float qsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
template <typename V>
__device__ __forceinline__ V qsqrtv(V x) {
  V r;
  r.x = qsqrt(x.x);  // two-element vectors, per element
  r.y = qsqrt(x.y);
  return r;
}

// van Leer's harmonic limited difference; evaluated without a branch (the
// quotient of the discarded side is selected away)
template <typename T>
__device__ __forceinline__ T vleer(T a, T b) {
  const T p = a * b;
  const T r = qdiv(T(2) * p, a + b);
  return p > T(0) ? r : T(0);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// mirror image of a ghost index across the low (idx < 0) or high (idx >= n) side
__device__ __forceinline__ int mirror_idx(int idx, int n) {
  return idx < 0 ? -1 - idx : (idx >= n ? 2 * n - 1 - idx : idx);
}

// Level-0 read of a centred departure with the outer boundary conditions
// (M: the level's bc).  bc 1: zero departure (the inflow state) beyond x_max, the nearest active
// cell elsewhere (zero-gradient outflow).  bc 2: zero departure (the
// background) beyond both flow ends, mirror images across the walls.  (For
// momenta only the ones normal to x read ghosts here, which hold the
// background at the flow ends in both modes.)
template <int M, typename T>
__device__ __forceinline__ T cread(const T *q, const Geo &G, int i, int j, int k) {
  if (M == 2) {
    if (i < 0 || i >= G.n[0]) return T(0);
    return q[lin(G, i, mirror_idx(j, G.n[1]), mirror_idx(k, G.n[2]))];
  }
  if (i >= G.n[0]) return T(0);
  i = i < 0 ? 0 : i;
  j = clampi(j, 0, G.n[1] - 1);
  k = clampi(k, 0, G.n[2] - 1);
  return q[lin(G, i, j, k)];
}

// Level-0 read of the velocity departure normal to faces of dimension d
// (active faces 0..n along d; M: the level's bc).  bc 1: zero beyond x_max, copies elsewhere.
// bc 2: zero (the wind) beyond both flow ends for x faces, mirror images
// across the flow ends for the tangential ones; across a wall the normal
// velocity is reversed (zero on the wall) and the tangential ones mirrored.
template <int M, typename T>
__device__ __forceinline__ T fread_bc(const T *v, const Geo &G, int d, int i, int j, int k) {
  if (M == 2) {
    T sgn = T(1);
    if (d == 0) {
      if (i < 0 || i > G.n[0]) return T(0);
    } else {
      i = mirror_idx(i, G.n[0]);
    }
    int id[3] = {i, j, k};
#pragma unroll
    for (int e = 1; e < 3; ++e) {
      if (d == e) {
        if (id[e] < 0) { id[e] = -id[e]; sgn = -sgn; }
        else if (id[e] > G.n[e]) { id[e] = 2 * G.n[e] - id[e]; sgn = -sgn; }
      } else {
        id[e] = mirror_idx(id[e], G.n[e]);
      }
    }
    return sgn * v[lin(G, id[0], id[1], id[2])];
  }
  if (d == 0) {
    if (i > G.n[0]) return T(0);
  } else if (i >= G.n[0]) {
    return T(0);
  }
  i = i < 0 ? 0 : i;
  j = clampi(j, 0, G.n[1] - (d == 1 ? 0 : 1));
  k = clampi(k, 0, G.n[2] - (d == 2 ? 0 : 1));
  return v[lin(G, i, j, k)];
}

// background of the wind along dimension d and of the transported quantities
__device__ __forceinline__ double vback(const Phys &P, int d) { return d == 0 ? -P.V : 0.0; }
__device__ __forceinline__ double qback(const Phys &P, int m) {
  return m == 0 ? P.rho0 : (m == 1 ? P.e0 : ((m == 2 || m == 3) ? -P.rho0 * P.V : 0.0));
}
// background specific value q0 / rho0
__device__ __forceinline__ double sback(const Phys &P, int m) {
  return m == 1 ? P.e0 / P.rho0 : ((m == 2 || m == 3) ? -P.V : 0.0);
}

// Neighbour exchange inside a wave through the data-parallel-primitive lane
// shifts: from_left gives every lane the value of the lane below it, from_right
// that of the lane above it (the end lanes receive 0).
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}

template <int CTRL>
__device__ __forceinline__ float dpp_t(float v) {
  return __builtin_bit_cast(float, dpp_i<CTRL>(__builtin_bit_cast(int, v)));
}

template <int CTRL>
__device__ __forceinline__ double dpp_t(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = dpp_i<CTRL>((int)b), hi = dpp_i<CTRL>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

constexpr int DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138;

template <typename T>
__device__ __forceinline__ T from_left(T v) { return dpp_t<DPP_WAVE_SHR1>(v); }

template <typename T>
__device__ __forceinline__ T from_right(T v) { return dpp_t<DPP_WAVE_SHL1>(v); }

// ------------------------------------------------------------------ init

// SplitMix64 finaliser (Steele, Lea & Flood 2014); output n of the stream
// with seed s is mix(s + (n+1) * 0x9e3779b97f4a7c15).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
  return z ^ (z >> 31);
}

template <typename T>
struct InitArgs {
  Box b;
  T *rho, *e, *vx, *vy, *vz;
  uint64_t seed;
  double amp;
};

// uniform background (zero departures) plus the density noise of the active
// cells: rho = rho0 (1 + A (2U - 1))
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_init(Geo G, Phys P, InitArgs<T> A) {
  int i, j, k;
  if (!thread_cell(A.b, i, j, k)) return;
  idx_t c = lin(G, i, j, k);
  double dr = 0.0;
  bool active = i >= 0 && j >= 0 && k >= 0 && i < G.n[0] && j < G.n[1] && k < G.n[2];
  if (active && A.amp != 0.0) {
    uint64_t a = ((uint64_t)k * (uint64_t)G.n[1] + (uint64_t)j) * (uint64_t)G.n[0] + (uint64_t)i;
    uint64_t n = ((uint64_t)G.level << 40) + a;
    uint64_t z = mix64(A.seed + (n + 1ULL) * 0x9e3779b97f4a7c15ULL);
    double U = (double)(z >> 11) * 0x1.0p-53;
    dr = P.rho0 * (A.amp * (2.0 * U - 1.0));
  }
  A.rho[c] = (T)dr;
  A.e[c] = T(0);
  A.vx[c] = T(0);
  A.vy[c] = T(0);
  A.vz[c] = T(0);
}

// ------------------------------------------------------------------ kick

template <typename T>
struct KickArgs {
  Box b;                     // union of the three face ranges
  int flo[3][3], fhi[3][3];  // [normal dir][dim] face ranges
  const T *q[NQ];            // rho, e (and the momenta when rebuilding)
  T *v[3];                   // face velocities written
  const T *vin[3];           // face velocities read (v itself, or the set a fused kick reads from)
  const double *dtp;
  double fac;
  Scal *slots;               // non-null: the step length from slots->smax (single-level runs)
  // with the compression fused (level 0): the compressed energy departures
  // (a buffer other than q[1], which every thread reads for the kick), the
  // compression's share of the step length, and the force log of the last
  // step's state (non-null log: the first block logs it, as k_compress2 does)
  T *eo;
  double cfac;
  Scal *log;
  const double *part;
  int npart;
  double *flog;
  int twice;                 // a fused finish applies the kick again (the next sub-step's first)
};

// Velocity source S(h) (eq. 15): each face velocity receives
// -h [ (gamma-1)(e_c - e_m) / (dx rho_face) + (Phi_c - Phi_m) / dx ],
// with Phi = -GM / sqrt(r^2 + eps^2) (eq. 16).  Since only the coordinate
// along the face normal differs between the two cells,
// (Phi_c - Phi_m)/dx = GM (x_c + x_m) / (d_c d_m (d_c + d_m)).
// REBUILD first sets the face velocity from the transported momenta,
// (P+_m + P-_c) / (rho_m + rho_c).  KICK = false skips the source.
template <typename T, bool REBUILD, bool KICK>
__global__ void __launch_bounds__(BX * BY) k_kick(Geo G, Phys P, KickArgs<T> A) {
  int i, j, k;
  if (!thread_cell_flat(A.b, i, j, k)) return;
  bool need = false;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    need |= i >= A.flo[d][0] && i < A.fhi[d][0] && j >= A.flo[d][1] && j < A.fhi[d][1] &&
            k >= A.flo[d][2] && k < A.fhi[d][2];
  const idx_t c = lin(G, i, j, k);
  // z faces kicked into another set: those outside their range go with them
  if (!REBUILD && A.v[2] != A.vin[2] &&
      !(i >= A.flo[2][0] && i < A.fhi[2][0] && j >= A.flo[2][1] && j < A.fhi[2][1] && k >= A.flo[2][2] &&
        k < A.fhi[2][2]))
    A.v[2][c] = A.vin[2][c];
  if (!need) return;
  const T h = (T)(A.fac * A.dtp[0]);
  const T rho0 = (T)P.rho0, gm1 = (T)P.gm1, GM = (T)P.GM, eps2 = (T)P.eps2, dx = (T)G.dx;
  const T *rho = A.q[0], *e = A.q[1];
  const T drc = rho[c], dec = e[c];
  const T xc[3] = {xcen<T>(G, 0, i), xcen<T>(G, 1, j), xcen<T>(G, 2, k)};
  const T r2c = xc[0] * xc[0] + xc[1] * xc[1] + xc[2] * xc[2] + eps2;
  const T dcen = qsqrt(r2c);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    bool in = i >= A.flo[d][0] && i < A.fhi[d][0] && j >= A.flo[d][1] && j < A.fhi[d][1] &&
              k >= A.flo[d][2] && k < A.fhi[d][2];
    if (!in) continue;
    const int im = i - (d == 0), jm = j - (d == 1), km = k - (d == 2);
    const idx_t m = c - dstride(G, d);
    const T drm = rho[m], dem = e[m];
    T vf;
    if (REBUILD) {
      const T *pm = A.q[2 + 2 * d], *pp = A.q[3 + 2 * d];
      const T ppm = pp[m], pmc = pm[c];
      const T vb = (T)vback(P, d);
      vf = qdiv(ppm + pmc - vb * (drm + drc), T(2) * rho0 + drm + drc);
    } else {
      vf = A.vin[d][c];
    }
    if (KICK) {
      const T rface = rho0 + T(0.5) * (drm + drc);
      const T gradp = qdiv(gm1 * (dec - dem), dx * rface);
      const T xm = xc[d] - dx;
      const T dm = qsqrt(r2c - xc[d] * xc[d] + xm * xm);
      const T gradphi = qdiv(GM * (xc[d] + xm), dm * dcen * (dm + dcen));
      vf = vf - h * (gradp + gradphi);
    }
    A.v[d][c] = vf;
  }
}

// The first kick and the compression of a finer level in one launch, two
// adjacent cells per thread as on level 0 (ub's x range counts pairs): a pair
// of the kick's union box kicks its low faces that lie in their ranges into
// A.v, reading the faces from A.vin, and compresses those of its cells that
// lie in the compression box cb into A.eo, from the six kicked faces around
// them.  The waves take 63 pairs of the box's flat numbering each and their
// last lane the pair after them, so that the high x face of a pair is the low
// face its next lane kicked (a cell of cb is never in the last face of its
// row); the high y and z faces the pair kicks again, by the expression of the
// cells above, with every distance formed from the cells' own coordinates (the
// same value).  A face of the union box outside its range is copied unkicked
// (what the separate kick leaves there).  Bound by memory: at 128^3 cells and
// their shell 59 us in FP64, where the kick and the compression apart took 48
// and 19, and 32 us in FP32, 35 with one cell per thread.
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_kick_compress_fine(Geo G, Phys P, KickArgs<T> A, Box cb, Box ub) {
#pragma clang fp contract(off)
  using V = typename lanes_of<T, 2>::type;
  int p, j, k;
  // no lane leaves before the exchange along x: a lane past the box takes
  // the box's first pair and writes nothing
  const bool inb = thread_cell_flat<BX - 1>(ub, p, j, k);
  const bool own = inb && threadIdx.x < BX - 1;
  if (!inb) {
    p = ub.lo[0];
    j = ub.lo[1];
    k = ub.lo[2];
  }
  const int i = 2 * p;
  const T h = (T)(A.fac * A.dtp[0]);
  const T rho0 = (T)P.rho0, gm1 = (T)P.gm1, GM = (T)P.GM, eps2 = (T)P.eps2, dx = (T)G.dx;
  const T *rho = A.q[0], *e = A.q[1];
  const idx_t c = lin(G, i, j, k);
  const int id[3] = {i, j, k};
  // bits: the pair's faces normal to d, at (jj, kk), that lie in their range
  auto in_range = [&](int d, int jj, int kk) -> int {
    if (jj < A.flo[d][1] || jj >= A.fhi[d][1] || kk < A.flo[d][2] || kk >= A.fhi[d][2]) return 0;
    return (i >= A.flo[d][0] && i < A.fhi[d][0] ? 1 : 0) + (i + 1 >= A.flo[d][0] && i + 1 < A.fhi[d][0] ? 2 : 0);
  };
  auto pick = [&](int m, V in, V out) -> V {
    out.x = m & 1 ? in.x : out.x;
    out.y = m & 2 ? in.y : out.y;
    return out;
  };
  V xcx;
  xcx.x = xcen<T>(G, 0, i);
  xcx.y = xcen<T>(G, 0, i + 1);
  const T xc[3] = {T(0), xcen<T>(G, 1, j), xcen<T>(G, 2, k)};
  auto dist = [&](V x, T y, T z) -> V { return qsqrtv(fmav<V>(x, x, V(fmav<T>(y, y, fmav<T>(z, z, eps2))))); };
  // the faces between cells m (below) and u (above) along d
  auto kicked = [&](V vf, V drm, V dem, V dru, V deu, V xm, V xu, V dm, V du) -> V {
    const V rface = fmav<V>(V(T(0.5)), drm + dru, V(rho0));
    const V gradp = qdiv(gm1 * (deu - dem), dx * rface);
    const V gradphi = qdiv(GM * (xu + xm), dm * du * (dm + du));
    return fmav<V>(V(-h), gradp + gradphi, vf);
  };
  const V drc = gldv<V>(rho, c), dec = gldv<V>(e, c);
  const V dcen = dist(xcx, xc[1], xc[2]);
  const T dprev = from_left(dcen.y);
  V vlo[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    vlo[d] = gldv<V>(A.vin[d], c);
    const int m = inb ? in_range(d, j, k) : 0;
    if (m) {
      V drm, dem, xm, xu, dm;
      if (d == 0) {
        xu = xcx;
        xm.x = xcen<T>(G, 0, i - 1);
        xm.y = xcx.x;
        drm.x = m & 1 ? rho[c - 1] : drc.x;
        dem.x = m & 1 ? e[c - 1] : dec.x;
        drm.y = drc.x;
        dem.y = dec.x;
        dm.y = dcen.x;
        // (the lane before holds the pair before, but for a row's first)
        if (threadIdx.x > 0 && p > ub.lo[0]) dm.x = dprev;
        else dm.x = dist(V(xm.x), xc[1], xc[2]).x;
      } else {
        const idx_t s = dstride(G, d);
        const T xd = xcen<T>(G, d, id[d] - 1);
        xu = V(xc[d]);
        xm = V(xd);
        drm = gldv<V>(rho, c - s);
        dem = gldv<V>(e, c - s);
        dm = d == 1 ? dist(xcx, xd, xc[2]) : dist(xcx, xc[1], xd);
      }
      vlo[d] = pick(m, kicked(vlo[d], drm, dem, drc, dec, xm, xu, dm, dcen), vlo[d]);
    }
    if (own) gstv<V>(A.v[d], c, vlo[d]);
  }
  V vhx;
  vhx.x = vlo[0].y;
  vhx.y = from_right(vlo[0].x);
  int m = 0;
  if (own && j >= cb.lo[1] && j < cb.hi[1] && k >= cb.lo[2] && k < cb.hi[2])
    m = (i >= cb.lo[0] && i < cb.hi[0] ? 1 : 0) + (i + 1 >= cb.lo[0] && i + 1 < cb.hi[0] ? 2 : 0);
  if (m) {
    V divv = T(0) + (vhx - vlo[0]);
#pragma unroll
    for (int d = 1; d < 3; ++d) {
      const idx_t s = dstride(G, d);
      V vhi = gldv<V>(A.vin[d], c + s);
      const int mh = in_range(d, id[1] + (d == 1), id[2] + (d == 2));
      if (mh) {
        const T xu = xcen<T>(G, d, id[d] + 1);
        const V du = d == 1 ? dist(xcx, xu, xc[2]) : dist(xcx, xc[1], xu);
        vhi = pick(mh, kicked(vhi, drc, dec, gldv<V>(rho, c + s), gldv<V>(e, c + s), V(xc[d]), V(xu), dcen, du), vhi);
      }
      divv += vhi - vlo[d];
    }
    const T dt = (T)(A.cfac * A.dtp[0]);
    const V a = T(0.5) * (T)P.gm1 * dt * qdiv(divv, V(dx));
    const V out = qdiv(fmav<V>(dec, T(1) - a, -(T(2) * a * (T)P.e0)), T(1) + a);
    if (m == 3) gstv<V>(A.eo, c, out);
    else if (m == 1) A.eo[c] = out.x;
    else A.eo[c + 1] = out.y;
  }
}

// ------------------------------------------------- artificial viscosity

template <typename T>
struct LevFaces {
  T *v[3];
};
template <typename T>
struct ViscArgs {
  int lo[3], hi[3];          // union of the ranges below
  int elo[3], ehi[3];        // cells whose energy changes
  int flo[3][3], fhi[3][3];  // [normal dir][dim] faces that change
  const T *rho;
  T *e;
  const T *v[3];
  T *vn[3];                  // new face velocities
  const double *dtp;
  double fac;
};

// Von Neumann-Richtmyer viscosity of ZEUS (Stone & Norman 1992) as the
// SubStep2 that the staging list of Sect. 3.3 names: per dimension d and cell
// c, dv = v_d(high face) - v_d(low face) and q_d = C2 rho dv^2 where dv < 0,
// else 0; e -= dt sum_d q_d dv / dx; v_d(face) -= dt (q_d(c) - q_d(c-1)) /
// (dx rho_face).  All from the values before the stage: the new velocities go
// to vn.  On level 0 the boundary faces (the injection face, walls under bc 2)
// keep their values, and cells and faces past the boundary read its ghosts.
template <typename T, int BC>
__global__ void __launch_bounds__(BX * BY) k_visc(Geo G, Phys P, ViscArgs<T> A) {
  int id[3];
  if (!thread_cell_flat(Box{{A.lo[0], A.lo[1], A.lo[2]}, {A.hi[0], A.hi[1], A.hi[2]}}, id[0], id[1], id[2])) return;
  const T dt = (T)(A.fac * A.dtp[0]);
  const T c2 = (T)P.visc, rho0 = (T)P.rho0, dx = (T)G.dx;
  auto rho_at = [&](int i, int j, int k) -> T { return BC ? cread<BC>(A.rho, G, i, j, k) : A.rho[lin(G, i, j, k)]; };
  auto v_at = [&](int d, int i, int j, int k) -> T {
    return BC ? fread_bc<BC>(A.v[d], G, d, i, j, k) : A.v[d][lin(G, i, j, k)];
  };
  // q_d and dv_d of the cell at p
  auto qd = [&](int d, const int *p, T &dv) -> T {
    const T lo = v_at(d, p[0], p[1], p[2]);
    const T hi = v_at(d, p[0] + (d == 0), p[1] + (d == 1), p[2] + (d == 2));
    dv = hi - lo;
    return dv < T(0) ? c2 * (rho0 + rho_at(p[0], p[1], p[2])) * dv * dv : T(0);
  };
  const idx_t c = lin(G, id[0], id[1], id[2]);
  bool ecell = true;
#pragma unroll
  for (int e = 0; e < 3; ++e) ecell = ecell && id[e] >= A.elo[e] && id[e] < A.ehi[e];
  if (ecell) {
    T de = T(0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      T dv;
      const T q = qd(d, id, dv);
      de += q * dv;
    }
    A.e[c] = A.e[c] - qdiv(dt * de, dx);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    bool in = true;
#pragma unroll
    for (int e = 0; e < 3; ++e) in = in && id[e] >= A.flo[d][e] && id[e] < A.fhi[d][e];
    if (!in) continue;
    const T vold = A.v[d][c];
    T vnew = vold;
    const bool fixed = BC && ((d == 0 && id[0] == G.n[0]) ||
                              (BC == 2 && d > 0 && (id[d] == 0 || id[d] == G.n[d])));
    if (!fixed) {
      int m[3] = {id[0] - (d == 0), id[1] - (d == 1), id[2] - (d == 2)};
      T dvc, dvm;
      const T qc = qd(d, id, dvc), qm = qd(d, m, dvm);
      const T rface = rho0 + T(0.5) * (rho_at(m[0], m[1], m[2]) + rho_at(id[0], id[1], id[2]));
      vnew = vold - qdiv(dt * (qc - qm), dx * rface);
    }
    A.vn[d][c] = vnew;
  }
}

// The new face velocities to their place, the three directions in one launch
// (two levels of 64^3: three launches of 4.7 us per level step -> one of 6.6).
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_copy_faces(Geo G, ViscArgs<T> A, LevFaces<T> out) {
  int id[3];
  if (!thread_cell_flat(Box{{A.lo[0], A.lo[1], A.lo[2]}, {A.hi[0], A.hi[1], A.hi[2]}}, id[0], id[1], id[2])) return;
  const idx_t c = lin(G, id[0], id[1], id[2]);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    bool in = true;
#pragma unroll
    for (int e = 0; e < 3; ++e) in = in && id[e] >= A.flo[d][e] && id[e] < A.fhi[d][e];
    if (in) out.v[d][c] = A.vn[d][c];
  }
}

// ------------------------------------------------------------ compression

template <typename T>
struct CellArgs {
  Box b;
  T *e;
  const T *v[3];
  const double *dtp;
  double fac;
  Scal *log;                 // non-null: clear log->smax and log a pending force (first block)
  const double *part;        // the force partials: three planes of npart values
  int npart;
  double *flog;
};

// Compressional heating (SubStep3): e <- e (1 - a) / (1 + a),
// a = (gamma - 1) dt div(v) / 2; for the departure de = e - e0:
// de <- (de (1 - a) - 2 a e0) / (1 + a).
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_compress(Geo G, Phys P, CellArgs<T> A) {
  int i, j, k;
  if (!thread_cell_flat(A.b, i, j, k)) return;
  const T dt = (T)(A.fac * A.dtp[0]);
  const idx_t c = lin(G, i, j, k);
  const T divv = qdiv((A.v[0][c + 1] - A.v[0][c]) + (A.v[1][c + G.sy] - A.v[1][c]) +
                           (A.v[2][c + G.sz] - A.v[2][c]),
                       (T)G.dx);
  const T a = T(0.5) * (T)P.gm1 * dt * divv;
  const T de = A.e[c];
  A.e[c] = qdiv(de * (T(1) - a) - T(2) * a * (T)P.e0, T(1) + a);
}

template <int NT>
__device__ void log_pending_body(const double *part, int n, Scal *S, double *flog);

// The same on level 0 with two adjacent cells per lane (even row length; the
// box's x range counts pairs): every field moves as one 8- or 16-byte access.
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_compress2(Geo G, Phys P, CellArgs<T> A) {
  using V = typename lanes_of<T, 2>::type;
  int p, j, k;
  if (thread_cell_flat(A.b, p, j, k)) {
    const T dt = (T)(A.fac * A.dtp[0]);
    const idx_t c = lin(G, 2 * p, j, k);
    const V vx0 = gldv<V>(A.v[0], c);
    V vx1;
    vx1.x = vx0.y;
    vx1.y = gld(A.v[0], c + 2);
    const V divv = qdiv((vx1 - vx0) + (gldv<V>(A.v[1], c + (idx_t)G.sy) - gldv<V>(A.v[1], c)) +
                            (gldv<V>(A.v[2], c + (idx_t)G.sz) - gldv<V>(A.v[2], c)),
                        V((T)G.dx));
    const V a = T(0.5) * (T)P.gm1 * dt * divv;
    const V de = gldv<V>(A.e, c);
    gstv<V>(A.e, c, qdiv(de * (T(1) - a) - T(2) * a * (T)P.e0, T(1) + a));
  }
  if (A.log && blockIdx.x == 0) {
    // the kick of this step has read the slots: clear them for this step's
    // end-of-step pass, and log the force of the last step's state
    for (int q = threadIdx.y * BX + threadIdx.x; q < NSLOT; q += BX * BY) A.log->smax[q] = 0ull;
    log_pending_body<BX * BY>(A.part, A.npart, A.log, A.flog);
  }
}

// ---------------------------------------------------- diffusion + heat

template <typename T>
struct DiffArgs {
  Box b;
  const T *rho, *e;
  T *eo;
  const double *hw;
  int hw_n[3], hw_lo[3];  // weight box extent and its first active index per dimension
  const double *dtp;
  double fac;
  int do_diff, do_heat;
  Scal *clear;  // non-null (level 0 after a fused kick and compression): the first block clears clear->smax
};

// departure of e/rho from e0/rho0
template <typename T>
__device__ __forceinline__ T dtemp(T dr, T de, T rho0, T e0) {
  return qdiv(rho0 * de - e0 * dr, rho0 * (rho0 + dr));
}

// Thermal diffusion (eqs. 19-22, energy flux down the gradient of e/rho with
// coefficient chi rho0) and heat release L dt w_c / dx^3 (Sect. 3.4), on a
// finer level (its ghost shell holds every neighbour).
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_diffuse_heat(Geo G, Phys P, DiffArgs<T> A) {
  int i, j, k;
  if (!thread_cell_flat(A.b, i, j, k)) return;
  const T dt = (T)(A.fac * A.dtp[0]);
  const T rho0 = (T)P.rho0, e0 = (T)P.e0;
  const idx_t c = lin(G, i, j, k);
  const T dec = A.e[c];
  T en = dec;
  if (A.do_diff) {
    const T Tc = dtemp(A.rho[c], dec, rho0, e0);
    T lap = T(0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const idx_t s = dstride(G, d);
      const T Tm = dtemp(A.rho[c - s], A.e[c - s], rho0, e0);
      const T Tp = dtemp(A.rho[c + s], A.e[c + s], rho0, e0);
      lap += (Tp - Tc) - (Tc - Tm);
    }
    en = dec + qdiv(dt * (T)(P.chi * P.rho0) * lap, (T)(G.dx * G.dx));
  }
  if (A.do_heat && A.hw_n[0] > 0) {
    // quadrant: the entries beyond a mirror plane are the images of the
    // level's cells and are heated as their cells are
    const int jj = (G.anch[1] && j < 0) ? -1 - j : j, kk = (G.anch[2] && k < 0) ? -1 - k : k;
    const int a = i - A.hw_lo[0], b = jj - A.hw_lo[1], d = kk - A.hw_lo[2];
    if (a >= 0 && b >= 0 && d >= 0 && a < A.hw_n[0] && b < A.hw_n[1] && d < A.hw_n[2] && i >= 0 && jj >= 0 &&
        kk >= 0 && i < G.n[0] && jj < G.n[1] && kk < G.n[2]) {
      const double w = A.hw[((long)d * A.hw_n[1] + b) * A.hw_n[0] + a];
      if (w != 0.0) en += (T)(P.L * (A.fac * A.dtp[0]) * w / (G.dx * G.dx * G.dx));
    }
  }
  A.eo[c] = en;
}

// The same on level 0, whose boundary conditions it applies on read, with two
// adjacent cells per lane (level-0 rows have an even length; the box's x
// range counts pairs): the pair's own fields and its y and z neighbours move
// as 8- or 16-byte accesses, the x neighbours of the pair are the other cell
// of the pair and one cell on each side.
template <typename T, int BC>
__device__ __forceinline__ void diffuse_heat2_body(Geo G, Phys P, DiffArgs<T> A, Blk bk) {
  using V = typename lanes_of<T, 2>::type;
  int p, j, k;
  const bool ok = thread_cell_flat(A.b, p, j, k, bk);
  if (A.clear && bk.id == 0) {
    // the kick of this step has read the slots: clear them for this step's
    // end-of-step pass
    for (int q = threadIdx.y * BX + threadIdx.x; q < NSLOT; q += BX * BY) A.clear->smax[q] = 0ull;
  }
  if (!ok) return;
  const int i = 2 * p;
  const T dt = (T)(A.fac * A.dtp[0]);
  const T rho0 = (T)P.rho0, e0 = (T)P.e0;
  const idx_t c = lin(G, i, j, k);
  const V de = gldv<V>(A.e, c);
  V en = de;
  if (A.do_diff) {
    auto tv = [&](V r, V e) -> V { return qdiv(rho0 * e - e0 * r, rho0 * (rho0 + r)); };
    const V Tc = tv(gldv<V>(A.rho, c), de);
    // x: past x_max (and past x_min under bc 2) the background, else the
    // nearest active cell (as k_diffuse_heat)
    V Tl, Tr;
    Tl.y = Tc.x;
    Tr.x = Tc.y;
    if (BC == 2 && i == 0) {
      Tl.x = T(0);
    } else {
      const idx_t cm = i > 0 ? c - 1 : c;
      Tl.x = dtemp(gld(A.rho, cm), gld(A.e, cm), rho0, e0);
    }
    Tr.y = i + 1 == G.n[0] - 1 ? T(0) : dtemp(gld(A.rho, c + 2), gld(A.e, c + 2), rho0, e0);
    V lap = V(0);
    lap += (Tr - Tc) - (Tc - Tl);
#pragma unroll
    for (int d = 1; d < 3; ++d) {
      const int id = d == 1 ? j : k;
      const idx_t s = dstride(G, d);
      const idx_t cm = id > 0 ? c - s : c, cp = id < G.n[d] - 1 ? c + s : c;
      const V Tm = tv(gldv<V>(A.rho, cm), gldv<V>(A.e, cm)), Tp = tv(gldv<V>(A.rho, cp), gldv<V>(A.e, cp));
      lap += (Tp - Tc) - (Tc - Tm);
    }
    en = de + qdiv(dt * (T)(P.chi * P.rho0) * lap, V((T)(G.dx * G.dx)));
  }
  if (A.do_heat && A.hw_n[0] > 0) {
    const int b = j - A.hw_lo[1], d = k - A.hw_lo[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int a = i + q - A.hw_lo[0];
      if (a >= 0 && b >= 0 && d >= 0 && a < A.hw_n[0] && b < A.hw_n[1] && d < A.hw_n[2]) {
        const double w = A.hw[((long)d * A.hw_n[1] + b) * A.hw_n[0] + a];
        if (w != 0.0) en[q] += (T)(P.L * (A.fac * A.dtp[0]) * w / (G.dx * G.dx * G.dx));
      }
    }
  }
  gstv<V>(A.eo, c, en);
}

template <typename T, int BC>
__global__ void __launch_bounds__(BX * BY) k_diffuse_heat2(Geo G, Phys P, DiffArgs<T> A) {
  diffuse_heat2_body<T, BC>(G, P, A, grid_blk());
}

// -------------------------------------------------------------- transport

template <typename T>
struct PassArgs {
  Box b;
  const T *qi[NQ];
  T *qo[NQ];
  const T *v[3];     // face velocity departures after the first kick
  const double *dtp;
  double fac;
  T *acc;            // this sub-step's frontier transfers of this level (fine levels) or null
  long astr;         // entries per quantity of acc: the level's largest face
  const T *fsum;     // transfers through the finer level's frontier (k_front_sum) or null
  long fstr;         // faces per quantity of fsum
};

// Frontier transfers.  A finer level stores its own transfers through its outer
// faces, each sub-step into a set of its own: acc[(2 dir + side) NQ + m][face].
// Before the coarse level's passes k_front_sum forms the transfers that replace
// theirs: per coarse face the sum of the four fine faces', each over the
// sub-steps, so that the walks read one value per face.  (Summed in the walks,
// with a read, add and write of one set per sub-step, the frontier's code made
// the fused x + y pass 160 KB, more than the instruction cache holds.)
template <typename T>
struct FrontArgs {
  const T *a, *b;  // the finer level's transfers of its first and second sub-step (null: one)
  T *out;
  long in_str, out_str;
};

template <typename T>
__global__ void __launch_bounds__(256) k_front_sum(Geo Gc, Geo Gf, FrontArgs<T> A) {
  const int ds = blockIdx.y, m = blockIdx.z, dir = ds >> 1;
  const int t1 = dir == 0 ? 1 : 0, t2 = dir == 2 ? 1 : 2;
  const unsigned c1 = (unsigned)Gc.cn[t1], f = blockIdx.x * 256 + threadIdx.x;
  if (f >= c1 * (unsigned)Gc.cn[t2]) return;
  const long fn = Gf.n[t1];
  const long i = ((long)ds * NQ + m) * A.in_str + 2 * (long)(f / c1) * fn + 2 * (f % c1);
  T s0 = A.a[i], s1 = A.a[i + 1], s2 = A.a[i + fn], s3 = A.a[i + fn + 1];
  if (A.b) {
    s0 += A.b[i];
    s1 += A.b[i + 1];
    s2 += A.b[i + fn];
    s3 += A.b[i + fn + 1];
  }
  A.out[((long)ds * NQ + m) * A.out_str + f] = (s0 + s1) + (s2 + s3);
}

// Cell of the x pass at row (j, k) and x: false where level 0's boundary
// holds the background (beyond x_max; under bc 2 beyond both flow ends), else
// the cell to read (the nearest active one under bc 1).
template <int BC>
__device__ __forceinline__ bool xcell_at(const Geo &G, int x, int j, int k, idx_t &c) {
  if (BC) {
    if (x >= G.n[0] || (BC == 2 && x < 0)) return false;
    x = x < 0 ? 0 : x;
  }
  c = lin(G, x, j, k);
  return true;
}

// Wave-tiled form of the x pass.  A wave holds 64 consecutive cells of one
// row, of which lanes 2..61 own their cell (tiles overlap by 4 cells): every
// lane forms the specific value of its cell and the limited difference there
// once, takes its neighbours' through lane shifts, computes the transfer
// through its left face, and the owning lanes take the right face's transfer
// from the lane above.  Arithmetic and its order are those of k_pass.
constexpr int XT = 60;

__host__ __device__ inline Box xtile_box(const Box &b) {
  Box v = b;
  const int ex = b.hi[0] - b.lo[0];
  v.lo[0] = 0;
  v.hi[0] = ex > 0 ? ((ex + XT - 1) / XT) * BX : 0;
  return v;
}

template <typename T, int BC>
__global__ void __launch_bounds__(BX * BY) k_xpass(Geo G, Phys P, PassArgs<T> A) {
  int iv, j, k;
  if (!thread_cell(xtile_box(A.b), iv, j, k)) return;
  const int lane = threadIdx.x;
  const int x = A.b.lo[0] - 2 + (iv / BX) * XT + lane;
  // lanes past the last cell's neighbours read that neighbour (never used)
  const int xl = min(x, A.b.hi[0] + 1);
  const bool owner = lane >= 2 && lane < 2 + XT && x < A.b.hi[0];
  const T dt = (T)(A.fac * A.dtp[0]);
  const T dx = (T)G.dx;
  const T mfac = dt * dx * dx, ivol = T(1) / (dx * dx * dx);
  const T rho0 = (T)P.rho0;
  const T vb = (T)vback(P, 0);
  idx_t c;
  const bool in = xcell_at<BC>(G, xl, j, k, c);
  // momenta tangential to x beyond a flow end under bc 2: the mirror cell's
  idx_t ct = c;
  bool int_ = in;
  if (BC == 2 && !in) {
    ct = lin(G, mirror_idx(xl, G.n[0]), j, k);
    int_ = true;
  }
  const T dr = in ? gld(A.qi[0], c) : T(0);
  const T irr = qdiv(T(1), rho0 * (rho0 + dr));
  // velocity departure on the left face (faces lo..hi are the ones used)
  const T da = gld(A.v[0], lin(G, clampi(x, A.b.lo[0], A.b.hi[0]), j, k));
  const T a = vb + da, nu = a * (dt / dx);
  const T hl = T(0.5) * (T(1) - nu), hh = T(0.5) * (T(1) + nu);
  const T M0 = rho0 * vb * mfac;
  auto left_face = [&](T sv) -> T {
    const T sm = from_left(sv), sp = from_right(sv);
    const T d = vleer(sp - sv, sv - sm);
    const T dm = from_left(d);
    const T lo = sm + dm * hl, hi = sv - d * hh;
    return a > T(0) ? lo : hi;
  };
  const T dM = (rho0 * da + left_face(dr) * a) * mfac;
  const T M = M0 + dM;

  // flux matching on the frontier of the finer level (its 4 faces over its 2
  // sub-cycles replace this level's transfer) and this level's own frontier
  bool fine_face = false;
  int side = 0;
  long fbase = 0;
  if (A.fsum) {
    const int a1 = j - G.co[1], a2 = k - G.co[2];
    const int lo = G.co[0], hi = G.co[0] + G.cn[0];
    if (a1 >= 0 && a2 >= 0 && a1 < G.cn[1] && a2 < G.cn[2] && (x == lo || x == hi)) {
      fine_face = true;
      side = (x == hi);
      fbase = (long)a2 * G.cn[1] + a1;
    }
  }
  long acc_i = -1;
  int acc_side = -1;
  if (A.acc && owner && j >= 0 && k >= 0 && j < G.n[1] && k < G.n[2] &&
      (x == 0 || x == G.n[0] - 1)) {
    acc_i = (long)k * G.n[1] + j;
    acc_side = (x == 0) ? 0 : 1;
  }
  const idx_t co = lin(G, x, j, k);
  auto finish = [&](int m, T own, T FL) {
    if (fine_face) {
      FL = A.fsum[((long)side * NQ + m) * A.fstr + fbase];
    }
    const T FR = from_right(FL);
    if (acc_side >= 0) A.acc[((long)acc_side * NQ + m) * A.astr + acc_i] = acc_side ? FR : FL;
    if (owner) gst(A.qo[m], co, own - (FR - FL) * ivol);
  };
  finish(0, dr, dM);

#pragma unroll 1
  for (int m = 1; m < NQ; ++m) {
    T sv, own;
    if (m >= 2) {
      // momentum P = rho v of a face velocity: its specific value is v itself
      const int d = (m - 2) >> 1;
      const idx_t off = (m & 1) ? dstride(G, d) : 0;
      if (d == 0) sv = in ? gld(A.v[d], c + off) : T(0);
      else sv = int_ ? gld(A.v[d], ct + off) : T(0);
      own = rho0 * sv + dr * ((T)vback(P, d) + sv);
    } else {
      const T dq = in ? gld(A.qi[m], c) : T(0);
      sv = (rho0 * dq - (T)qback(P, m) * dr) * irr;
      own = dq;
    }
    finish(m, own, (T)sback(P, m) * dM + left_face(sv) * M);
  }
}

// Row form of the x pass for level 0 when a row has at most 64 R cells and R
// divides it: one wave holds a whole row, lane l the R consecutive cells
// R l .. R l + R - 1, so the neighbours of a cell are in its own lane or, at
// the lane's ends, in the adjacent lane (one lane shift per exchanged value
// for R cells).  The boundary conditions give what lies beyond the row: at
// x_min the outflow copy (the specific value of cell -1 is that of cell 0,
// the limited difference there is zero); at x_max, cells n, n+1 hold zero
// departures and the injection face carries no departure transfer.  Cells
// past n inside the wave are those ghost cells.  Arithmetic and its order are
// those of k_xpass.
__host__ __device__ inline Box xrow_box(const Box &b) {
  Box v = b;
  v.lo[0] = 0;
  v.hi[0] = (b.hi[0] > b.lo[0]) ? BX : 0;
  return v;
}

// lane shift with a fill value for the lane that has no source
template <int CTRL>
__device__ __forceinline__ float dpp_fill(float v, float fill) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, fill),
                                                               __builtin_bit_cast(int, v), CTRL, 0xf, 0xf,
                                                               false));
}

template <int CTRL>
__device__ __forceinline__ double dpp_fill(double v, double fill) {
  const long long b = __builtin_bit_cast(long long, v), f = __builtin_bit_cast(long long, fill);
  const int lo = __builtin_amdgcn_update_dpp((int)f, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(f >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// the value of the cell before each of the lane's R cells (fill for cell -1)
template <typename T, int R>
__device__ __forceinline__ void row_left(const T (&v)[R], T (&out)[R], T fill) {
  out[0] = dpp_fill<DPP_WAVE_SHR1>(v[R - 1], fill);
#pragma unroll
  for (int r = 1; r < R; ++r) out[r] = v[r - 1];
}

// the value of the cell after each of the lane's R cells (fill past the wave)
template <typename T, int R>
__device__ __forceinline__ void row_right(const T (&v)[R], T (&out)[R], T fill) {
#pragma unroll
  for (int r = 0; r + 1 < R; ++r) out[r] = v[r + 1];
  out[R - 1] = dpp_fill<DPP_WAVE_SHL1>(v[0], fill);
}

// R consecutive entries from an R-aligned index (R a power of two)
template <typename T, int R>
__device__ __forceinline__ void row_load(const T *p, idx_t c, T (&out)[R]) {
  typedef T vec __attribute__((ext_vector_type(R)));
  const vec w = *reinterpret_cast<const vec *>(reinterpret_cast<const char *>(p) +
                                                (unsigned)c * (unsigned)sizeof(T));
#pragma unroll
  for (int r = 0; r < R; ++r) out[r] = w[r];
}

// the same from any index
template <typename T, int R>
__device__ __forceinline__ void row_load_any(const T *p, idx_t c, T (&out)[R]) {
  typedef T vec __attribute__((ext_vector_type(R), aligned(sizeof(T))));
  const vec w = *reinterpret_cast<const vec *>(reinterpret_cast<const char *>(p) +
                                                (unsigned)c * (unsigned)sizeof(T));
#pragma unroll
  for (int r = 0; r < R; ++r) out[r] = w[r];
}

template <typename T, int R>
__device__ __forceinline__ void row_store(T *p, idx_t c, const T (&v)[R]) {
  typedef T vec __attribute__((ext_vector_type(R)));
  vec w;
#pragma unroll
  for (int r = 0; r < R; ++r) w[r] = v[r];
  *reinterpret_cast<vec *>(reinterpret_cast<char *>(p) + (unsigned)c * (unsigned)sizeof(T)) = w;
}

// x pass of one level-0 row held by one wave, R cells per lane (lane l owns
// cells R l .. R l + R - 1; lanes past the row end hold zero departures, the
// inflow state beyond x_max): from the row's density and left-face velocity
// departures (dr, da, set by the caller) the mass transfers through every left
// face, then per quantity its transfers and updated departures.
template <typename T, int R>
struct XRow {
  T dr[R], da[R];
  T dt, dx, rho0, ivol, mfac, M0, irr[R], a[R], hl[R], hh[R], dM[R], M[R];

  // face velocities and Courant numbers of the row
  __device__ __forceinline__ void flow(const Geo &G, const Phys &P, T dt_) {
#pragma clang fp contract(off)
    dt = dt_;
    dx = (T)G.dx;
    mfac = dt * dx * dx;
    const T cour = dt / dx;
    ivol = T(1) / (dx * dx * dx);
    rho0 = (T)P.rho0;
    const T vb = (T)vback(P, 0);
    M0 = rho0 * vb * mfac;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      a[r] = vb + da[r];
      const T nu = a[r] * cour;
      hl[r] = fmav<T>(T(-0.5), nu, T(0.5));  // (1 -+ nu)/2, exact halvings of the rounded 1 -+ nu
      hh[r] = fmav<T>(T(0.5), nu, T(0.5));
    }
  }
  // the mass transfers through the left faces (departures dm_)
  __device__ __forceinline__ void take_mass(const T (&dm_)[R]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      dM[r] = dm_[r];
      M[r] = M0 + dM[r];
    }
  }
  template <bool BG = false>
  __device__ __forceinline__ void mass() {
#pragma clang fp contract(off)
    T fv[R], dm_[R];
    left_faces<BG>(dr, fv);
#pragma unroll
    for (int r = 0; r < R; ++r) dm_[r] = fmav<T>(fv[r], a[r], rho0 * da[r]) * mfac;
    take_mass(dm_);
  }
  __device__ __forceinline__ void recip() {
#pragma clang fp contract(off)
#pragma unroll
    for (int r = 0; r < R; ++r) irr[r] = qdiv(T(1), rho0 * (rho0 + dr[r]));
  }
  __device__ __forceinline__ void begin(const Geo &G, const Phys &P, T dt_) {
    flow(G, P, dt_);
    recip();
    mass();
  }
  // left-face value of the upwind van Leer reconstruction of s, per cell (BG:
  // the background before the row's first cell, else a copy of that cell)
  template <bool BG = false>
  __device__ __forceinline__ void left_faces(const T (&sv)[R], T (&fv)[R]) const {
#pragma clang fp contract(off)
    T sl[R], sr[R], d[R], dl[R];
    row_left<T, R>(sv, sl, BG ? T(0) : sv[0]);
    row_right<T, R>(sv, sr, T(0));
#pragma unroll
    for (int r = 0; r < R; ++r) d[r] = vleer(sr[r] - sv[r], sv[r] - sl[r]);
    row_left<T, R>(d, dl, T(0));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // both upwind values, then a select (a branch per face costs more)
      const T lo = fmav<T>(dl[r], hl[r], sl[r]), hi = fmav<T>(-d[r], hh[r], sv[r]);
      fv[r] = a[r] > T(0) ? lo : hi;
    }
  }
  // specific value and own departure of quantity m >= 1 from its input: the
  // energy departure (m = 1) or the face velocity whose momentum it is
  __device__ __forceinline__ void quantity(const Phys &P, int m, const T (&in)[R], T (&sv)[R],
                                           T (&own)[R]) const {
#pragma clang fp contract(off)
    if (m >= 2) {
      // momentum P = rho v of a face velocity: its specific value is v itself
      const T vbd = (T)vback(P, (m - 2) >> 1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        sv[r] = in[r];
        own[r] = fmav<T>(dr[r], vbd + sv[r], rho0 * sv[r]);
      }
    } else {
      const T q0 = (T)qback(P, m);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        sv[r] = fmav<T>(rho0, in[r], -(q0 * dr[r])) * irr[r];
        own[r] = in[r];
      }
    }
  }
  // transfers of quantity m through the left faces
  template <bool BG = false>
  __device__ __forceinline__ void transfers(const Phys &P, int m, const T (&sv)[R], T (&F)[R]) const {
#pragma clang fp contract(off)
    T fv[R];
    left_faces<BG>(sv, fv);
    const T s0 = (T)sback(P, m);
#pragma unroll
    for (int r = 0; r < R; ++r) F[r] = fmav<T>(s0, dM[r], fv[r] * M[r]);
  }
  // updated departures from the left-face transfers (none through x_max)
  __device__ __forceinline__ void update(const T (&own)[R], const T (&FL)[R], T (&out)[R]) const {
#pragma clang fp contract(off)
    T FR[R];
    row_right<T, R>(FL, FR, T(0));
#pragma unroll
    for (int r = 0; r < R; ++r) out[r] = fmav<T>(-(FR[r] - FL[r]), ivol, own[r]);
  }
};

// input of quantity m >= 1 of the row of level 0 at index c (first cell of the
// lane): the energy departure, or the face velocity whose momentum it is (the
// right x face from the next lane's left face, zero past x_max)
template <typename T, int R>
__device__ __forceinline__ void xrow_input(const Geo &G, const PassArgs<T> &A, int m, idx_t c, bool live,
                                           const T (&da)[R], T (&in)[R]) {
  if (m == 3) {
    row_right<T, R>(da, in, T(0));
    return;
  }
  if (m == 2) {
#pragma unroll
    for (int r = 0; r < R; ++r) in[r] = da[r];
    return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) in[r] = T(0);
  if (!live) return;
  if (m == 1) {
    row_load<T, R>(A.qi[1], c, in);
  } else {
    const int d = (m - 2) >> 1;
    row_load<T, R>(A.v[d], c + ((m & 1) ? dstride(G, d) : 0), in);
  }
}

template <typename T, int R>
__global__ void __launch_bounds__(BX * BY) k_xrow(Geo G, Phys P, PassArgs<T> A) {
  int lane, j, k;
  if (!thread_cell(xrow_box(A.b), lane, j, k)) return;
  const int n = G.n[0];
  const int x0 = R * lane;
  const bool live = x0 < n;  // the lane's cells are active (R divides n)
  const idx_t c = lin(G, x0, j, k);
  XRow<T, R> X;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    X.dr[r] = T(0);
    X.da[r] = T(0);
  }
  if (live) {
    row_load<T, R>(A.qi[0], c, X.dr);
    row_load<T, R>(A.v[0], c, X.da);  // left faces x0 .. x0+R-1 (all <= n - 1)
  }
  X.begin(G, P, (T)(A.fac * A.dtp[0]));
  // flux matching on the frontier of the finer level
  const bool ov = A.fsum && j - G.co[1] >= 0 && k - G.co[2] >= 0 && j - G.co[1] < G.cn[1] && k - G.co[2] < G.cn[2];
  const int flo = G.co[0], fhi = G.co[0] + G.cn[0];
  const long fbase = (long)(k - G.co[2]) * G.cn[1] + (j - G.co[1]);
  auto finish = [&](int m, const T (&own)[R], T (&FL)[R]) {
    if (ov) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int x = x0 + r;
        if (x == flo || x == fhi) {
          FL[r] = A.fsum[((long)(x == fhi) * NQ + m) * A.fstr + fbase];
        }
      }
    }
    T out[R];
    X.update(own, FL, out);
    if (live) row_store<T, R>(A.qo[m], c, out);
  };
  {
    T F[R];
#pragma unroll
    for (int r = 0; r < R; ++r) F[r] = X.dM[r];
    finish(0, X.dr, F);
  }

#pragma unroll 1
  for (int m = 1; m < NQ; ++m) {
    T in[R], sv[R], own[R], F[R];
    xrow_input<T, R>(G, A, m, c, live, X.da, in);
    X.quantity(P, m, in, sv, own);
    X.transfers(P, m, sv, F);
    finish(m, own, F);
  }
}

// Row form of the x pass on a finer level (no boundary conditions: the
// stored row holds the ghost cells): one wave per row, lane l the R cells
// xs + R l .. xs + R l + R - 1 from the R-aligned start xs <= lo - 2, so that
// the wave covers the cells [lo - 2, hi + 2) every update of [lo, hi) reads.
// The arithmetic is XRow's (that of k_xpass); the cells outside [lo, hi) are
// computed and not written, and the frontier transfers are taken (the finer
// level's sums at the covered box's faces) and accumulated (this level's own
// at faces 0 and n) as k_xpass does.
template <typename T, int R>
__global__ void __launch_bounds__(BX * BY) k_xrow_fine(Geo G, Phys P, PassArgs<T> A, int xs) {
  int lane, j, k;
  if (!thread_cell_flat(xrow_box(A.b), lane, j, k)) return;
  const int n = G.n[0];
  const int x0 = xs + R * lane;
  // the lane's cells lie within the row's padded storage, which starts px
  // entries before x = 0 (loads past it are not made; the padding is read as
  // the neighbours of cells outside the range the update reads)
  const int px = (int)(G.off - (long)G.g * (G.sy + G.sz));
  const bool live = x0 >= -px && x0 + R <= (int)G.sy - px;
  const idx_t c = lin(G, x0, j, k);
  XRow<T, R> X;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    X.dr[r] = T(0);
    X.da[r] = T(0);
  }
  if (live) {
    row_load<T, R>(A.qi[0], c, X.dr);
    row_load<T, R>(A.v[0], c, X.da);
  }
  X.begin(G, P, (T)(A.fac * A.dtp[0]));
  const bool ov = A.fsum && j - G.co[1] >= 0 && k - G.co[2] >= 0 && j - G.co[1] < G.cn[1] && k - G.co[2] < G.cn[2];
  const int flo = G.co[0], fhi = G.co[0] + G.cn[0];
  const long fbase = (long)(k - G.co[2]) * G.cn[1] + (j - G.co[1]);
  const bool accrow = A.acc && j >= 0 && k >= 0 && j < G.n[1] && k < G.n[2];
  const long acc_i = (long)k * G.n[1] + j;
  // the lane's cells all inside the updated range: one vector store
  const bool inner = x0 >= A.b.lo[0] && x0 + R <= A.b.hi[0];
  auto finish = [&](int m, const T (&own)[R], T (&FL)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int x = x0 + r;
      if (ov && (x == flo || x == fhi)) {
        FL[r] = A.fsum[((long)(x == fhi) * NQ + m) * A.fstr + fbase];
      }
      if (accrow && (x == 0 || x == n)) A.acc[((long)(x == n) * NQ + m) * A.astr + acc_i] = FL[r];
    }
    T out[R];
    X.update(own, FL, out);
    if (inner) {
      row_store<T, R>(A.qo[m], c, out);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (x0 + r >= A.b.lo[0] && x0 + r < A.b.hi[0]) A.qo[m][c + r] = out[r];
    }
  };
  {
    T F[R];
#pragma unroll
    for (int r = 0; r < R; ++r) F[r] = X.dM[r];
    finish(0, X.dr, F);
  }

#pragma unroll 1
  for (int m = 1; m < NQ; ++m) {
    T in[R], sv[R], own[R], F[R];
    xrow_input<T, R>(G, A, m, c, live, X.da, in);
    X.quantity(P, m, in, sv, own);
    X.transfers(P, m, sv, F);
    finish(m, own, F);
  }
}

// Streaming form of the y and z passes.  A thread owns one column segment
// [c0, c1) along DIR (lanes along x, so every load is coalesced) and walks it
// once: each cell is loaded once (one iteration ahead of its use), each limited
// difference and each face transfer is computed once, and the cell is written
// as soon as its right face is known.  The eight quantities are split over two
// waves of the block: one moves rho, e, P-x, P+x, the other P-y, P+y, P-z, P+z
// (both compute the mass transfers they scale).  A lane may own W = 2 adjacent
// columns, whose cells then move as one 8- or 16-byte access.
template <typename T>
struct MarchArgs {
  int lo[3], hi[3];   // cells to update; DIR is the walked dimension
  int chunk;          // cells per segment
  const T *qi[NQ];
  T *qo[NQ];
  const T *v;         // face velocity departure normal to DIR
  const double *dtp;
  double fac;
  T *acc;
  long astr;
  const T *fsum;
  long fstr;
};

// Transported quantities of group GRP of NG (u = 0.. of the group; entries
// past the group's count are unused): two groups {e, P-x, P+x} and {P-y, P+y,
// P-z, P+z}, or four groups {e}, {P-x, P+x}, {P-y, P+y}, {P-z, P+z}.  Every
// group also transports the density (its mass transfers carry the others);
// the first one stores it.
// NG = 3 is the one group {e, P+y} of the neighbour row a fused z finish
// walks for the y faces of its first row.
constexpr int group_q(int NG, int GRP, int u) {
  return NG == 2 ? (GRP ? 4 + u : (u < 3 ? 1 + u : 1))
                 : (NG == 3 ? (u == 1 ? 5 : 1) : (GRP == 0 ? 1 : (u < 2 ? 2 * GRP + u : 1)));
}
constexpr int group_n(int NG, int GRP) { return NG == 2 ? (GRP ? 4 : 3) : (NG == 3 ? 2 : (GRP ? 2 : 1)); }

// Rows of a column read from the transported set (the y and z passes): the
// raw departures of row c (w[0] the density, w[1..] the group's quantities)
// through level 0's boundary rules.  bc 1 clamps c to the active range; bc 2:
// across a wall (DIR is y or z) every quantity takes its mirror image, and the
// two momenta normal to the wall swap and change sign.
template <typename T, typename V, int DIR, int BC, int GRP, int NG>
struct ColSrc {
  const T *rho;
  const T *qin[4];
  idx_t base, st;
  int n;
  __device__ __forceinline__ V ld(int u, int c) const {  // u < 0: the density
    constexpr bool walls = BC == 2;
    // group wg holds P-, P+ normal to DIR at u = pa, pa + 1
    constexpr int wg = NG == 2 ? 1 : (DIR == 1 ? 2 : 3);
    constexpr int pa = NG == 2 ? ((DIR == 1) ? 0 : 2) : 0;
    const T *q = u < 0 ? rho : qin[u];
    if (walls && (c < 0 || c >= n)) {
      // rows c0-2 .. c1+1 have a mirror image in the active range for n >= 2;
      // the row c1+2 fetched past the last one (never used) may not (n = 2)
      // and is kept in range
      const idx_t m = base + clampi(mirror_idx(c, n), 0, n - 1) * st;
      if (GRP == wg && (u == pa || u == pa + 1)) return -gldv<V>(qin[u ^ 1], m);
      return gldv<V>(q, m);
    }
    if (BC) c = clampi(c, 0, n - 1);
    return gldv<V>(q, base + c * st);
  }
  __device__ __forceinline__ void get(int c, V (&w)[5]) {
    w[0] = ld(-1, c);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < group_n(NG, GRP)) w[u + 1] = ld(u, c);
  }
};

// Transfers through the frontier faces normal to DIR (y or z) of a walk's
// columns, W adjacent ones per lane (FR, bit 0: the level may have a finer one,
// whose transfers fsum holds; bit 1: a coarser one, for which it stores its own):
// few faces of a walk lie on a frontier, so one branch per row asks, and the
// lanes beside it access past the buffer's end.
template <typename T, int W, int DIR, int FR>
struct FaceFront {
  Buf s, a;
  unsigned sq, aq;     // bytes between quantities
  unsigned so[W], ao;  // the columns' entries, low side, quantity 0
  int lo, hi, f0, f1;  // frontier faces: the finer level's, this level's own
  int c0, c1;          // the faces whose transfers this walk stores
  template <typename A>
  __device__ __forceinline__ FaceFront(const Geo &G, const A &M, int x0, int t, bool put, int c0_, int c1_) {
    constexpr int T2 = DIR == 1 ? 2 : 1;
    constexpr unsigned B = sizeof(T);
    c0 = c0_;
    c1 = c1_;
    constexpr int none = -0x40000000;  // no face
    if constexpr ((FR & 1) != 0) {
      lo = M.fsum ? G.co[DIR] : none;
      hi = M.fsum ? G.co[DIR] + G.cn[DIR] : none;
      sq = (unsigned)M.fstr * B;
      s = make_buf(M.fsum + 2 * DIR * NQ * M.fstr, 2 * NQ * sq);
      const int a2 = t - G.co[T2];
#pragma unroll
      for (int q = 0; q < W; ++q) {
        const int a1 = x0 + q - G.co[0];
        const bool in = a1 >= 0 && a1 < G.cn[0] && a2 >= 0 && a2 < G.cn[T2];
        so[q] = in ? (unsigned)(a2 * G.cn[0] + a1) * B : BUF_NONE;
      }
    }
    if constexpr ((FR & 2) != 0) {
      f0 = M.acc ? 0 : none;
      f1 = M.acc ? G.n[DIR] : none;
      aq = (unsigned)M.astr * B;
      a = make_buf(M.acc + 2 * DIR * NQ * M.astr, 2 * NQ * aq);
      const bool in = put && x0 >= 0 && x0 < G.n[0] && t >= 0 && t < G.n[T2];
      ao = in ? (unsigned)(t * G.n[0] + x0) * B : BUF_NONE;
    }
  }
  __device__ __forceinline__ bool is(int f) const {
    return ((FR & 1) && (f == lo || f == hi)) || ((FR & 2) && (f == f0 || f == f1));
  }
  // the transfer of quantity m through such a face, given the pass's own
  template <typename V>
  __device__ __forceinline__ V get(int m, int f, V F) const {
    T v[W];
    from_lanes<V, T, W>(F, v);
    if constexpr ((FR & 1) != 0) {
      const bool on = f == lo || f == hi;
#pragma unroll
      for (int q = 0; q < W; ++q) {
        T w;
        buf_load(s, on ? so[q] : BUF_NONE, (m + (f == hi ? NQ : 0)) * sq, w);
        v[q] = on && so[q] != BUF_NONE ? w : v[q];
      }
    }
    if constexpr ((FR & 2) != 0) {
      const bool on = (f == f0 || f == f1) && f >= c0 && f < c1;
#pragma unroll
      for (int q = 0; q < W; ++q)
        buf_store(a, on ? ao + q * (unsigned)sizeof(T) : BUF_NONE, (m + (f != 0 ? NQ : 0)) * aq, v[q]);
    }
    return to_lanes<V, T, W>(v);
  }
};

// One column segment [c0, c1) of the quantity group GRP of NG at in-plane
// position (i, t), W adjacent columns per lane.  The rows come from src, in
// increasing order c0-2, c0-1, ..., each requested one iteration ahead of its
// use; lanes that are not live (past the row end) neither read nor write.
// FR: the level's frontier transfers (X), as FaceFront's.
template <typename T, int DIR, int BC, int GRP, int FR, int W, int NG, typename Src, typename Sink>
__device__ __forceinline__ void march_column(const Geo &G, const Phys &P, const MarchArgs<T> &A, int i, int t, int c0,
                                             int c1, Src &src, Sink &snk, bool live,
                                             const FaceFront<T, W, DIR, FR> &X) {
  // the transfer through a segment's first face is formed before the walk and
  // again, by the segment below, inside it: with no implicit contraction and
  // the fused products written out, both give the same value, so the results
  // do not depend on where segments start
#pragma clang fp contract(off)
  using V = typename lanes_of<T, W>::type;  // the W adjacent columns of a lane
  constexpr int TD = (DIR == 1) ? 2 : 1;
  const T dt = (T)(A.fac * A.dtp[0]);
  const T dx = (T)G.dx;
  const T mfac = dt * dx * dx, ivol = T(1) / (dx * dx * dx), cour = dt / dx;
  const T rho0 = (T)P.rho0;
  const T vb = (T)vback(P, DIR);
  const T M0 = rho0 * vb * mfac;
  const idx_t st = dstride(G, DIR);
  int id3[3];
  id3[0] = i;
  id3[TD] = t;
  id3[DIR] = 0;
  const idx_t base = lin(G, id3[0], id3[1], id3[2]);
  auto cidx = [&](int c) -> idx_t {
    if (BC) c = clampi(c, 0, G.n[DIR] - 1);
    return base + c * st;
  };
  constexpr int mq[4] = {group_q(NG, GRP, 0), group_q(NG, GRP, 1), group_q(NG, GRP, 2), group_q(NG, GRP, 3)};
  constexpr int nq = group_n(NG, GRP);
  // the momenta across the wind (P-y .. P+z) have a zero background, and
  // only x carries a background velocity: those terms are dropped outright
  constexpr bool zq[4] = {mq[0] >= 4, mq[1] >= 4, mq[2] >= 4, mq[3] >= 4};
  constexpr bool wind = DIR == 0;
  T q0[4], sb[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    q0[u] = (T)qback(P, mq[u]);
    sb[u] = (T)sback(P, mq[u]);
  }

  // final transfers of the walk's face f, given the solver's values (the
  // density belongs to the first group)
  auto fix = [&](int f, V (&F)[5]) {
    if constexpr (FR != 0) {
      if (X.is(f)) {
        if (!GRP) F[0] = X.get(0, f, F[0]);
#pragma unroll
        for (int u = 0; u < nq; ++u) F[u + 1] = X.get(mq[u], f, F[u + 1]);
      }
    }
  };
  // the face's weights hl = (1 - nu)/2, hh = (1 + nu)/2 are exact halvings
  auto upwind = [&](V sl, V dl, V sr, V dr, V a, V hl, V hh) -> V {
    const V lo = fmav<V>(dl, hl, sl), hi = fmav<V>(-dr, hh, sr);
    return a > T(0) ? lo : hi;
  };
  // numerator of the departure of quantity u's specific value from raw
  // departures (q, rho): times 1/(rho0 rho) it is the value
  auto numer = [&](int u, V q, V r) -> V { return zq[u] ? rho0 * q : fmav<V>(V(rho0), q, -(q0[u] * r)); };
  // limited difference at a cell of value s from its left neighbour's value sl
  // and its right neighbour's numerator and reciprocal (xr, ir): the right
  // difference takes the neighbour's value unrounded, the left one the values
  auto limited = [&](V xr, V ir, V s, V sl) -> V { return vleer(fmav<V>(xr, ir, -s), s - sl); };
  // Courant weights of a face: (1 -+ nu)/2, exact halvings of the rounded 1 -+ nu
  auto weights = [&](V a, V &hl, V &hh) {
    const V nu = a * cour;
    hl = fmav<V>(V(-0.5), nu, V(0.5));
    hh = fmav<V>(V(0.5), nu, V(0.5));
  };
  // velocity departure on face c (normal to DIR)
  auto face = [&](int c) -> V { return live ? gldv<V>(A.v, base + c * st) : V(0); };

  // window: departures of the specific values at c, c+1 (s0, s1; index 0 is
  // the density departure), limited difference at c (d0), transfer through
  // face c (F0); raw departures of cells c, c+1, c+2 (w0, w1, w2) and the
  // velocity departure on face c+1 (va), all fetched at least one iteration
  // ahead of their use
  V s0[5], s1[5], d0[5], F0[5], w0[5], w1[5], w2[5];
  V va;
  {
    // the density (u = 0) is its own value: numerator the raw departure,
    // reciprocal 1
    V rm2[5], rm1[5], sm2[5], sm1[5], x0[5], x1[5];
    src.get(c0 - 2, rm2);
    src.get(c0 - 1, rm1);
    src.get(c0, w0);
    src.get(c0 + 1, w1);
    const V ir_m2 = qdiv(V(1), rho0 * (rho0 + rm2[0])), ir_m1 = qdiv(V(1), rho0 * (rho0 + rm1[0]));
    const V ir_0 = qdiv(V(1), rho0 * (rho0 + w0[0])), ir_p1 = qdiv(V(1), rho0 * (rho0 + w1[0]));
    sm2[0] = rm2[0]; sm1[0] = rm1[0]; s0[0] = x0[0] = w0[0]; s1[0] = x1[0] = w1[0];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u >= nq) break;
      sm2[u + 1] = numer(u, rm2[u + 1], rm2[0]) * ir_m2;
      sm1[u + 1] = numer(u, rm1[u + 1], rm1[0]) * ir_m1;
      x0[u + 1] = numer(u, w0[u + 1], w0[0]);
      x1[u + 1] = numer(u, w1[u + 1], w1[0]);
      s0[u + 1] = x0[u + 1] * ir_0;
      s1[u + 1] = x1[u + 1] * ir_p1;
    }
    const V da = face(c0);
    const V a = wind ? vb + da : da;
    V hl, hh;
    weights(a, hl, hh);
    V dM = V(0), M = V(0);
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      if (u > nq) break;
      const V dm1 = limited(x0[u], u ? ir_0 : V(1), sm1[u], sm2[u]);
      d0[u] = limited(x1[u], u ? ir_p1 : V(1), s0[u], sm1[u]);
      const V fv = upwind(sm1[u], dm1, s0[u], d0[u], a, hl, hh);
      if (u == 0) {
        dM = fmav<V>(fv, a, rho0 * da) * mfac;
        M = wind ? M0 + dM : dM;
        F0[0] = dM;
      } else {
        F0[u] = zq[u - 1] ? fv * M : fmav<V>(V(sb[u - 1]), dM, fv * M);
      }
    }
    fix(c0, F0);
    src.get(c0 + 2, w2);
    va = face(c0 + 1);
  }
  for (int c = c0; c < c1; ++c) {
    const idx_t ic = cidx(c);
    // next iteration's rows: cell c+3 and face c+2 (one row past the last
    // needed one, c1+1, is fetched and not used: no branch splits the body)
    V nn[5];
    src.get(c + 3, nn);
    const V vn = face(min(c + 2, c1));
    const V ir2 = qdiv(V(1), rho0 * (rho0 + w2[0]));
    V s2[5], x2[5];
    s2[0] = x2[0] = w2[0];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u < nq) {
        x2[u + 1] = numer(u, w2[u + 1], w2[0]);
        s2[u + 1] = x2[u + 1] * ir2;
      }
    }
    const V da = va;
    const V a = wind ? vb + da : da;
    V hl, hh;
    weights(a, hl, hh);
    V dM = V(0), M = V(0), F1[5];
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      if (u > nq) break;
      const V d1 = limited(x2[u], u ? ir2 : V(1), s1[u], s0[u]);
      const V fv = upwind(s0[u], d0[u], s1[u], d1, a, hl, hh);
      if (u == 0) {
        dM = fmav<V>(fv, a, rho0 * da) * mfac;
        M = wind ? M0 + dM : dM;
        F1[0] = dM;
      } else {
        F1[u] = zq[u - 1] ? fv * M : fmav<V>(V(sb[u - 1]), dM, fv * M);
      }
      if (FR == 0) {
        snk.put(u, ic, fmav<V>(-(F1[u] - F0[u]), V(ivol), w0[u]));
        F0[u] = F1[u];
      }
      d0[u] = d1;
      s0[u] = s1[u];
      s1[u] = s2[u];
    }
    if constexpr (FR != 0) {
      fix(c + 1, F1);
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        if (u > nq) break;
        snk.put(u, ic, fmav<V>(-(F1[u] - F0[u]), V(ivol), w0[u]));
        F0[u] = F1[u];
      }
    }
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      w0[u] = w1[u];
      w1[u] = w2[u];
      w2[u] = nn[u];
    }
    va = vn;
    snk.done(c);
  }
}

// The usual sink of a column walk: cell c's new departures of the group's
// quantities (u = 1..) and, for the first group, of the density (u = 0) go to
// the output set.
template <typename T, typename V, int GRP, int NG>
struct OutSink {
  T *q[5];
  bool live;
  __device__ __forceinline__ OutSink(const MarchArgs<T> &A, bool lv) : live(lv) {
    q[0] = A.qo[0];
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u + 1] = A.qo[group_q(NG, GRP, u)];
  }
  __device__ __forceinline__ void put(int u, idx_t ic, V val) {
    if ((u > 0 || GRP == 0) && live) gstv<V>(q[u], ic, val);
  }
  __device__ __forceinline__ void done(int) {}
};

// The sink of a walk over a finer level of the quadrant, whose rows and planes
// start at the mirror planes: the images of the cells within the ghost shell's
// width of a plane are stored beside them (P-_d of an image is -P+_d of its
// cell, d the plane's normal), so that the next pass finds its neighbours
// beyond the planes and no launch sets them.
template <typename T, int DIR, int GRP, int NG>
struct ImageSink {
  const MarchArgs<T> *A;
  int c, t, g;  // the walk's cell, its transverse index, the shell's width
  idx_t sy, sz;
  bool live;
  __device__ __forceinline__ ImageSink(const Geo &G, const MarchArgs<T> &M, int c0, int t_, bool lv)
      : A(&M), c(c0), t(t_), g(G.g), sy((idx_t)G.sy), sz((idx_t)G.sz), live(lv) {}
  __device__ __forceinline__ void put(int u, idx_t ic, T val) {
    if (!((u > 0 || GRP == 0) && live)) return;
    const int m = u == 0 ? 0 : group_q(NG, GRP, u - 1);
    const int my = m == 4 || m == 5 ? 9 - m : m, mz = m == 6 || m == 7 ? 13 - m : m;
    const T vy = my != m ? -val : val, vz = mz != m ? -val : val;
    const int j = DIR == 1 ? c : t, k = DIR == 1 ? t : c;
    const idx_t iy = ic - (1 + 2 * j) * sy, iz = (1 + 2 * k) * sz;
    gst(A->qo[m], ic, val);
    if (j < g) gst(A->qo[my], iy, vy);
    if (k < g) {
      gst(A->qo[mz], ic - iz, vz);
      if (j < g) gst(A->qo[my != m ? my : mz], iy - iz, my != m ? vy : vz);
    }
  }
  __device__ __forceinline__ void done(int) { ++c; }
};

template <typename T, int DIR, int BC, int FR, int W, bool ANCH = false>
__global__ void __launch_bounds__(256) k_march(Geo G, Phys P, MarchArgs<T> A) {
  constexpr int TD = (DIR == 1) ? 2 : 1;
  const int lane = threadIdx.x, ty = threadIdx.y;
  // threadIdx.y is the same across a wave (blockDim.x is one wave): reading it
  // from the first lane makes the quantity group, and so every field pointer,
  // a scalar
  const int grp = __builtin_amdgcn_readfirstlane(ty) & 1;
  int i, t, ch;
  if (W == 1) {
    // one column per lane: the (x, transverse) columns of the box numbered x
    // fastest, each wave taking 64 consecutive ones (rows that are not a
    // multiple of 64 long share waves), two waves' worth per block
    const unsigned ex = (unsigned)(A.hi[0] - A.lo[0]), et = (unsigned)(A.hi[TD] - A.lo[TD]);
    const unsigned nt2 = (ex * et + 127) / 128;
    const unsigned h = blockIdx.x;
    ch = (int)(h / nt2);
    const unsigned f = (h % nt2) * 128 + (unsigned)(ty >> 1) * 64 + (unsigned)lane;
    if (f >= ex * et) return;
    i = A.lo[0] + (int)(f % ex);
    t = A.lo[TD] + (int)(f / ex);
  } else {
    const int nbx = (A.hi[0] - A.lo[0] + 64 * W - 1) / (64 * W);
    const int ntb = (A.hi[TD] - A.lo[TD] + 1) / 2;
    const unsigned h = blockIdx.x;
    const int bx = (int)(h % (unsigned)nbx);
    const unsigned r1 = h / (unsigned)nbx;
    const int tb = (int)(r1 % (unsigned)ntb);
    ch = (int)(r1 / (unsigned)ntb);
    i = A.lo[0] + (bx * 64 + lane) * W;  // the lane's first column (W divides the extent)
    t = A.lo[TD] + tb * 2 + (ty >> 1);
    if (i >= A.hi[0] || t >= A.hi[TD]) return;
  }
  const int c0 = A.lo[DIR] + ch * A.chunk;
  const int c1 = min(c0 + A.chunk, A.hi[DIR]);
  if (c0 >= c1) return;
  using V = typename lanes_of<T, W>::type;
  int id3[3];
  id3[0] = i;
  id3[TD] = t;
  id3[DIR] = 0;
  const idx_t base = lin(G, id3[0], id3[1], id3[2]);
  const FaceFront<T, W, DIR, FR> X(G, A, i, t, true, c0, c1);
  auto walk = [&](auto gc) {
    constexpr int g = decltype(gc)::value;
    ColSrc<T, V, DIR, BC, g, 2> src{A.qi[0], {A.qi[group_q(2, g, 0)], A.qi[group_q(2, g, 1)], A.qi[group_q(2, g, 2)],
                                              A.qi[group_q(2, g, 3)]}, base, dstride(G, DIR), G.n[DIR]};
    if constexpr (ANCH) {
      ImageSink<T, DIR, g, 2> snk(G, A, c0, t, true);
      march_column<T, DIR, BC, g, FR, W, 2>(G, P, A, i, t, c0, c1, src, snk, true, X);
    } else {
      OutSink<T, V, g, 2> snk(A, true);
      march_column<T, DIR, BC, g, FR, W, 2>(G, P, A, i, t, c0, c1, src, snk, true, X);
    }
  };
  if (grp) walk(std::integral_constant<int, 1>{});
  else walk(std::integral_constant<int, 0>{});
}

// Fused x and y passes with the density's work done once per plane.  Every
// quantity group needs the density's transfers: the mass transfers through the
// x faces of each row, the row's x-updated density and the y pass's reciprocal
// 1/(rho0 rho), and the mass transfers through the y faces.  The first wave of
// a block (the density leader) computes them one row ahead of the march and
// hands them to the block's waves (itself included) through LDS, so that the
// waves move only their own quantities; the reciprocal of each row past the
// segment's first ones is formed by the second wave, a row behind the leader
// (whose step is the longest of the four).  Row r sits in slot r mod XY_RS, face
// f in slot f mod XY_FS; one barrier per row orders the hand-over.  The
// arithmetic of every value is that of the separate passes (k_xrow, k_march).
//
// A wave holds a tile of 64 W consecutive cells of a row, W per lane.  What the
// lane shifts bring in at a tile's ends is wrong for a few cells: a tile that
// starts inside a row is exact from its third cell, and one that ends inside it
// up to its fifth from the end (P+x of a cell is read from the next lane's left
// face), so tiles overlap and each stores its exact pairs of cells.  At level
// 0's row ends the tile's own ends are the boundary rules: before x = 0 the
// lane shift fills in the outflow copy (or the background), and the cells past
// x = n - 1 are the row's padding, which holds zero departures, the inflow
// state.  The cells a row has past its whole tiles take half or a quarter of a
// wave where they fit, two or four planes' to a wave.
constexpr int XY_RS = 8, XY_FS = 4;

template <typename T, int W>
struct XyShare {
  T *rows;   // [XY_RS][3][W][64]: x-face mass transfers, x-updated density, 1/(rho0 rho)
  T *faces;  // [XY_FS][W][64]: y-face mass transfers
  int lane;
  using V = typename lanes_of<T, W>::type;
  __device__ __forceinline__ T &row(int r, int f, int q) const {
    return rows[(((r & (XY_RS - 1)) * 3 + f) * W + q) * 64 + lane];
  }
  __device__ __forceinline__ T &face(int f, int q) const { return faces[((f & (XY_FS - 1)) * W + q) * 64 + lane]; }
  __device__ __forceinline__ V rowv(int r, int f) const {
    T a[W];
#pragma unroll
    for (int q = 0; q < W; ++q) a[q] = row(r, f, q);
    return to_lanes<V, T, W>(a);
  }
  __device__ __forceinline__ V facev(int f) const {
    T a[W];
#pragma unroll
    for (int q = 0; q < W; ++q) a[q] = face(f, q);
    return to_lanes<V, T, W>(a);
  }
  __device__ __forceinline__ void put_face(int f, V v) const {
    T a[W];
    from_lanes<V, T, W>(v, a);
#pragma unroll
    for (int q = 0; q < W; ++q) face(f, q) = a[q];
  }
};

// What a level's rows are, by XB: 1, 4 level 0 under boundary mode 1 with rows of
// one tile and of several, 2 under mode 2, 0 a finer level, 3 a finer level of
// the quadrant.  (Under 1 the lanes past the row's end compute zero departures,
// as they read; they store them over the zeros of the row's padding, so that no
// lane is kept from storing: 128^3 FP64 69 -> 62 us.)  Rows beyond a mirror plane or wall
// are the images of the level's own: their x pass is that of the row they
// mirror, and the momenta across the plane swap and change sign.
constexpr bool xy_mirror_lo(int XB) { return XB == 2 || XB == 3; }
constexpr bool xy_mirror_hi(int XB) { return XB == 2; }

// The lane's place and the block's: plane t, cells x0 .. x0 + W - 1, whose
// loads start at xl (x0 kept inside the row's storage); put: the lane stores its
// results.
// (edge: the cell of a pair of which only that one lies in the stored range, or
// -1; any_edge: on any lane of the wave)
struct XyLane {
  int t, x0, xl;
  bool put, any_edge;
  int edge;
};

template <typename T, int W, int XB>
struct XyGrid {
  const Geo *G;
  int rmax;  // finer levels: the last row that may be read
  XyLane L;
  __device__ __forceinline__ int row(int r) const {
    const int n = G->n[1];
    if (XB == 1 || XB == 4) return clampi(r, 0, n - 1);
    // (a row past the ones the walk uses may have no image: kept in range)
    if (XB == 2) return clampi(mirror_idx(r, n), 0, n - 1);
    if (XB == 3 && r < 0) return -1 - r;
    return min(r, rmax);
  }
  // row r is an image
  __device__ __forceinline__ bool image(int r) const {
    return (xy_mirror_lo(XB) && r < 0) || (xy_mirror_hi(XB) && r >= G->n[1]);
  }
  __device__ __forceinline__ idx_t at(int r) const { return lin(*G, L.xl, row(r), L.t); }
  // momenta tangential to x (their velocities): past the flow end x_max under
  // bc 2 the last cell's value, read by the lane after it one entry early (an
  // odd index; what it then reads for the cell after that, the row's padding, is
  // not used: it enters the first one's limited difference only, whose other
  // factor, the difference of two equal values, is zero)
  __device__ __forceinline__ idx_t tangential() const { return L.x0 == G->n[0] ? -1 : 0; }
};

// Frontier transfers of a walk (FR, bit 0: the level has a finer one whose
// transfers B.fsum holds; bit 1: it has a coarser one and stores its own).  A
// lane has at most one x face on the finer level's frontier (face x0 + fq) and
// at most one on the level's own (face x0: levels have an even count of cells and
// lanes start at even ones); the lanes that have none, and the rows that lie
// beside the frontier, access past the buffer's end, so that the walk's steps
// stay free of branches.
template <typename T, int W, int FR>
struct XyFront {
  FaceFront<T, W, 1, FR> y;  // the y faces
  Buf xs, xa;            // fsum and acc, x faces
  unsigned xsq, xaq;     // bytes between quantities
  unsigned fo, ao;       // the lane's x entry, quantity 0, row 0 of the level
  int fq, lo, hi;        // rows of the covered box
  __device__ __forceinline__ XyFront(const Geo &G, const PassArgs<T> &A, const XyLane &L, int c0, int c1)
      : y(G, A, L.x0, L.t, L.put, c0, c1) {
    constexpr unsigned B = sizeof(T);
    if constexpr (FR & 1) {
      lo = G.co[1];
      hi = G.co[1] + G.cn[1];
      xsq = (unsigned)A.fstr * B;
      xs = make_buf(A.fsum, 2 * NQ * xsq);
      const int a2 = L.t - G.co[2];
      const bool in = a2 >= 0 && a2 < G.cn[2];
      const int l = G.co[0] - L.x0, h = l + G.cn[0];
      const bool is_l = l >= 0 && l < W, is_h = h >= 0 && h < W;
      fq = in && is_l ? l : in && is_h ? h : -1;
      fo = fq >= 0 ? (is_h ? NQ * xsq : 0u) + (unsigned)(a2 * G.cn[1]) * B : BUF_NONE;
    }
    if constexpr (FR & 2) {
      xaq = (unsigned)A.astr * B;
      xa = make_buf(A.acc, 2 * NQ * xaq);
      const bool in = L.put && L.t >= 0 && L.t < G.n[2];
      const bool is_l = L.x0 == 0, is_h = L.x0 == G.n[0];
      ao = in && (is_l || is_h) ? (is_h ? NQ * xaq : 0u) + (unsigned)(L.t * G.n[1]) * B : BUF_NONE;
    }
  }
  // the finer level's transfer of quantity m through the lane's x face of row
  // rr (any value where it has none)
  __device__ __forceinline__ T fine_x(int m, int rr) const {
    T v;
    buf_load(xs, rr >= lo && rr < hi ? fo + (unsigned)(rr - lo) * (unsigned)sizeof(T) : BUF_NONE, m * xsq, v);
    return v;
  }
  // the transfers F of quantity m through the x faces of row r (rr the row it
  // is read from, fine its fine_x): the finer level's on its frontier, and into
  // this level's own set on rows [c0, c1)
  __device__ __forceinline__ void row(const Geo &G, int m, int r, int rr, int c0, int c1, T fine, T (&F)[W]) const {
    if constexpr (FR & 1) {
      const int q0 = rr >= lo && rr < hi ? fq : -1;
#pragma unroll
      for (int q = 0; q < W; ++q) F[q] = q0 == q ? fine : F[q];
    }
    if constexpr (FR & 2) {
      const bool in = r >= c0 && r < c1 && r >= 0 && r < G.n[1];
      buf_store(xa, in ? ao + (unsigned)r * (unsigned)sizeof(T) : BUF_NONE, m * xaq, F[0]);
    }
  }
};

// inputs of one row's x pass: its density and x-face velocity departures
template <typename T, int W, int XB>
__device__ __forceinline__ idx_t xy_row_in(const XyGrid<T, W, XB> &Q, const PassArgs<T> &A, int r, T (&dr)[W],
                                           T (&da)[W]) {
  const idx_t c = Q.at(r);
  row_load<T, W>(A.qi[0], c, dr);
  row_load<T, W>(A.v[0], c, da);
  return c;
}

// the leader's x pass of the density of row r: left-face mass transfers and
// x-updated departure into the row's slot, with ir also the reciprocal (under
// FR the update takes the frontier's transfers, the slot the pass's own,
// which the other quantities' transfers are formed from)
template <typename T, int W, int XB, int FR>
__device__ __forceinline__ typename lanes_of<T, W>::type xy_lead_row(const XyGrid<T, W, XB> &Q, const Phys &P, T dt,
                                                                     const XyShare<T, W> &S, int r, const T (&dr)[W],
                                                                     const T (&da)[W], const PassArgs<T> &A,
                                                                     const XyFront<T, W, FR> &X, int c0, int c1, T fine,
                                                                     bool ir = true) {
  XRow<T, W> R;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    R.dr[q] = dr[q];
    R.da[q] = da[q];
  }
  R.flow(*Q.G, P, dt);
  R.template mass<XB == 2>();
  T out[W];
  if constexpr (FR != 0) {
    T F[W];
#pragma unroll
    for (int q = 0; q < W; ++q) F[q] = R.dM[q];
    X.row(*Q.G, 0, r, Q.row(r), c0, c1, fine, F);
    R.update(R.dr, F, out);
  } else {
    R.update(R.dr, R.dM, out);
  }
#pragma unroll
  for (int q = 0; q < W; ++q) {
    S.row(r, 0, q) = R.dM[q];
    S.row(r, 1, q) = out[q];
    if (ir) S.row(r, 2, q) = qdiv(T(1), R.rho0 * (R.rho0 + out[q]));
  }
  return to_lanes<typename lanes_of<T, W>::type, T, W>(out);
}

// Rows of a column for the y pass of a group's own quantities: the x pass of
// those quantities on the tile's rows, with the row's mass transfers taken from
// the leader; the inputs of the next row are loaded while the y pass uses this
// one.
template <typename T, int W, int GRP, int NG, int XB, int FR>
struct XyOwn {
  using V = typename lanes_of<T, W>::type;
  const XyGrid<T, W, XB> &Q;
  const Phys &P;
  const PassArgs<T> &A;
  const XyFront<T, W, FR> &X;
  T dt;
  int c0, c1;
  T dr[W], da[W], in[4][W], fn[4];  // inputs of the next row

  __device__ __forceinline__ void load(int r) {
    const idx_t c = xy_row_in<T, W, XB>(Q, A, r, dr, da);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u < group_n(NG, GRP)) {
        const int m = group_q(NG, GRP, u);
        if (m == 1) row_load<T, W>(A.qi[1], c, in[u]);
        if (m >= 4) {
          const int d = (m - 2) >> 1;
          const idx_t f = c + ((m & 1) ? dstride(*Q.G, d) : 0);
          if constexpr (XB == 2) row_load_any<T, W>(A.v[d], f + Q.tangential(), in[u]);
          else row_load<T, W>(A.v[d], f, in[u]);
        }
        if (FR & 1) fn[u] = X.fine_x(m, Q.row(r));
      }
    }
  }
  __device__ __forceinline__ void get(int r, const XyShare<T, W> &S, V (&w)[4]) {
    constexpr int nq = group_n(NG, GRP);
    constexpr int m[4] = {group_q(NG, GRP, 0), group_q(NG, GRP, 1), group_q(NG, GRP, 2), group_q(NG, GRP, 3)};
    XRow<T, W> R;
#pragma unroll
    for (int q = 0; q < W; ++q) {
      R.dr[q] = dr[q];
      R.da[q] = da[q];
    }
    R.flow(*Q.G, P, dt);
    if (m[0] == 1) R.recip();  // the energy's specific value
    T dm[W];
#pragma unroll
    for (int q = 0; q < W; ++q) dm[q] = S.row(r, 0, q);
    R.take_mass(dm);
    T own[4][W], F[4][W];
#pragma unroll
    for (int u = 0; u < nq; ++u) {
      T inq[W], sv[W];
      if (m[u] == 3) {
        row_right<T, W>(R.da, inq, T(0));  // the right face of a cell is the next one's left
      } else {
#pragma unroll
        for (int q = 0; q < W; ++q) inq[q] = m[u] == 2 ? R.da[q] : in[u][q];
      }
      R.quantity(P, m[u], inq, sv, own[u]);
      if (XB == 2 && m[u] < 4) R.template transfers<true>(P, m[u], sv, F[u]);
      else R.template transfers<false>(P, m[u], sv, F[u]);
    }
    if constexpr (FR != 0)
#pragma unroll
      for (int u = 0; u < nq; ++u) X.row(*Q.G, m[u], r, Q.row(r), c0, c1, fn[u], F[u]);
#pragma unroll
    for (int u = 0; u < nq; ++u) {
      T out[W];
      R.update(own[u], F[u], out);
      w[u] = to_lanes<V, T, W>(out);
    }
    if constexpr (xy_mirror_lo(XB) && m[0] == 4) {
      const bool im = Q.image(r);
      const V pm = w[0], pp = w[1];
      w[0] = im ? -pp : pm;
      w[1] = im ? -pm : pp;
    }
    load(r + 1);
  }
};

// One plane's y segment [c0, c1) of group GRP's own quantities; with LEAD
// also the density (its x pass one row ahead, its y-face transfers one face
// ahead, its update).  Each row is one step that ends in a barrier, so every
// wave of the block meets the same barriers.  The values a step hands to the
// next live in rings of three slots whose roles turn with the step's phase
// (its row's distance from c0, mod 3), so that no value is copied from step
// to step.  Under FR the transfers through the frontiers' x faces are taken and
// stored without a branch (XyFront), those through its few y faces in one per
// row.
template <typename T, int W, int GRP, int NG, bool LEAD, int XB, int FR>
__device__ __forceinline__ void xy_shared_group(const XyGrid<T, W, XB> &Q, const Phys &P, const PassArgs<T> &A,
                                                const MarchArgs<T> &M, T dt, int c0, int c1,
                                                const XyShare<T, W> &S) {
  // a segment's first face is formed here and, by the segment below, in its
  // walk: as in march_column, no implicit contraction, the fused products
  // written out, so that both give the same value
#pragma clang fp contract(off)
  using V = typename lanes_of<T, W>::type;
  constexpr int nq = group_n(NG, GRP);
  constexpr int mq[4] = {group_q(NG, GRP, 0), group_q(NG, GRP, 1), group_q(NG, GRP, 2), group_q(NG, GRP, 3)};
  constexpr bool zq[4] = {mq[0] >= 4, mq[1] >= 4, mq[2] >= 4, mq[3] >= 4};
  const Geo &G = *Q.G;
  const T dx = (T)G.dx;
  const T mfac = dt * dx * dx, ivol = T(1) / (dx * dx * dx), cour = dt / dx;
  const T rho0 = (T)P.rho0;
  const idx_t st = (idx_t)G.sy;
  const idx_t base = lin(G, Q.L.xl, 0, Q.L.t);
  const int t = Q.L.t, x0 = Q.L.x0;
  const XyFront<T, W, FR> X(G, A, Q.L, c0, c1);
  T q0[4], sb[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    q0[u] = (T)qback(P, mq[u]);
    sb[u] = (T)sback(P, mq[u]);
  }
  // the face's weights hl = (1 - nu)/2, hh = (1 + nu)/2 are exact halvings
  // of the rounded 1 -+ nu
  auto upwind = [&](V sl, V dl, V sr, V dr, V a) -> V {
    const V nu = a * cour;
    const V hl = fmav<V>(V(-0.5), nu, V(0.5)), hh = fmav<V>(V(0.5), nu, V(0.5));
    const V lo = fmav<V>(dl, hl, sl), hi = fmav<V>(-dr, hh, sr);
    return a > T(0) ? lo : hi;
  };
  // numerator of a specific value's departure (times 1/(rho0 rho) the value)
  // and the limited difference at a cell from its right neighbour's numerator
  // and reciprocal: the arithmetic of march_column
  auto numer = [&](int u, V q, V r) -> V { return zq[u] ? rho0 * q : fmav<V>(V(rho0), q, -(q0[u] * r)); };
  auto limited = [&](V xr, V ir, V s, V sl) -> V { return vleer(fmav<V>(xr, ir, -s), s - sl); };
  auto face = [&](int c) -> V { return gldv<V>(M.v, base + c * st); };
  // mass transfer through a y face from the density around it
  auto mass_y = [&](V a, V sl, V dl, V sr, V dr) -> V {
    return fmav<V>(upwind(sl, dl, sr, dr, a), a, rho0 * a) * mfac;
  };
  auto store = [&](int m, int j, idx_t ic, auto val) {
    using V = decltype(val);
    gstv<V>(M.qo[m], ic, val);
    if constexpr (XB == 3) {  // the images beyond the mirror planes (as ImageSink)
      const int my = m == 4 || m == 5 ? 9 - m : m, mz = m == 6 || m == 7 ? 13 - m : m;
      const V vy = my != m ? -val : val, vz = mz != m ? -val : val;
      const idx_t iy = ic - (1 + 2 * j) * (idx_t)G.sy, iz = (1 + 2 * t) * (idx_t)G.sz;
      if (j < G.g) gstv<V>(M.qo[my], iy, vy);
      if (t < G.g) {
        gstv<V>(M.qo[mz], ic - iz, vz);
        if (j < G.g) gstv<V>(M.qo[my != m ? my : mz], iy - iz, my != m ? vy : vz);
      }
    }
  };

  // leader rings: x-updated density of rows c+1 .. c+3 (rr), its limited
  // difference at c+1 (rd), the mass transfers of faces c, c+1 (rm), the
  // velocity departure of face c+2 (rv); inputs of row c+4 (ldr, lda); under
  // FR the density's transfer through face c (rf)
  V rr[3], rd[3], rm[3], rv[3], rf = V(0);
  T ldr[W], lda[W], lfn = T(0);
  auto lead_in = [&](int r) {  // inputs of the leader's next row
    xy_row_in<T, W, XB>(Q, A, r, ldr, lda);
    if constexpr ((FR & 1) != 0) lfn = X.fine_x(0, Q.row(r));
  };
  // own rings: specific values at c, c+1 (ss), limited difference at c (sd),
  // transfer through face c (sF), x-updated departures of rows c .. c+2 (sw),
  // velocity departure of face c+1 (sv)
  XyOwn<T, W, GRP, NG, XB, FR> src{Q, P, A, X, dt, c0, c1};
  V ss[3][4], sd[3][4], sF[3][4], sw[3][4], sv[3];
  // rows c0-2 .. c0+3 of the density, c0-2 .. c0+2 of the own quantities, one
  // row behind it so that the waves work side by side; in a loop (the code of
  // one row, not of six), each row's inputs loaded a row ahead
  {
    V w[6], wm2[4], wm1[4];
    src.load(c0 - 2);
    if constexpr (LEAD) lead_in(c0 - 2);
#pragma unroll 1
    for (int k = 0; k < 6; ++k) {
      if constexpr (LEAD) {
        T cdr[W], cda[W];
        const T cfn = lfn;
#pragma unroll
        for (int q = 0; q < W; ++q) {
          cdr[q] = ldr[q];
          cda[q] = lda[q];
        }
        lead_in(c0 - 1 + k);
#pragma unroll
        for (int i = 0; i < 5; ++i) w[i] = w[i + 1];
        w[5] = xy_lead_row<T, W, XB, FR>(Q, P, dt, S, c0 - 2 + k, cdr, cda, A, X, c0, c1, cfn, true);
      }
      __syncthreads();
      if (k < 5) {
#pragma unroll
        for (int u = 0; u < nq; ++u) {
          wm2[u] = wm1[u];
          wm1[u] = sw[0][u];
          sw[0][u] = sw[1][u];
          sw[1][u] = sw[2][u];
        }
        src.get(c0 - 2 + k, S, sw[2]);
      }
    }
    if constexpr (LEAD) {
      const V r_m2 = w[0], r_m1 = w[1], r_0 = w[2];
#pragma unroll
      for (int k = 0; k < 3; ++k) rr[k] = w[3 + k];
      const V d_m1 = vleer(r_0 - r_m1, r_m1 - r_m2);
      const V d_0 = vleer(rr[0] - r_0, r_0 - r_m1);
      rm[0] = mass_y(face(c0), r_m1, d_m1, r_0, d_0);
      S.put_face(c0, rm[0]);
      rd[0] = vleer(rr[1] - rr[0], rr[0] - r_0);
      rm[1] = mass_y(face(c0 + 1), r_0, d_0, rr[0], rd[0]);
      S.put_face(c0 + 1, rm[1]);
      rv[0] = face(min(c0 + 2, c1));
      rf = rm[0];
      if constexpr (FR != 0)
        if (X.y.is(c0)) rf = X.y.get(0, c0, rf);
    }
    __syncthreads();
    const V r_m2 = S.rowv(c0 - 2, 1), r_m1 = S.rowv(c0 - 1, 1), r_0 = S.rowv(c0, 1), r_p1 = S.rowv(c0 + 1, 1);
    const V i_m2 = S.rowv(c0 - 2, 2), i_m1 = S.rowv(c0 - 1, 2), i_0 = S.rowv(c0, 2), i_p1 = S.rowv(c0 + 1, 2);
    const V a = face(c0);
    const V dM = S.facev(c0);
#pragma unroll
    for (int u = 0; u < nq; ++u) {
      const V sm2 = numer(u, wm2[u], r_m2) * i_m2, sm1 = numer(u, wm1[u], r_m1) * i_m1;
      const V y0 = numer(u, sw[0][u], r_0), y1 = numer(u, sw[1][u], r_p1);
      ss[0][u] = y0 * i_0;
      ss[1][u] = y1 * i_p1;
      const V dm1 = limited(y0, i_0, sm1, sm2);
      sd[0][u] = limited(y1, i_p1, ss[0][u], sm1);
      const V fv = upwind(sm1, dm1, ss[0][u], sd[0][u], a);
      sF[0][u] = zq[u] ? fv * dM : fmav<V>(V(sb[u]), dM, fv * dM);
    }
    if constexpr (FR != 0)
      if (X.y.is(c0))
#pragma unroll
        for (int u = 0; u < nq; ++u) sF[0][u] = X.y.get(mq[u], c0, sF[0][u]);
    sv[0] = face(c0 + 1);
  }

  // row c in phase K0: ring slot K0 holds the oldest value, K1 the next, K2
  // the newest (or the free slot)
  auto step = [&](auto phase, int c) {
    constexpr int K0 = decltype(phase)::value, K1 = (K0 + 1) % 3, K2 = (K0 + 2) % 3;
    const idx_t ic = base + c * st;
    {
      const V r2 = S.rowv(c + 2, 1), ir2 = S.rowv(c + 2, 2);
      const V a = sv[K0];
      sv[K1] = face(min(c + 2, c1));
      const V dM = S.facev(c + 1);
#pragma unroll
      for (int u = 0; u < nq; ++u) {
        const V x2 = numer(u, sw[K2][u], r2);
        ss[K2][u] = x2 * ir2;
        sd[K1][u] = limited(x2, ir2, ss[K1][u], ss[K0][u]);
        const V fv = upwind(ss[K0][u], sd[K0][u], ss[K1][u], sd[K1][u], a);
        sF[K1][u] = zq[u] ? fv * dM : fmav<V>(V(sb[u]), dM, fv * dM);
      }
      if constexpr (FR != 0)
        if (X.y.is(c + 1))
#pragma unroll
          for (int u = 0; u < nq; ++u) sF[K1][u] = X.y.get(mq[u], c + 1, sF[K1][u]);
      V out[4];
#pragma unroll
      for (int u = 0; u < nq; ++u) out[u] = fmav<V>(-(sF[K1][u] - sF[K0][u]), V(ivol), sw[K0][u]);
      if (XB == 1 || Q.L.put) {
#pragma unroll
        for (int u = 0; u < nq; ++u) store(mq[u], c, ic, out[u]);
      }
      if constexpr (W == 2 && (XB == 0 || XB == 3)) {
        if (Q.L.any_edge && Q.L.edge >= 0) {
#pragma unroll
          for (int u = 0; u < nq; ++u) store(mq[u], c, ic + Q.L.edge, Q.L.edge ? out[u].y : out[u].x);
        }
      }
      src.get(c + 3, S, sw[K0]);
    }
    if constexpr (GRP == 1) {
      // the reciprocal of row c+3 (its density came from the leader a step
      // ago), for the y walk one step later; the leader carries more work
#pragma unroll
      for (int q = 0; q < W; ++q) S.row(c + 3, 2, q) = qdiv(T(1), rho0 * (rho0 + S.row(c + 3, 1, q)));
    }
    if constexpr (LEAD) {
      V F1 = rm[K1];
      if constexpr (FR != 0)
        if (X.y.is(c + 1)) F1 = X.y.get(0, c + 1, F1);
      const V out = fmav<V>(-(F1 - (FR ? rf : rm[K0])), V(ivol), S.rowv(c, 1));
      if (XB == 1 || Q.L.put) store(0, c, ic, out);
      if constexpr (W == 2 && (XB == 0 || XB == 3)) {
        if (Q.L.any_edge && Q.L.edge >= 0) store(0, c, ic + Q.L.edge, Q.L.edge ? out.y : out.x);
      }
      if (FR) rf = F1;
      rd[K1] = vleer(rr[K2] - rr[K1], rr[K1] - rr[K0]);
      rm[K2] = mass_y(rv[K0], rr[K0], rd[K0], rr[K1], rd[K1]);
      S.put_face(c + 2, rm[K2]);
      rv[K1] = face(min(c + 3, c1));
      rr[K0] = xy_lead_row<T, W, XB, FR>(Q, P, dt, S, c + 4, ldr, lda, A, X, c0, c1, lfn, false);
      lead_in(c + 5);
    }
    __syncthreads();
  };
  for (int c = c0; c < c1; c += 3) {
    step(std::integral_constant<int, 0>(), c);
    if (c + 1 < c1) step(std::integral_constant<int, 1>(), c + 1);
    if (c + 2 < c1) step(std::integral_constant<int, 2>(), c + 2);
  }
}

// Cells a tile (W = 2) stores: from its third to the fifth from its end, in
// pairs; the tails of a half or a quarter of a wave likewise.  A level-0 row's first tile stores its
// first two cells too (XY_EDGE), and one in which the row ends all up to the
// end: the cells past it are in the tile's lanes, or (under bc 1, in a whole
// tile) what the lane shifts bring in.
constexpr int XY_TILE = 2 * BX - 6, XY_EDGE = 2;
constexpr int xy_tail_cells(int parts) { return 2 * BX / parts - 6; }

// The tiles of rows of the cells [lo, hi): whole ones, then the cells past them
// in tiles of a half or a quarter of a wave, two or four planes to a wave (parts
// of a wave; 0: none).
struct XyTiles {
  int lo, hi;    // even: the pairs stored
  int xlo, xhi;  // and the cells of them, where the range ends inside a pair
  int ntiles, parts;
  long blocks(int np) const { return (long)np * ntiles + (parts ? (np + parts - 1) / parts : 0); }
};

template <typename T, int W, int XB, int FR>
__device__ __forceinline__ void xyshared_body(Geo G, Phys P, PassArgs<T> A, MarchArgs<T> M, XyTiles B, Blk bk) {
  constexpr int NG = 4;
  __shared__ T rows[XY_RS * 3 * W * 64];
  __shared__ T faces[XY_FS * W * 64];
  const int lane = threadIdx.x;
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.y);
  // blocks: of each y segment the planes' tiles, whole ones first
  const int np = M.hi[2] - M.lo[2], whole = np * B.ntiles, tails = B.parts ? (np + B.parts - 1) / B.parts : 0;
  const int ch = (int)(bk.id / (unsigned)(whole + tails)), w = (int)(bk.id % (unsigned)(whole + tails));
  const int c0 = M.lo[1] + ch * M.chunk;
  const int c1 = min(c0 + M.chunk, M.hi[1]);
  if (c0 >= c1) return;  // the whole block
  XyGrid<T, W, XB> Q;
  Q.G = &G;
  Q.rmax = G.n[1] + G.g - 2;
  constexpr bool level0 = XB != 0 && XB != 3;
  const bool whole_tile = w < whole;
  const int k = whole_tile ? w / np : B.ntiles;
  const int shift = whole_tile ? 6 : (B.parts == 2 ? 5 : 4);  // lanes of a tile: 64, 32 or 16
  const int lx = lane & ((1 << shift) - 1);
  const int p = whole_tile ? w % np : B.parts * (w - whole) + (lane >> shift);
  const int xs = B.lo + XY_TILE * k + (level0 ? XY_EDGE : 0) - 2;  // the tile's first cell
  Q.L.t = M.lo[2] + min(p, np - 1);  // (a part past the last plane walks it again, storing nothing)
  Q.L.x0 = xs + W * lx;
  const int px = (int)(G.off - (long)G.g * (G.sy + G.sz));
  Q.L.xl = clampi(Q.L.x0, -px, (int)G.sy - px - W);
  // the lanes after the tile's inexact first pair (the row's own end: none) and
  // before its inexact last two (none where the row ends in the tile)
  const int cells = W << shift;
  const bool ends = level0 && xs + cells >= G.n[0] + (XB == 2 || !whole_tile ? 2 : 0);
  Q.L.put = p < np && (lx >= 1 || (level0 && k == 0)) && (ends || lx < (1 << shift) - 2) && Q.L.x0 < B.hi;
  Q.L.edge = -1;
  if (!level0 && Q.L.put && (Q.L.x0 < B.xlo || Q.L.x0 + 1 >= B.xhi)) {
    Q.L.edge = Q.L.x0 < B.xlo ? 1 : 0;
    Q.L.put = false;
  }
  Q.L.any_edge = !level0 && __any(Q.L.edge >= 0);
  const T dt = (T)(A.fac * A.dtp[0]);
  const XyShare<T, W> S{rows, faces, lane};
  if (grp == 0) xy_shared_group<T, W, 0, NG, true, XB, FR>(Q, P, A, M, dt, c0, c1, S);
  else if (grp == 1) xy_shared_group<T, W, 1, NG, false, XB, FR>(Q, P, A, M, dt, c0, c1, S);
  else if (grp == 2) xy_shared_group<T, W, 2, NG, false, XB, FR>(Q, P, A, M, dt, c0, c1, S);
  else xy_shared_group<T, W, 3, NG, false, XB, FR>(Q, P, A, M, dt, c0, c1, S);
}

template <typename T, int W, int XB, int FR>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_xyshared(Geo G, Phys P, PassArgs<T> A, MarchArgs<T> M, XyTiles B) {
  xyshared_body<T, W, XB, FR>(G, P, A, M, B, grid_blk());
}

// ------------------------------------------------------------ CommUp

// The five state fields of one CommUp or CommMean in one launch: field f
// takes blocks [start[f], start[f+1]).
template <typename T>
struct UpArgs {
  const T *Q[NSTATE];  // coarse fields: rho, e, vx, vy, vz
  T *out[NSTATE];      // fine fields
  Box b;               // coarse hosts of the fine entries (every field)
  // hosts whose eight children are all active fine cells ([0, n/2) along each
  // axis, relative to b.lo) are not enumerated: the shell around them is, in
  // three parts -- the planes outside them (all rows), the rows outside them
  // in their planes, the hosts outside them in their rows
  int in_lo[3], in_n[3];
  unsigned c1, c2, nshell;
  unsigned nb;         // blocks per field of the shell
  // quadrant: then blocks that set the images of the active entries next to
  // the planes, numbered with j <= g first (all k), then j > g with k <= g
  unsigned ni;         // blocks per field of these
};

// A state entry (i, j, k) >= the mirror planes of a quadrant level: the images
// beyond them, val at the mirror position (a cell j at -1 - j, a face normal to
// the plane j at -j, reversed), within the ghost shell; stag: the field's face
// axis or -1.
template <typename T>
__device__ __forceinline__ void put_images(const Geo &G, T *a, int stag, int i, int j, int k, T val) {
  const int jm = stag == 1 ? -j : -1 - j, km = stag == 2 ? -k : -1 - k;
  const bool y = jm < 0 && jm >= -G.g, z = km < 0 && km >= -G.g;
  if (y) a[lin(G, i, jm, k)] = stag == 1 ? -val : val;
  if (z) a[lin(G, i, j, km)] = stag == 2 ? -val : val;
  if (y && z) a[lin(G, i, jm, km)] = stag >= 1 ? -val : val;
}

// element f of a five-entry argument array, for a wave-uniform f (a select
// chain rather than an indexed load of the kernel's arguments)
template <typename P>
__device__ __forceinline__ P pick5(const P (&a)[NSTATE], int f) {
  return f == 0 ? a[0] : f == 1 ? a[1] : f == 2 ? a[2] : f == 3 ? a[3] : a[4];
}

// CommUp (Sect. 3.2.1, Fig. 2): every fine entry outside the fine active set
// from the 27 coarse entries around its host, interpolating along z, then y,
// then x.  The background is uniform, so departures interpolate like values.
// One thread per coarse host: its eight fine children share the 27 coarse
// neighbours and, since the limited slope of a 1-D step does not depend on
// which half of the host a child takes, every slope is formed once for both
// children (19 slopes instead of 8 x 13).  A.b counts hosts relative to the
// covered coarse box (host H = Gc.co + h).
template <typename T, int CBC>
__global__ void __launch_bounds__(BX * BY) k_commup(Geo Gc, Geo Gf, UpArgs<T> UA) {
  const int fld = (int)(blockIdx.x / (UA.nb + UA.ni));
  struct {
    const T *Q;
    T *out;
    int stag;
  } A{pick5(UA.Q, fld), pick5(UA.out, fld), fld >= 2 ? fld - 2 : -1};
  int h[3];
  {
    unsigned f = (blockIdx.x % (UA.nb + UA.ni)) * (BX * BY) + threadIdx.y * BX + threadIdx.x;
    if (f >= UA.nb * (BX * BY)) {
      f -= UA.nb * (BX * BY);
      const unsigned nx = (unsigned)(Gf.n[0] + (A.stag == 0)), ny = (unsigned)(Gf.n[1] + (A.stag == 1)),
                     nz = (unsigned)(Gf.n[2] + (A.stag == 2)), w = (unsigned)min(Gf.g + 1, (int)ny),
                     wz = (unsigned)min(Gf.g + 1, (int)nz);
      const unsigned n1 = nx * w * nz, n2 = nx * (ny - w) * wz;
      if (f >= n1 + n2) return;
      const bool lo = f < n1;
      const unsigned g = lo ? f : f - n1, rows = lo ? w : ny - w;
      const int i = (int)(g % nx), j = (int)(g / nx % rows + (lo ? 0 : w)), k = (int)(g / (nx * rows));
      put_images(Gf, A.out, A.stag, i, j, k, A.out[lin(Gf, i, j, k)]);
      return;
    }
    if (f >= UA.nshell) return;
    const unsigned X = (unsigned)(UA.b.hi[0] - UA.b.lo[0]), Y = (unsigned)(UA.b.hi[1] - UA.b.lo[1]);
    unsigned x, y, z;
    if (f < UA.c1) {
      z = f / (X * Y);
      y = (f % (X * Y)) / X;
      x = f % X;
      if ((int)z >= UA.in_lo[2]) z += UA.in_n[2];
    } else if (f < UA.c2) {
      const unsigned g = f - UA.c1, ny = Y - UA.in_n[1];
      z = UA.in_lo[2] + g / (ny * X);
      y = (g % (ny * X)) / X;
      x = g % X;
      if ((int)y >= UA.in_lo[1]) y += UA.in_n[1];
    } else {
      const unsigned g = f - UA.c2, nx = X - UA.in_n[0];
      z = UA.in_lo[2] + g / (UA.in_n[1] * nx);
      y = UA.in_lo[1] + (g % (UA.in_n[1] * nx)) / nx;
      x = g % nx;
      if ((int)x >= UA.in_lo[0]) x += UA.in_n[0];
    }
    h[0] = UA.b.lo[0] + (int)x;
    h[1] = UA.b.lo[1] + (int)y;
    h[2] = UA.b.lo[2] + (int)z;
  }
  // children 2h, 2h+1 along each axis; the host is skipped when all eight are
  // active entries (which the fine level owns)
  bool inner = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int hi = Gf.n[d] + (d == A.stag ? 1 : 0);
    if (2 * h[d] < 0 || 2 * h[d] + 1 >= hi) inner = false;
  }
  if (inner) return;
  const int H0 = Gc.co[0] + h[0], H1 = Gc.co[1] + h[1], H2 = Gc.co[2] + h[2];
  auto C = [&](int a, int b, int cc) -> T {
    const int ci = H0 + a, cj = H1 + b, ck = H2 + cc;
    if (CBC) {
      if (A.stag < 0) return cread<CBC>(A.Q, Gc, ci, cj, ck);
      return fread_bc<CBC>(A.Q, Gc, A.stag, ci, cj, ck);
    }
    return A.Q[lin(Gc, ci, cj, ck)];
  };
  // both children of one 1-D step of the prolongation, from three
  // consecutive coarse values around the host: on centred axes a quarter
  // coarse cell either side of the host centre with van Leer's limited slope;
  // along a face field's own axis the even child is the host face, the odd
  // one the mean of the host face and the next
  auto up2 = [&](bool stag_axis, T m, T c, T p, T &lo, T &hi) {
    if (stag_axis) {
      lo = c;
      hi = T(0.5) * (c + p);
    } else {
      const T sl = vleer(p - c, c - m);
      lo = c + sl * T(-0.25);
      hi = c + sl * T(0.25);
    }
  };
  T qz[2][3][3];  // [z child][x offset][y offset]
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) up2(A.stag == 2, C(a - 1, b - 1, -1), C(a - 1, b - 1, 0), C(a - 1, b - 1, 1),
                                    qz[0][a][b], qz[1][a][b]);
  T r[2][2][3];  // [z child][y child][x offset]
#pragma unroll
  for (int o2 = 0; o2 < 2; ++o2)
#pragma unroll
    for (int a = 0; a < 3; ++a) up2(A.stag == 1, qz[o2][a][0], qz[o2][a][1], qz[o2][a][2], r[o2][0][a], r[o2][1][a]);
#pragma unroll
  for (int o2 = 0; o2 < 2; ++o2)
#pragma unroll
    for (int o1 = 0; o1 < 2; ++o1) {
      T v[2];
      up2(A.stag == 0, r[o2][o1][0], r[o2][o1][1], r[o2][o1][2], v[0], v[1]);
      const int k = 2 * h[2] + o2, j = 2 * h[1] + o1;
#pragma unroll
      for (int o0 = 0; o0 < 2; ++o0) {
        const int i = 2 * h[0] + o0;
        const int id[3] = {i, j, k};
        bool in = true, active = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          if (id[d] < -Gf.g || id[d] >= Gf.s[d] - Gf.g) in = false;
          if (id[d] < 0 || id[d] >= Gf.n[d] + (d == A.stag ? 1 : 0)) active = false;
        }
        if (in && !active) {
          A.out[lin(Gf, i, j, k)] = v[o0];
          if (UA.ni) put_images(Gf, A.out, A.stag, i, j, k, v[o0]);
        }
      }
    }
}

// ------------------------------------------------------ quadrant images
// The entries of a finer level beyond an anchored face (the perturber's mirror
// plane, Sect. 3.4) as the mirror images of the level's own entries:
// dst = sgn src at the mirror position -- cell j < 0 takes cell -1-j, a face
// normal to the plane j < 0 takes face -j.  One launch per plane, every
// listed field at each position.
template <typename T>
struct MirArgs {
  T *dst[NQ];
  const T *src[NQ];
  T sgn[NQ];
  int face[NQ];  // the field lives on the faces normal to the plane
  int nf;
  int d;         // the plane's normal (1 or 2)
  Box b;         // the entries beyond the plane
};

template <typename T>
__global__ void __launch_bounds__(BX * BY) k_mirror(Geo G, MirArgs<T> A) {
  int i, j, k;
  if (!thread_cell_flat(A.b, i, j, k)) return;
  const int id[3] = {i, j, k};
  const int m = id[A.d];  // < 0
  const idx_t c = lin(G, i, j, k), sd = dstride(G, A.d);
  for (int f = 0; f < A.nf; ++f) {
    const idx_t src = A.face[f] ? c - 2 * m * sd : c + (-1 - 2 * m) * sd;
    A.dst[f][c] = A.sgn[f] * A.src[f][src];
  }
}

// ------------------------------------------------------------ CommMean

template <typename T>
struct MeanArgs {
  const T *Q[NSTATE];      // fine fields
  T *out[NSTATE];          // coarse fields
  Box b;                   // covered coarse cells, relative to the covered box (faces: one more
                           // along their normal)
  unsigned start[NSTATE + 1];
};

// CommMean (Sect. 3.2.2): covered coarse cells take the mean of their 8 fine
// cells, covered coarse faces the mean of their 4 coincident fine faces.
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_commmean(Geo Gf, Geo Gc, MeanArgs<T> MA) {
  const unsigned h = blockIdx.x;
  const int fld = h < MA.start[1] ? 0 : h < MA.start[2] ? 1 : h < MA.start[3] ? 2 : h < MA.start[4] ? 3 : 4;
  const unsigned s0 = fld == 0 ? 0u : fld == 1 ? MA.start[1] : fld == 2 ? MA.start[2] : fld == 3 ? MA.start[3] : MA.start[4];
  const unsigned s1 = fld == 0 ? MA.start[1] : fld == 1 ? MA.start[2] : fld == 2 ? MA.start[3] : fld == 3 ? MA.start[4]
                                                                                                 : MA.start[5];
  struct {
    const T *Q;
    T *out;
    int stag;
  } A{pick5(MA.Q, fld), pick5(MA.out, fld), fld >= 2 ? fld - 2 : -1};
  Box bb = MA.b;
  bb.hi[0] += A.stag == 0 ? 1 : 0;
  bb.hi[1] += A.stag == 1 ? 1 : 0;
  bb.hi[2] += A.stag == 2 ? 1 : 0;
  int I, J, K;
  if (!thread_cell_flat(bb, I, J, K, Blk{h - s0, s1 - s0})) return;
  const idx_t f = lin(Gf, 2 * I, 2 * J, 2 * K);
  const T *q = A.Q;
  T val;
  if (A.stag < 0) {
    const idx_t sx = 1, sy = (idx_t)Gf.sy, sz = (idx_t)Gf.sz;
    val = (((q[f] + q[f + sx]) + (q[f + sy] + q[f + sx + sy])) +
           ((q[f + sz] + q[f + sx + sz]) + (q[f + sy + sz] + q[f + sx + sy + sz]))) * T(0.125);
  } else {
    const idx_t e1 = (A.stag == 0) ? (idx_t)Gf.sy : 1;
    const idx_t e2 = (A.stag == 2) ? (idx_t)Gf.sy : (idx_t)Gf.sz;
    val = ((q[f] + q[f + e1]) + (q[f + e2] + q[f + e1 + e2])) * T(0.25);
  }
  const int ci = Gc.co[0] + I, cj = Gc.co[1] + J, ck = Gc.co[2] + K;
  A.out[lin(Gc, ci, cj, ck)] = val;
  // a quadrant level's images of the cells overwritten (level 0 stores none)
  if (Gc.level > 0 && Gc.anch[1]) put_images(Gc, A.out, A.stag, ci, cj, ck, val);
}

// -------------------------------------------------------------- reductions

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

template <typename T>
struct RedArgs {
  Box b;
  const T *rho, *e, *v[3];
  double *part;              // per-block partials: three planes of npart values
  double *spart;             // per-block maximum signal speeds
  int npart;                 // partial slots per plane (the blocks of the one-cell-per-thread grid)
  Scal *S;
  int cov_lo[3], cov_hi[3];  // covered cells (empty if no finer level)
};

template <typename T>
__device__ __forceinline__ bool is_covered(const RedArgs<T> &A, int i, int j, int k) {
  return i >= A.cov_lo[0] && i < A.cov_hi[0] && j >= A.cov_lo[1] && j < A.cov_hi[1] && k >= A.cov_lo[2] &&
         k < A.cov_hi[2];
}

// block sum of three values into part[q * blocks + block]; fixed order for a fixed grid
__device__ void block_sum3(double a, double b, double c, double *part, int npart, Blk bk = grid_blk()) {
  __shared__ double sh[3][BX * BY / 64];
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int t = threadIdx.y * BX + threadIdx.x;
  const int w = t / 64, l = t % 64;
  if (l == 0) {
    sh[0][w] = a;
    sh[1][w] = b;
    sh[2][w] = c;
  }
  __syncthreads();
  if (t == 0) {
    const long blk = bk.id;
    double s0 = 0, s1 = 0, s2 = 0;
    for (int q = 0; q < BX * BY / 64; ++q) {
      s0 += sh[0][q];
      s1 += sh[1][q];
      s2 += sh[2][q];
    }
    // three planes of one value per block (coalesced for the final sum)
    const long nb = npart;
    part[blk] = s0;
    part[nb + blk] = s1;
    part[2 * nb + blk] = s2;
  }
}

// Force of the gas on the perturber, eq. 18: G M (rho - rho0) dV r /
// (r^2+eps^2)^{3/2} over uncovered active cells, in FP64 (the uniform part
// sums to zero by symmetry).
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_force(Geo G, Phys P, RedArgs<T> A) {
  int i, j, k;
  const bool ok = thread_cell(A.b, i, j, k);
  double fx = 0.0, fy = 0.0, fz = 0.0;
  if (ok && !is_covered(A, i, j, k)) {
    const double x = xcen<double>(G, 0, i), y = xcen<double>(G, 1, j), z = xcen<double>(G, 2, k);
    const double d2 = x * x + y * y + z * z + P.eps2;
    const double vol = G.dx * G.dx * G.dx;
    const double w = P.GM * (double)A.rho[lin(G, i, j, k)] * vol / (d2 * sqrt(d2));
    fx = w * x;
    fy = w * y;
    fz = w * z;
  }
  block_sum3(fx, fy, fz, A.part, A.npart);
}

// mass, internal energy and kinetic energy (face velocities averaged to
// centres), FP64
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_totals(Geo G, Phys P, RedArgs<T> A) {
  int i, j, k;
  const bool ok = thread_cell(A.b, i, j, k);
  double m = 0.0, ei = 0.0, ek = 0.0;
  if (ok && !is_covered(A, i, j, k)) {
    const idx_t c = lin(G, i, j, k);
    const double vol = G.dx * G.dx * G.dx;
    const double r = P.rho0 + (double)A.rho[c];
    double v2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double vc = vback(P, d) + 0.5 * ((double)A.v[d][c] + (double)A.v[d][c + dstride(G, d)]);
      v2 += vc * vc;
    }
    m = r * vol;
    ei = (P.e0 + (double)A.e[c]) * vol;
    ek = 0.5 * r * v2 * vol;
  }
  block_sum3(m, ei, ek, A.part, A.npart);
}

// fixed-order sum of the partials of all levels (one block)
struct FinalArgs {
  const double *part[MAXLEV];
  int npart[MAXLEV];
  int nl;
  double *out;   // 3 doubles
  Scal *S;       // with flog: append (out, t) to the ring
  double *flog;
};

// The one-block kernels that finish a reduction run FT threads: each reads
// its partials (blocks t, t+FT, ...) eight at a time, so that all partials
// of a 128^3 level are in flight at once; the order of the sum is fixed.
constexpr int FT = 1024;
constexpr int FW = FT / 64;

// thread 0: the wave sums sh (in wave order) into out, then the log entry
__device__ void final3_finish(const FinalArgs &A, const double (*sh)[FW]) {
  for (int q = 0; q < 3; ++q) {
    double t = 0.0;
    for (int v = 0; v < FW; ++v) t += sh[q][v];
    A.out[q] = t * (A.out == A.S->totals ? A.S->tmul : A.S->fmul[q]);
  }
  if (A.flog) {
    const unsigned int n = A.S->nlog;
    double *e = A.flog + 4 * (size_t)(n % FLOG);
    for (int q = 0; q < 3; ++q) e[q] = A.out[q];
    e[3] = A.S->t;
    A.S->nlog = n + 1;
    A.S->pending = 0;
  }
}

__device__ void final3_body(const FinalArgs &A) {
  __shared__ double sh[3][FW];
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  for (int l = 0; l < A.nl; ++l) {
    const double *p = A.part[l];
    const int n = A.npart[l];
    int b = threadIdx.x;
    for (; b + 7 * FT < n; b += 8 * FT) {
      double x[8][3];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < 3; ++q) x[u][q] = p[(size_t)q * n + b + u * FT];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s0 += x[u][0];
        s1 += x[u][1];
        s2 += x[u][2];
      }
    }
    for (; b < n; b += FT) {
      s0 += p[b];
      s1 += p[(size_t)n + b];
      s2 += p[2 * (size_t)n + b];
    }
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  const int w = threadIdx.x / 64;
  if (threadIdx.x % 64 == 0) {
    sh[0][w] = s0;
    sh[1][w] = s1;
    sh[2][w] = s2;
  }
  __syncthreads();
  if (threadIdx.x == 0) final3_finish(A, sh);
  __syncthreads();
}

__global__ void __launch_bounds__(FT) k_final3(FinalArgs A) { final3_body(A); }

// A pending end-of-step force (single-level runs): the fixed-order sum of the
// three planes of partials by the NT threads of one block, into S->force and
// the log at the time S->tlog of its state; every thread calls it.
template <int NT>
__device__ void log_pending_body(const double *part, int n, Scal *S, double *flog) {
  constexpr int NW = NT / 64;
  __shared__ double sh[3][NW];
  const int tid = threadIdx.y * blockDim.x + threadIdx.x;
  if (!S->pending) return;  // the same value for every thread of the block
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  int b = tid;
  for (; b + 7 * NT < n; b += 8 * NT) {
    double x[8][3];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) x[u][q] = part[(size_t)q * n + b + u * NT];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      s0 += x[u][0];
      s1 += x[u][1];
      s2 += x[u][2];
    }
  }
  for (; b < n; b += NT) {
    s0 += part[b];
    s1 += part[(size_t)n + b];
    s2 += part[2 * (size_t)n + b];
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  if (tid % 64 == 0) {
    sh[0][tid / 64] = s0;
    sh[1][tid / 64] = s1;
    sh[2][tid / 64] = s2;
  }
  __syncthreads();
  if (tid == 0) {
    const unsigned int k = S->nlog;
    double *e = flog + 4 * (size_t)(k % FLOG);
    for (int q = 0; q < 3; ++q) {
      double t = 0.0;
      for (int v = 0; v < NW; ++v) t += sh[q][v];
      t *= S->fmul[q];
      S->force[q] = t;
      e[q] = t;
    }
    e[3] = S->tlog;
    S->nlog = k + 1;
    S->pending = 0;
  }
}

__global__ void __launch_bounds__(FT) k_log_pending(const double *part, int n, Scal *S, double *flog) {
  log_pending_body<FT>(part, n, S, flog);
}

// Signal speed c_s + |v| of an active cell, the largest over its six faces,
// and whether its density and energy are positive and finite.
template <typename T>
__device__ __forceinline__ double cell_signal(const Geo &G, const Phys &P, const RedArgs<T> &A, idx_t c,
                                              int &bad) {
  const double r = P.rho0 + (double)A.rho[c], en = P.e0 + (double)A.e[c];
  if (!(r > 0.0) || !(en > 0.0) || !isfinite(r) || !isfinite(en)) bad = 1;
  const double cs = sqrt(P.gamma * P.gm1 * en / r);
  double vm = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double a = fabs(vback(P, d) + (double)A.v[d][c]);
    const double b = fabs(vback(P, d) + (double)A.v[d][c + dstride(G, d)]);
    vm = fmax(vm, fmax(a, b));
  }
  const double sig = cs + vm;
  if (!isfinite(sig)) bad = 1;
  return sig;
}

// block maximum of the signal speeds into spart[block]; a bad cell raises
// the health flag
__device__ void block_signal(double sig, int bad, double *spart, Scal *S, Blk bk = grid_blk()) {
  sig = wave_max(bad ? 0.0 : sig);
  const bool anybad = __any(bad);
  __shared__ double sh[BX * BY / 64];
  const int t = threadIdx.y * BX + threadIdx.x;
  if ((t % 64) == 0) {
    sh[t / 64] = sig;
    if (anybad) atomicOr(&S->health, 1);
  }
  __syncthreads();
  if (t == 0) {
    double m = sh[0];
    for (int q = 1; q < BX * BY / 64; ++q) m = fmax(m, sh[q]);
    spart[bk.id] = m;
    // the same maximum into this block's slot (m >= 0, so the order of the
    // bits is that of the values)
    if (S)
      __hip_atomic_fetch_max(&S->smax[bk.id & (NSLOT - 1)], (unsigned long long)__double_as_longlong(m),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Largest signal speed over the active cells and their faces (per block,
// reduced by the final kernel), and the health check.
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_signal(Geo G, Phys P, RedArgs<T> A) {
  int i, j, k;
  const bool ok = thread_cell(A.b, i, j, k);
  double sig = 0.0;
  int bad = 0;
  if (ok) sig = cell_signal(G, P, A, lin(G, i, j, k), bad);
  block_signal(sig, bad, A.spart, A.S);
}

// End of a step: the force partials of eq. 18 (as k_force) and the signal
// speed partials of the next step's time step (as k_signal) in one pass over
// the state, which both read.
template <typename T>
__global__ void __launch_bounds__(BX * BY) k_post(Geo G, Phys P, RedArgs<T> A) {
  int i, j, k;
  const bool ok = thread_cell(A.b, i, j, k);
  double fx = 0.0, fy = 0.0, fz = 0.0, sig = 0.0;
  int bad = 0;
  if (ok) {
    const idx_t c = lin(G, i, j, k);
    sig = cell_signal(G, P, A, c, bad);
    if (!is_covered(A, i, j, k)) {
      const double x = xcen<double>(G, 0, i), y = xcen<double>(G, 1, j), z = xcen<double>(G, 2, k);
      const double d2 = x * x + y * y + z * z + P.eps2;
      const double vol = G.dx * G.dx * G.dx;
      const double w = P.GM * (double)A.rho[c] * vol / (d2 * sqrt(d2));
      fx = w * x;
      fy = w * y;
      fz = w * z;
    }
  }
  block_sum3(fx, fy, fz, A.part, A.npart);
  block_signal(sig, bad, A.spart, A.S);
}

// Level-0 form of the kick (rows of even length, as every level-0 mesh has):
// one thread per pair of adjacent active cells (the box's x range counts
// pairs) computes the faces on the low side of both cells and, for the last
// cells along a dimension, also the boundary face n there (the injection face
// at x_max carries the wind), so the grid is exactly the active box.  The
// pair's own fields and its y and z neighbours move as 8- or 16-byte
// accesses; the two low x faces take the cell before the pair and the pair
// itself.  With POST (the last kernel of a single-level step) it also forms
// the end-of-step reductions of k_post: the force partials of its cells, and
// the signal speed c_s + |v| of every pair of an active cell and one of its
// faces, taken at the face's owner (the cell on its high side, or the last
// cell for face n), which holds both adjacent cells' densities and energies.
// A block then covers the cells of up to two blocks of the one-cell-per-thread
// grid whose blocks k_post and the final sums count: it writes its partials to
// slot blockIdx.x and zeros to slot gridDim.x + blockIdx.x (when that is below
// npart).  With COMP (the first kick of a step) it then compresses its cells
// as k_compress2 does, from the kicked velocities of their six faces: the high
// faces that other threads own (x face i+2, y face j+1, z face k+1) it kicks
// again itself with their owners' arithmetic (they are not written); the
// compressed energy goes to A.eo.
// (five waves per SIMD: the FP64 end-of-step form fits 93 registers with no
// spill, against 104 and four waves unconstrained)
template <typename T, int BCM, bool REBUILD, bool KICK, bool POST, bool COMP>
__device__ __forceinline__ void kick0p_body(Geo G, Phys P, KickArgs<T> A, RedArgs<T> R, Blk bk) {
  using V = typename lanes_of<T, 2>::type;
  int p, j, k;
  const bool ok = thread_cell_flat(A.b, p, j, k, bk);
  // with COMP in FP64, a block whose threads all hold pairs (the same for
  // all its threads) hands each pair's low y faces to the pairs below them in
  // the block, which then need not kick their high y faces again (128^3: the
  // FP64 step 0.7 % faster; in FP32, where the kick is cheap, no faster)
  const int tid = threadIdx.y * BX + threadIdx.x;
  const int exb = A.b.hi[0] - A.b.lo[0];
  const long fl = (long)(j - A.b.lo[1]) * exb + (p - A.b.lo[0]);
  const bool full = COMP && sizeof(T) == 8 && fl - tid + BX * BY <= (long)exb * (A.b.hi[1] - A.b.lo[1]);
  const bool yx = full && tid + exb < BX * BY;
  double fx = 0.0, fy = 0.0, fz = 0.0;
  T sig = T(0);
  int bad = 0;
  // the step length: as dt_body (one level), from the slots of the last
  // end-of-step pass; the first thread records it and advances the time
  double dtk = 0.0;
  if (A.slots) {
    __shared__ double shs[BX * BY / 64];
    double m = 0.0;
    for (int q = tid; q < NSLOT; q += BX * BY) m = fmax(m, __longlong_as_double((long long)A.slots->smax[q]));
    m = wave_max(m);
    if (tid % 64 == 0) shs[tid / 64] = m;
    __syncthreads();
    double smax = shs[0];
#pragma unroll
    for (int q = 1; q < BX * BY / 64; ++q) smax = fmax(smax, shs[q]);
    double dtl = G.dx / smax;
    if (P.chi > 0.0) dtl = fmin(dtl, G.dx * G.dx / (6.0 * P.chi));
    dtk = P.cfl * dtl;
    if (bk.id == 0 && threadIdx.x == 0 && threadIdx.y == 0) {
      A.slots->dtl[0] = P.cfl * dtl;
      A.slots->dt[0] = dtk;
      A.slots->t += dtk;
    }
  }
  if (POST && bk.id == 0 && threadIdx.x == 0 && threadIdx.y == 0) {
    R.S->tlog = R.S->t;  // the force partials of this state await the log
    R.S->pending = 1;
  }
  if (ok) {
    const int i = 2 * p;
    const T h = (T)(A.fac * (A.slots ? dtk : A.dtp[0]));
    const T rho0 = (T)P.rho0, gm1 = (T)P.gm1, GM = (T)P.GM, eps2 = (T)P.eps2, dx = (T)G.dx;
    const T *rho = A.q[0], *e = A.q[1];
    const int id[3] = {i, j, k};
    const idx_t c = lin(G, i, j, k);
    const V drc = gldv<V>(rho, c), dec = gldv<V>(e, c);
    V xcx;
    xcx.x = xcen<T>(G, 0, i);
    xcx.y = xcen<T>(G, 0, i + 1);
    const T yc = xcen<T>(G, 1, j), zc = xcen<T>(G, 2, k);
    // squared softened distance of cells at (xv, y, z): every cell's distance
    // is formed by this one expression, whichever thread needs it
    auto r2of = [&](V xv, T y, T z) -> V { return xv * xv + y * y + z * z + eps2; };
    const V r2c = r2of(xcx, yc, zc);
    const V dcen = qsqrtv(r2c);
    const T gg = (T)(P.gamma * P.gm1), e0 = (T)P.e0;
    // pair p-1 is the lane before, unless this is the wave's first lane (BX is
    // the wave width) or p the row's first pair (flat tiles)
    const int lane = threadIdx.x;
    auto sound1 = [&](T dr, T de) -> T {
      const T r = rho0 + dr, en = e0 + de;
      if (!(r > T(0)) || !(en > T(0)) || !isfinite(r) || !isfinite(en)) bad = 1;
      return qsqrt(qdiv(gg * en, r));
    };
    auto sound = [&](V dr, V de) -> V {
      V s;
      s.x = sound1(dr.x, de.x);
      s.y = sound1(dr.y, de.y);
      return s;
    };
    auto vmax = [&](V a) { sig = fmax(sig, fmax(a.x, a.y)); };
    auto vabs = [&](V a) -> V {
      V r;
      r.x = fabs(a.x);
      r.y = fabs(a.y);
      return r;
    };
    V cs_own = V(0);
    if (POST) cs_own = sound(drc, dec);
    const T csprev = POST ? dpp_fill<DPP_WAVE_SHR1>(cs_own.y, T(0)) : T(0);
    // the kick of a face pair: cells below (drm, dem) and above (dcr, der) the
    // faces, the coordinate along d of the cell above (xr; the cell below is
    // at xr - dx) and the distances of the cells below (dm) and above (dr_)
    auto kickv = [&](int d, V vf, V drm, V dem, V dcr, V der, V xr, V dm, V dr_) -> V {
      if (KICK) {
        const V rface = rho0 + T(0.5) * (drm + dcr);
        const V gradp = qdiv(gm1 * (der - dem), dx * rface);
        const V xm = xr - dx;
        const V gradphi = qdiv(GM * (xr + xm), dm * dr_ * (dm + dr_));
        vf = vf - h * (gradp + gradphi);
      }
      return vf;
    };
    // the own cells' distances and sound speeds shifted by one lane: lane l
    // gets pair l-1's second cell, cell i-1 (lane 0 forms it itself)
    const T dprev = dpp_fill<DPP_WAVE_SHR1>(dcen.y, T(0));
    auto rebuild = [&](int d, V ppm, V pmc, V drm, V dcr) -> V {
      const T vb = (T)vback(P, d);
      return qdiv(ppm + pmc - vb * (drm + dcr), T(2) * rho0 + drm + dcr);
    };
    // kicked velocities of the low faces of both cells and, with COMP, of
    // their high faces
    V vlo[3], vhi[3];
    // x: faces i and i+1; below them cell i-1 (the own cell i again at x = 0,
    // the background under bc 2) and cell i
    {
      V drm, dem, ppm;
      drm.y = drc.x;
      dem.y = dec.x;
      const T *pm = A.q[2], *pp = A.q[3];
      if (i > 0) {
        drm.x = gld(rho, c - 1);
        dem.x = gld(e, c - 1);
      } else if (BCM == 2) {
        drm.x = T(0);
        dem.x = T(0);
      } else {
        drm.x = drc.x;
        dem.x = dec.x;
      }
      V vf;
      if (REBUILD) {
        const V ppc = gldv<V>(pp, c);
        ppm.y = ppc.x;
        ppm.x = i > 0 ? gld(pp, c - 1) : (BCM == 2 ? T(0) : ppc.x);
        vf = rebuild(0, ppm, gldv<V>(pm, c), drm, drc);
      } else {
        vf = gldv<V>(A.vin[0], c);
      }
      V dmx;
      dmx.y = dcen.x;
      if (i > 0 && lane > 0) {
        dmx.x = dprev;
      } else {
        V xb;
        xb.x = xcen<T>(G, 0, i - 1);  // cell i-1 (a ghost position at x = 0)
        xb.y = xb.x;
        dmx.x = qsqrtv(r2of(xb, yc, zc)).x;
      }
      vf = kickv(0, vf, drm, dem, drc, dec, xcx, dmx, dcen);
      gstv<V>(A.v[0], c, vf);
      vlo[0] = vf;
      if (POST) {
        const V a = vabs((T)vback(P, 0) + vf);
        vmax(a + cs_own);
        if (i > 0) sig = fmax(sig, a.x + (lane > 0 ? csprev : sound1(drm.x, dem.x)));
        sig = fmax(sig, a.y + cs_own.x);
      }
      if (i + 1 == G.n[0] - 1) {
        A.v[0][c + 2] = T(0);  // injection face at x_max carries the wind
        if (POST) sig = fmax(sig, fabs((T)vback(P, 0)) + cs_own.y);
      }
    }
    // y and z: the low faces of both cells, then face n after the last ones
#pragma unroll
    for (int d = 1; d < 3; ++d) {
      const idx_t sd = dstride(G, d);
      const T xd = d == 1 ? yc : zc;
      const T *pm = A.q[2 + 2 * d], *pp = A.q[3 + 2 * d];
      if (BCM == 2 && id[d] == 0) {
        gstv<V>(A.v[d], c, V(0));  // a wall: no normal velocity
        vlo[d] = V(0);
        if (POST) vmax(cs_own);
      } else {
        const idx_t cm = id[d] > 0 ? c - sd : c;
        const V drm = gldv<V>(rho, cm), dem = gldv<V>(e, cm);
        V vf = REBUILD ? rebuild(d, gldv<V>(pp, cm), gldv<V>(pm, c), drm, drc) : gldv<V>(A.vin[d], c);
        // the cell below id (a ghost position at id = 0)
        const T xb = xcen<T>(G, d, id[d] - 1);
        const V dmb = qsqrtv(d == 1 ? r2of(xcx, xb, zc) : r2of(xcx, yc, xb));
        vf = kickv(d, vf, drm, dem, drc, dec, V(xd), dmb, dcen);
        gstv<V>(A.v[d], c, vf);
        vlo[d] = vf;
        if (POST) {
          const V a = vabs((T)vback(P, d) + vf);
          vmax(a + cs_own);
          if (id[d] > 0) vmax(a + sound(drm, dem));
        }
      }
      if (id[d] == G.n[d] - 1) {
        const idx_t cf = c + sd;
        if (BCM == 2) {
          gstv<V>(A.v[d], cf, V(0));  // a wall
          vhi[d] = V(0);
          if (POST) vmax(cs_own);
        } else {
          // both sides read the last cells (zero-gradient outflow)
          const T xr = xcen<T>(G, d, id[d] + 1);
          const V dr_ = qsqrtv(d == 1 ? r2of(xcx, xr, zc) : r2of(xcx, yc, xr));
          V vf = REBUILD ? rebuild(d, gldv<V>(pp, c), gldv<V>(pm, c), drc, drc) : gldv<V>(A.vin[d], cf);
          vf = kickv(d, vf, drc, dec, drc, dec, V(xr), dcen, dr_);
          gstv<V>(A.v[d], cf, vf);
          vhi[d] = vf;
          if (POST) vmax(vabs((T)vback(P, d) + vf) + cs_own);
        }
      } else if (COMP && !(d == 1 && yx)) {
        // face id+1: the low face of the next cells, kicked as their thread
        // does (the own cells below it)
        const idx_t cn = c + sd;
        const T xn = xcen<T>(G, d, id[d] + 1);
        const V r2n = d == 1 ? r2of(xcx, xn, zc) : r2of(xcx, yc, xn);
        vhi[d] = kickv(d, gldv<V>(A.vin[d], cn), drc, dec, gldv<V>(rho, cn), gldv<V>(e, cn), V(xn), dcen,
                       qsqrtv(r2n));
      }
    }
    if (COMP && full) {
      // the pairs above in the block: their low y faces (every thread of a
      // full block is here)
      __shared__ V ylo[BX * BY];
      ylo[tid] = vlo[1];
      __syncthreads();
      if (yx && id[1] != G.n[1] - 1) vhi[1] = ylo[tid + exb];
    }
    if (COMP) {
      // x face i+2: the injection face (a zero departure) at x_max, else the
      // first face of the next pair: the next lane's (it holds that pair
      // unless this is the wave's last lane; a lane past the box holds none,
      // but then this pair is the row's last), else kicked here as the next
      // pair's thread does
      const T vnext = dpp_fill<DPP_WAVE_SHL1>(vlo[0].x, T(0));
      V vx1;
      vx1.x = vlo[0].y;
      if (i + 2 == G.n[0]) {
        vx1.y = T(0);
      } else if (lane < BX - 1) {
        vx1.y = vnext;
      } else {
        const idx_t cn = c + 2;
        const T xn = xcen<T>(G, 0, i + 2);
        const V xnv = V(xn);
        vx1.y = kickv(0, V(gld(A.vin[0], cn)), V(drc.y), V(dec.y), V(gld(rho, cn)), V(gld(e, cn)), xnv,
                      V(dcen.y), qsqrtv(r2of(xnv, yc, zc))).x;
      }
      // compression over the step (as k_compress2)
      const T dtc = (T)(A.cfac * (A.slots ? dtk : A.dtp[0]));
      const V divv = qdiv((vx1 - vlo[0]) + (vhi[1] - vlo[1]) + (vhi[2] - vlo[2]), V(dx));
      const V a = T(0.5) * gm1 * dtc * divv;
      gstv<V>(A.eo, c, qdiv(dec * (T(1) - a) - T(2) * a * (T)P.e0, T(1) + a));
    }
    if (POST) {
      // force of the gas in these cells on the perturber, eq. 18: each cell's
      // term in the storage type, the sum in FP64
      const V w = qdiv(GM * drc * (dx * dx * dx), r2c * dcen);
      fx = (double)(w.x * xcx.x) + (double)(w.y * xcx.y);
      fy = (double)(w.x * yc) + (double)(w.y * yc);
      fz = (double)(w.x * zc) + (double)(w.y * zc);
      if (!isfinite(sig)) bad = 1;
    }
  }
  if (COMP && A.log && bk.id == 0) log_pending_body<BX * BY>(A.part, A.npart, A.log, A.flog);
  if (POST) {
    block_sum3(fx, fy, fz, R.part, R.npart, bk);
    block_signal((double)sig, bad, R.spart, R.S, bk);
    if (threadIdx.x == 0 && threadIdx.y == 0)
      for (unsigned z = bk.n + bk.id; z < (unsigned)R.npart; z += bk.n) {
        R.part[z] = 0.0;
        R.part[R.npart + z] = 0.0;
        R.part[2 * (size_t)R.npart + z] = 0.0;
        R.spart[z] = 0.0;
      }
  }
}

template <typename T, int BCM, bool REBUILD, bool KICK, bool POST, bool COMP = false>
__global__ void __launch_bounds__(BX * BY) __attribute__((amdgpu_waves_per_eu(5)))
k_kick0p(Geo G, Phys P, KickArgs<T> A, RedArgs<T> R) {
  kick0p_body<T, BCM, REBUILD, KICK, POST, COMP>(G, P, A, R, grid_blk());
}

// ------------------------------------------ z pass fused with the step's end
//
// The z pass, the velocity rebuild and the second half kick S(dt/2) of eq. 15
// in one launch: of a level-0 step without a finer level (bc 1), with the
// end-of-step reductions, or of a finer level's step, with its frontier
// transfers and within its margins.  One block per (band of ZF_TY rows, z
// segment), 3 ZF_TY + 1 waves (or one more, zf_zwave), each lane holding two
// adjacent cells of a row; long rows take several blocks, whose tiles overlap
// by a pair, and short ones share a wave, two or four bands to a block:
//  - per band row two walker waves stream the z pass's column segments
//    (march_column, groups {rho, e, P-x, P+x} and {P-y, P+y, P-z, P+z}), and
//    one more walker takes the row below the band ({rho, e, P+y}: the first
//    row's y faces need that row's new values);
//  - per band row one finisher wave takes each plane's new departures from
//    LDS and does what k_kick0p's end-of-step form does: rebuilds the face
//    velocities of its cells' low faces (and of the boundary faces after the
//    last cells), kicks them, forms the signal speeds and the force partials.
// Walkers write plane k into one of two LDS buffers and a barrier hands it
// over: the finishers work on plane k while the walkers compute plane k+1.
// The walk starts one plane below the segment, so that the segment's first
// z faces have their lower cells.  Only the new density and energy (written
// by the first group's walkers) and the face velocities reach HBM; the eight
// transported fields of the z pass never do.  Bound by instruction issue and
// the latency of a plane (one block per CU in FP64, two in FP32).  The z pass
// and the rebuild apart, and this: a finer level of 128^3 and its shell 92 + 58
// -> 83 us (FP64), 48 + 26 -> 48 us (FP32); a level 0 of 200 x 184 x 152, 188 +
// 115 -> 240 us (FP64).  Rows that share a wave against one row to a wave: 64^3
// 26 -> 20 us, 64 x 256 x 256 239 -> 140 us (FP64).
constexpr int ZF_TY = 2;
template <typename T>
constexpr bool zf_share() {
  return sizeof(T) == 8;
}
constexpr bool zf_level0(int XB) { return XB == 1 || XB == 4; }
// In FP64 a finer level's z faces of both rows are an eighth wave's: the seven
// others load the four SIMDs unevenly (a walker and a finisher on two of them).
// 92 -> 83 us at 128^3 and their shell; on level 0, where the walkers carry
// more, 77 -> 79, and not used.
template <typename T, int XB>
constexpr bool zf_zwave() {
  return sizeof(T) == 8 && !zf_level0(XB);
}
template <typename T, int XB>
constexpr int zf_waves() {
  return 3 * ZF_TY + (zf_zwave<T, XB>() ? 2 : 1);
}

// LDS planes: [2 buffers][ZF_TY + 1 row slots (slot 0: the row below the
// band)][NQ quantities, then the cells' sound speeds and distances from the
// perturber][2 * 64 cells]
constexpr int ZF_CS = NQ, ZF_DIST = NQ + 1, ZF_NQ = NQ + 2;
template <typename T>
struct ZfLds {
  T *base;
  __device__ __forceinline__ T *at(int buf, int r, int m) const {
    return base + ((buf * (ZF_TY + 1) + r) * ZF_NQ + m) * 128;
  }
};

// A walker's sink: the plane's new departures into its row slot of the
// current buffer, the density and energy of a band row (OUT) also to the
// output set -- for the segment's own planes only: the plane below it
// belongs to the segment below, whose block writes it (the same value: see
// march_column; one writer per plane); done() hands the plane over.
// In FP64 the walkers also take a share of the finisher's work on their
// plane (the finisher's work per plane is about twice a walker's, and every
// plane ends in a barrier): the first group the cells' sound speeds (from the
// new density and energy), the second group (and the walker of the row below)
// the cells' distances from the perturber, and the second group the force
// partials of the segment's planes -- with the finisher's expressions, into
// LDS for the finisher of the row and of the row above.  (In FP32 the extra
// registers this costs the walkers lower the occupancy from four waves per
// SIMD to three, which costs more than the balance gains: the finisher keeps
// that work.)
template <typename T>
struct ZfWork {
  const Geo *G;
  const Phys *P;
  bool put;                           // the lane's cells are the block's
  typename lanes_of<T, 2>::type xcx;  // x of the lane's two cells
  T yc;                               // y of the row
  double *fx, *fy, *fz;
  int *bad;
};

template <typename T, int XB, int GRP, int NG, bool OUT>
struct ZfSink {
  using V = typename lanes_of<T, 2>::type;
  ZfLds<T> L;
  T *rho_out, *e_out;
  int r, row, x0, buf, plane, c0;  // x0: the pair's place in the LDS rows
  bool live;
  ZfWork<T> W;
  V drc;
  __device__ __forceinline__ void put(int u, idx_t ic, V val) {
    if (zf_share<T>() && u == 0 && (GRP == 1 || NG == 3)) {
      // distances of the plane's cells (and, second group, their force terms)
      const T zcen = xcen<T>(*W.G, 2, plane);
      const T eps2 = (T)W.P->eps2;
      const V r2c = W.xcx * W.xcx + W.yc * W.yc + zcen * zcen + eps2;
      const V dcen = qsqrtv(r2c);
      *reinterpret_cast<V *>(L.at(buf, r, ZF_DIST) + x0) = dcen;
      if (zf_level0(XB) && GRP == 1 && W.put && plane >= c0) {
        const T GM = (T)W.P->GM, dx = (T)W.G->dx;
        const V w = qdiv(GM * val * (dx * dx * dx), r2c * dcen);
        *W.fx += (double)(w.x * W.xcx.x) + (double)(w.y * W.xcx.y);
        *W.fy += (double)(w.x * W.yc) + (double)(w.y * W.yc);
        *W.fz += (double)(w.x * zcen) + (double)(w.y * zcen);
      }
    }
    if (u == 0 && GRP != 0) return;  // the first group holds the density
    const int m = u == 0 ? 0 : group_q(NG, GRP, u - 1);
    *reinterpret_cast<V *>(L.at(buf, r, m) + x0) = val;
    if (OUT && m <= 1 && W.put && plane >= c0) {
      T *out = m == 0 ? rho_out : e_out;
      gstv<V>(out, ic, val);
      if constexpr (XB == 3) {  // the images beyond the mirror planes
        const idx_t iy = ic - (1 + 2 * row) * (idx_t)W.G->sy, z = (1 + 2 * plane) * (idx_t)W.G->sz;
        if (row < W.G->g) gstv<V>(out, iy, val);
        if (plane < W.G->g) {
          gstv<V>(out, ic - z, val);
          if (row < W.G->g) gstv<V>(out, iy - z, val);
        }
      }
    }
    if (zf_level0(XB) && zf_share<T>() && GRP == 0 && m == 0) drc = val;
    if (zf_level0(XB) && zf_share<T>() && GRP == 0 && m == 1) {
      // sound speeds of the plane's cells (the health check on live lanes)
      const T rho0 = (T)W.P->rho0, e0 = (T)W.P->e0, gg = (T)(W.P->gamma * W.P->gm1);
      V cs;
      {
        const T rr = rho0 + drc.x, en = e0 + val.x;
        if (live && (!(rr > T(0)) || !(en > T(0)) || !isfinite(rr) || !isfinite(en))) *W.bad = 1;
        cs.x = qsqrt(qdiv(gg * en, rr));
      }
      {
        const T rr = rho0 + drc.y, en = e0 + val.y;
        if (live && (!(rr > T(0)) || !(en > T(0)) || !isfinite(rr) || !isfinite(en))) *W.bad = 1;
        cs.y = qsqrt(qdiv(gg * en, rr));
      }
      *reinterpret_cast<V *>(L.at(buf, r, ZF_CS) + x0) = cs;
    }
  }
  __device__ __forceinline__ void done(int) {
    __syncthreads();
    buf ^= 1;
    ++plane;
  }
};

template <typename T, int XB, int FR, int GRP, int NG, bool OUT>
__device__ __forceinline__ void zf_walk(const Geo &G, const Phys &P, const MarchArgs<T> &M, ZfLds<T> L, int r, int row,
                                        int x0, int xl, int s0, bool live, int cs, int c0, int c1, ZfWork<T> W) {
  using V = typename lanes_of<T, 2>::type;
  constexpr int BC = zf_level0(XB) ? 1 : 0;
  const idx_t base = lin(G, xl, row, 0);
  const T *qi = M.qi[0];
  ColSrc<T, V, 2, BC, GRP, NG> src{qi, {M.qi[group_q(NG, GRP, 0)], M.qi[group_q(NG, GRP, 1)],
                                        M.qi[group_q(NG, GRP, 2)], M.qi[group_q(NG, GRP, 3)]},
                                   base, (idx_t)G.sz, G.n[2]};
  ZfSink<T, XB, GRP, NG, OUT> snk{L, M.qo[0], M.qo[1], r, row, s0, 0, cs, c0, live, W, V(0)};
  const FaceFront<T, 2, 2, FR> X(G, M, x0, row, W.put && (OUT || (GRP == 1 && NG == 2)), c0, c1);
  march_column<T, 2, BC, GRP, FR, 2, NG>(G, P, M, xl, row, cs, c1, src, snk, live, X);
}

// Cells of a row a tile adds to the one before it (whose last pair it walks
// again, for the x faces of its first pair).
constexpr int ZF_TILE = 2 * BX - 2;

// Tiles of rows of the cells [lo, hi): whole ones, the rest in a tile of a
// half or a quarter of a wave where it fits, two or four bands to a block.
inline XyTiles zf_tiles(int lo, int hi) {
  XyTiles B{lo, hi, lo, hi, 0, 0};
  for (int left = hi - lo; left > (B.ntiles ? 2 : 0); left -= ZF_TILE) {
    B.parts = left <= BX / 2 ? 4 : left <= BX ? 2 : 0;
    if (B.parts) break;
    ++B.ntiles;
  }
  return B;
}

// XB: 1 a level-0 row in one whole tile, 4 other level-0 rows, 0 a finer level
// (no reductions; the faces written are those of K's ranges), 3 a finer level
// between mirror planes (the images beyond them are stored too).  FR: as
// FaceFront's.
template <typename T, int XB, int FR>
__device__ __forceinline__ void zfinish_body(Geo G, Phys P, MarchArgs<T> M, KickArgs<T> K, RedArgs<T> R, XyTiles B,
                                             Blk bk) {
  constexpr bool L0 = zf_level0(XB), share = zf_share<T>(), zwave = zf_zwave<T, XB>();
  using V = typename lanes_of<T, 2>::type;
  __shared__ __align__(16) T zl[2 * (ZF_TY + 1) * ZF_NQ * 128];
  __shared__ double sh[5][zf_waves<T, XB>()];
  const ZfLds<T> L{zl};
  const int lane = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.y);
  // block -> (row band, z segment): each XCD (block h runs on XCD h % 8)
  // takes one contiguous range of bands through all segments
  const int z0 = L0 ? 0 : M.lo[2], z1 = L0 ? G.n[2] : M.hi[2];
  const int y0 = L0 ? 0 : M.lo[1], y1 = L0 ? G.n[1] : M.hi[1];
  const int nch = (z1 - z0 + M.chunk - 1) / M.chunk;
  const unsigned N = bk.n, h = bk.id;
  const unsigned q8 = N / 8, r8 = N % 8, xcd = h % 8, s8 = h / 8;
  const unsigned Lg = (xcd < r8) ? xcd * (q8 + 1) + s8 : r8 * (q8 + 1) + (xcd - r8) * q8 + s8;
  const int unit = (int)(Lg / (unsigned)nch), ch = (int)(Lg % (unsigned)nch);
  const int c0 = z0 + ch * M.chunk, c1 = min(c0 + M.chunk, z1);
  const int cs = c0 > z0 ? c0 - 1 : z0;  // first plane walked
  // the lane's band and pair of cells; in: of the box, put: the block's own
  int band = unit, lx = lane, tile = 0;
  if (XB != 1) {
    const int nb = (y1 - y0 + ZF_TY - 1) / ZF_TY, whole = nb * B.ntiles;
    if (unit < whole) {
      tile = unit / nb;
      band = unit - tile * nb;
    } else {
      const int shift = B.parts == 2 ? 5 : 4;  // lanes of a part
      lx = lane & ((1 << shift) - 1);
      tile = B.ntiles;
      band = B.parts * (unit - whole) + (lane >> shift);
    }
  }
  const int j0 = y0 + band * ZF_TY;
  const int x0 = (L0 ? 0 : B.lo) + ZF_TILE * tile + 2 * lx;
  const bool in = x0 < (L0 ? G.n[0] : B.hi) && (XB == 1 || j0 < y1);
  const bool put = in && (XB == 1 || lx > 0 || tile == 0);
  // lanes past the row end read the row's first cells (in bounds, unused),
  // rows past the box its last one
  const int xl = in ? x0 : (L0 ? 0 : B.lo);
  const int s0 = 2 * lane;
  double fx = 0.0, fy = 0.0, fz = 0.0;
  T sig = T(0);
  int bad = 0;
  if (L0 && bk.id == 0 && lane == 0 && wv == 0) {
    R.S->tlog = R.S->t;  // the force partials of this state await the log
    R.S->pending = 1;
  }
  if (wv <= 2 * ZF_TY) {
    V xw;
    xw.x = xcen<T>(G, 0, x0);
    xw.y = xcen<T>(G, 0, x0 + 1);
    if (wv == 0) {
      // the row below the band (row 0 again for the first band: its sound
      // speeds and distances are not used there)
      const int jb = XB == 1 ? max(j0 - 1, y0) : clampi(j0 - 1, y0, y1 - 1);
      zf_walk<T, XB, FR, 0, 3, false>(G, P, M, L, 0, jb, x0, xl, s0, in, cs, c0, c1,
                                      ZfWork<T>{&G, &P, put, xw, xcen<T>(G, 1, jb), &fx, &fy, &fz, &bad});
    } else {
      const int y = (wv - 1) >> 1;
      const bool row = j0 + y < y1;
      const int j = min(j0 + y, y1 - 1);
      const ZfWork<T> W{&G, &P, put && row, xw, xcen<T>(G, 1, j), &fx, &fy, &fz, &bad};
      if ((wv - 1) & 1) zf_walk<T, XB, FR, 1, 2, false>(G, P, M, L, 1 + y, j, x0, xl, s0, in, cs, c0, c1, W);
      else zf_walk<T, XB, FR, 0, 2, true>(G, P, M, L, 1 + y, j, x0, xl, s0, in, cs, c0, c1, W);
    }
  } else {
    // finishers: cells x0, x0 + 1 of the rows j
    const int i = x0;
    // finer levels: the faces within their ranges
    auto in_range = [&](int d, int j, int k) {
      return L0 || (j >= K.flo[d][1] && j < K.fhi[d][1] && k >= K.flo[d][2] && k < K.fhi[d][2]);
    };
    const T h = (T)(K.fac * K.dtp[0]), h2 = !L0 && K.twice ? h : T(0);
    const T rho0 = (T)P.rho0, gm1 = (T)P.gm1, GM = (T)P.GM, eps2 = (T)P.eps2, dx = (T)G.dx;
    const T gg = (T)(P.gamma * P.gm1), e0 = (T)P.e0;
    V xcx;
    xcx.x = xcen<T>(G, 0, i);
    xcx.y = xcen<T>(G, 0, i + 1);
    auto r2of = [&](V xv, T yy, T zz) -> V { return xv * xv + yy * yy + zz * zz + eps2; };
    auto sound1 = [&](T dr, T de) -> T {
      const T rr = rho0 + dr, en = e0 + de;
      if (!(rr > T(0)) || !(en > T(0)) || !isfinite(rr) || !isfinite(en)) bad = 1;
      return qsqrt(qdiv(gg * en, rr));
    };
    auto sound = [&](V dr, V de) -> V {
      V s;
      s.x = sound1(dr.x, de.x);
      s.y = sound1(dr.y, de.y);
      return s;
    };
    auto vmax = [&](V a) { sig = fmax(sig, fmax(a.x, a.y)); };
    auto vabs = [&](V a) -> V {
      V o;
      o.x = fabs(a.x);
      o.y = fabs(a.y);
      return o;
    };
    // A rebuilt face velocity a / b before its kick.  On level 0 the quotient is
    // rounded, then kicked, as k_kick0p's pairs are; a finer level's dividend
    // and reciprocal go into the kick's multiply-add unrounded, as in k_kick: in
    // FP32 the quotient's own rounding made the velocities of 4 x 128^3 2.5 %
    // noisier (rms of vz over 40 steps 9.75e-11 against 9.50e-11).
    struct Quot {
      V a, r;
    };
    auto rebuild = [&](int d, V ppm, V pmc, V drm, V dcr) -> Quot {
      const T vb = (T)vback(P, d);
      const V a = ppm + pmc - vb * (drm + dcr), b = T(2) * rho0 + drm + dcr;
      return L0 ? Quot{qdiv(a, b), V(1)} : Quot{a, qdiv(V(T(1)), b)};
    };
    auto kickv = [&](Quot f, V drm, V dem, V dcr, V der, V xr, V dm, V dr_) -> V {
      const V rface = rho0 + T(0.5) * (drm + dcr);
      const V gradp = qdiv(gm1 * (der - dem), dx * rface);
      const V xm = xr - dx;
      const V gradphi = qdiv(GM * (xr + xm), dm * dr_ * (dm + dr_));
      if constexpr (L0) return f.a - h * (gradp + gradphi);
      const V g = gradp + gradphi;
      return fmav<V>(V(-h2), g, fmav<V>(f.a, f.r, -(h * g)));
    };
    // the faces normal to d at row j, plane k and (XB 3) their images: a face's
    // image lies as far beyond the plane, normal velocities change sign
    auto put_face = [&](int d, idx_t c, int j, int k, V v) {
      auto at = [&](int jj, int kk, V w) {
        if (in_range(d, jj, kk)) gstv<V>(K.v[d], c + (jj - j) * (idx_t)G.sy + (kk - k) * (idx_t)G.sz, w);
      };
      at(j, k, v);
      if constexpr (XB == 3) {
        const int jm = d == 1 ? -j : -1 - j, km = d == 2 ? -k : -1 - k;
        if (jm < 0) at(jm, k, d == 1 ? -v : v);
        if (km < 0) {
          at(j, km, d == 2 ? -v : v);
          if (jm < 0) at(jm, km, d == 0 ? v : -v);
        }
      }
    };
    auto ldv = [&](int buf, int rr, int m) -> V { return *reinterpret_cast<const V *>(L.at(buf, rr, m) + s0); };
    // the cells below the z faces: new departures, sound speeds and
    // distances of the plane before
    struct Below {
      V r = V(0), e = V(0), p = V(0), c = V(0), d = V(0);
    };
    // plane k of band row y: its x and y faces (XY), its z faces (Z)
    auto plane = [&](auto XY, auto Z, int y, int k, int buf, Below &zb) {
      const int j = j0 + y, r = 1 + y;
      const bool own = put && j < y1;
      if (!(in && j < y1)) return;
      const T yc = xcen<T>(G, 1, j);
      const V drc = ldv(buf, r, 0), dec = ldv(buf, r, 1);
      const T zcen = xcen<T>(G, 2, k);
      V dcen, cs_own, r2c;
      if (share) {
        dcen = ldv(buf, r, ZF_DIST);  // the walkers' distances and sound speeds
        if (L0) cs_own = ldv(buf, r, ZF_CS);
      } else {
        r2c = r2of(xcx, yc, zcen);
        dcen = qsqrtv(r2c);
        if (L0) cs_own = sound(drc, dec);
      }
      V ppz;
      if (Z) ppz = ldv(buf, r, 7);
      const T csprev = L0 && XY ? dpp_fill<DPP_WAVE_SHR1>(cs_own.y, T(0)) : T(0);
      const T dprev = XY ? dpp_fill<DPP_WAVE_SHR1>(dcen.y, T(0)) : T(0);
      if (k >= c0 && (XB == 1 || own)) {
        const idx_t c = lin(G, i, j, k);
        // x: faces i and i+1; below them cell i-1 (the cell itself at x = 0) and cell i
        if constexpr (XY) {
          V drm, dem, ppm;
          drm.y = drc.x;
          dem.y = dec.x;
          const V ppc = ldv(buf, r, 3);
          ppm.y = ppc.x;
          if (lx > 0) {
            drm.x = L.at(buf, r, 0)[s0 - 1];
            dem.x = L.at(buf, r, 1)[s0 - 1];
            ppm.x = L.at(buf, r, 3)[s0 - 1];
          } else {
            drm.x = drc.x;
            dem.x = dec.x;
            ppm.x = ppc.x;
          }
          const Quot f0 = rebuild(0, ppm, ldv(buf, r, 2), drm, drc);
          V dmx;
          dmx.y = dcen.x;
          if (lx > 0) {
            dmx.x = dprev;
          } else {
            V xb;
            xb.x = xcen<T>(G, 0, i - 1);  // cell i-1 (a ghost position at x = 0)
            xb.y = xb.x;
            dmx.x = qsqrtv(r2of(xb, yc, zcen)).x;
          }
          const V vf = kickv(f0, drm, dem, drc, dec, xcx, dmx, dcen);
          put_face(0, c, j, k, vf);
          if constexpr (L0) {
            const V a = vabs((T)vback(P, 0) + vf);
            vmax(a + cs_own);
            if (lx > 0) sig = fmax(sig, a.x + csprev);
            sig = fmax(sig, a.y + cs_own.x);
            if (i + 1 == G.n[0] - 1) {
              K.v[0][c + 2] = T(0);  // injection face at x_max carries the wind
              sig = fmax(sig, fabs((T)vback(P, 0)) + cs_own.y);
            }
          }
        }
        // y: face j (the row below from slot r-1; the row itself at y = 0),
        // and face n after the last row
        if constexpr (XY) {
          const V pmy = ldv(buf, r, 4), ppy = ldv(buf, r, 5);
          const bool lo = j > y0;
          const V drm = lo ? ldv(buf, r - 1, 0) : drc, dem = lo ? ldv(buf, r - 1, 1) : dec;
          const Quot f0 = rebuild(1, lo ? ldv(buf, r - 1, 5) : ppy, pmy, drm, drc);
          // the row below: its walkers' distances and sound speeds (the ghost
          // row's distance at y = 0)
          const V dmb = share && lo ? ldv(buf, r - 1, ZF_DIST) : qsqrtv(r2of(xcx, xcen<T>(G, 1, j - 1), zcen));
          V vf = kickv(f0, drm, dem, drc, dec, V(yc), dmb, dcen);
          if (XB == 3 && !lo) vf = V(0);  // the mirror plane
          put_face(1, c, j, k, vf);
          if constexpr (L0) {
            const V a = vabs(vf);
            vmax(a + cs_own);
            if (lo) vmax(a + (share ? ldv(buf, r - 1, ZF_CS) : sound(drm, dem)));
          }
          if (L0 && j == G.n[1] - 1) {
            const T xr = xcen<T>(G, 1, j + 1);
            const V dr_ = qsqrtv(r2of(xcx, xr, zcen));
            const V vh = kickv(rebuild(1, ppy, pmy, drc, drc), drc, dec, drc, dec, V(xr), dcen, dr_);
            gstv<V>(K.v[1], c + (idx_t)G.sy, vh);
            vmax(vabs(vh) + cs_own);
          }
        }
        // z: face k (the plane before from the walk's previous plane; the
        // plane itself at z = 0), and face n after the last plane
        if constexpr (Z) {
          const V pmz = ldv(buf, r, 6);
          const bool lo = k > z0;
          const V drm = lo ? zb.r : drc, dem = lo ? zb.e : dec;
          const Quot f0 = rebuild(2, lo ? zb.p : ppz, pmz, drm, drc);
          const V dmb = lo ? zb.d : qsqrtv(r2of(xcx, yc, xcen<T>(G, 2, k - 1)));
          V vf = kickv(f0, drm, dem, drc, dec, V(zcen), dmb, dcen);
          if (XB == 3 && !lo) vf = V(0);
          put_face(2, c, j, k, vf);
          if constexpr (L0) {
            const V a = vabs(vf);
            vmax(a + cs_own);
            if (lo) vmax(a + zb.c);
          }
          if (L0 && k == G.n[2] - 1) {
            const T xr = xcen<T>(G, 2, k + 1);
            const V dr_ = qsqrtv(r2of(xcx, yc, xr));
            const V vh = kickv(rebuild(2, ppz, pmz, drc, drc), drc, dec, drc, dec, V(xr), dcen, dr_);
            gstv<V>(K.v[2], c + (idx_t)G.sz, vh);
            vmax(vabs(vh) + cs_own);
          }
        }
        // force of the gas in these cells on the perturber, eq. 18: each
        // cell's term in the storage type, the sum in FP64 (in FP64 formed by
        // the second group's walker)
        if (L0 && !share) {
          const V w = qdiv(GM * drc * (dx * dx * dx), r2c * dcen);
          fx += (double)(w.x * xcx.x) + (double)(w.y * xcx.y);
          fy += (double)(w.x * yc) + (double)(w.y * yc);
          fz += (double)(w.x * zcen) + (double)(w.y * zcen);
        }
      }
      if (Z) {
        zb.r = drc;
        zb.e = dec;
        zb.p = ppz;
        if (L0) zb.c = cs_own;
        zb.d = dcen;
      }
    };
    const std::true_type yes{};
    const std::false_type no{};
    if (zwave && wv == zf_waves<T, XB>() - 1) {
      Below zb[ZF_TY];
      for (int k = cs; k < c1; ++k) {
        __syncthreads();
#pragma unroll
        for (int y = 0; y < ZF_TY; ++y) plane(no, yes, y, k, (k - cs) & 1, zb[y]);
      }
    } else {
      const std::bool_constant<!zwave> z{};
      Below zb;
      for (int k = cs; k < c1; ++k) {
        __syncthreads();
        plane(yes, z, wv - 1 - 2 * ZF_TY, k, (k - cs) & 1, zb);
      }
    }
    if (!isfinite(sig)) bad = 1;
  }
  if (!L0) return;
  // block sums of the force partials and maximum of the signal speeds (every
  // wave takes part; walkers contribute zeros), written to the block's slot;
  // the slots of the one-cell-per-thread grid past the launch are zeroed
  fx = wave_sum(fx);
  fy = wave_sum(fy);
  fz = wave_sum(fz);
  double sg = wave_max(bad ? 0.0 : (double)sig);
  const bool anybad = __any(bad);
  if (lane == 0) {
    sh[0][wv] = fx;
    sh[1][wv] = fy;
    sh[2][wv] = fz;
    sh[3][wv] = sg;
    if (anybad) atomicOr(&R.S->health, 1);
  }
  __syncthreads();
  if (lane == 0 && wv == 0) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, m = 0.0;
    for (int w = 0; w < zf_waves<T, XB>(); ++w) {
      s0 += sh[0][w];
      s1 += sh[1][w];
      s2 += sh[2][w];
      m = fmax(m, sh[3][w]);
    }
    const long nb = R.npart;
    R.part[bk.id] = s0;
    R.part[nb + bk.id] = s1;
    R.part[2 * nb + bk.id] = s2;
    R.spart[bk.id] = m;
    __hip_atomic_fetch_max(&R.S->smax[bk.id & (NSLOT - 1)], (unsigned long long)__double_as_longlong(m),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (unsigned z = bk.n + bk.id + (unsigned)(wv * 64 + lane) * bk.n; z < (unsigned)R.npart;
       z += bk.n * 64u * zf_waves<T, XB>()) {
    R.part[z] = 0.0;
    R.part[R.npart + z] = 0.0;
    R.part[2 * (size_t)R.npart + z] = 0.0;
    R.spart[z] = 0.0;
  }
}

template <typename T, int XB, int FR>
__global__ void __launch_bounds__((64 * zf_waves<T, XB>())) k_zfinish(Geo G, Phys P, MarchArgs<T> M, KickArgs<T> K, RedArgs<T> R,
                                                            XyTiles B) {
  zfinish_body<T, XB, FR>(G, P, M, K, R, B, grid_blk());
}

struct DtArgs {
  // advance: 0 set dt, 1 set dt and advance the time, 2 per-level limits only
  double dx[MAXLEV];
  const double *part[MAXLEV];  // per-block maximum signal speeds of each level
  int npart[MAXLEV];
  int nl;
  int advance;
};

// coarse step cfl * min_l 2^l min(dx_l / smax_l, dx_l^2 / (6 chi)) (eq. 55, xi = 2)
// thread 0: the step lengths from each level's largest signal speed smax
__device__ void dt_finish(const Phys &P, const DtArgs &A, Scal *S, const double *smax) {
  double best = INFINITY;
  for (int l = 0; l < A.nl; ++l) {
    double dtl = A.dx[l] / smax[l];
    if (P.chi > 0.0) dtl = fmin(dtl, A.dx[l] * A.dx[l] / (6.0 * P.chi));
    S->dtl[l] = P.cfl * dtl;  // the level's own limit (for the sub-cycling criterion)
    dtl = ldexp(dtl, l);
    best = fmin(best, dtl);
  }
  if (A.advance == 2) return;  // limits only: the host sets the schedule
  const double dt0 = P.cfl * best;
  for (int l = 0; l < A.nl; ++l) S->dt[l] = ldexp(dt0, -l);
  if (A.advance) S->t += dt0;
}

__device__ void dt_body(const Phys &P, const DtArgs &A, Scal *S) {
  __shared__ double sh[FW];
  __shared__ double smax[MAXLEV];
  for (int l = 0; l < A.nl; ++l) {
    const double *p = A.part[l];
    const int n = A.npart[l];
    double m = 0.0;
    int b = threadIdx.x;
    for (; b + 7 * FT < n; b += 8 * FT) {
      double x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = p[b + u * FT];
#pragma unroll
      for (int u = 0; u < 8; ++u) m = fmax(m, x[u]);
    }
    for (; b < n; b += FT) m = fmax(m, p[b]);
    m = wave_max(m);
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = sh[0];
      for (int v = 1; v < FW; ++v) t = fmax(t, sh[v]);
      smax[l] = t;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) dt_finish(P, A, S, smax);
}

__global__ void __launch_bounds__(FT) k_dt_final(Phys P, DtArgs A, Scal *S) { dt_body(P, A, S); }

// Between two steps: the force of the state just reached (logged at its
// time), then the next step's time step from the same state's signal speeds.
// One pass reads the partials of both (the force planes and the signal
// speeds of a block side by side, all in flight together); the sums keep the
// order of final3_body and the maxima are those of dt_body.
template <bool do_force, bool do_dt>
__global__ void __launch_bounds__(FT) k_step_final(Phys P, FinalArgs F, DtArgs D, Scal *S) {
  __shared__ double sh[3][FW];
  __shared__ double shm[MAXLEV][FW];
  __shared__ double smax[MAXLEV];
  const int t = threadIdx.x, w = t / 64;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  for (int l = 0; l < D.nl; ++l) {
    const double *p = F.part[l], *q = D.part[l];
    const int n = D.npart[l];
    double m = 0.0;
    int b = t;
    for (; b + 7 * FT < n; b += 8 * FT) {
      double x[8][3], y[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (do_force)
#pragma unroll
          for (int c = 0; c < 3; ++c) x[u][c] = p[(size_t)c * n + b + u * FT];
        if (do_dt) y[u] = q[b + u * FT];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (do_force) {
          s0 += x[u][0];
          s1 += x[u][1];
          s2 += x[u][2];
        }
        if (do_dt) m = fmax(m, y[u]);
      }
    }
    for (; b < n; b += FT) {
      if (do_force) {
        s0 += p[b];
        s1 += p[(size_t)n + b];
        s2 += p[2 * (size_t)n + b];
      }
      if (do_dt) m = fmax(m, q[b]);
    }
    m = wave_max(m);
    if (t % 64 == 0) shm[l][w] = m;
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  if (t % 64 == 0) {
    sh[0][w] = s0;
    sh[1][w] = s1;
    sh[2][w] = s2;
  }
  __syncthreads();
  if (t != 0) return;
  if (do_force) final3_finish(F, sh);
  if (do_dt) {
    for (int l = 0; l < D.nl; ++l) {
      double v = shm[l][0];
      for (int u = 1; u < FW; ++u) v = fmax(v, shm[l][u]);
      smax[l] = v;
    }
    dt_finish(P, D, S, smax);
  }
}

__global__ void k_zero(unsigned int *p, size_t n) {
  size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; t < n; t += stride) p[t] = 0u;
}

// every stored entry (level 0 stores cells 0..n-1 and faces 0..n)
Box full_box(const Geo &G) {
  Box b;
  for (int d = 0; d < 3; ++d) {
    b.lo[d] = -G.g;
    b.hi[d] = G.s[d] - G.g;
  }
  return b;
}
Box active_box(const Geo &G) {
  Box b;
  for (int d = 0; d < 3; ++d) {
    b.lo[d] = 0;
    b.hi[d] = G.n[d];
  }
  return b;
}
Box uniform_box(const Geo &G, int lo_off, int hi_off) {
  Box b;
  for (int d = 0; d < 3; ++d) {
    b.lo[d] = -G.g + lo_off;
    b.hi[d] = G.n[d] + G.g - hi_off;
  }
  return b;
}

// A finer level's launch computes only the entries within its stage's margin
// G.mg of the active range (the entries later stages and the level's
// observers need); the range [lo, hi) along d, of cells or (face) of faces
// normal to d, is cut to it.
inline void clip_margin(const Geo &G, int d, bool face, int &lo, int &hi) {
  lo = max(lo, -G.mg[d]);
  hi = min(hi, G.n[d] + G.mg[d] + (face ? 1 : 0));
}
inline Box clip_cells(const Geo &G, Box b) {
  for (int d = 0; d < 3; ++d) clip_margin(G, d, false, b.lo[d], b.hi[d]);
  return b;
}

template <typename T>
inline T *tp(void *p) {
  return reinterpret_cast<T *>(p);
}

}  // namespace

// launch only non-empty grids
// While a recorder is set (the engine's dry run of a step), every launch that
// is not one of the batched stages marks the recording failed and is not made.
#define DFK_LAUNCH(K, GR, BL, ST, ...)                                      \
  do {                                                                      \
    if (g_rec) {                                                            \
      g_rec->failed = true;                                                 \
      break;                                                                \
    }                                                                       \
    dim3 g_ = (GR);                                                         \
    if (!empty_grid(g_)) hipLaunchKernelGGL(K, g_, BL, 0, ST, __VA_ARGS__); \
  } while (0)

thread_local Recorder *g_rec = nullptr;

// in a recording: add the launch of stage kind `kind` with its arguments
template <typename E>
bool record(int kind, const E &e) {
  if (!g_rec) return false;
  if (e.nblk == 0) return true;  // an empty launch is no launch
  JobRec r;
  r.kind = kind;
  r.nblk = e.nblk;
  r.bytes.resize(sizeof(E));
  std::memcpy(r.bytes.data(), &e, sizeof(E));
  g_rec->recs.push_back(std::move(r));
  return true;
}

// ============================================================ batched jobs
// One launch for one stage of several single-level runs (the engine's batched
// step): run r owns the blocks [start[r], start[r+1]) of the launch, each
// run's count padded to a multiple of 8 so that its blocks keep their XCD
// placement (block h on XCD h % 8), and its launch arguments are entry r of
// the table; block b runs as block b - start[r] of the run's own launch.  The
// bodies are those of the single-run kernels, so a run's results do not
// depend on the other runs in the launch.
template <typename T>
struct KcJob {
  Geo G;
  Phys P;
  KickArgs<T> A;
  RedArgs<T> R;
  unsigned nblk;
};
template <typename T>
struct DiffJob {
  Geo G;
  Phys P;
  DiffArgs<T> A;
  unsigned nblk;
};
template <typename T>
struct XyJob {
  Geo G;
  Phys P;
  PassArgs<T> A;
  MarchArgs<T> M;
  XyTiles B;
  unsigned nblk;
};
template <typename T>
struct ZfJob {
  Geo G;
  Phys P;
  MarchArgs<T> M;
  KickArgs<T> K;
  RedArgs<T> R;
  XyTiles B;
  unsigned nblk;
};
struct LogJob {
  const double *part;
  int npart;
  Scal *S;
  double *flog;
  unsigned nblk;
};

// stage kinds of the batched launches (dfk.h), per storage type and form
template <typename T>
constexpr int jk_kc(int bc) {
  return (sizeof(T) == 4 ? JK_KC_F1 : JK_KC_D1) + (bc == 2 ? 1 : 0);
}
template <typename T>
constexpr int jk_df(int bc) {
  return (sizeof(T) == 4 ? JK_DF_F1 : JK_DF_D1) + (bc == 2 ? 1 : 0);
}
template <typename T>
constexpr int jk_xy(int n) {  // the k_xyshared form transport_xy_t takes for rows of n cells
  return (sizeof(T) == 4 ? JK_XY_F1 : JK_XY_D1) + (n > BX ? 1 : 0);
}
template <typename T>
constexpr int jk_zf(bool one) {  // one: the row in one whole tile
  return (sizeof(T) == 4 ? JK_ZF_F1 : JK_ZF_D1) + (one ? 0 : 1);
}

template <typename E>
struct JobTab {
  const E *__restrict__ e;
  const unsigned *__restrict__ start;  // n + 1 block offsets
  int n;
};

// the run of block b and the block's place in the run's launch; false for a
// padding block
template <typename E>
__device__ __forceinline__ bool job_of(const JobTab<E> &t, unsigned b, int &r, Blk &bk) {
  int lo = 0, hi = t.n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (t.start[mid] <= b) lo = mid;
    else hi = mid;
  }
  r = lo;
  bk.id = b - t.start[lo];
  bk.n = t.e[lo].nblk;
  return bk.id < bk.n;
}

template <typename T, int BCM>
__global__ void __launch_bounds__(BX * BY) __attribute__((amdgpu_waves_per_eu(5)))
k_kick_compress_jobs(JobTab<KcJob<T>> t) {
  int r;
  Blk bk;
  if (!job_of(t, blockIdx.x, r, bk)) return;
  const KcJob<T> &J = t.e[r];
  kick0p_body<T, BCM, false, true, false, true>(J.G, J.P, J.A, J.R, bk);
}

template <typename T, int BC>
__global__ void __launch_bounds__(BX * BY) k_diffuse_heat2_jobs(JobTab<DiffJob<T>> t) {
  int r;
  Blk bk;
  if (!job_of(t, blockIdx.x, r, bk)) return;
  const DiffJob<T> &J = t.e[r];
  diffuse_heat2_body<T, BC>(J.G, J.P, J.A, bk);
}

template <typename T, int W>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_xyshared_jobs(JobTab<XyJob<T>> t) {
  int r;
  Blk bk;
  if (!job_of(t, blockIdx.x, r, bk)) return;
  const XyJob<T> &J = t.e[r];
  xyshared_body<T, W, 1, 0>(J.G, J.P, J.A, J.M, J.B, bk);
}

template <typename T, int XB>
__global__ void __launch_bounds__((64 * zf_waves<T, XB>())) k_zfinish_jobs(JobTab<ZfJob<T>> t) {
  int r;
  Blk bk;
  if (!job_of(t, blockIdx.x, r, bk)) return;
  const ZfJob<T> &J = t.e[r];
  zfinish_body<T, XB, 0>(J.G, J.P, J.M, J.K, J.R, J.B, bk);
}

__global__ void __launch_bounds__(FT) k_log_pending_jobs(JobTab<LogJob> t) {
  const LogJob &J = t.e[blockIdx.x];
  log_pending_body<FT>(J.part, J.npart, J.S, J.flog);
}

// ======================================================================
// launchers (templated on the storage type, dispatched on P.fp32)

template <typename T>
static void init_state_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, uint64_t seed,
                         double amp) {
  InitArgs<T> A;
  A.b = full_box(G);
  A.rho = tp<T>(B.q[cur][0]);
  A.e = tp<T>(B.q[cur][1]);
  A.vx = tp<T>(B.v[0]);
  A.vy = tp<T>(B.v[1]);
  A.vz = tp<T>(B.v[2]);
  A.seed = seed;
  A.amp = amp;
  DFK_LAUNCH(k_init<T>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
}
void init_state(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, uint64_t seed, double amp) {
  if (P.fp32) init_state_t<float>(st, G, P, B, cur, seed, amp);
  else init_state_t<double>(st, G, P, B, cur, seed, amp);
}

template <typename T>
static RedArgs<T> red_args(const Geo &G, LevBufs &B, int cur, Scal *S);

template <typename T>
static void kick_t(hipStream_t st, const Geo &G, const Phys &P, void *const *q, void *const *v, const double *dtp,
                   double fac, bool rebuild, bool do_kick, LevBufs *post = nullptr, Scal *S = nullptr,
                   Scal *slots = nullptr, void *vz = nullptr) {
  KickArgs<T> A{};
  A.slots = nullptr;
  for (int d = 0; d < 3; ++d)
    for (int e = 0; e < 3; ++e) {
      if (G.bc) {
        A.flo[d][e] = 0;
        A.fhi[d][e] = G.n[e] + (d == e ? 1 : 0);
      } else if (!rebuild) {
        A.flo[d][e] = -G.g + (d == e ? 1 : 0);
        A.fhi[d][e] = G.n[e] + G.g;
      } else {
        A.flo[d][e] = -G.g + (d == e ? 3 : 2);
        A.fhi[d][e] = G.n[e] + G.g - 3;
      }
      if (!G.bc) clip_margin(G, e, d == e, A.flo[d][e], A.fhi[d][e]);
    }
  for (int e = 0; e < 3; ++e) {
    A.b.lo[e] = min(A.flo[0][e], min(A.flo[1][e], A.flo[2][e]));
    A.b.hi[e] = max(A.fhi[0][e], max(A.fhi[1][e], A.fhi[2][e]));
  }
  for (int m = 0; m < NQ; ++m) A.q[m] = tp<T>(q[m]);
  for (int d = 0; d < 3; ++d) {
    A.v[d] = tp<T>(v[d]);
    A.vin[d] = A.v[d];
  }
  if (vz) A.v[2] = tp<T>(vz);
  A.dtp = dtp;
  A.fac = fac;
  const dim3 bl(BX, BY);
  if (G.bc) {
    // level 0: one thread per pair of active cells (boundary faces by the
    // last cells)
    A.b = active_box(G);
    RedArgs<T> R{};
    if (post) R = red_args<T>(G, *post, 0, S);
    A.b.hi[0] = G.n[0] / 2;  // level-0 rows have an even length
    A.slots = slots;
    const dim3 gr = grid_of_flat(A.b);
    if (G.bc == 2) {
      if (rebuild && do_kick && post) DFK_LAUNCH((k_kick0p<T, 2, true, true, true>), gr, bl, st, G, P, A, R);
      else if (rebuild && do_kick) DFK_LAUNCH((k_kick0p<T, 2, true, true, false>), gr, bl, st, G, P, A, R);
      else if (rebuild) DFK_LAUNCH((k_kick0p<T, 2, true, false, false>), gr, bl, st, G, P, A, R);
      else DFK_LAUNCH((k_kick0p<T, 2, false, true, false>), gr, bl, st, G, P, A, R);
    } else {
      if (rebuild && do_kick && post) DFK_LAUNCH((k_kick0p<T, 1, true, true, true>), gr, bl, st, G, P, A, R);
      else if (rebuild && do_kick) DFK_LAUNCH((k_kick0p<T, 1, true, true, false>), gr, bl, st, G, P, A, R);
      else if (rebuild) DFK_LAUNCH((k_kick0p<T, 1, true, false, false>), gr, bl, st, G, P, A, R);
      else DFK_LAUNCH((k_kick0p<T, 1, false, true, false>), gr, bl, st, G, P, A, R);
    }
    return;
  }
  const dim3 gr = grid_of_flat(A.b);
  {
    if (rebuild && do_kick) DFK_LAUNCH((k_kick<T, true, true>), gr, bl, st, G, P, A);
    else if (rebuild) DFK_LAUNCH((k_kick<T, true, false>), gr, bl, st, G, P, A);
    else DFK_LAUNCH((k_kick<T, false, true>), gr, bl, st, G, P, A);
  }
}

void kick(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp, double fac,
          Scal *slots, void *vz) {
  if (!G.bc) slots = nullptr;  // the slots belong to level 0
  if (P.fp32) kick_t<float>(st, G, P, B.q[cur], B.v, dtp, fac, false, true, nullptr, nullptr, slots, vz);
  else kick_t<double>(st, G, P, B.q[cur], B.v, dtp, fac, false, true, nullptr, nullptr, slots, vz);
}

template <typename T>
static void kick_compress_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp,
                            double kfac, double cfac, Scal *slots, double *flog) {
  KickArgs<T> A{};
  A.b = active_box(G);
  A.b.hi[0] = G.n[0] / 2;  // cell pairs: level-0 rows have an even length
  for (int m = 0; m < NQ; ++m) A.q[m] = tp<T>(B.q[cur][m]);
  for (int d = 0; d < 3; ++d) {
    A.v[d] = tp<T>(B.vk[d]);
    A.vin[d] = tp<T>(B.v[d]);
  }
  A.dtp = dtp;
  A.fac = kfac;
  A.slots = slots;
  A.eo = tp<T>(B.etmp);
  A.cfac = cfac;
  A.log = slots;
  A.part = B.part;
  A.npart = (int)part_count(G);
  A.flog = flog;
  RedArgs<T> R{};
  const dim3 gr = grid_of_flat(A.b), bl(BX, BY);
  if (record(jk_kc<T>(G.bc), KcJob<T>{G, P, A, R, gr.x})) return;
  if (G.bc == 2) DFK_LAUNCH((k_kick0p<T, 2, false, true, false, true>), gr, bl, st, G, P, A, R);
  else DFK_LAUNCH((k_kick0p<T, 1, false, true, false, true>), gr, bl, st, G, P, A, R);
}
template <typename T>
static void kick_compress_fine_t(hipStream_t st, const Geo &Gk, const Geo &Gc, const Phys &P, LevBufs &B, int cur,
                                 const double *dtp, double kfac, double cfac, void *const *vk) {
  KickArgs<T> A{};
  // the kick's face ranges within Gk's margins (as kick_t), the compression's
  // cells within Gc's (as compress_t)
  for (int d = 0; d < 3; ++d)
    for (int e = 0; e < 3; ++e) {
      A.flo[d][e] = -Gk.g + (d == e ? 1 : 0);
      A.fhi[d][e] = Gk.n[e] + Gk.g;
      clip_margin(Gk, e, d == e, A.flo[d][e], A.fhi[d][e]);
    }
  Box ub;
  for (int e = 0; e < 3; ++e) {
    ub.lo[e] = min(A.flo[0][e], min(A.flo[1][e], A.flo[2][e]));
    ub.hi[e] = max(A.fhi[0][e], max(A.fhi[1][e], A.fhi[2][e]));
  }
  const Box cb = clip_cells(Gc, uniform_box(Gc, 0, 1));
  for (int e = 0; e < 3; ++e) {
    ub.lo[e] = min(ub.lo[e], cb.lo[e]);
    ub.hi[e] = max(ub.hi[e], cb.hi[e]);
  }
  // pairs of cells (rows are padded to even bounds)
  ub.lo[0] = (ub.lo[0] - (ub.lo[0] & 1)) / 2;
  ub.hi[0] = (ub.hi[0] + (ub.hi[0] & 1)) / 2;
  for (int m = 0; m < NQ; ++m) A.q[m] = tp<T>(B.q[cur][m]);
  for (int d = 0; d < 3; ++d) {
    A.v[d] = tp<T>(vk[d]);
    A.vin[d] = tp<T>(B.v[d]);
  }
  A.dtp = dtp;
  A.fac = kfac;
  A.eo = tp<T>(B.etmp);
  A.cfac = cfac;
  DFK_LAUNCH(k_kick_compress_fine<T>, grid_of_flat<BX - 1>(ub), dim3(BX, BY), st, Gk, P, A, cb, ub);
}
void kick_compress_fine(hipStream_t st, const Geo &Gk, const Geo &Gc, const Phys &P, LevBufs &B, int cur,
                        const double *dtp, double kfac, double cfac, void *const *vk) {
  if (P.fp32) kick_compress_fine_t<float>(st, Gk, Gc, P, B, cur, dtp, kfac, cfac, vk);
  else kick_compress_fine_t<double>(st, Gk, Gc, P, B, cur, dtp, kfac, cfac, vk);
}

void kick_compress(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp, double kfac,
                   double cfac, Scal *slots, double *flog) {
  if (P.fp32) kick_compress_t<float>(st, G, P, B, cur, dtp, kfac, cfac, slots, flog);
  else kick_compress_t<double>(st, G, P, B, cur, dtp, kfac, cfac, slots, flog);
}

void rebuild_kick(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int src, const double *dtp,
                  double fac, bool do_kick, Scal *post) {
  LevBufs *pb = (post && G.bc && do_kick) ? &B : nullptr;
  if (P.fp32) kick_t<float>(st, G, P, B.q[src], B.v, dtp, fac, true, do_kick, pb, post);
  else kick_t<double>(st, G, P, B.q[src], B.v, dtp, fac, true, do_kick, pb, post);
}

template <typename T>
static void compress_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp,
                       double fac, Scal *log, double *flog) {
  CellArgs<T> A;
  A.b = G.bc ? active_box(G) : clip_cells(G, uniform_box(G, 0, 1));
  A.e = tp<T>(B.q[cur][1]);
  for (int d = 0; d < 3; ++d) A.v[d] = tp<T>(B.v[d]);
  A.dtp = dtp;
  A.fac = fac;
  A.log = log;
  A.part = B.part;
  A.npart = (int)part_count(G);
  A.flog = flog;
  if (G.bc) {
    A.b.hi[0] = G.n[0] / 2;  // cell pairs: level-0 rows have an even length
    DFK_LAUNCH(k_compress2<T>, grid_of_flat(A.b), dim3(BX, BY), st, G, P, A);
    return;
  }
  DFK_LAUNCH(k_compress<T>, grid_of_flat(A.b), dim3(BX, BY), st, G, P, A);
}
void compress(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp, double fac,
              Scal *log, double *flog) {
  if (!G.bc) log = nullptr;  // the slots and the log belong to level 0
  if (P.fp32) compress_t<float>(st, G, P, B, cur, dtp, fac, log, flog);
  else compress_t<double>(st, G, P, B, cur, dtp, fac, log, flog);
}

template <typename T>
static void viscosity_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp,
                        double fac) {
  ViscArgs<T> A;
  for (int e = 0; e < 3; ++e) {
    A.elo[e] = G.bc ? 0 : -G.g;
    A.ehi[e] = G.bc ? G.n[e] : G.n[e] + G.g - 1;
    if (!G.bc) clip_margin(G, e, false, A.elo[e], A.ehi[e]);
  }
  for (int d = 0; d < 3; ++d)
    for (int e = 0; e < 3; ++e) {
      if (G.bc) {
        A.flo[d][e] = 0;
        A.fhi[d][e] = G.n[e] + (d == e ? 1 : 0);
      } else {
        A.flo[d][e] = -G.g + (d == e ? 1 : 0);
        A.fhi[d][e] = G.n[e] + G.g - 1;
        clip_margin(G, e, d == e, A.flo[d][e], A.fhi[d][e]);
      }
    }
  for (int e = 0; e < 3; ++e) {
    A.lo[e] = min(A.elo[e], min(A.flo[0][e], min(A.flo[1][e], A.flo[2][e])));
    A.hi[e] = max(A.ehi[e], max(A.fhi[0][e], max(A.fhi[1][e], A.fhi[2][e])));
  }
  A.rho = tp<T>(B.q[cur][0]);
  A.e = tp<T>(B.q[cur][1]);
  for (int d = 0; d < 3; ++d) {
    A.v[d] = tp<T>(B.v[d]);
    A.vn[d] = tp<T>(B.q[1 - cur][2 + d]);
  }
  A.dtp = dtp;
  A.fac = fac;
  Box ub;
  for (int e = 0; e < 3; ++e) {
    ub.lo[e] = A.lo[e];
    ub.hi[e] = A.hi[e];
  }
  if (G.bc == 2) DFK_LAUNCH((k_visc<T, 2>), grid_of_flat(ub), dim3(BX, BY), st, G, P, A);
  else if (G.bc) DFK_LAUNCH((k_visc<T, 1>), grid_of_flat(ub), dim3(BX, BY), st, G, P, A);
  else DFK_LAUNCH((k_visc<T, 0>), grid_of_flat(ub), dim3(BX, BY), st, G, P, A);
  LevFaces<T> out;
  for (int d = 0; d < 3; ++d) out.v[d] = tp<T>(B.v[d]);
  DFK_LAUNCH((k_copy_faces<T>), grid_of_flat(ub), dim3(BX, BY), st, G, A, out);
}

void viscosity(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp, double fac) {
  if (!(P.visc > 0.0)) return;
  if (P.fp32) viscosity_t<float>(st, G, P, B, cur, dtp, fac);
  else viscosity_t<double>(st, G, P, B, cur, dtp, fac);
}

template <typename T>
static void diffuse_heat_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp,
                           double fac, bool do_diff, bool do_heat, Scal *clear) {
  DiffArgs<T> A;
  A.clear = G.bc ? clear : nullptr;
  A.b = G.bc ? active_box(G) : clip_cells(G, uniform_box(G, 1, 1));
  A.rho = tp<T>(B.q[cur][0]);
  A.e = tp<T>(B.q[cur][1]);
  A.eo = tp<T>(B.etmp);
  A.hw = B.hw;
  for (int d = 0; d < 3; ++d) {
    A.hw_n[d] = B.hw_n[d];
    A.hw_lo[d] = G.anch[d] ? 0 : G.n[d] / 2 - B.hw_n[d] / 2;
  }
  A.dtp = dtp;
  A.fac = fac;
  A.do_diff = do_diff && P.chi > 0.0;
  A.do_heat = do_heat && P.L != 0.0;
  if (G.bc) {
    A.b.hi[0] = G.n[0] / 2;  // cell pairs: level-0 rows have an even length
    if (record(jk_df<T>(G.bc), DiffJob<T>{G, P, A, grid_of_flat(A.b).x})) return;
    if (G.bc == 2) DFK_LAUNCH((k_diffuse_heat2<T, 2>), grid_of_flat(A.b), dim3(BX, BY), st, G, P, A);
    else DFK_LAUNCH((k_diffuse_heat2<T, 1>), grid_of_flat(A.b), dim3(BX, BY), st, G, P, A);
  } else {
    DFK_LAUNCH(k_diffuse_heat<T>, grid_of_flat(A.b), dim3(BX, BY), st, G, P, A);
  }
}
void diffuse_heat(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, const double *dtp,
                  double fac, bool do_diff, bool do_heat, Scal *clear) {
  if (P.fp32) diffuse_heat_t<float>(st, G, P, B, cur, dtp, fac, do_diff, do_heat, clear);
  else diffuse_heat_t<double>(st, G, P, B, cur, dtp, fac, do_diff, do_heat, clear);
}

// Segment length of a walking launch over ext cells with cols blocks per layer
// of segments.
//
// walk_cells, for the fused x + y and z passes, which are bound by instruction
// issue and latency: a block's time is its segment's rows plus a prologue of
// `rows`, and a launch takes that times the rounds of `fill` blocks it makes
// (the blocks that run at once).  The length of least time is taken: on small
// meshes the shortest whose blocks run in one round, on larger ones whole
// rounds.  Beside other runs' launches (share) the fill is a part of the GPU
// and segments are not made longer than the default.
// seg_cells, for the streaming y and z passes, which are bound by memory: the
// default unless it leaves the GPU unfilled.
// Per step, with the default length and so: 32^3 107 -> 34 us (FP64), 56 -> 29
// (FP32); 64^3 104 -> 54, 54 -> 42; 96^3 148 -> 118, 89 -> 78; two levels of
// 32^3 203 -> 157, 219 -> 142.
static int seg_cells(const Segs &s, int ext, long cols, long fill, int lo) {
  if (s.cells > 0) return min(ext, s.cells);
  const long nseg = fill / s.share / max(cols, 1L);  // layers of segments a fill holds
  int c = min(ext, s.dflt);
  if (nseg >= 1) c = min(c, (int)((ext + nseg - 1) / nseg));
  return min(ext, max(c, lo));
}
static int walk_cells(const Segs &s, int ext, long cols, long fill, int rows) {
  if (s.cells > 0 || s.share > 1) return seg_cells(s, ext, cols, fill, 2);
  int best = ext;
  double least = 0.0;
  for (int nseg = 1; nseg <= (ext + 1) / 2; ++nseg) {
    const int c = (ext + nseg - 1) / nseg;
    double rounds = (double)(cols * ((ext + c - 1) / c)) / (double)fill;
    if (rounds < 4.0) rounds = std::ceil(rounds);
    const double time = rounds * (c + rows);
    if (nseg == 1 || time < least) {
      least = time;
      best = c;
    }
  }
  return best;
}
// Blocks of a fill, the best of 1/2 to 2 times as many over single-level cubes
// of 24 to 128 cells, whose rows take one tile (the forms of longer rows and of
// finer levels, whose registers allow other numbers of waves, take the same
// figures): the fused x + y pass two blocks per CU in FP64 and four in FP32,
// the fused z pass one and two, the streaming walks two; and the rows that the
// fused passes' prologues take: for the z pass 5 to 12 do equally well, with 2
// the finer levels of 128^3 (142 planes before their second sub-step) took
// segments of 12 planes, 104 us per level step against 92, and a level 0 of
// 200 x 184 x 152 in FP32 151 us against 134.
constexpr long XY_FILL64 = 512, XY_FILL32 = 1024, ZF_FILL64 = 256, ZF_FILL32 = 512, MARCH_FILL = 512;
constexpr int XY_ROWS = 5, ZF_ROWS = 8;

static size_t largest_face(const int *n) {
  return std::max((size_t)n[0] * n[1], std::max((size_t)n[0] * n[2], (size_t)n[1] * n[2]));
}
size_t front_faces(const Geo &G) { return largest_face(G.cn); }
size_t level_faces(const Geo &G) { return largest_face(G.n); }
template <typename T>
static void front_sums_t(hipStream_t st, const Geo &Gc, LevBufs &Bc, const Geo &Gf, LevBufs &Bf, bool two) {
  const FrontArgs<T> A{tp<T>(Bf.acc[0]), two ? tp<T>(Bf.acc[1]) : nullptr, tp<T>(Bc.fsum), (long)level_faces(Gf),
                       (long)front_faces(Gc)};
  DFK_LAUNCH(k_front_sum<T>, dim3((unsigned)((front_faces(Gc) + 255) / 256), 6, NQ), dim3(256), st, Gc, Gf, A);
}
void front_sums(hipStream_t st, const Geo &Gc, const Phys &P, LevBufs &Bc, const Geo &Gf, LevBufs &Bf, bool two) {
  if (P.fp32) front_sums_t<float>(st, Gc, Bc, Gf, Bf, two);
  else front_sums_t<double>(st, Gc, Bc, Gf, Bf, two);
}

template <typename T, int BC, int FR, int W>
static void march_launch(hipStream_t st, int dir, const Geo &G, const Phys &P, const MarchArgs<T> &M, dim3 gr,
                         dim3 bl) {
  if (dir == 1) DFK_LAUNCH((k_march<T, 1, BC, FR, W>), gr, bl, st, G, P, M);
  else DFK_LAUNCH((k_march<T, 2, BC, FR, W>), gr, bl, st, G, P, M);
}

template <typename T>
static void transport_pass_t(hipStream_t st, int dir, const Geo &G, const Phys &P, LevBufs &B, int src,
                             const double *dtp, double fac, const Segs &segs,
                             int sub) {
  PassArgs<T> A;
  if (G.bc) {
    A.b = active_box(G);
  } else {
    // in-bounds ranges that cover every entry the active cells depend on
    for (int d = 0; d < 3; ++d) {
      if (d == dir || (dir != 0 && d < dir)) {
        A.b.lo[d] = -G.g + 2;
        A.b.hi[d] = G.n[d] + G.g - 3;
      } else {
        A.b.lo[d] = -G.g;
        A.b.hi[d] = G.n[d] + G.g - 1;
      }
    }
    A.b = clip_cells(G, A.b);
    // the z walk of a quadrant level stores the images beyond the planes itself
    if (dir == 2 && G.anch[1]) A.b.lo[1] = A.b.lo[2] = 0;
  }
  for (int m = 0; m < NQ; ++m) {
    A.qi[m] = tp<T>(B.q[src][m]);
    A.qo[m] = tp<T>(B.q[1 - src][m]);
  }
  for (int d = 0; d < 3; ++d) A.v[d] = tp<T>(B.v[d]);
  A.dtp = dtp;
  A.fac = fac;
  A.acc = G.level > 0 ? tp<T>(B.acc[sub]) : nullptr;
  A.astr = (long)level_faces(G);
  A.fsum = tp<T>(B.fsum);
  A.fstr = (long)front_faces(G);
  if (dir == 0) {
    const dim3 bl(BX, BY);
    const int n = G.n[0];
    if (G.bc == 2) DFK_LAUNCH((k_xpass<T, 2>), grid_of(xtile_box(A.b)), bl, st, G, P, A);
    else if (G.bc && n <= BX) DFK_LAUNCH((k_xrow<T, 1>), grid_of(xrow_box(A.b)), bl, st, G, P, A);
    else if (G.bc && n <= 2 * BX && n % 2 == 0) DFK_LAUNCH((k_xrow<T, 2>), grid_of(xrow_box(A.b)), bl, st, G, P, A);
    else if (G.bc && n <= 4 * BX && n % 4 == 0) DFK_LAUNCH((k_xrow<T, 4>), grid_of(xrow_box(A.b)), bl, st, G, P, A);
    else if (G.bc) DFK_LAUNCH((k_xpass<T, 1>), grid_of(xtile_box(A.b)), bl, st, G, P, A);
    else {
      // finer levels: a row per wave when the cells the update reads, from an
      // aligned start, fit 64 R of them (in FP64 R <= 2: four cells per lane
      // take 138 registers, and the overlapping tiles were faster); else the
      // overlapping tiles
      const int x1 = A.b.hi[0] + 2;
      auto start = [&](int R) { return A.b.lo[0] - 2 - (((A.b.lo[0] - 2) % R) + R) % R; };
      if (x1 - start(1) <= BX) DFK_LAUNCH((k_xrow_fine<T, 1>), grid_of_flat(xrow_box(A.b)), bl, st, G, P, A, start(1));
      else if (x1 - start(2) <= 2 * BX)
        DFK_LAUNCH((k_xrow_fine<T, 2>), grid_of_flat(xrow_box(A.b)), bl, st, G, P, A, start(2));
      else if (sizeof(T) == 4 && x1 - start(4) <= 4 * BX)
        DFK_LAUNCH((k_xrow_fine<T, 4>), grid_of_flat(xrow_box(A.b)), bl, st, G, P, A, start(4));
      else DFK_LAUNCH((k_xpass<T, 0>), grid_of(xtile_box(A.b)), bl, st, G, P, A);
    }
    return;
  }
  MarchArgs<T> M;
  for (int d = 0; d < 3; ++d) {
    M.lo[d] = A.b.lo[d];
    M.hi[d] = A.b.hi[d];
  }
  const int ext = M.hi[dir] - M.lo[dir];
  if (ext <= 0) return;
  for (int m = 0; m < NQ; ++m) {
    M.qi[m] = A.qi[m];
    M.qo[m] = A.qo[m];
  }
  M.v = A.v[dir];
  M.dtp = A.dtp;
  M.fac = A.fac;
  M.acc = A.acc;
  M.astr = A.astr;
  M.fsum = A.fsum;
  M.fstr = A.fstr;
  const int td = (dir == 1) ? 2 : 1;
  const long ntb = (M.hi[td] - M.lo[td] + 1) / 2;
  const long ncol = (long)(M.hi[0] - M.lo[0]) * (M.hi[td] - M.lo[td]);
  const bool front = M.acc || M.fsum;
  // level 0 without frontier transfers: two adjacent columns per lane (its
  // rows start 128-byte aligned and the x extent is even) in FP32, and in FP64
  // for the z pass (its 16-byte accesses halve the address and load work per
  // byte; the FP64 y pass is fused with the x pass or keeps one column)
  const int w = ((sizeof(T) == 4 || dir == 2) && G.bc && !front && (M.hi[0] - M.lo[0]) % 2 == 0 &&
                 M.lo[0] % 2 == 0)
                    ? 2
                    : 1;
  const long nbx = (M.hi[0] - M.lo[0] + 64 * w - 1) / (64 * w);
  // one column per lane: blocks of 128 consecutive columns (k_march)
  const long cols = w == 1 ? (ncol + 127) / 128 : nbx * ntb;
  M.chunk = seg_cells(segs, ext, cols, MARCH_FILL, 2);
  const long nch = (ext + M.chunk - 1) / M.chunk;
  const dim3 gr((unsigned)(cols * nch)), bl(64, 4);
  if (!G.bc) {
    // finer levels always carry frontier transfers
    if (dir == 2 && G.anch[1]) DFK_LAUNCH((k_march<T, 2, 0, 3, 1, true>), gr, bl, st, G, P, M);
    else march_launch<T, 0, 3, 1>(st, dir, G, P, M, gr, bl);
  } else if (G.bc == 2) {
    if (front) march_launch<T, 2, 1, 1>(st, dir, G, P, M, gr, bl);
    else if (w == 2) march_launch<T, 2, 0, 2>(st, dir, G, P, M, gr, bl);
    else march_launch<T, 2, 0, 1>(st, dir, G, P, M, gr, bl);
  } else {
    if (front) march_launch<T, 1, 1, 1>(st, dir, G, P, M, gr, bl);
    else if (w == 2) march_launch<T, 1, 0, 2>(st, dir, G, P, M, gr, bl);
    else march_launch<T, 1, 0, 1>(st, dir, G, P, M, gr, bl);
  }
}
// tiles of a level-0 row of n cells: one while the row and, under bc 2, the
// cell past it fit its lanes; else whole tiles as long as more cells are left
// than the last one's, a part of a wave for the rest where it fits with the two
// cells before and past it
static XyTiles row_tiles(int n, int bc) {
  XyTiles B{0, n, 0, n, 1, 0};
  const int past = bc == 2 ? 2 : 0;
  if (n + past <= 2 * BX) return B;
  int left = n - (XY_TILE + XY_EDGE);
  for (; left + past > 2 * BX - 2; left -= XY_TILE) ++B.ntiles;
  if (left + 4 <= BX / 2) B.parts = 4;
  else if (left + 4 <= BX) B.parts = 2;
  else ++B.ntiles;
  return B;
}

template <typename T>
static void transport_xy_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int src, const double *dtp,
                           double fac, const Segs &segs) {
  const int n = G.n[0];
  PassArgs<T> A;
  A.b = active_box(G);
  for (int m = 0; m < NQ; ++m) {
    A.qi[m] = tp<T>(B.q[src][m]);
    A.qo[m] = tp<T>(B.q[1 - src][m]);
  }
  for (int d = 0; d < 3; ++d) A.v[d] = tp<T>(B.v[d]);
  A.dtp = dtp;
  A.fac = fac;
  // under a finer level: flux matching on its frontier (level 0 accumulates
  // nothing)
  A.acc = nullptr;
  A.fsum = tp<T>(B.fsum);
  A.fstr = (long)front_faces(G);
  MarchArgs<T> M;
  for (int d = 0; d < 3; ++d) {
    M.lo[d] = A.b.lo[d];
    M.hi[d] = A.b.hi[d];
  }
  for (int m = 0; m < NQ; ++m) {
    M.qi[m] = A.qo[m];
    M.qo[m] = A.qo[m];
  }
  M.v = A.v[1];
  M.dtp = dtp;
  M.fac = fac;
  M.acc = nullptr;
  M.fsum = A.fsum;
  M.fstr = A.fstr;
  // one block of four waves per (plane, y segment, tile)
  const bool one = n + (G.bc == 2 ? 1 : 0) <= BX;  // one cell per lane holds the row
  const XyTiles Bt = one ? XyTiles{0, n, 0, n, 1, 0} : row_tiles(n, G.bc);
  const long cols = Bt.blocks(G.n[2]);
  M.chunk = walk_cells(segs, G.n[1], cols, sizeof(T) == 8 ? XY_FILL64 : XY_FILL32, XY_ROWS);
  const long nch = (G.n[1] + M.chunk - 1) / M.chunk;
  const dim3 gr((unsigned)(cols * nch)), bl(64, 4);
  const bool many = Bt.ntiles > 1 || Bt.parts;
  const int fr = A.fsum ? 1 : 0;
  if (!fr && G.bc == 1 && !many && record(jk_xy<T>(n), XyJob<T>{G, P, A, M, Bt, gr.x})) return;
  auto go = [&](auto w, auto xb) {
    constexpr int W = decltype(w)::value, XB = decltype(xb)::value;
    if (fr) DFK_LAUNCH((k_xyshared<T, W, XB, 1>), gr, bl, st, G, P, A, M, Bt);
    else DFK_LAUNCH((k_xyshared<T, W, XB, 0>), gr, bl, st, G, P, A, M, Bt);
  };
  const std::integral_constant<int, 1> c1{};
  const std::integral_constant<int, 2> c2{};
  if (G.bc == 2 && one) go(c1, c2);
  else if (G.bc == 2) go(c2, c2);
  else if (one) go(c1, c1);
  else if (!many) go(c2, c1);
  else go(c2, std::integral_constant<int, 4>{});
}
void transport_xy(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int src, const double *dtp, double fac,
                  const Segs &segs) {
  if (P.fp32) transport_xy_t<float>(st, G, P, B, src, dtp, fac, segs);
  else transport_xy_t<double>(st, G, P, B, src, dtp, fac, segs);
}

template <typename T>
static void transport_xy_fine_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int src,
                                const double *dtp, double fac, const Segs &segs,
                                int sub) {
  PassArgs<T> A;
  // the y pass's box (x, y two cells inside the stored box, z all of it),
  // within G's margins
  for (int d = 0; d < 3; ++d) {
    A.b.lo[d] = d < 2 ? -G.g + 2 : -G.g;
    A.b.hi[d] = d < 2 ? G.n[d] + G.g - 3 : G.n[d] + G.g - 1;
  }
  A.b = clip_cells(G, A.b);
  if (G.anch[1]) A.b.lo[1] = A.b.lo[2] = 0;  // quadrant: from the mirror planes
  for (int m = 0; m < NQ; ++m) {
    A.qi[m] = tp<T>(B.q[src][m]);
    A.qo[m] = tp<T>(B.q[1 - src][m]);
  }
  for (int d = 0; d < 3; ++d) A.v[d] = tp<T>(B.v[d]);
  A.dtp = dtp;
  A.fac = fac;
  A.acc = tp<T>(B.acc[sub]);
  A.astr = (long)level_faces(G);
  A.fsum = tp<T>(B.fsum);
  A.fstr = (long)front_faces(G);
  MarchArgs<T> M;
  for (int d = 0; d < 3; ++d) {
    M.lo[d] = A.b.lo[d];
    M.hi[d] = A.b.hi[d];
  }
  const int ext = M.hi[1] - M.lo[1];
  if (ext <= 0 || M.hi[0] <= M.lo[0] || M.hi[2] <= M.lo[2]) return;
  for (int m = 0; m < NQ; ++m) {
    M.qi[m] = A.qi[m];
    M.qo[m] = A.qo[m];
  }
  M.v = A.v[1];
  M.dtp = dtp;
  M.fac = fac;
  M.acc = A.acc;
  M.astr = A.astr;
  M.fsum = A.fsum;
  M.fstr = A.fstr;
  // pairs of cells: whole tiles, then the row's last cells in tiles of a part of
  // a wave.  A box that the margin bounds is extended to whole pairs (what that
  // adds is not read); one that the stored shell bounds is not, since on small
  // meshes CommUp reads the entries beyond it as they were.
  XyTiles Bt;
  Bt.lo = A.b.lo[0] - (A.b.lo[0] & 1);
  Bt.hi = A.b.hi[0] + (A.b.hi[0] & 1);
  Bt.xlo = A.b.lo[0] == -G.g + 2 ? A.b.lo[0] : Bt.lo;
  Bt.xhi = A.b.hi[0] == G.n[0] + G.g - 3 ? A.b.hi[0] : Bt.hi;
  const int ex = Bt.hi - Bt.lo, np = M.hi[2] - M.lo[2];
  Bt.ntiles = ex / XY_TILE;
  const int tail = ex - Bt.ntiles * XY_TILE;
  Bt.parts = tail == 0 || tail > xy_tail_cells(2) ? 0 : tail > xy_tail_cells(4) ? 2 : 4;
  if (tail && !Bt.parts) ++Bt.ntiles;
  Segs xs = segs;
  if (xs.cells) xs.cells = max(xs.cells, 16);  // each segment x-updates four rows beyond its own
  const long cols = Bt.blocks(np);
  M.chunk = walk_cells(xs, ext, cols, sizeof(T) == 8 ? XY_FILL64 : XY_FILL32, XY_ROWS);
  const int nseg = (ext + M.chunk - 1) / M.chunk;
  const dim3 gr((unsigned)(cols * nseg)), bl(64, 4);
  if (G.anch[1] && A.fsum) DFK_LAUNCH((k_xyshared<T, 2, 3, 3>), gr, bl, st, G, P, A, M, Bt);
  else if (G.anch[1]) DFK_LAUNCH((k_xyshared<T, 2, 3, 2>), gr, bl, st, G, P, A, M, Bt);
  else if (A.fsum) DFK_LAUNCH((k_xyshared<T, 2, 0, 3>), gr, bl, st, G, P, A, M, Bt);
  else DFK_LAUNCH((k_xyshared<T, 2, 0, 2>), gr, bl, st, G, P, A, M, Bt);
}
void transport_xy_fine(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int src, const double *dtp,
                       double fac, const Segs &segs, int sub) {
  if (P.fp32) transport_xy_fine_t<float>(st, G, P, B, src, dtp, fac, segs, sub);
  else transport_xy_fine_t<double>(st, G, P, B, src, dtp, fac, segs, sub);
}

bool transport_z_finish_fits(const Geo &G) {
  return G.bc == 1 && !G.has_fine;  // (level-0 rows have an even length)
}

template <typename T>
static bool transport_z_finish_t(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, void *const *vin, int src,
                                 const double *dtp, double fac, double kfac, Scal *S, const Segs &segs) {
  // the walk reads the z-face velocities the finish rewrites: they must be
  // another set (the first kick's, when it was fused with the compression)
  if (!transport_z_finish_fits(G) || !S || vin[2] == B.v[2]) return false;
  MarchArgs<T> M{};
  const Box b = active_box(G);
  for (int d = 0; d < 3; ++d) {
    M.lo[d] = b.lo[d];
    M.hi[d] = b.hi[d];
  }
  const XyTiles Bt = zf_tiles(0, G.n[0]);
  const long cols = Bt.blocks((G.n[1] + ZF_TY - 1) / ZF_TY);
  M.chunk = walk_cells(segs, G.n[2], cols, sizeof(T) == 8 ? ZF_FILL64 : ZF_FILL32, ZF_ROWS);
  for (int m = 0; m < NQ; ++m) {
    M.qi[m] = tp<T>(B.q[src][m]);
    M.qo[m] = tp<T>(B.q[1 - src][m]);
  }
  M.v = tp<T>(vin[2]);
  M.dtp = dtp;
  M.fac = fac;
  M.acc = nullptr;
  M.fsum = nullptr;
  KickArgs<T> K{};
  for (int d = 0; d < 3; ++d) {
    K.v[d] = tp<T>(B.v[d]);
    K.vin[d] = K.v[d];
  }
  K.dtp = dtp;
  K.fac = kfac;
  const RedArgs<T> R = red_args<T>(G, B, 1 - src, S);
  const long nch = (G.n[2] + M.chunk - 1) / M.chunk;
  const long nblk = cols * nch;
  if (nblk > R.npart) return false;  // every block needs a partial slot
  const bool one = Bt.ntiles == 1 && !Bt.parts && G.n[1] % ZF_TY == 0;
  if (record(jk_zf<T>(one), ZfJob<T>{G, P, M, K, R, Bt, (unsigned)nblk})) return true;
  const dim3 gr((unsigned)nblk), bl(64, zf_waves<T, 1>());
  if (one) DFK_LAUNCH((k_zfinish<T, 1, 0>), gr, bl, st, G, P, M, K, R, Bt);
  else DFK_LAUNCH((k_zfinish<T, 4, 0>), gr, bl, st, G, P, M, K, R, Bt);
  return true;
}

bool transport_z_finish_fine_fits(const Geo &G, const Phys &P) {
  if (G.bc || P.visc > 0.0) return false;
  for (int d = 0; d < 3; ++d)
    if (G.mg[d] > G.g - 4) return false;
  return true;
}

template <typename T>
static void transport_z_finish_fine_t(hipStream_t st, const Geo &Gz, const Geo &G, const Phys &P, LevBufs &B,
                                      const void *vz, void *vzo, bool twice, int src, const double *dtp, double fac,
                                      double kfac, const Segs &segs, int sub) {
  MarchArgs<T> M{};
  for (int d = 0; d < 3; ++d) {
    M.lo[d] = -Gz.mg[d];
    M.hi[d] = Gz.n[d] + Gz.mg[d];
  }
  if (G.anch[1]) M.lo[1] = M.lo[2] = 0;  // quadrant: from the mirror planes
  // whole pairs of cells, as the fused x + y pass of the level stores
  const XyTiles Bt = zf_tiles(M.lo[0] - (M.lo[0] & 1), M.hi[0] + (M.hi[0] & 1));
  const int ext = M.hi[2] - M.lo[2];
  const long cols = Bt.blocks((M.hi[1] - M.lo[1] + ZF_TY - 1) / ZF_TY);
  M.chunk = walk_cells(segs, ext, cols, sizeof(T) == 8 ? ZF_FILL64 : ZF_FILL32, ZF_ROWS);
  for (int m = 0; m < NQ; ++m) {
    M.qi[m] = tp<T>(B.q[src][m]);
    M.qo[m] = tp<T>(B.q[1 - src][m]);
  }
  M.v = reinterpret_cast<const T *>(vz);
  M.dtp = dtp;
  M.fac = fac;
  M.acc = tp<T>(B.acc[sub]);
  M.astr = (long)level_faces(G);
  M.fsum = tp<T>(B.fsum);
  M.fstr = (long)front_faces(G);
  KickArgs<T> K{};
  for (int d = 0; d < 3; ++d) {
    K.v[d] = tp<T>(B.v[d]);
    K.vin[d] = K.v[d];
    for (int e = 0; e < 3; ++e) {
      K.flo[d][e] = -G.mg[e];
      K.fhi[d][e] = G.n[e] + G.mg[e] + (d == e ? 1 : 0);
    }
  }
  K.v[2] = tp<T>(vzo);
  K.dtp = dtp;
  K.fac = kfac;
  K.twice = twice;
  const RedArgs<T> R{};
  const dim3 gr((unsigned)(cols * ((ext + M.chunk - 1) / M.chunk))), bl(64, zf_waves<T, 0>());
  if (G.anch[1] && M.fsum) DFK_LAUNCH((k_zfinish<T, 3, 3>), gr, bl, st, Gz, P, M, K, R, Bt);
  else if (G.anch[1]) DFK_LAUNCH((k_zfinish<T, 3, 2>), gr, bl, st, Gz, P, M, K, R, Bt);
  else if (M.fsum) DFK_LAUNCH((k_zfinish<T, 0, 3>), gr, bl, st, Gz, P, M, K, R, Bt);
  else DFK_LAUNCH((k_zfinish<T, 0, 2>), gr, bl, st, Gz, P, M, K, R, Bt);
}
void transport_z_finish_fine(hipStream_t st, const Geo &Gz, const Geo &G, const Phys &P, LevBufs &B, const void *vz,
                             void *vzo, bool twice, int src, const double *dtp, double fac, double kfac,
                             const Segs &segs, int sub) {
  if (P.fp32) transport_z_finish_fine_t<float>(st, Gz, G, P, B, vz, vzo, twice, src, dtp, fac, kfac, segs, sub);
  else transport_z_finish_fine_t<double>(st, Gz, G, P, B, vz, vzo, twice, src, dtp, fac, kfac, segs, sub);
}
bool transport_z_finish(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, void *const *vin, int src,
                        const double *dtp, double fac, double kfac, Scal *S, const Segs &segs) {
  if (P.fp32) return transport_z_finish_t<float>(st, G, P, B, vin, src, dtp, fac, kfac, S, segs);
  return transport_z_finish_t<double>(st, G, P, B, vin, src, dtp, fac, kfac, S, segs);
}

void transport_pass(hipStream_t st, int dir, const Geo &G, const Phys &P, LevBufs &B, int src, const double *dtp,
                    double fac, const Segs &segs, int sub) {
  if (P.fp32) transport_pass_t<float>(st, dir, G, P, B, src, dtp, fac, segs, sub);
  else transport_pass_t<double>(st, dir, G, P, B, src, dtp, fac, segs, sub);
}

// each thread moves four 16-byte words (loads first), block b the words
// [1024 b, 1024 b + 1024)
__global__ void __launch_bounds__(256) k_copy16(uint4 *dst, const uint4 *src, size_t n) {
  const size_t base = (size_t)blockIdx.x * 1024 + threadIdx.x;
  uint4 w[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (base + 256 * u < n) w[u] = src[base + 256 * u];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (base + 256 * u < n) dst[base + 256 * u] = w[u];
}

void log_pending(hipStream_t st, const Geo &G, LevBufs &B, Scal *S, double *flog) {
  const LogJob J{(const double *)B.part, (int)part_count(G), S, flog, 1u};
  if (record(JK_LOG, J)) return;
  DFK_LAUNCH(k_log_pending, dim3(1), dim3(FT), st, J.part, J.npart, S, flog);
}

void set_recorder(Recorder *r) { g_rec = r; }

size_t job_entry_size(int kind) {
  switch (kind) {
    case JK_KC_D1: case JK_KC_D2: return sizeof(KcJob<double>);
    case JK_KC_F1: case JK_KC_F2: return sizeof(KcJob<float>);
    case JK_DF_D1: case JK_DF_D2: return sizeof(DiffJob<double>);
    case JK_DF_F1: case JK_DF_F2: return sizeof(DiffJob<float>);
    case JK_XY_D1: case JK_XY_D2: return sizeof(XyJob<double>);
    case JK_XY_F1: case JK_XY_F2: return sizeof(XyJob<float>);
    case JK_ZF_D1: case JK_ZF_D2: return sizeof(ZfJob<double>);
    case JK_ZF_F1: case JK_ZF_F2: return sizeof(ZfJob<float>);
    case JK_LOG: return sizeof(LogJob);
    default: return 0;
  }
}

template <typename E>
static JobTab<E> tab_of(const void *entries, const unsigned *start, int n) {
  return JobTab<E>{reinterpret_cast<const E *>(entries), start, n};
}

void launch_jobs(hipStream_t st, int kind, const void *entries, const unsigned *start, int n, unsigned nblocks) {
  const dim3 gr(nblocks), bl(BX, BY), xb(64, 4), zb(64, zf_waves<double, 1>());
  switch (kind) {
    case JK_KC_D1: DFK_LAUNCH((k_kick_compress_jobs<double, 1>), gr, bl, st, tab_of<KcJob<double>>(entries, start, n)); break;
    case JK_KC_D2: DFK_LAUNCH((k_kick_compress_jobs<double, 2>), gr, bl, st, tab_of<KcJob<double>>(entries, start, n)); break;
    case JK_KC_F1: DFK_LAUNCH((k_kick_compress_jobs<float, 1>), gr, bl, st, tab_of<KcJob<float>>(entries, start, n)); break;
    case JK_KC_F2: DFK_LAUNCH((k_kick_compress_jobs<float, 2>), gr, bl, st, tab_of<KcJob<float>>(entries, start, n)); break;
    case JK_DF_D1: DFK_LAUNCH((k_diffuse_heat2_jobs<double, 1>), gr, bl, st, tab_of<DiffJob<double>>(entries, start, n)); break;
    case JK_DF_D2: DFK_LAUNCH((k_diffuse_heat2_jobs<double, 2>), gr, bl, st, tab_of<DiffJob<double>>(entries, start, n)); break;
    case JK_DF_F1: DFK_LAUNCH((k_diffuse_heat2_jobs<float, 1>), gr, bl, st, tab_of<DiffJob<float>>(entries, start, n)); break;
    case JK_DF_F2: DFK_LAUNCH((k_diffuse_heat2_jobs<float, 2>), gr, bl, st, tab_of<DiffJob<float>>(entries, start, n)); break;
    case JK_XY_D1: DFK_LAUNCH((k_xyshared_jobs<double, 1>), gr, xb, st, tab_of<XyJob<double>>(entries, start, n)); break;
    case JK_XY_D2: DFK_LAUNCH((k_xyshared_jobs<double, 2>), gr, xb, st, tab_of<XyJob<double>>(entries, start, n)); break;
    case JK_XY_F1: DFK_LAUNCH((k_xyshared_jobs<float, 1>), gr, xb, st, tab_of<XyJob<float>>(entries, start, n)); break;
    case JK_XY_F2: DFK_LAUNCH((k_xyshared_jobs<float, 2>), gr, xb, st, tab_of<XyJob<float>>(entries, start, n)); break;
    case JK_ZF_D1: DFK_LAUNCH((k_zfinish_jobs<double, 1>), gr, zb, st, tab_of<ZfJob<double>>(entries, start, n)); break;
    case JK_ZF_D2: DFK_LAUNCH((k_zfinish_jobs<double, 4>), gr, zb, st, tab_of<ZfJob<double>>(entries, start, n)); break;
    case JK_ZF_F1: DFK_LAUNCH((k_zfinish_jobs<float, 1>), gr, zb, st, tab_of<ZfJob<float>>(entries, start, n)); break;
    case JK_ZF_F2: DFK_LAUNCH((k_zfinish_jobs<float, 4>), gr, zb, st, tab_of<ZfJob<float>>(entries, start, n)); break;
    case JK_LOG: DFK_LAUNCH(k_log_pending_jobs, gr, dim3(FT), st, tab_of<LogJob>(entries, start, n)); break;
    default: break;
  }
}

void stream_copy(hipStream_t st, void *dst, const void *src, size_t n16) {
  if (n16 == 0) return;
  const size_t blocks = (n16 + 1023) / 1024;
  DFK_LAUNCH(k_copy16, dim3((unsigned)blocks), dim3(256), st, reinterpret_cast<uint4 *>(dst),
                     reinterpret_cast<const uint4 *>(src), n16);
}

void zero(hipStream_t st, void *p, size_t bytes) {
  const size_t n = bytes / 4;
  if (n == 0 || !p) return;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  DFK_LAUNCH(k_zero, dim3((unsigned)blocks), dim3(256), st, reinterpret_cast<unsigned int *>(p), n);
}

// floor(i / 2)
static int fdiv2_host(int i) { return (i >= 0) ? i / 2 : -((1 - i) / 2); }

template <typename T>
static void commup_t(hipStream_t st, const Geo &Gc, LevBufs &Bc, int curc, const Geo &Gf, LevBufs &Bf, int curf) {
  UpArgs<T> A;
  for (int f = 0; f < NSTATE; ++f) {
    A.Q[f] = tp<T>(f == 0 ? Bc.q[curc][0] : (f == 1 ? Bc.q[curc][1] : Bc.v[f - 2]));
    A.out[f] = tp<T>(f == 0 ? Bf.q[curf][0] : (f == 1 ? Bf.q[curf][1] : Bf.v[f - 2]));
  }
  // hosts of the stored fine entries [-g, n+g) along each axis (from the
  // mirror plane along an anchored one: the entries beyond it are the fine
  // level's own images, which the same launch sets)
  for (int d = 0; d < 3; ++d) {
    A.b.lo[d] = Gf.anch[d] ? 0 : fdiv2_host(-Gf.g);
    A.b.hi[d] = fdiv2_host(Gf.s[d] - Gf.g - 1) + 1;
  }
  // the inner hosts, relative to b.lo (every fine child an active cell)
  unsigned ext[3];
  for (int d = 0; d < 3; ++d) {
    ext[d] = (unsigned)(A.b.hi[d] - A.b.lo[d]);
    const int lo = std::max(0, -A.b.lo[d]), hi = std::min((int)ext[d], Gf.n[d] / 2 - A.b.lo[d]);
    A.in_lo[d] = lo;
    A.in_n[d] = std::max(0, hi - lo);
  }
  if (A.in_n[0] == 0 || A.in_n[1] == 0 || A.in_n[2] == 0) A.in_n[0] = A.in_n[1] = A.in_n[2] = 0;
  A.c1 = (ext[2] - A.in_n[2]) * ext[0] * ext[1];
  A.c2 = A.c1 + A.in_n[2] * (ext[1] - A.in_n[1]) * ext[0];
  A.nshell = A.c2 + A.in_n[2] * A.in_n[1] * (ext[0] - A.in_n[0]);
  A.nb = (A.nshell + BX * BY - 1) / (BX * BY);
  A.ni = 0;
  if (Gf.anch[1]) {
    const unsigned w = (unsigned)Gf.g + 1;  // an upper bound over the fields
    A.ni = (unsigned)(Gf.n[0] + 1) * w * (unsigned)(Gf.n[1] + Gf.n[2] + 2);
    A.ni = (A.ni + BX * BY - 1) / (BX * BY);
  }
  const dim3 gr((A.nb + A.ni) * NSTATE);
  if (Gc.bc == 2) DFK_LAUNCH((k_commup<T, 2>), gr, dim3(BX, BY), st, Gc, Gf, A);
  else if (Gc.bc) DFK_LAUNCH((k_commup<T, 1>), gr, dim3(BX, BY), st, Gc, Gf, A);
  else DFK_LAUNCH((k_commup<T, 0>), gr, dim3(BX, BY), st, Gc, Gf, A);
}
void commup(hipStream_t st, const Geo &Gc, const Phys &P, LevBufs &Bc, int curc, const Geo &Gf, LevBufs &Bf,
            int curf) {
  if (P.fp32) commup_t<float>(st, Gc, Bc, curc, Gf, Bf, curf);
  else commup_t<double>(st, Gc, Bc, curc, Gf, Bf, curf);
}

template <typename T>
static void mirror_q_t(hipStream_t st, const Geo &G, LevBufs &B, int set) {
  for (int d = 1; d < 3; ++d) {
    if (!G.anch[d]) continue;
    MirArgs<T> A{};
    A.nf = NQ;
    for (int m = 0; m < NQ; ++m) {
      // the momenta normal to the plane swap and change sign: P-_d of an
      // image is -P+_d of its cell
      const int pair = (m == 2 + 2 * d) ? m + 1 : ((m == 3 + 2 * d) ? m - 1 : m);
      A.dst[m] = tp<T>(B.q[set][m]);
      A.src[m] = tp<T>(B.q[set][pair]);
      A.sgn[m] = pair != m ? T(-1) : T(1);
      A.face[m] = 0;
    }
    A.d = d;
    for (int e = 0; e < 3; ++e) {
      A.b.lo[e] = -G.g;
      A.b.hi[e] = e == d ? 0 : G.s[e] - G.g;
    }
    DFK_LAUNCH(k_mirror<T>, grid_of_flat(A.b), dim3(BX, BY), st, G, A);
  }
}

void mirror_q(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int set) {
  if (G.bc || !(G.anch[1] || G.anch[2])) return;
  if (P.fp32) mirror_q_t<float>(st, G, B, set);
  else mirror_q_t<double>(st, G, B, set);
}

template <typename T>
static void commmean_t(hipStream_t st, const Geo &Gf, LevBufs &Bf, int curf, const Geo &Gc, LevBufs &Bc,
                       int curc) {
  MeanArgs<T> A;
  A.start[0] = 0;
  for (int f = 0; f < NSTATE; ++f) {
    const int stag = f >= 2 ? f - 2 : -1;
    A.Q[f] = tp<T>(f == 0 ? Bf.q[curf][0] : (f == 1 ? Bf.q[curf][1] : Bf.v[f - 2]));
    A.out[f] = tp<T>(f == 0 ? Bc.q[curc][0] : (f == 1 ? Bc.q[curc][1] : Bc.v[f - 2]));
    Box b;
    for (int d = 0; d < 3; ++d) {
      A.b.lo[d] = b.lo[d] = 0;
      A.b.hi[d] = Gc.cn[d];
      b.hi[d] = Gc.cn[d] + (d == stag ? 1 : 0);
    }
    A.start[f + 1] = A.start[f] + grid_of_flat(b).x;
  }
  DFK_LAUNCH(k_commmean<T>, dim3(A.start[NSTATE]), dim3(BX, BY), st, Gf, Gc, A);
}
void commmean(hipStream_t st, const Geo &Gf, const Phys &P, LevBufs &Bf, int curf, const Geo &Gc, LevBufs &Bc,
              int curc) {
  if (P.fp32) commmean_t<float>(st, Gf, Bf, curf, Gc, Bc, curc);
  else commmean_t<double>(st, Gf, Bf, curf, Gc, Bc, curc);
}

size_t part_count(const Geo &G) {
  const Box b = active_box(G);
  return (size_t)grid_of(b).x;
}

template <typename T>
static RedArgs<T> red_args(const Geo &G, LevBufs &B, int cur, Scal *S) {
  RedArgs<T> A;
  A.b = active_box(G);
  A.rho = tp<T>(B.q[cur][0]);
  A.e = tp<T>(B.q[cur][1]);
  for (int d = 0; d < 3; ++d) A.v[d] = tp<T>(B.v[d]);
  A.part = B.part;
  A.npart = (int)part_count(G);
  A.spart = B.part + 3 * (size_t)A.npart;
  A.S = S;
  for (int d = 0; d < 3; ++d) {
    A.cov_lo[d] = G.has_fine ? G.co[d] : 0;
    A.cov_hi[d] = G.has_fine ? G.co[d] + G.cn[d] : 0;
  }
  return A;
}

void signal_speed(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, Scal *S) {
  if (P.fp32) {
    RedArgs<float> A = red_args<float>(G, B, cur, S);
    DFK_LAUNCH(k_signal<float>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  } else {
    RedArgs<double> A = red_args<double>(G, B, cur, S);
    DFK_LAUNCH(k_signal<double>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  }
}

static DtArgs dt_args(const Geo *G, const LevBufs *B, int nl, int advance) {
  DtArgs A;
  for (int l = 0; l < MAXLEV; ++l) {
    A.dx[l] = l < nl ? G[l].dx : 0.0;
    A.part[l] = l < nl ? B[l].part + 3 * part_count(G[l]) : nullptr;
    A.npart[l] = l < nl ? (int)part_count(G[l]) : 0;
  }
  A.nl = nl;
  A.advance = advance;
  return A;
}

void dt_final(hipStream_t st, const Geo *G, const LevBufs *B, int nl, const Phys &P, Scal *S, int advance) {
  DFK_LAUNCH(k_dt_final, dim3(1), dim3(FT), st, P, dt_args(G, B, nl, advance), S);
}

void post_partials(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur, Scal *S) {
  if (P.fp32) {
    RedArgs<float> A = red_args<float>(G, B, cur, S);
    DFK_LAUNCH(k_post<float>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  } else {
    RedArgs<double> A = red_args<double>(G, B, cur, S);
    DFK_LAUNCH(k_post<double>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  }
}

static FinalArgs final_args(double *const *parts, const int *nparts, int nl, Scal *S, int slot, double *flog) {
  FinalArgs A;
  for (int l = 0; l < MAXLEV; ++l) {
    A.part[l] = l < nl ? parts[l] : nullptr;
    A.npart[l] = l < nl ? nparts[l] : 0;
  }
  A.nl = nl;
  A.out = slot == 1 ? S->totals : S->force;
  A.S = S;
  A.flog = slot == 2 ? flog : nullptr;
  return A;
}

void step_final(hipStream_t st, const Geo *G, LevBufs *B, int nl, const Phys &P, Scal *S, double *flog,
                int do_force, int do_dt) {
  double *parts[MAXLEV];
  int np[MAXLEV];
  for (int l = 0; l < nl; ++l) {
    parts[l] = B[l].part;
    np[l] = (int)part_count(G[l]);
  }
  const FinalArgs F = final_args(parts, np, nl, S, 2, flog);
  const DtArgs D = dt_args(G, B, nl, do_dt == 2 ? 2 : 1);
  if (do_force && do_dt) DFK_LAUNCH((k_step_final<true, true>), dim3(1), dim3(FT), st, P, F, D, S);
  else if (do_force) DFK_LAUNCH((k_step_final<true, false>), dim3(1), dim3(FT), st, P, F, D, S);
  else if (do_dt) DFK_LAUNCH((k_step_final<false, true>), dim3(1), dim3(FT), st, P, F, D, S);
}

int force_partials(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur) {
  if (P.fp32) {
    RedArgs<float> A = red_args<float>(G, B, cur, nullptr);
    DFK_LAUNCH(k_force<float>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  } else {
    RedArgs<double> A = red_args<double>(G, B, cur, nullptr);
    DFK_LAUNCH(k_force<double>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  }
  return (int)part_count(G);
}

int totals_partials(hipStream_t st, const Geo &G, const Phys &P, LevBufs &B, int cur) {
  if (P.fp32) {
    RedArgs<float> A = red_args<float>(G, B, cur, nullptr);
    DFK_LAUNCH(k_totals<float>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  } else {
    RedArgs<double> A = red_args<double>(G, B, cur, nullptr);
    DFK_LAUNCH(k_totals<double>, grid_of(A.b), dim3(BX, BY), st, G, P, A);
  }
  return (int)part_count(G);
}

void force_final(hipStream_t st, double *const *parts, const int *nparts, int nl, Scal *S, int slot,
                 double *flog) {
  DFK_LAUNCH(k_final3, dim3(1), dim3(FT), st, final_args(parts, nparts, nl, S, slot, flog));
}

}  // namespace dfk
