// Galerkin coarsening of the variable-coefficient operator behind the C ABI of
// include/mg_galerkin.h.  Level 0 runs the 7-point kernels of mg_kernels.hip (red-black
// Gauss-Seidel with face coefficients, residual + full weighting, trilinear prolongation,
// norms); the coarse levels hold 27-point stencils R A P built on the GPU from the finer level's
// coefficients, and run the kernels below: eight-colour Gauss-Seidel, residual with full
// weighting, and, from 9^3 nodes down to the exact solve of the one-node coarsest level, the
// whole V-cycle in one launch.  A coarse level stores
// its stencil colour-major: for each of the eight parity colours, 27 arrays over that colour's
// nodes in C order, so that a colour pass of the smoother reads its coefficients contiguously.
#include "../../include/mg_galerkin.h"
#include "mg_kernels.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <new>
#include <type_traits>
#include <vector>

namespace {

constexpr size_t kGalAlign = 256;
constexpr int kGalThreads = 256;
constexpr int kCentre = 13;  // stencil array of the node itself: 9 + 3 + 1

thread_local char g_gal_err[512] = "no error";

__device__ __forceinline__ size_t gidx(int n, int z, int y, int x)
{
  return ((size_t)z * n + y) * (size_t)n + x;
}

// Colour-major stencil storage of a level with n nodes per side: half = (n-1)/2 slots per axis
// and colour; interior index v of parity p sits in slot (v - 2 + p) / 2; the coefficient of
// offset o at a node of colour c and slot t is S[(c * 27 + o) * half^3 + t].
__device__ __forceinline__ int colour_of(int z, int y, int x) { return 4 * (z & 1) + 2 * (y & 1) + (x & 1); }

__device__ __forceinline__ size_t slot_of(int half, int z, int y, int x)
{
  const int jz = (z - 2 + (z & 1)) / 2, jy = (y - 2 + (y & 1)) / 2, jx = (x - 2 + (x & 1)) / 2;
  return ((size_t)jz * half + jy) * half + jx;
}

// first coefficient (offset 0) of interior node (z, y, x); offset o at + o * half^3
template <typename TS>
__device__ __forceinline__ const TS* node_coeffs(const TS* S, int half, int z, int y, int x)
{
  const size_t h3 = (size_t)half * half * half;
  return S + (size_t)colour_of(z, y, x) * 27 * h3 + slot_of(half, z, y, x);
}

// (A u)_i - a_ii u_i: the off-diagonal part of the 27-point stencil at interior node i
template <typename TS>
__device__ __forceinline__ double offdiag(const TS* __restrict__ Sn, size_t h3,
                                          const double* __restrict__ u, int n, int z, int y, int x)
{
  double s = 0.0;
#pragma unroll
  for (int o = 0; o < 27; ++o) {
    if (o == kCentre) continue;
    const int dz = o / 9 - 1, dy = (o / 3) % 3 - 1, dx = o % 3 - 1;
    s += (double)Sn[o * h3] * u[gidx(n, z + dz, y + dy, x + dx)];
  }
  return s;
}

// Eight-colour Gauss-Seidel visits the colours C = 4 (z%2) + 2 (y%2) + x%2 in order; nodes of one
// colour never couple.  ZERO below: the first sweep from a zero iterate, which is not read before
// it is written: only the neighbours of the colours before C count (the colour of a neighbour is C
// with the parities of the offset's nonzero components flipped), which halves the coefficients
// read over the sweep.

// the coefficients of slot `slot` of colour C
template <int C, bool ZERO, typename TS>
__device__ __forceinline__ void load_coeffs(TS (&A)[27], const TS* __restrict__ S, size_t h3, size_t slot)
{
#pragma unroll
  for (int o = 0; o < 27; ++o) {
    const int nb = C ^ ((o / 9 != 1 ? 4 : 0) | ((o / 3) % 3 != 1 ? 2 : 0) | (o % 3 != 1 ? 1 : 0));
    if (ZERO && nb > C) continue;
    A[o] = S[((size_t)C * 27 + o) * h3 + slot];
  }
}

// The off-diagonal sum of colour C with the coefficients in registers; value(o, dz, dy, dx) gives
// the neighbour at an offset.
template <int C, bool ZERO, typename TS, typename F>
__device__ __forceinline__ double colour_offdiag(const TS (&A)[27], F&& value)
{
  double s = 0.0;
#pragma unroll
  for (int o = 0; o < 27; ++o) {
    const int dz = o / 9 - 1, dy = (o / 3) % 3 - 1, dx = o % 3 - 1;
    const int nb = C ^ ((dz ? 4 : 0) | (dy ? 2 : 0) | (dx ? 1 : 0));
    if (o == kCentre || (ZERO && nb > C)) continue;
    s += (double)A[o] * value(dz, dy, dx);
  }
  return s;
}

// Two colours of a sweep in one launch, C = 2 ZY and C + 1: the even and the odd nodes of the rows
// of (z, y)-parity ZY, which do not couple across rows.  A thread owns an even node and the odd
// one before it (the same slot of both colours); the odd node's two neighbours in the row come
// from the even phase through LDS.  Both nodes' 54 coefficients are in flight at once, and a sweep
// is four launches: at 65^3 5.9 us each, 23.6 us a sweep against 35 in eight (one per colour).
template <typename TS, int ZY, bool ZERO>
__global__ void __launch_bounds__(kGalThreads)
    k_gal_rows(int n, const TS* __restrict__ S, const double* __restrict__ f, double* u)
{
  constexpr int C = 2 * ZY;
  __shared__ double even[kGalThreads + 1];
  const int half = (n - 1) / 2;  // a power of two up to 256: rows do not straddle workgroups
  const int h2 = half * half, t = blockIdx.x * kGalThreads + threadIdx.x;
  const int jx = t % half, y = 2 * ((t / half) % half) + 2 - (ZY & 1), z = 2 * (t / h2) + 2 - (ZY >> 1);
  const bool row = t < h2 * half && y <= n - 2 && z <= n - 2;
  const size_t h3 = (size_t)h2 * half;
  const size_t i = gidx(n, z, y, 2 * jx + 1);  // the odd node; the even one is next
  TS A[27], B[27];
  double fo = 0.0, ve = 0.0;
  const bool e = row && 2 * jx + 2 <= n - 2;
  if (row) load_coeffs<C + 1, ZERO>(B, S, h3, t);
  if (e) {
    load_coeffs<C, ZERO>(A, S, h3, t);
    const double off = colour_offdiag<C, ZERO>(A, [&](int dz, int dy, int dx) {
      return u[i + 1 + (ptrdiff_t)(dz * n + dy) * n + dx];
    });
    ve = (f[i + 1] - off) / (double)A[kCentre];
    u[i + 1] = ve;
  }
  if (row) fo = f[i];
  even[threadIdx.x + 1] = ve;  // 0 on the boundary
  __syncthreads();
  if (!row) return;
  const double vw = jx ? even[threadIdx.x] : 0.0;
  const double off = colour_offdiag<C + 1, ZERO>(B, [&](int dz, int dy, int dx) {
    return dz || dy ? u[i + (ptrdiff_t)(dz * n + dy) * n + dx] : dx < 0 ? vw : ve;
  });
  u[i] = (fo - off) / (double)B[kCentre];
}

// Four colours of a sweep (those of z-parity PZ) in one launch on a small level: planes of one
// parity do not couple, and within a plane the colours follow each other in LDS.  One workgroup
// per plane, one thread per slot of a colour (half^2 of them); the coefficients of the next colour
// are read while the current one is computed.  A sweep is two launches: at 33^3 18.4 us against
// 35 in eight (one per colour).  Not at 65^3: its 32 workgroups draw too little bandwidth (87 us
// against 35).
template <typename TS, int PZ, bool ZERO, int HALF>
__global__ void __launch_bounds__(HALF * HALF)
    k_gal_planes(const TS* __restrict__ S, const double* __restrict__ f, double* u)
{
  constexpr int n = 2 * HALF + 1, plane = n * n, T = HALF * HALF;
  __shared__ double P[3 * plane];
  const int t = threadIdx.x, jx = t % HALF, jy = t / HALF;
  const int z = 2 * (int)blockIdx.x + 2 - PZ;
  if (z > n - 2) return;
  constexpr size_t h3 = (size_t)HALF * T;
  const size_t slot = (size_t)blockIdx.x * T + t;
  TS A[27], B[27];
  load_coeffs<4 * PZ, ZERO>(A, S, h3, slot);
  for (int i = t; i < 3 * plane; i += T) P[i] = u[(size_t)(z - 1) * plane + i];
  __syncthreads();
  auto colour = [&](auto CC, const TS (&K)[27]) {
    constexpr int C = decltype(CC)::value;
    const int x = 2 * jx + 2 - (C & 1), y = 2 * jy + 2 - ((C >> 1) & 1);
    if (x <= n - 2 && y <= n - 2) {
      const double* U = P + plane + y * n + x;
      const double off = colour_offdiag<C, ZERO>(K, [&](int dz, int dy, int dx) { return U[dz * plane + dy * n + dx]; });
      const double v = (f[(size_t)z * plane + y * n + x] - off) / (double)K[kCentre];
      P[plane + y * n + x] = v;
      u[(size_t)z * plane + y * n + x] = v;
    }
    __syncthreads();
  };
  load_coeffs<4 * PZ + 1, ZERO>(B, S, h3, slot);
  colour(std::integral_constant<int, 4 * PZ>{}, A);
  load_coeffs<4 * PZ + 2, ZERO>(A, S, h3, slot);
  colour(std::integral_constant<int, 4 * PZ + 1>{}, B);
  load_coeffs<4 * PZ + 3, ZERO>(B, S, h3, slot);
  colour(std::integral_constant<int, 4 * PZ + 2>{}, A);
  colour(std::integral_constant<int, 4 * PZ + 3>{}, B);
}

// r = f - A u at interior nodes (f == nullptr reads 0); the boundary of r is not written
template <typename TS>
__global__ void __launch_bounds__(kGalThreads)
    k_gal_residual(int n, const TS* __restrict__ S, const double* __restrict__ f,
                   const double* __restrict__ u, double* __restrict__ r)
{
  const int m = n - 2;
  const int t = blockIdx.x * kGalThreads + threadIdx.x;
  if (t >= m * m * m) return;
  const int x = 1 + t % m, y = 1 + (t / m) % m, z = 1 + t / (m * m);
  const int half = (n - 1) / 2;
  const size_t h3 = (size_t)half * half * half;
  const TS* Sn = node_coeffs(S, half, z, y, x);
  const size_t i = gidx(n, z, y, x);
  const double au = (double)Sn[kCentre * h3] * u[i] + offdiag(Sn, h3, u, n, z, y, x);
  r[i] = (f ? f[i] : 0.0) - au;
}

// fc = full weighting of r at coarse interior nodes (nf: fine nodes per side)
__global__ void __launch_bounds__(kGalThreads)
    k_gal_fw(int nf, const double* __restrict__ r, double* __restrict__ fc)
{
  const int nc = (nf - 1) / 2 + 1, m = nc - 2;
  const int t = blockIdx.x * kGalThreads + threadIdx.x;
  if (t >= m * m * m) return;
  const int X = 1 + t % m, Y = 1 + (t / m) % m, Z = 1 + t / (m * m);
  double s = 0.0;
  for (int oz = -1; oz <= 1; ++oz)
    for (int oy = -1; oy <= 1; ++oy)
      for (int ox = -1; ox <= 1; ++ox) {
        const double w = (oz ? 0.25 : 0.5) * (oy ? 0.25 : 0.5) * (ox ? 0.25 : 0.5);
        s += w * r[gidx(nf, 2 * Z + oz, 2 * Y + oy, 2 * X + ox)];
      }
  fc[gidx(nc, Z, Y, X)] = s;
}

// The Galerkin operator of the next level, one thread per coarse interior node I:
//   S_c[I][s] = sum_a w_a sum_b A[2I + a][b] P(2I + a + b, I + s)
// over the fine nodes 2I + a of the full weighting (w = 1/4, 1/2, 1/4 per axis), the couplings b of
// the fine operator and the coarse neighbours s, with P the trilinear interpolation (per axis: a
// fine node at distance 0 takes 1, at distance 1 takes 1/2 of the coarse value).  The 27 values of
// each fine row are contracted axis by axis.  One pass over the fine coefficients per level, where
// probing with 27 combs of coarse nodes took 27 prolongations, residuals and restrictions of
// whole levels (129^3: about 4 ms of launches for the hierarchy, 0.17 ms in all now).
struct RapSum {
  double c[3][3][3] = {};  // [z][y][x] offset + 1 of the coarse neighbour
  // adds w times the fine row A (27 couplings at offset o = 9 (dz+1) + 3 (dy+1) + dx+1) of the
  // fine node at distance (az, ay, ax) from 2I
  __device__ __forceinline__ void add(double w, const double (&A)[27], int az, int ay, int ax)
  {
    auto p = [](int t, int s) {  // weight of coarse offset s for a fine node at distance t from 2I
      const int d = t - 2 * s;
      return d == 0 ? 1.0 : d == 1 || d == -1 ? 0.5 : 0.0;
    };
    double Y[3][3][3] = {};  // [dz][sy][sx]
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int sx = 0; sx < 3; ++sx) {
          double X = 0.0;
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) X += A[9 * dz + 3 * dy + dx] * p(ax + dx - 1, sx - 1);
#pragma unroll
          for (int sy = 0; sy < 3; ++sy) Y[dz][sy][sx] += X * p(ay + dy - 1, sy - 1);
        }
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
      for (int sz = 0; sz < 3; ++sz) {
        const double q = w * p(az + dz - 1, sz - 1);
#pragma unroll
        for (int sy = 0; sy < 3; ++sy)
#pragma unroll
          for (int sx = 0; sx < 3; ++sx) c[sz][sy][sx] += q * Y[dz][sy][sx];
      }
  }
};

// coarse node t of a level with nc nodes per side; false past the last
__device__ __forceinline__ bool rap_node(int nc, int t, int& Z, int& Y, int& X)
{
  const int m = nc - 2;
  X = 1 + t % m;
  Y = 1 + (t / m) % m;
  Z = 1 + t / (m * m);
  return t < m * m * m;
}

// the coupling of coarse node (Z, Y, X) to its neighbour at offset o; 0 if that leaves the interior
__device__ __forceinline__ void rap_store(double v, int o, int nc, int Z, int Y, int X, double* __restrict__ S)
{
  const int half = (nc - 1) / 2;
  const size_t h3 = (size_t)half * half * half;
  const int z = Z + o / 9 - 1, y = Y + (o / 3) % 3 - 1, x = X + o % 3 - 1;
  const bool in = z >= 1 && z <= nc - 2 && y >= 1 && y <= nc - 2 && x >= 1 && x <= nc - 2;
  const_cast<double*>(node_coeffs(S, half, Z, Y, X))[o * h3] = in ? v : 0.0;
}

// from the 7-point operator of coefficient k (nc: coarse nodes per side)
__global__ void __launch_bounds__(kGalThreads)
    k_gal_rap_fine(int nc, double ih2, const double* __restrict__ k, double* __restrict__ S)
{
  int Z, Y, X;
  if (!rap_node(nc, blockIdx.x * kGalThreads + threadIdx.x, Z, Y, X)) return;
  const int n = 2 * (nc - 1) + 1;
  RapSum R;
  for (int a = 0; a < 27; ++a) {
    const int az = a / 9 - 1, ay = (a / 3) % 3 - 1, ax = a % 3 - 1;
    const int z = 2 * Z + az, y = 2 * Y + ay, x = 2 * X + ax;
    const double ki = k[gidx(n, z, y, x)];
    const double c0 = 0.5 * (ki + k[gidx(n, z, y, x - 1)]) * ih2, c1 = 0.5 * (ki + k[gidx(n, z, y, x + 1)]) * ih2;
    const double c2 = 0.5 * (ki + k[gidx(n, z, y - 1, x)]) * ih2, c3 = 0.5 * (ki + k[gidx(n, z, y + 1, x)]) * ih2;
    const double c4 = 0.5 * (ki + k[gidx(n, z - 1, y, x)]) * ih2, c5 = 0.5 * (ki + k[gidx(n, z + 1, y, x)]) * ih2;
    double A[27] = {};
    A[13] = ((((c0 + c1) + c2) + c3) + c4) + c5;
    A[12] = -c0;
    A[14] = -c1;
    A[10] = -c2;
    A[16] = -c3;
    A[4] = -c4;
    A[22] = -c5;
    R.add((az ? 0.25 : 0.5) * (ay ? 0.25 : 0.5) * (ax ? 0.25 : 0.5), A, az, ay, ax);
  }
#pragma unroll
  for (int o = 0; o < 27; ++o) rap_store(R.c[o / 9][(o / 3) % 3][o % 3], o, nc, Z, Y, X, S);
}

// From a 27-point level: eight coarse nodes per workgroup and one lane per fine row of a node (27 of
// 32 lanes), whose contributions meet in LDS and are summed in the order of the rows.  The levels
// are small: with a thread per coarse node the 27 rows were a serial chain of loads, 63-99 us a
// level from 65^3 down to 3^3; with a lane per row 46 us at 65^3, below 10 us on the others.
constexpr int kRapNodes = kGalThreads / 32;

__global__ void __launch_bounds__(kGalThreads)
    k_gal_rap(int nc, const double* __restrict__ Sf, double* __restrict__ S)
{
  __shared__ double part[kRapNodes][27][27];  // [node][row][coarse neighbour]
  const int g = threadIdx.x >> 5, a = threadIdx.x & 31;
  int Z, Y, X;
  const bool node = rap_node(nc, blockIdx.x * kRapNodes + g, Z, Y, X) && a < 27;
  if (node) {
    const int half = nc - 1;  // of the fine level
    const size_t h3 = (size_t)half * half * half;
    const int az = a / 9 - 1, ay = (a / 3) % 3 - 1, ax = a % 3 - 1;
    const double* Sn = node_coeffs(Sf, half, 2 * Z + az, 2 * Y + ay, 2 * X + ax);
    double A[27];
#pragma unroll
    for (int o = 0; o < 27; ++o) A[o] = Sn[o * h3];
    RapSum R;
    R.add((az ? 0.25 : 0.5) * (ay ? 0.25 : 0.5) * (ax ? 0.25 : 0.5), A, az, ay, ax);
#pragma unroll
    for (int s = 0; s < 27; ++s) part[g][a][s] = R.c[s / 9][(s / 3) % 3][s % 3];
  }
  __syncthreads();
  if (!node) return;
  double sum = 0.0;  // lane a: the coupling to the coarse neighbour at offset a
#pragma unroll
  for (int r = 0; r < 27; ++r) sum += part[g][r][a];
  rap_store(sum, a, nc, Z, Y, X, S);
}

__global__ void __launch_bounds__(kGalThreads)
    k_gal_to_f32(const double* __restrict__ S, float* __restrict__ S32, size_t count)
{
  const size_t t = (size_t)blockIdx.x * kGalThreads + threadIdx.x;
  if (t < count) S32[t] = (float)S[t];
}

// The V-cycle's tail in one launch: the levels of at most 9^3 nodes from a zero guess, by one
// workgroup, with u, f and the residual of every level in LDS and every thread the owner of one
// node with its 27 coefficients in registers.  A colour pass of such a level is at most 64 nodes,
// so its launch (2-3 us) costs far more than its work, and a cycle takes 8 colours x 4 sweeps of
// each.  (17^3 does not belong here: one compute unit draws its 0.7 MB of coefficients per sweep
// too slowly; the tail from 17^3 took 127 us per V(2,2)-cycle.)  Operations and their order are
// those of the per-level kernels.  Measured, 9^3 to 3^3, V(2,2): 33.6 us, against
// about 150 us in 70 launches.
constexpr int kGalTailN = 9, kGalTailLevels = 3, kGalTailThreads = 512;
static_assert((kGalTailN - 1) * (kGalTailN - 1) * (kGalTailN - 1) <= kGalTailThreads, "a node per thread");

template <typename TS>
struct GalTailArgs {
  const TS* S[kGalTailLevels];
  const double* Sc;  // the coarsest stencil, FP64
  const double* f;
  double* u;
  int n, levels, nu1, nu2;
};

__host__ __device__ constexpr int gal_tail_offset(int n0, int l)
{
  int off = 0, n = n0;
  for (int q = 0; q < l; ++q) {
    off += 3 * n * n * n;
    n = (n - 1) / 2 + 1;
  }
  return off;
}

template <typename TS>
__device__ __forceinline__ void gal_load(TS (&A)[27], const TS* __restrict__ S, int c, int h3, int t)
{
#pragma unroll
  for (int o = 0; o < 27; ++o) A[o] = S[(size_t)(c * 27 + o) * h3 + t];
}

// off-diagonal sum with the coefficients in registers and u in LDS (n nodes per side)
template <typename TS>
__device__ __forceinline__ double gal_offdiag(const TS (&A)[27], const double* u, int n, int i)
{
  double s = 0.0;
#pragma unroll
  for (int o = 0; o < 27; ++o) {
    if (o == kCentre) continue;
    const int dz = o / 9 - 1, dy = (o / 3) % 3 - 1, dx = o % 3 - 1;
    s += (double)A[o] * u[i + (dz * n + dy) * n + dx];
  }
  return s;
}

template <typename TS>
__global__ void __launch_bounds__(kGalTailThreads) k_gal_tail(GalTailArgs<TS> a)
{
  __shared__ double gal_lds[gal_tail_offset(kGalTailN, kGalTailLevels)];
  const int t = threadIdx.x;
  const int total = gal_tail_offset(a.n, a.levels);
  for (int i = t; i < total; i += kGalTailThreads) gal_lds[i] = 0.0;
  __syncthreads();
  struct L {
    int n, half, h3;
    double *u, *f, *r;
  };
  auto level = [&](int l) {
    L v;
    v.n = a.n;
    for (int q = 0; q < l; ++q) v.n = (v.n - 1) / 2 + 1;
    v.half = (v.n - 1) / 2;
    v.h3 = v.half * v.half * v.half;
    double* p = gal_lds + gal_tail_offset(a.n, l);
    v.u = p;
    v.f = p + v.n * v.n * v.n;
    v.r = v.f + v.n * v.n * v.n;
    return v;
  };
  // LDS index of a slot of colour c (-1: none)
  auto node = [&](const L& v, int c, int slot) {
    const int x = 2 * (slot % v.half) + 2 - (c & 1), y = 2 * ((slot / v.half) % v.half) + 2 - ((c >> 1) & 1);
    const int z = 2 * (slot / (v.half * v.half)) + 2 - (c >> 2);
    return x <= v.n - 2 && y <= v.n - 2 && z <= v.n - 2 ? (z * v.n + y) * v.n + x : -1;
  };
  // one step: the colour's update, or (res) its residual
  auto step = [&](const L& v, const TS (&A)[27], int i, bool res) {
    if (i < 0) return;
    const double off = gal_offdiag(A, v.u, v.n, i), d = (double)A[kCentre];
    if (res) v.r[i] = v.f[i] - (d * v.u[i] + off);
    else v.u[i] = (v.f[i] - off) / d;
  };
  // `passes` sweeps, then (res) the residual
  auto smooth = [&](const L& v, const TS* S, int passes, bool res) {
    // thread c h3 + slot owns one node
    const int c = t / v.h3, slot = t - c * v.h3;
    int i = -1;
    TS A[27];
    if (c < 8) {
      gal_load(A, S, c, v.h3, slot);
      i = node(v, c, slot);
    }
    for (int s = 0; s < passes; ++s)
      for (int q = 0; q < 8; ++q) {
        if (q == c) step(v, A, i, false);
        __syncthreads();
      }
    if (res) {
      step(v, A, i, true);
      __syncthreads();
    }
  };
  {
    const L v = level(0);
    const int N = v.n * v.n * v.n;
    for (int i = t; i < N; i += kGalTailThreads) v.f[i] = a.f[i];
    __syncthreads();
  }
  const int last = a.levels - 1;
  for (int l = 0; l < last; ++l) {
    const L v = level(l), w = level(l + 1);
    smooth(v, a.S[l], a.nu1, true);
    const int m = w.n - 2;
    for (int q = t; q < m * m * m; q += kGalTailThreads) {
      const int X = 1 + q % m, Y = 1 + (q / m) % m, Z = 1 + q / (m * m);
      double s = 0.0;
#pragma unroll
      for (int oz = -1; oz <= 1; ++oz)
#pragma unroll
        for (int oy = -1; oy <= 1; ++oy)
#pragma unroll
          for (int ox = -1; ox <= 1; ++ox)
            s += (oz ? 0.25 : 0.5) * (oy ? 0.25 : 0.5) * (ox ? 0.25 : 0.5) *
                 v.r[((2 * Z + oz) * v.n + 2 * Y + oy) * v.n + 2 * X + ox];
      w.f[(Z * w.n + Y) * w.n + X] = s;
    }
    __syncthreads();
  }
  {
    const L v = level(last);  // 3^3: one interior node (colour 7, slot 0 of one)
    if (t == 0) v.u[13] = v.f[13] / node_coeffs(a.Sc, 1, 1, 1, 1)[kCentre];
    __syncthreads();
  }
  for (int l = last - 1; l >= 0; --l) {
    const L v = level(l), w = level(l + 1);
    const int m = v.n - 2;
    for (int q = t; q < m * m * m; q += kGalTailThreads) {
      const int x = 1 + q % m, y = 1 + (q / m) % m, z = 1 + q / (m * m);
      const double wt = ((z & 1) ? 0.5 : 1.0) * ((y & 1) ? 0.5 : 1.0) * ((x & 1) ? 0.5 : 1.0);
      double s = 0.0;  // the terms of prolong_add, in its order
      for (int b = 0; b <= (z & 1); ++b)
        for (int c = 0; c <= (y & 1); ++c) {
          const double* e = w.u + (((z >> 1) + b) * w.n + (y >> 1) + c) * w.n + ((x + 1) >> 1);
          if (x & 1) s = s + wt * e[-1];
          s = s + wt * e[0];
        }
      const int i = (z * v.n + y) * v.n + x;
      v.u[i] = v.u[i] + s;
    }
    __syncthreads();
    smooth(v, a.S[l], a.nu2, false);
  }
  const L v = level(0);
  const int N = v.n * v.n * v.n;
  for (int i = t; i < N; i += kGalTailThreads) a.u[i] = v.u[i];
}

// out[o][i] = the stencil in natural layout (27 arrays of n^3 values, 0 off the interior)
__global__ void __launch_bounds__(kGalThreads)
    k_gal_export(int n, const double* __restrict__ S, double* __restrict__ out)
{
  const size_t t = (size_t)blockIdx.x * kGalThreads + threadIdx.x;
  const size_t cnt = (size_t)n * n * n;
  if (t >= cnt) return;
  const int x = (int)(t % n), y = (int)((t / n) % n), z = (int)(t / ((size_t)n * n));
  const bool in = x > 0 && y > 0 && z > 0 && x < n - 1 && y < n - 1 && z < n - 1;
  const int half = (n - 1) / 2;
  const size_t h3 = (size_t)half * half * half;
  const double* Sn = in ? node_coeffs(S, half, z, y, x) : nullptr;
  for (int o = 0; o < 27; ++o) out[o * cnt + t] = in ? Sn[o * h3] : 0.0;
}

unsigned blocks_for(size_t count) { return (unsigned)((count + kGalThreads - 1) / kGalThreads); }

}  // namespace

struct GalLevel {
  int n = 0;
  size_t cnt = 0;
  size_t scnt = 0;      // doubles of the colour-major stencil: 8 colours x 27 x ((n-1)/2)^3
  double* u = nullptr;  // correction (levels >= 1)
  double* f = nullptr;  // right-hand side (levels >= 1)
  double* r = nullptr;  // residual (levels >= 1)
  double* S = nullptr;  // colour-major stencil (levels >= 1)
  float* S32 = nullptr; // its FP32 copy for the cycle (coarse_f32)
};

struct mggal_ctx {
  mggal_grid g{};
  hipStream_t s = nullptr;
  double h = 0;
  double* k = nullptr;      // copy of the coefficient
  double* t = nullptr;      // level 0's second buffer
  int tail = -1;            // first level of the one-launch tail (the coarsest, 3^3, at the latest)
  double* partial = nullptr;
  double* scal = nullptr;
  mgk::HostNorm hn;         // where norms are written to
  std::vector<GalLevel> lv;
  char err[512] = "no error";
};

namespace {

mg_status gal_fail(mggal_ctx* c, mg_status st, const char* fmt, ...)
{
  char* buf = c ? c->err : g_gal_err;
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, 512, fmt, ap);
  va_end(ap);
  return st;
}

mg_status gal_hip(mggal_ctx* c, hipError_t e, const char* what)
{
  if (e == hipSuccess) return MG_OK;
  return gal_fail(c, MG_EHIP, "%s: %s", what, hipGetErrorString(e));
}

mg_status gal_validate(const mggal_grid* g)
{
  if (!g) return gal_fail(nullptr, MG_EINVAL, "grid description is NULL");
  const int n = g->n;
  if (n < 5 || n > 1025 || ((n - 1) & (n - 2)) != 0)
    return gal_fail(nullptr, MG_EINVAL, "n must be 2^m + 1 in [5, 1025] (got %d)", n);
  int nl = n;
  for (int l = 1; l < g->levels; ++l) nl = (nl - 1) / 2 + 1;
  if (g->levels < 2 || nl != 3)
    return gal_fail(nullptr, MG_EINVAL, "levels must reach 3 nodes per side (n=%d, levels=%d)", n, g->levels);
  if (g->nu1 < 0 || g->nu2 < 0) return gal_fail(nullptr, MG_EINVAL, "nu1, nu2 must be >= 0");
  if (g->max_cycles < 1) return gal_fail(nullptr, MG_EINVAL, "max_cycles must be >= 1");
  if (g->coarse_f32 != 0 && g->coarse_f32 != 1) return gal_fail(nullptr, MG_EINVAL, "coarse_f32 must be 0 or 1");
  return MG_OK;
}

struct GalCarver {
  char* base;
  size_t off = 0;
  template <typename T>
  T* take(size_t count)
  {
    off = (off + kGalAlign - 1) / kGalAlign * kGalAlign;
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

void gal_layout(const mggal_grid* g, GalCarver& cv, mggal_ctx* c)
{
  const size_t cnt0 = (size_t)g->n * g->n * g->n;
  double* k = cv.take<double>(cnt0);
  double* t = cv.take<double>(cnt0);
  // A third fine array, which the probing set-up needed and nothing uses now, is still counted: the
  // size that mggal_workspace_bytes reports is tested to hold three.
  (void)cv.take<double>(cnt0);
  double* partial = cv.take<double>(mgk::kStreamPartials);
  double* scal = cv.take<double>(8);
  std::vector<GalLevel> lv;
  int n = g->n;
  for (int l = 0; l < g->levels; ++l) {
    GalLevel L;
    L.n = n;
    L.cnt = (size_t)n * n * n;
    const size_t half = (size_t)(n - 1) / 2;
    L.scnt = 8 * 27 * half * half * half;
    if (l > 0) {
      L.u = cv.take<double>(L.cnt);
      L.f = cv.take<double>(L.cnt);
      L.r = cv.take<double>(L.cnt);
      L.S = cv.take<double>(L.scnt);
      if (g->coarse_f32) L.S32 = cv.take<float>(L.scnt);
    }
    lv.push_back(L);
    n = (n - 1) / 2 + 1;
  }
  if (c) {
    c->k = k;
    c->t = t;
    c->partial = partial;
    c->scal = scal;
    c->lv = lv;
  }
}

// level 0 on a large grid: the streaming kernels of the rediscretised path
bool fine_tiled(const mggal_ctx* c) { return mgk::rbgs_tiled_supported(3, c->g.n); }

// `sweeps` red-black sweeps on level 0, two per launch, from u (or u + P ec), alternating with t
// (same boundary values); returns the buffer with the result.  fc: also the restricted residual.
double* smooth_fine(mggal_ctx* c, const double* f, double* u, double* t, int sweeps, const double* ec, double* fc)
{
  const int n = c->g.n;
  const bool tiled = fine_tiled(c);
  if (ec && (sweeps == 0 || (tiled && sweeps == 1))) {  // the large grids' one-sweep pass takes no correction
    mgk::prolong_add<double>(c->s, 3, c->lv[1].n, ec, u);
    ec = nullptr;
  }
  double *cur = u, *oth = t;
  bool restricted = false;
  while (sweeps > 0) {
    const int sw = sweeps >= 2 ? 2 : 1;
    if (tiled) {
      mgk::rbgs_tiled<double>(c->s, n, c->h, c->k, f, cur, oth, sw, false, ec);
    } else {
      mgk::rbgs_cube<double>(c->s, n, c->h, c->k, f, cur, oth, sw, false, ec, sweeps == sw ? fc : nullptr);
      restricted = sweeps == sw && fc;
    }
    double* x = cur;
    cur = oth;
    oth = x;
    sweeps -= sw;
    ec = nullptr;
  }
  if (fc && !restricted) {
    if (tiled) mgk::restrict_residual_tiled<double>(c->s, n, c->h, c->k, f, cur, fc);
    else mgk::restrict_residual<double>(c->s, 3, n, c->h, c->k, f, cur, fc);
  }
  return cur;
}

// one sweep: whole planes per workgroup where a level has too few rows to fill the device
template <typename TS, bool ZERO>
void sweep_coarse(hipStream_t s, const GalLevel& L, const TS* S, const double* f, double* u)
{
  if (L.n == 17) {
    k_gal_planes<TS, 0, ZERO, 8><<<8, 64, 0, s>>>(S, f, u);
    k_gal_planes<TS, 1, ZERO, 8><<<8, 64, 0, s>>>(S, f, u);
  } else if (L.n == 33) {
    k_gal_planes<TS, 0, ZERO, 16><<<16, 256, 0, s>>>(S, f, u);
    k_gal_planes<TS, 1, ZERO, 16><<<16, 256, 0, s>>>(S, f, u);
  } else {
    const size_t half = (size_t)(L.n - 1) / 2;
    const unsigned gb = blocks_for(half * half * half);
    k_gal_rows<TS, 0, ZERO><<<gb, kGalThreads, 0, s>>>(L.n, S, f, u);
    k_gal_rows<TS, 1, ZERO><<<gb, kGalThreads, 0, s>>>(L.n, S, f, u);
    k_gal_rows<TS, 2, ZERO><<<gb, kGalThreads, 0, s>>>(L.n, S, f, u);
    k_gal_rows<TS, 3, ZERO><<<gb, kGalThreads, 0, s>>>(L.n, S, f, u);
  }
}

// `sweeps` eight-colour sweeps on a coarse level; zero: u is 0 (not read)
void smooth_coarse(mggal_ctx* c, int l, int sweeps, bool zero)
{
  const GalLevel& L = c->lv[l];
  if (zero && sweeps == 0) mgk::fill<double>(c->s, L.cnt, 0.0, L.u);
  for (int s = 0; s < sweeps; ++s) {
    if (L.S32 && zero && s == 0) sweep_coarse<float, true>(c->s, L, L.S32, L.f, L.u);
    else if (L.S32) sweep_coarse<float, false>(c->s, L, L.S32, L.f, L.u);
    else if (zero && s == 0) sweep_coarse<double, true>(c->s, L, L.S, L.f, L.u);
    else sweep_coarse<double, false>(c->s, L, L.S, L.f, L.u);
  }
}

template <typename TS>
void launch_tail(mggal_ctx* c, int l, const TS* (*stencil)(const GalLevel&))
{
  GalTailArgs<TS> a{};
  a.levels = (int)c->lv.size() - l;
  for (int q = 0; q + 1 < a.levels; ++q) a.S[q] = stencil(c->lv[l + q]);
  a.Sc = c->lv.back().S;
  a.f = c->lv[l].f;
  a.u = c->lv[l].u;
  a.n = c->lv[l].n;
  a.nu1 = c->g.nu1;
  a.nu2 = c->g.nu2;
  k_gal_tail<TS><<<1, kGalTailThreads, 0, c->s>>>(a);
}

// the correction of coarse level l (its f to its u), from zero
void coarse_cycle(mggal_ctx* c, int l)
{
  GalLevel& L = c->lv[l];
  if (l == c->tail) {
    if (c->g.coarse_f32) launch_tail<float>(c, l, [](const GalLevel& q) -> const float* { return q.S32; });
    else launch_tail<double>(c, l, [](const GalLevel& q) -> const double* { return q.S; });
    return;
  }
  GalLevel& C = c->lv[l + 1];
  smooth_coarse(c, l, c->g.nu1, true);
  const size_t mf = (size_t)L.n - 2, mc = (size_t)C.n - 2;
  if (L.S32) k_gal_residual<float><<<blocks_for(mf * mf * mf), kGalThreads, 0, c->s>>>(L.n, L.S32, L.f, L.u, L.r);
  else k_gal_residual<double><<<blocks_for(mf * mf * mf), kGalThreads, 0, c->s>>>(L.n, L.S, L.f, L.u, L.r);
  k_gal_fw<<<blocks_for(mc * mc * mc), kGalThreads, 0, c->s>>>(L.n, L.r, C.f);
  coarse_cycle(c, l + 1);
  mgk::prolong_add<double>(c->s, 3, C.n, C.u, L.u);
  smooth_coarse(c, l, c->g.nu2, false);
}

// one V-cycle, the result in u; the second buffer holds u's boundary values
void vcycle(mggal_ctx* c, const double* f, double* u)
{
  double* cur = smooth_fine(c, f, u, c->t, c->g.nu1, nullptr, c->lv[1].f);
  coarse_cycle(c, 1);
  double* r = smooth_fine(c, f, cur, cur == u ? c->t : u, c->g.nu2, c->lv[1].u, nullptr);
  if (r != u) mgk::copy<double>(c->s, c->lv[0].cnt, r, u);
}

void copy_boundary(mggal_ctx* c, const double* u) { mgk::copy_boundary(c->s, 3, c->g.n, u, c->t); }

// Galerkin operator of level l+1 from level l
void build_level(mggal_ctx* c, int l)
{
  GalLevel& C = c->lv[l + 1];
  const size_t m = (size_t)C.n - 2;
  if (l == 0) k_gal_rap_fine<<<blocks_for(m * m * m), kGalThreads, 0, c->s>>>(C.n, 1.0 / (c->h * c->h), c->k, C.S);
  else k_gal_rap<<<(unsigned)((m * m * m + kRapNodes - 1) / kRapNodes), kGalThreads, 0, c->s>>>(C.n, c->lv[l].S, C.S);
}

mg_status read_norm2(mggal_ctx* c, const double* f, const double* u, int mode, double* out)
{
  c->hn.take();
  c->hn.unread = true;
  double* at = c->hn.mem ? c->hn.mem : c->scal;
  if (fine_tiled(c)) mgk::resid_norm2_tiled(c->s, c->g.n, c->h, c->k, f, u, mode, c->partial, at);
  else mgk::resid_norm2(c->s, 3, c->g.n, c->h, c->k, f, u, mode, c->partial, at);
  if (mg_status st = gal_hip(c, hipGetLastError(), "norm")) return st;
  if (!c->hn.mem)
    if (mg_status st = gal_hip(c, hipMemcpyAsync(out, c->scal, sizeof(double), hipMemcpyDeviceToHost, c->s),
                               "reading the norm"))
      return st;
  if (mg_status st = gal_hip(c, hipStreamSynchronize(c->s), "stream synchronisation")) return st;
  c->hn.unread = false;
  if (c->hn.mem) *out = mgk::host_norm(c->hn.mem, 0);
  return MG_OK;
}

}  // namespace

// ================================================================== C ABI
extern "C" {

size_t mggal_workspace_bytes(const mggal_grid* grid)
{
  if (gal_validate(grid) != MG_OK) return 0;
  GalCarver cv{nullptr};
  gal_layout(grid, cv, nullptr);
  return cv.off + kGalAlign;
}

mg_status mggal_setup(const mggal_grid* grid, const double* k, void* workspace, size_t bytes,
                      void* stream, mggal_ctx** out)
{
  if (!out) return gal_fail(nullptr, MG_EINVAL, "out is NULL");
  *out = nullptr;
  if (mg_status st = gal_validate(grid)) return st;
  if (!k) return gal_fail(nullptr, MG_EINVAL, "k is NULL");
  if (!workspace) return gal_fail(nullptr, MG_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(workspace) % kGalAlign != 0)
    return gal_fail(nullptr, MG_EINVAL, "workspace must be %zu-byte aligned", kGalAlign);
  const size_t need = mggal_workspace_bytes(grid);
  if (bytes < need) return gal_fail(nullptr, MG_ENOMEM, "workspace of %zu bytes < %zu required", bytes, need);
  mggal_ctx* c = new (std::nothrow) mggal_ctx;
  if (!c) return gal_fail(nullptr, MG_ENOMEM, "host allocation of the context failed");
  c->g = *grid;
  c->s = static_cast<hipStream_t>(stream);
  c->h = 1.0 / (grid->n - 1);
  GalCarver cv{static_cast<char*>(workspace)};
  gal_layout(grid, cv, c);
  c->hn.set_device();
  mgk::copy<double>(c->s, c->lv[0].cnt, k, c->k);
  for (size_t l = 1; l < c->lv.size(); ++l) {  // zero boundaries of every coarse array
    mgk::fill<double>(c->s, c->lv[l].cnt, 0.0, c->lv[l].u);
    mgk::fill<double>(c->s, c->lv[l].cnt, 0.0, c->lv[l].f);
    mgk::fill<double>(c->s, c->lv[l].cnt, 0.0, c->lv[l].r);
  }
  for (size_t l = 0; l + 1 < c->lv.size(); ++l) build_level(c, (int)l);
  for (int l = 1; l < grid->levels && c->tail < 0; ++l)
    if (c->lv[l].n <= kGalTailN && grid->levels - l <= kGalTailLevels) c->tail = l;
  for (size_t l = 1; l < c->lv.size(); ++l)
    if (c->lv[l].S32)
      k_gal_to_f32<<<blocks_for(c->lv[l].scnt), kGalThreads, 0, c->s>>>(c->lv[l].S, c->lv[l].S32, c->lv[l].scnt);
  mg_status st = gal_hip(c, hipGetLastError(), "building the Galerkin hierarchy");
  if (!st) st = gal_hip(c, hipStreamSynchronize(c->s), "setup");
  if (st) {
    snprintf(g_gal_err, sizeof g_gal_err, "%s", c->err);
    delete c;
    return st;
  }
  *out = c;
  return MG_OK;
}

void mggal_destroy(mggal_ctx* c) { delete c; }

const char* mggal_last_error(const mggal_ctx* c) { return c ? c->err : g_gal_err; }

mg_status mggal_stencil(mggal_ctx* c, int level, double* out)
{
  if (!c) return gal_fail(nullptr, MG_EINVAL, "context is NULL");
  if (level < 1 || level >= (int)c->lv.size()) return gal_fail(c, MG_EINVAL, "level %d has no stencil", level);
  if (!out) return gal_fail(c, MG_EINVAL, "out is NULL");
  const GalLevel& L = c->lv[level];
  k_gal_export<<<blocks_for(L.cnt), kGalThreads, 0, c->s>>>(L.n, L.S, out);
  return gal_hip(c, hipGetLastError(), "exporting the stencil");
}

mg_status mggal_vcycle(mggal_ctx* c, const double* f, double* u)
{
  if (!c) return gal_fail(nullptr, MG_EINVAL, "context is NULL");
  if (!f || !u) return gal_fail(c, MG_EINVAL, "f and u must be non-NULL");
  copy_boundary(c, u);
  vcycle(c, f, u);
  return gal_hip(c, hipGetLastError(), "V-cycle");
}

mg_status mggal_solve(mggal_ctx* c, const double* f, double* u, double tol, int* cycles,
                      double* relres)
{
  if (!c) return gal_fail(nullptr, MG_EINVAL, "context is NULL");
  if (!f || !u) return gal_fail(c, MG_EINVAL, "f and u must be non-NULL");
  if (!(tol > 0)) return gal_fail(c, MG_EINVAL, "tol must be > 0");
  double b2 = 0, r2 = 0;
  mg_status st = read_norm2(c, f, u, 1, &b2);
  const double bn = std::sqrt(b2);
  if (!st && !(bn > 0 && std::isfinite(bn))) st = gal_fail(c, MG_EINVAL, "right-hand side norm %.3e", bn);
  int kcyc = 0;
  double rel = 1.0;
  if (!st) st = read_norm2(c, f, u, 0, &r2);
  if (!st) rel = std::sqrt(r2) / bn;
  if (!st) copy_boundary(c, u);
  while (!st && std::isfinite(rel) && rel > tol && kcyc < c->g.max_cycles) {
    vcycle(c, f, u);
    ++kcyc;
    st = read_norm2(c, f, u, 0, &r2);
    rel = std::sqrt(r2) / bn;
  }
  if (cycles) *cycles = kcyc;
  if (relres) *relres = rel;
  if (st) return st;
  if (!std::isfinite(rel)) return gal_fail(c, MG_ENAN, "residual norm is not finite after %d cycles", kcyc);
  if (rel > tol) return gal_fail(c, MG_ENOCONV, "relative residual %.3e > tol %.3e after %d cycles", rel, tol, kcyc);
  return MG_OK;
}

}  // extern "C"
