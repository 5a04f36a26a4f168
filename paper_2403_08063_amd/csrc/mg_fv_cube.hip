// Damped-Jacobi sweeps of the cell-centred finite-volume scheme on small levels (16^3 to
// 64^3 cells) in one launch, on gfx950: as mg_fv_tiled.hip, 2 or 3 sweeps with the prolongation before
// or the restriction after them and the norm of the input's residual, but from boxes in LDS.
//
// The plane-marching kernel takes ten plane steps of 2-3 us on such a level before its chunks are
// through, however few they are.  Here a workgroup computes an 8^3 cube of the result from the box
// of cells within S (with the restriction S + 1) of it: the iterate in two LDS buffers, f of the
// thread's cells in registers, a barrier between the sweeps.  Sweep j is exact j cells inside the
// box; the redundant work costs less than the marching kernel's latency.
// Every cell takes the single passes' operations in their order: results are bitwise equal.
// Measured, V(3,3): pre-smoothing with restriction (and norm) 6.2, 7.4 and 19.2 us at 16^3, 32^3 and
// 64^3, post-smoothing with prolongation 7.9, 8.3 and 14.8 us; the marching kernel took 20 and 30,
// 23 and 24 us at 32^3 and 64^3.
#include "mg_kernels.h"

#include <type_traits>

namespace mgk {
namespace {

template <int V>
using IC = std::integral_constant<int, V>;

enum { kRead = 0, kZero = 1, kProlong = 2 };

struct FvCubeArgs {
  const double *u, *f, *ec;
  double *out, *fc, *partial;
  int N;
  double ih2, coef;
};

constexpr int kFvCube = 8;  // cells per side of a workgroup's part of the result

template <int S, int IN, bool RES, bool NORM>
struct FvCube {
  static constexpr int H = S + (RES ? 1 : 0);
  static constexpr int B = kFvCube + 2 * H, N3 = B * B * B;  // box
  static constexpr int R = B - 2, CELLS = R * R * R;         // cells a sweep can update
  static constexpr int THREADS = 512;
  static constexpr int K = (CELLS + THREADS - 1) / THREADS;
  static constexpr int EB = B / 2 + 3;                       // coarse cells around the box per side
  static_assert(H <= 4 && kFvCube * kFvCube * kFvCube == THREADS, "one result cell per thread");

  struct Shared {
    double a[N3], b[N3];
    double e[IN == kProlong ? EB * EB * EB : 1];
    double red[NORM ? THREADS / 64 : 1];
  };

  __device__ __forceinline__ static void run(const FvCubeArgs& g, Shared& sh)
  {
    const int N = g.N, m = N + 2, t = threadIdx.x;
    const int bx = 1 + kFvCube * (int)blockIdx.x - H, by = 1 + kFvCube * (int)blockIdx.y - H,
              bz = 1 + kFvCube * (int)blockIdx.z - H;  // the box's first cell
    auto at = [&](int z, int y, int x) { return ((size_t)z * m + y) * (size_t)m + x; };

    // the thread's cells: LDS offset, f, and which of them and of their neighbours count
    int pos[K];
    double f[K];
    unsigned faces[K];  // bits 0-5: neighbour -x .. +z is a ghost; bit 6: a cell of the domain
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int q = min(t + i * THREADS, CELLS - 1);
      const int lx = 1 + q % R, ly = 1 + (q / R) % R, lz = 1 + q / (R * R);
      const int x = bx + lx, y = by + ly, z = bz + lz;
      const bool in = t + i * THREADS < CELLS && x >= 1 && x <= N && y >= 1 && y <= N && z >= 1 && z <= N;
      pos[i] = (lz * B + ly) * B + lx;
      faces[i] = (x == 1 ? 1u : 0u) | (x == N ? 2u : 0u) | (y == 1 ? 4u : 0u) | (y == N ? 8u : 0u) |
                 (z == 1 ? 16u : 0u) | (z == N ? 32u : 0u) | (in ? 64u : 0u);
      f[i] = in ? g.f[at(z, y, x)] : 0.0;
    }
    const int Nc = N / 2;
    const int ex = (bx >> 1) - 1, ey = (by >> 1) - 1, ez = (bz >> 1) - 1;  // first coarse cell of sh.e
    if constexpr (IN == kProlong) {
      // outside the domain the correction is minus the adjacent cell, per axis
      for (int q = t; q < EB * EB * EB; q += THREADS) {
        int c[3] = {ex + q % EB, ey + (q / EB) % EB, ez + q / (EB * EB)};
        double sign = 1.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          if (c[d] < 1 || c[d] > Nc) sign = -sign;
          c[d] = min(max(c[d], 1), Nc);
        }
        sh.e[q] = sign * g.ec[((size_t)c[2] * (Nc + 2) + c[1]) * (size_t)(Nc + 2) + c[0]];
      }
      __syncthreads();
    }
    for (int q = t; q < N3; q += THREADS) {
      const int x = bx + q % B, y = by + (q / B) % B, z = bz + q / (B * B);
      const bool stored = x >= 0 && x <= N + 1 && y >= 0 && y <= N + 1 && z >= 0 && z <= N + 1;
      double v = IN == kZero || !stored ? 0.0 : g.u[at(z, y, x)];
      if constexpr (IN == kProlong) {
        if (x >= 1 && x <= N && y >= 1 && y <= N && z >= 1 && z <= N) {
          // 8 terms in the order z, y, x, the parent (X = (x + 1) / 2) first, then its neighbour on
          // the cell's side
          const int X = ((x + 1) >> 1) - ex, Y = ((y + 1) >> 1) - ey, Z = ((z + 1) >> 1) - ez;
          const int dx = (x & 1) ? -1 : 1, dy = (y & 1) ? -EB : EB, dz = (z & 1) ? -EB * EB : EB * EB;
          const double* p = sh.e + (Z * EB + Y) * EB + X;
          double s = 0.0;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const double w = (j & 4 ? 0.25 : 0.75) * (j & 2 ? 0.25 : 0.75) * (j & 1 ? 0.25 : 0.75);
            s += w * p[(j & 4 ? dz : 0) + (j & 2 ? dy : 0) + (j & 1 ? dx : 0)];
          }
          v = v + s;
        }
      }
      sh.a[q] = v;
      sh.b[q] = v;  // positions that no sweep updates (ghosts) are read from either buffer
    }
    __syncthreads();

    // (A u) at the thread's cell i; a ghost neighbour enters as 2 g - u_i
    auto apply = [&](const double* s, int i) {
      const int p = pos[i];
      const unsigned fl = faces[i];
      const double c = s[p];
      double v[6] = {s[p - 1], s[p + 1], s[p - B], s[p + B], s[p - B * B], s[p + B * B]};
#pragma unroll
      for (int d = 0; d < 6; ++d)
        if ((fl >> d) & 1u) v[d] = 2.0 * v[d] - c;
      double r = c - v[0];
#pragma unroll
      for (int d = 1; d < 6; ++d) r = r + (c - v[d]);
      return r * g.ih2;
    };
    double sumsq = 0.0;
    double *src = sh.a, *dst = sh.b;
#pragma unroll
    for (int j = 0; j < S; ++j) {
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const double r = f[i] - (IN == kZero && j == 0 ? 0.0 : apply(src, i));
        const double v = src[pos[i]] + g.coef * r;
        if (faces[i] & 64u) dst[pos[i]] = v;
        if (NORM && j == 0) {
          // the cells of this workgroup's cube
          const int q = t + i * THREADS;
          const int lx = 1 + q % R, ly = 1 + (q / R) % R, lz = 1 + q / (R * R);
          const bool mine = (faces[i] & 64u) && lx >= H && lx < H + kFvCube && ly >= H && ly < H + kFvCube &&
                            lz >= H && lz < H + kFvCube;
          if (mine) sumsq += r * r;
        }
      }
      __syncthreads();
      double* x = src;
      src = dst;
      dst = x;
    }
    {
      const int lx = t % kFvCube, ly = (t / kFvCube) % kFvCube, lz = t / (kFvCube * kFvCube);
      g.out[at(bz + H + lz, by + H + ly, bx + H + lx)] = src[((H + lz) * B + H + ly) * B + H + lx];
    }
    if constexpr (RES) {
      // residuals of the cells, then the mean of 8 children
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const double r = f[i] - apply(src, i);
        if (faces[i] & 64u) dst[pos[i]] = r;
      }
      __syncthreads();
      constexpr int C = kFvCube / 2;
      if (t < C * C * C) {
        const int X = t % C, Y = (t / C) % C, Z = t / (C * C);
        const double* r = dst + ((H + 2 * Z) * B + H + 2 * Y) * B + H + 2 * X;
        double s = 0.0;
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
          for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) s += r[(dz * B + dy) * B + dx];
        const size_t mc = (size_t)Nc + 2;
        g.fc[((size_t)(1 + C * blockIdx.z + Z) * mc + 1 + C * blockIdx.y + Y) * mc + 1 + C * blockIdx.x + X] = s / 8.0;
      }
    }
    if constexpr (NORM) {
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) sumsq += __shfl_xor(sumsq, o, 64);
      if ((t & 63) == 0) sh.red[t >> 6] = sumsq;
      __syncthreads();
      if (t == 0) {
        double tot = 0.0;
        for (int w = 0; w < THREADS / 64; ++w) tot += sh.red[w];
        g.partial[(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = tot;
      }
    }
  }
};

template <int S, int IN, bool RES, bool NORM>
__global__ void __launch_bounds__(512) k_fv_cube(FvCubeArgs g)
{
  __shared__ typename FvCube<S, IN, RES, NORM>::Shared sh;
  FvCube<S, IN, RES, NORM>::run(g, sh);
}

}  // namespace

bool fv_cube_supported(int N) { return N >= 16 && N <= 64; }

int fv_cube_sweeps(hipStream_t s, int N, double h, double omega, int sweeps, const double* u,
                   const double* f, const double* ec, double* out, double* fc, double* partial, bool norm)
{
  const int c = N / kFvCube;
  const FvCubeArgs g{u, f, ec, out, fc, partial, N, 1.0 / (h * h), omega * (h * h / 6.0)};
  auto go = [&](auto sc) {
    constexpr int S = decltype(sc)::value;
    const dim3 grid(c, c, c);
    if (ec) k_fv_cube<S, kProlong, false, false><<<grid, 512, 0, s>>>(g);
    else if (!u && fc) k_fv_cube<S, kZero, true, false><<<grid, 512, 0, s>>>(g);
    else if (!u) k_fv_cube<S, kZero, false, false><<<grid, 512, 0, s>>>(g);
    else if (fc && norm) k_fv_cube<S, kRead, true, true><<<grid, 512, 0, s>>>(g);
    else if (fc) k_fv_cube<S, kRead, true, false><<<grid, 512, 0, s>>>(g);
    else k_fv_cube<S, kRead, false, false><<<grid, 512, 0, s>>>(g);
  };
  if (sweeps == 3) go(IC<3>{});
  else go(IC<2>{});
  return c * c * c;
}

}  // namespace mgk
