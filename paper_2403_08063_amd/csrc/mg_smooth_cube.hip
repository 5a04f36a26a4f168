// Red-black Gauss-Seidel on small 3D levels (up to 65^3 nodes) in one launch, on gfx950.
//
// One launch performs S (1 or 2) sweeps, out of place, from u, from a zero guess or from u + P e,
// and, for the pre-smoothing, restricts the residual of the result.  A level of this size is bound
// by launch latency: ten launches of 3-13 us per smoothing step and level, each a fraction of a
// microsecond of work.  (The plane-marching kernel of the large levels is no remedy here: its
// pipeline takes a dozen plane steps of 1.5-2 us before the first plane is final.)
//
// A workgroup computes an 8^3 cube of the result from a box around it: half-sweep j is exact j + 1
// nodes inside the box, so the box reaches H = 2S nodes beyond what has to be final -- the cube
// or, for the restriction onto the cube's 4^3 coarse nodes, one node (two above) more.  The box of
// u (and of k) is staged in LDS once; every thread owns up to K nodes of each colour, their f in
// registers, through all half-sweeps, with a barrier between them.  The redundant work (a 19^3 box
// per 8^3 cube) is cheap next to a launch: at 65^3 the 512 cubes run in one round.
// Operations and their order are those of the per-colour kernels (bitwise equal).
// Measured, FP64 V(2,2): at 65^3 the pre-smoothing with the restriction 20 us (27 in five
// launches, and ten launch gaps a step more), the post-smoothing 13.5 us (27); at 33^3 10 and 8.3
// us (18, 17).  Forcing two workgroups per compute unit on the restriction (64 VGPRs) spills: 28 us.
#include "mg_kernels.h"
#include "mg_stencil.h"

#include <type_traits>

namespace mgk {
namespace {

template <int V>
using IC = std::integral_constant<int, V>;

enum { kInRead = 0, kInZero = 1, kInProlong = 2 };

template <typename T>
struct CubeArgs {
  const T *u, *f, *k, *ec;
  T *out, *fc;
  int n, tiles;
  T h2, ih2;
};

constexpr int kCube = 8;  // nodes per side of a workgroup's part of the result

template <typename T, bool VAR, int S, int IN, bool RES>
struct Cube {
  static constexpr int H = 2 * S;
  static constexpr int LO = H + (RES ? 1 : 0);              // box index of the cube's first node
  static constexpr int B = LO + kCube + H + (RES ? 2 : 0);  // box nodes per side
  static constexpr int N3 = B * B * B;
  static constexpr int R = B - 2, HX = (R + 1) / 2;         // nodes that can be updated; per row and colour
  static constexpr int COUNT = HX * R * R;
  static constexpr int THREADS = 1024;
  static constexpr int K = (COUNT + THREADS - 1) / THREADS;
  static constexpr int RB = kCube + 1;                      // residual nodes per side (RES)
  static constexpr int EB = (B + 1) / 2 + 1;                // coarse nodes around the box per side
  static_assert(RB * RB * RB <= THREADS && EB * EB * EB <= 2 * THREADS, "one or two per thread");

  struct Shared {
    T u[N3];
    T k[VAR ? N3 : 1];
    T r[RES ? RB * RB * RB : 1];
    T e[IN == kInProlong ? EB * EB * EB : 1];
  };

  __device__ __forceinline__ static void run(const CubeArgs<T>& a, Shared& sh)
  {
    const int n = a.n, t = threadIdx.x;
    const int ox = 1 + kCube * (int)blockIdx.x, oy = 1 + kCube * (int)blockIdx.y, oz = 1 + kCube * (int)blockIdx.z;
    const int bx = ox - LO, by = oy - LO, bz = oz - LO;  // the box's first node
    auto node = [&](int z, int y, int x) { return ((size_t)z * n + y) * (size_t)n + x; };
    auto inside = [&](int z, int y, int x) {
      return x >= 1 && x <= n - 2 && y >= 1 && y <= n - 2 && z >= 1 && z <= n - 2;
    };

    // the thread's nodes: LDS offset (-1: none) and f; box coordinates are recovered from the offset
    int at[2][K];
    T h2f[2][K];
    const int par = bx + by + bz;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int q = t + i * THREADS;
        const int row = q / HX, z = 1 + row / R, y = 1 + row % R;
        const int x = 1 + ((1 + par + y + z + c) & 1) + 2 * (q % HX);
        const bool in = q < COUNT && x <= R && inside(bz + z, by + y, bx + x);
        at[c][i] = in ? (z * B + y) * B + x : -1;
        h2f[c][i] = in ? a.h2 * a.f[node(bz + z, by + y, bx + x)] : T(0);
      }
    T fr = T(0);  // RES: f of the thread's residual node
    if constexpr (RES) {
      if (t < RB * RB * RB) {
        const int x = ox + t % RB, y = oy + (t / RB) % RB, z = oz + t / (RB * RB);
        if (inside(z, y, x)) fr = a.f[node(z, y, x)];
      }
    }
    const int ex = bx >> 1, ey = by >> 1, ez = bz >> 1;  // first coarse node of sh.e
    if constexpr (IN == kInProlong) {
      const int nc = (n - 1) / 2 + 1;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int q = t + i * THREADS;
        if (q < EB * EB * EB) {
          const int X = ex + q % EB, Y = ey + (q / EB) % EB, Z = ez + q / (EB * EB);
          const bool in = X >= 0 && X < nc && Y >= 0 && Y < nc && Z >= 0 && Z < nc;
          sh.e[q] = in ? a.ec[((size_t)Z * nc + Y) * (size_t)nc + X] : T(0);
        }
      }
      __syncthreads();
    }
    // P e at an interior node, in the terms and order of corrected_at
    auto correction = [&](int z, int y, int x) -> T {
      const T wt = ((z & 1) ? T(0.5) : T(1)) * ((y & 1) ? T(0.5) : T(1)) * ((x & 1) ? T(0.5) : T(1));
      const int sx = x & 1, sy = (y & 1) ? EB : 0, sz = (z & 1) ? EB * EB : 0;
      const T* e = sh.e + (((z >> 1) - ez) * EB + ((y >> 1) - ey)) * EB + (((x + 1) >> 1) - ex);
      T s = T(0);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const bool in = (c == 0 || (z & 1)) && (b == 0 || (y & 1));
          const T* q = e + (c ? sz : 0) + (b ? sy : 0);
          const T e0 = q[-sx], e1 = q[0];
          if (in && sx) s = s + wt * e0;
          if (in) s = s + wt * e1;
        }
      return s;
    };
    for (int q = t; q < N3; q += THREADS) {
      const int x = bx + q % B, y = by + (q / B) % B, z = bz + q / (B * B);
      const bool in = x >= 0 && x < n && y >= 0 && y < n && z >= 0 && z < n;
      T v = IN == kInZero || !in ? T(0) : a.u[node(z, y, x)];
      // colour 1 only: the first half-sweep overwrites colour 0 without reading its old value
      if (IN == kInProlong && ((x + y + z) & 1) && inside(z, y, x)) v = v + correction(z, y, x);
      sh.u[q] = v;
      if constexpr (VAR) sh.k[q] = in ? a.k[node(z, y, x)] : T(1);
    }
    __syncthreads();

#pragma unroll
    for (int j = 0; j < H; ++j) {
      const int c = j & 1;
      T v[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int p = max(at[c][i], (B + 1) * B + 1);
        const T xm = sh.u[p - 1], xp = sh.u[p + 1], ym = sh.u[p - B], yp = sh.u[p + B];
        const T zm = sh.u[p - B * B], zp = sh.u[p + B * B];
        if constexpr (!VAR) {
          v[i] = gs_const<T, 3>(h2f[c][i], xm, xp, ym, yp, zm, zp);
        } else {
          v[i] = gs_var<T, 3>(h2f[c][i], sh.k[p], xm, sh.k[p - 1], xp, sh.k[p + 1], ym, sh.k[p - B], yp,
                              sh.k[p + B], zm, sh.k[p - B * B], zp, sh.k[p + B * B]);
        }
      }
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (at[c][i] >= 0) sh.u[at[c][i]] = v[i];
      __syncthreads();
    }

    if constexpr (RES) {
      if (t < RB * RB * RB) {
        const int lx = t % RB, ly = (t / RB) % RB, lz = t / (RB * RB);
        const int p = ((LO + lz) * B + LO + ly) * B + LO + lx;
        const T xm = sh.u[p - 1], xp = sh.u[p + 1], ym = sh.u[p - B], yp = sh.u[p + B];
        const T zm = sh.u[p - B * B], zp = sh.u[p + B * B];
        T au;
        if constexpr (!VAR) {
          au = au_const<T, 3>(a.ih2, sh.u[p], xm, xp, ym, yp, zm, zp);
        } else {
          au = au_var<T, 3>(a.ih2, sh.u[p], sh.k[p], xm, sh.k[p - 1], xp, sh.k[p + 1], ym, sh.k[p - B], yp,
                            sh.k[p + B], zm, sh.k[p - B * B], zp, sh.k[p + B * B]);
        }
        sh.r[t] = fr - au;
      }
    }
    // the cube of the result
    if (t < kCube * kCube * kCube) {
      const int lx = t % kCube, ly = (t / kCube) % kCube, lz = t / (kCube * kCube);
      if (inside(oz + lz, oy + ly, ox + lx))
        a.out[node(oz + lz, oy + ly, ox + lx)] = sh.u[((LO + lz) * B + LO + ly) * B + LO + lx];
    }
    if constexpr (RES) {
      __syncthreads();
      constexpr int C = kCube / 2;
      if (t < C * C * C) {
        // coarse node (X, Y, Z) lies at the cube's odd offsets: fine node ox + 1 + 2 i
        const int i = t % C, j = (t / C) % C, l = t / (C * C);
        const int nc = (n - 1) / 2 + 1;
        const int X = (ox + 1) / 2 + i, Y = (oy + 1) / 2 + j, Z = (oz + 1) / 2 + l;
        if (X <= nc - 2 && Y <= nc - 2 && Z <= nc - 2) {
          constexpr T w[3] = {T(0.25), T(0.5), T(0.25)};
          T s = T(0);
#pragma unroll
          for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
              for (int dx = 0; dx < 3; ++dx)
                s = s + (w[dx] * w[dy] * w[dz]) * sh.r[((2 * l + dz) * RB + 2 * j + dy) * RB + 2 * i + dx];
          a.fc[((size_t)Z * nc + Y) * (size_t)nc + X] = s;
        }
      }
    }
  }
};

template <typename T, bool VAR, int S, int IN, bool RES>
__global__ void __launch_bounds__(1024) k_rbgs_cube(CubeArgs<T> a)
{
  __shared__ typename Cube<T, VAR, S, IN, RES>::Shared sh;
  Cube<T, VAR, S, IN, RES>::run(a, sh);
}

}  // namespace

bool rbgs_cube_supported(int dim, int n) { return dim == 3 && n <= 65; }

template <typename T>
void rbgs_cube(hipStream_t s, int n, double h, const T* k, const T* f, const T* u, T* out, int sweeps,
               bool zero, const T* ec, T* fc)
{
  const int tiles = (n - 2 + kCube - 1) / kCube;
  const CubeArgs<T> a{u, f, k, ec, out, fc, n, tiles, (T)(h * h), (T)(1.0 / (h * h))};
  auto go = [&](auto vc, auto sc, auto ic, auto rc) {
    k_rbgs_cube<T, decltype(vc)::value, decltype(sc)::value, decltype(ic)::value, decltype(rc)::value>
        <<<dim3(tiles, tiles, tiles), 1024, 0, s>>>(a);
  };
  auto in = [&](auto vc, auto sc) {
    if (ec) go(vc, sc, IC<kInProlong>{}, std::false_type{});
    else if (zero && fc) go(vc, sc, IC<kInZero>{}, std::true_type{});
    else if (zero) go(vc, sc, IC<kInZero>{}, std::false_type{});
    else if (fc) go(vc, sc, IC<kInRead>{}, std::true_type{});
    else go(vc, sc, IC<kInRead>{}, std::false_type{});
  };
  if (k && sweeps == 2) in(std::true_type{}, IC<2>{});
  else if (k) in(std::true_type{}, IC<1>{});
  else if (sweeps == 2) in(std::false_type{}, IC<2>{});
  else in(std::false_type{}, IC<1>{});
}

template void rbgs_cube<double>(hipStream_t, int, double, const double*, const double*, const double*, double*,
                                int, bool, const double*, double*);
template void rbgs_cube<float>(hipStream_t, int, double, const float*, const float*, const float*, float*, int,
                               bool, const float*, float*);

}  // namespace mgk
