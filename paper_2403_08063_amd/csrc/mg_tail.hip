// Coarse tail of the V-cycle in one launch.
//
// Below a few ten thousand interior nodes per level a kernel launch costs more than the
// work it carries (the V-cycle's coarse levels are launch-latency bound, the GPU analogue
// of the coarse-grid overhead the paper measures in Sect. 6).  One workgroup of 1024
// threads therefore runs the complete V(nu1, nu2)-cycle on all levels from `first` down to
// the coarsest, with workgroup barriers between the dependent phases: zero guess,
// red-black half-sweeps, residual + full-weighting restriction, the coarsest solve,
// prolongation + correction, post-smoothing.  Every phase evaluates the same point
// formulas in the same order as the multi-kernel path (mg_stencil.h), so the result is
// bitwise identical to launching the per-level kernels.
#include "mg_kernels.h"
#include "mg_stencil.h"

namespace mgk {
namespace {

constexpr int kTailThreads = 1024;

// Work items of a phase: an nx x ny (x nz) box, enumerated over power-of-two padded x and
// y extents so that a thread index splits into coordinates by shifts and masks (an integer
// division costs tens of instructions, more than a tail phase's arithmetic).
__device__ __forceinline__ int ceil_log2(int v) { return v <= 1 ? 0 : 32 - __clz(v - 1); }

template <typename F>
__device__ __forceinline__ void for_box(int nx, int ny, int nz, F&& body)
{
  const int lx = ceil_log2(nx), ly = ceil_log2(ny);
  const int total = (1 << (lx + ly)) * nz;
  for (int t = threadIdx.x; t < total; t += blockDim.x) {
    const int x = t & ((1 << lx) - 1), y = (t >> lx) & ((1 << ly) - 1), z = t >> (lx + ly);
    if (x < nx && y < ny) body(x, y, z);
  }
}

template <typename T, int DIM, bool VAR>
__device__ void tail_half_sweep(const TailLevel<T>& L, int colour)
{
  const int n = L.n;
  const int half = (n - 1) / 2;  // nodes of one colour in a row, rounded up
  const size_t sy = (size_t)n, sz = (size_t)n * n;
  for_box(half, n - 2, DIM == 3 ? n - 2 : 1, [&](int q, int yy, int zz) {
    const int y = 1 + yy;
    const int z = DIM == 3 ? 1 + zz : 0;
    const int x = 1 + ((1 + y + z + colour) & 1) + 2 * q;
    if (x > n - 2) return;
    const size_t i = ((size_t)z * n + y) * (size_t)n + x;
    L.u[i] = gs_at<T, DIM, VAR>(L.f, L.u, L.k, i, sy, sz, L.h2);
  });
  __syncthreads();
}

template <typename T, int DIM, bool VAR>
__global__ void __launch_bounds__(kTailThreads) k_tail(TailArgs<T> a)
{
  __shared__ double b[1024];
  const int last = a.nlev - 1;
  for (int l = 0; l < last; ++l) {
    const TailLevel<T>& L = a.lv[l];
    const size_t N = DIM == 3 ? (size_t)L.n * L.n * L.n : (size_t)L.n * L.n;
    for (size_t i = threadIdx.x; i < N; i += blockDim.x) L.u[i] = T(0);
    __syncthreads();
    for (int s = 0; s < a.nu1; ++s) {
      tail_half_sweep<T, DIM, VAR>(L, 0);
      tail_half_sweep<T, DIM, VAR>(L, 1);
    }
    const TailLevel<T>& C = a.lv[l + 1];
    const int nc = C.n, mc = nc - 2;
    const int cnt = DIM == 3 ? mc * mc * mc : mc * mc;
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      const int X = 1 + t % mc;
      const int Y = 1 + (t / mc) % mc;
      const int Z = DIM == 3 ? 1 + t / (mc * mc) : 0;
      C.f[((size_t)Z * nc + Y) * (size_t)nc + X] =
          restrict_at<T, DIM, VAR>(L.f, L.u, L.k, L.n, L.ih2, X, Y, Z);
    }
    __syncthreads();
  }
  coarsest_apply<T>(DIM, a.lv[last].n, a.ainv, a.lv[last].f, a.lv[last].u, b);
  for (int l = last - 1; l >= 0; --l) {
    const TailLevel<T>& L = a.lv[l];
    const TailLevel<T>& C = a.lv[l + 1];
    const int nc = C.n, mf = L.n - 2;
    const int rows = DIM == 3 ? mf * mf : mf;
    const int pairs = nc - 1;
    for (int t = threadIdx.x; t < rows * pairs; t += blockDim.x) {
      const int r = t / pairs, c = 1 + (t - r * pairs);
      const int y = 1 + r % mf;
      const int z = DIM == 3 ? 1 + r / mf : 0;
      prolong_pair<T, DIM>(C.u, L.u, nc, c, y, z);
    }
    __syncthreads();
    for (int s = 0; s < a.nu2; ++s) {
      tail_half_sweep<T, DIM, VAR>(L, 0);
      tail_half_sweep<T, DIM, VAR>(L, 1);
    }
  }
}

// The same cycle with the levels in LDS (dynamic): per level u, k (variable coefficient), the
// residual r and, below the first level, f.
//
// The phases form a serial chain of some 40 half-sweeps and transfers over at most 4096 nodes, so
// their latency is what counts: LDS reads, a barrier and, in the version before this one, mostly
// index arithmetic (64-bit, repeated in every phase) and 27 residuals per coarse node.  Here a
// thread keeps the nodes it owns on a level (K of each colour), their LDS offsets, h^2 f and the
// face coefficients in registers through the sweeps; the residual is formed once per node; only
// the colour that the first post-smoothing half-sweep reads takes the coarse correction; and the
// levels of at most 64 kWaveK nodes per colour run in the first wave alone, where the order of
// LDS accesses replaces the barriers.  Operations and their order are those of the per-level
// kernels.  Measured per cycle: 17^3 to 3^3 21.6 us (FP64, constant coefficient; 30.2 before),
// 38.4 us with a variable coefficient (51.4), 65^2 to 3^2 24.2 us (31.6).
constexpr int kBlockK = 2;  // nodes of a colour per thread on the levels of the whole workgroup
constexpr int kWaveK = 3;   // and, at most, on the levels of one wave
static_assert(2 * kBlockK * kTailThreads >= kTailMaxNodes, "a thread's share of the first level");

template <typename T>
struct LdsLevel {
  T *u, *k, *r, *f;
  int n;
};

template <typename T, int DIM, bool VAR>
__device__ __forceinline__ LdsLevel<T> lds_level(unsigned char* base, const TailArgs<T>& a, int l)
{
  int off = 0;
  for (int q = 0; q < l; ++q) {
    const int n = a.lv[q].n, N = DIM == 3 ? n * n * n : n * n;
    off += N * (2 + (VAR ? 1 : 0) + (q ? 1 : 0));
  }
  const int n = a.lv[l].n, N = DIM == 3 ? n * n * n : n * n;
  T* p = reinterpret_cast<T*>(base) + off;
  LdsLevel<T> L;
  L.u = p;
  L.r = p + N;
  L.k = VAR ? p + 2 * N : nullptr;
  L.f = l ? p + (VAR ? 3 : 2) * N : nullptr;
  L.n = n;
  return L;
}

// The steps of a level by the workgroup (WAVE = false) or the first wave, K nodes of each colour
// per thread.
template <typename T, int DIM, bool VAR, bool WAVE, int K>
struct TailRun {
  static constexpr int THREADS = WAVE ? 64 : kTailThreads;
  // coefficients in registers; those of more than two FP64 nodes would exceed them: from LDS
  static constexpr bool KREG = VAR && (K == 1 || sizeof(T) == 4);

  __device__ __forceinline__ static void sync()
  {
    if constexpr (WAVE) {
      // one wave's LDS accesses execute in program order; keep the compiler to it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
    }
  }

  // The nodes of colour c that this thread owns: LDS offsets (-1: none).
  __device__ __forceinline__ static void own(const TailLevel<T>& G, int c, int (&at)[K])
  {
    const int n = G.n, half = (n - 1) / 2, m = n - 2;
    const int count = half * m * (DIM == 3 ? m : 1);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int q = (int)threadIdx.x + i * THREADS;
      const int row = (int)__umulhi((unsigned)q, G.div_half), t = q - row * half;
      const int zz = DIM == 3 ? (int)__umulhi((unsigned)row, G.div_m) : 0;
      const int y = 1 + row - zz * m, z = DIM == 3 ? 1 + zz : 0;
      const int x = 1 + ((1 + y + z + c) & 1) + 2 * t;
      at[i] = q < count && x <= n - 2 ? (z * n + y) * n + x : -1;
    }
  }

  // the node, or an interior node in place of none
  __device__ __forceinline__ static int at_or_any(const LdsLevel<T>& L, int p)
  {
    return max(p, (DIM == 3 ? L.n * L.n : 0) + L.n + 1);
  }

  struct Nodes {
    int at[2][K];
    T h2f[2][K], f[2][K];
    T c[KREG ? 2 : 1][KREG ? K : 1][2 * DIM], ck[KREG ? 2 : 1][KREG ? K : 1];
  };

  // k at a node and its neighbours
  __device__ __forceinline__ static void faces(const LdsLevel<T>& L, int p, T& kp, T (&k)[2 * DIM])
  {
    const int sy = L.n, sz = L.n * L.n;
    const int off[6] = {-1, 1, -sy, sy, -sz, sz};
    kp = L.k[p];
#pragma unroll
    for (int d = 0; d < 2 * DIM; ++d) k[d] = L.k[p + off[d]];
  }

  // per node: offsets, f and, with a variable coefficient, k around it
  __device__ __forceinline__ static void setup(const TailLevel<T>& G, const LdsLevel<T>& L, const T* f, Nodes& N)
  {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      own(G, c, N.at[c]);
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int p = at_or_any(L, N.at[c][i]);
        N.f[c][i] = f[p];
        N.h2f[c][i] = G.h2 * N.f[c][i];
        if constexpr (KREG) faces(L, p, N.ck[c][i], N.c[c][i]);
      }
    }
  }

  __device__ __forceinline__ static void node_k(const LdsLevel<T>& L, const Nodes& N, int c, int i, T& kp, T (&k)[2 * DIM])
  {
    if constexpr (KREG) {
      kp = N.ck[c][i];
#pragma unroll
      for (int d = 0; d < 2 * DIM; ++d) k[d] = N.c[c][i][d];
    } else {
      faces(L, at_or_any(L, N.at[c][i]), kp, k);
    }
  }

  // All of a thread's loads come before its stores (a store between them would make the compiler
  // wait out one node's LDS latency after another's); a node that is not there reads node `p0`.
  __device__ __forceinline__ static void half_sweep(const TailLevel<T>& G, const LdsLevel<T>& L, const Nodes& N, int c)
  {
    const int sy = L.n, sz = L.n * L.n;
    T v[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int p = at_or_any(L, N.at[c][i]);
      const T xm = L.u[p - 1], xp = L.u[p + 1], ym = L.u[p - sy], yp = L.u[p + sy];
      const T zm = DIM == 3 ? L.u[p - sz] : T(0), zp = DIM == 3 ? L.u[p + sz] : T(0);
      if constexpr (!VAR) {
        v[i] = gs_const<T, DIM>(N.h2f[c][i], xm, xp, ym, yp, zm, zp);
      } else {
        T k[2 * DIM], kp;
        node_k(L, N, c, i, kp, k);
        v[i] = gs_var<T, DIM>(N.h2f[c][i], kp, xm, k[0], xp, k[1], ym, k[2], yp, k[3], zm,
                              DIM == 3 ? k[2 * DIM - 2] : T(0), zp, DIM == 3 ? k[2 * DIM - 1] : T(0));
      }
    }
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (N.at[c][i] >= 0) L.u[N.at[c][i]] = v[i];
    sync();
  }

  __device__ __forceinline__ static void residuals(const TailLevel<T>& G, const LdsLevel<T>& L, const Nodes& N)
  {
    const int sy = L.n, sz = L.n * L.n;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T v[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int p = at_or_any(L, N.at[c][i]);
        const T ui = L.u[p];
        const T xm = L.u[p - 1], xp = L.u[p + 1], ym = L.u[p - sy], yp = L.u[p + sy];
        const T zm = DIM == 3 ? L.u[p - sz] : T(0), zp = DIM == 3 ? L.u[p + sz] : T(0);
        T au;
        if constexpr (!VAR) {
          au = au_const<T, DIM>(G.ih2, ui, xm, xp, ym, yp, zm, zp);
        } else {
          T k[2 * DIM], kp;
          node_k(L, N, c, i, kp, k);
          au = au_var<T, DIM>(G.ih2, ui, kp, xm, k[0], xp, k[1], ym, k[2], yp, k[3], zm,
                              DIM == 3 ? k[2 * DIM - 2] : T(0), zp, DIM == 3 ? k[2 * DIM - 1] : T(0));
        }
        v[i] = N.f[c][i] - au;
      }
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (N.at[c][i] >= 0) L.r[N.at[c][i]] = v[i];
    }
    sync();
  }

  // coarse f = full weighting of r (restrict_at's order); up to 2 K coarse nodes per thread
  __device__ __forceinline__ static void restrict_to(const TailLevel<T>& Gc, const LdsLevel<T>& L, const LdsLevel<T>& C)
  {
    const int nc = C.n, mc = nc - 2, nf = L.n;
    const int count = mc * mc * (DIM == 3 ? mc : 1);
    for (int q = threadIdx.x; q < count; q += THREADS) {
      const int row = mc == 1 ? q : (int)__umulhi((unsigned)q, Gc.div_m);
      const int zz = DIM == 3 ? (mc == 1 ? row : (int)__umulhi((unsigned)row, Gc.div_m)) : 0;
      const int X = 1 + q - row * mc, Y = 1 + row - zz * mc, Z = DIM == 3 ? 1 + zz : 0;
      const T* r = L.r + ((DIM == 3 ? 2 * Z * nf : 0) + 2 * Y) * nf + 2 * X;
      constexpr T w[3] = {T(0.25), T(0.5), T(0.25)};
      T s = T(0);
#pragma unroll
      for (int oz = (DIM == 3 ? -1 : 0); oz <= (DIM == 3 ? 1 : 0); ++oz)
#pragma unroll
        for (int oy = -1; oy <= 1; ++oy)
#pragma unroll
          for (int ox = -1; ox <= 1; ++ox)
            s = s + (w[ox + 1] * w[oy + 1] * (DIM == 3 ? w[oz + 1] : T(1))) * r[(oz * nf + oy) * nf + ox];
      C.f[(Z * nc + Y) * nc + X] = s;
    }
    sync();
  }

  // u += P e on colour 1 (on both colours if no half-sweep overwrites colour 0 unread), with
  // corrected_at's terms and order
  __device__ __forceinline__ static void correct(const TailLevel<T>& G, const LdsLevel<T>& L, const LdsLevel<T>& C,
                                                 const Nodes& N, bool both)
  {
    const int n = L.n, nc = C.n;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (c == 0 && !both) continue;
      T v[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int p = at_or_any(L, N.at[c][i]);
        const int row = (int)__umulhi((unsigned)p, G.div_n), x = p - row * n;
        const int z = DIM == 3 ? (int)__umulhi((unsigned)row, G.div_n) : 0, y = row - z * n;
        // an even index takes one coarse value with weight 1, an odd one two with weight 1/2: the
        // terms that are not there are read (from the node's own coarse cell) and left out
        const T wz = DIM == 3 ? ((z & 1) ? T(0.5) : T(1)) : T(1), wy = (y & 1) ? T(0.5) : T(1);
        const T wx = (x & 1) ? T(0.5) : T(1), wt = wz * wy * wx;
        const int oz = DIM == 3 && (z & 1) ? nc * nc : 0, oy = (y & 1) ? nc : 0, ox = (x & 1) ? 1 : 0;
        const T* e = C.u + ((DIM == 3 ? z >> 1 : 0) * nc + (y >> 1)) * nc + ((x + 1) >> 1);
        T s = T(0);
#pragma unroll
        for (int a = 0; a < (DIM == 3 ? 2 : 1); ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const bool in = (a == 0 || (z & 1)) && (b == 0 || (y & 1));
            const T* q = e + (a ? oz : 0) + (b ? oy : 0);
            const T e0 = q[-ox], e1 = q[0];
            if (in && (x & 1)) s = s + wt * e0;
            if (in) s = s + wt * e1;
          }
        v[i] = L.u[p] + s;
      }
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (N.at[c][i] >= 0) L.u[N.at[c][i]] = v[i];
    }
    sync();
  }

  // pre-smoothing from zero, residual and restriction on level l
  __device__ __forceinline__ static void down(unsigned char* base, const TailArgs<T>& a, int l)
  {
    const LdsLevel<T> L = lds_level<T, DIM, VAR>(base, a, l), C = lds_level<T, DIM, VAR>(base, a, l + 1);
    const TailLevel<T>& G = a.lv[l];
    Nodes N;
    setup(G, L, l ? L.f : G.f, N);
    for (int s = 0; s < a.nu1; ++s) {
      half_sweep(G, L, N, 0);
      half_sweep(G, L, N, 1);
    }
    residuals(G, L, N);
    restrict_to(a.lv[l + 1], L, C);
  }

  // correction and post-smoothing on level l
  __device__ __forceinline__ static void up(unsigned char* base, const TailArgs<T>& a, int l)
  {
    const LdsLevel<T> L = lds_level<T, DIM, VAR>(base, a, l), C = lds_level<T, DIM, VAR>(base, a, l + 1);
    const TailLevel<T>& G = a.lv[l];
    Nodes N;
    setup(G, L, l ? L.f : G.f, N);
    correct(G, L, C, N, a.nu2 == 0);
    for (int s = 0; s < a.nu2; ++s) {
      half_sweep(G, L, N, 0);
      half_sweep(G, L, N, 1);
    }
  }

  // the coarsest solve, a row of the inverse per thread (coarsest_apply's order)
  __device__ __forceinline__ static void coarsest(const LdsLevel<T>& L, const TailArgs<T>& a, double* b)
  {
    const int n = L.n, m1 = n - 2;
    const int m = DIM == 3 ? m1 * m1 * m1 : m1 * m1;
    for (int q = threadIdx.x; q < m; q += THREADS) {
      int z, y, x;
      unknown_to_node(DIM, n, q, z, y, x);
      b[q] = (double)L.f[(z * n + y) * n + x];
    }
    sync();
    for (int q = threadIdx.x; q < m; q += THREADS) {
      double s = 0.0;
      for (int c = 0; c < m; ++c) s += a.ainv[(size_t)c * m + q] * b[c];
      int z, y, x;
      unknown_to_node(DIM, n, q, z, y, x);
      L.u[(z * n + y) * n + x] = (T)s;
    }
    sync();
  }
};

template <typename T, int DIM, bool VAR>
__global__ void __launch_bounds__(kTailThreads) k_tail_lds(TailArgs<T> a)
{
  extern __shared__ __align__(16) unsigned char tail_lds[];
  __shared__ double b[1024];
  // zero guesses (boundaries included) and coefficients of every level
  for (int l = 0; l < a.nlev; ++l) {
    const LdsLevel<T> L = lds_level<T, DIM, VAR>(tail_lds, a, l);
    const int N = DIM == 3 ? L.n * L.n * L.n : L.n * L.n;
    for (int i = threadIdx.x; i < N; i += kTailThreads) {
      L.u[i] = T(0);
      if constexpr (VAR) L.k[i] = a.lv[l].k[i];
    }
  }
  __syncthreads();
  using Block = TailRun<T, DIM, VAR, false, kBlockK>;
  using Wave = TailRun<T, DIM, VAR, true, kWaveK>;
  using Small = TailRun<T, DIM, VAR, true, 1>;
  const int last = a.nlev - 1;
  // first level of the first wave, and of one node of a colour per lane (the coarsest at the latest)
  auto nodes = [&](int l) { return (a.lv[l].n - 1) / 2 * (a.lv[l].n - 2) * (DIM == 3 ? a.lv[l].n - 2 : 1); };
  int lw = 0, l1 = 0;
  while (lw < last && nodes(lw) > 64 * kWaveK) ++lw;
  for (l1 = lw; l1 < last && nodes(l1) > 64;) ++l1;
  // A coarsest level of up to 64 unknowns is solved by the first wave, a larger one (up to 1024) by
  // the workgroup: a wave would take m / 64 chains of m loads one after the other (V(2,2) at 113^3,
  // 216 unknowns: 173 us with the wave, 125 so; at 121^2 on three levels, 841: 985 and 107).
  const int mc = a.lv[last].n - 2;
  const bool wide = mc * mc * (DIM == 3 ? mc : 1) > 64;
  for (int l = 0; l < lw; ++l) Block::down(tail_lds, a, l);
  LdsLevel<T> Lc = lds_level<T, DIM, VAR>(tail_lds, a, last);
  if (last == 0) Lc.f = a.lv[0].f;
  if (threadIdx.x < 64) {
    for (int l = lw; l < l1; ++l) Wave::down(tail_lds, a, l);
    for (int l = l1; l < last; ++l) Small::down(tail_lds, a, l);
    if (!wide) Wave::coarsest(Lc, a, b);
  }
  if (wide) {
    __syncthreads();
    Block::coarsest(Lc, a, b);
  }
  if (threadIdx.x < 64) {
    for (int l = last - 1; l >= l1; --l) Small::up(tail_lds, a, l);
    for (int l = l1 - 1; l >= lw; --l) Wave::up(tail_lds, a, l);
  }
  __syncthreads();
  for (int l = lw - 1; l >= 0; --l) Block::up(tail_lds, a, l);
  const LdsLevel<T> L0 = lds_level<T, DIM, VAR>(tail_lds, a, 0);
  const int N0 = DIM == 3 ? L0.n * L0.n * L0.n : L0.n * L0.n;
  for (int i = threadIdx.x; i < N0; i += kTailThreads) a.lv[0].u[i] = L0.u[i];
}

// LDS of the levels, bytes
template <typename T>
size_t tail_lds_bytes(int dim, const TailArgs<T>& a)
{
  const bool var = a.lv[0].k != nullptr;
  size_t vals = 0;
  for (int q = 0; q < a.nlev; ++q) {
    const size_t n = (size_t)a.lv[q].n;
    vals += (dim == 3 ? n * n * n : n * n) * (2 + (var ? 1 : 0) + (q ? 1 : 0));
  }
  return vals * sizeof(T);
}

// dynamic LDS the tail may take next to its static 8 KB (gfx950: 160 KB per CU)
constexpr size_t kTailLdsMax = 152 * 1024;

template <typename Kernel>
bool allow_lds(Kernel kern, size_t bytes)
{
  if (bytes > kTailLdsMax) return false;
  static int granted[64] = {0};  // per device: 1 granted, -1 refused
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  if (granted[dev] == 0)
    granted[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kTailLdsMax) == hipSuccess ? 1 : -1;
  return granted[dev] == 1;
}

template <typename T, int DIM, bool VAR>
void launch_tail(hipStream_t s, const TailArgs<T>& a)
{
  const size_t bytes = tail_lds_bytes<T>(DIM, a);
  auto kl = k_tail_lds<T, DIM, VAR>;
  if (allow_lds(kl, bytes)) kl<<<1, kTailThreads, bytes, s>>>(a);
  else k_tail<T, DIM, VAR><<<1, kTailThreads, 0, s>>>(a);
}

}  // namespace

bool tail_fits(int dim, int n)
{
  const long long m = n - 2;
  return (dim == 3 ? m * m * m : m * m) <= kTailMaxNodes;
}

template <typename T>
void tail_cycle(hipStream_t s, int dim, TailArgs<T> a)
{
  // q / d = umulhi(q, ceil(2^32 / d)) for the indices here (q d < 2^32; d > 1)
  auto reciprocal = [](int d) { return d > 1 ? (unsigned)((0x100000000ull + d - 1) / d) : 0u; };
  for (int q = 0; q < a.nlev; ++q) {
    a.lv[q].div_half = reciprocal((a.lv[q].n - 1) / 2);
    a.lv[q].div_m = reciprocal(a.lv[q].n - 2);
    a.lv[q].div_n = reciprocal(a.lv[q].n);
  }
  const bool var = a.lv[0].k != nullptr;
  if (dim == 3) {
    if (var) launch_tail<T, 3, true>(s, a);
    else launch_tail<T, 3, false>(s, a);
  } else {
    if (var) launch_tail<T, 2, true>(s, a);
    else launch_tail<T, 2, false>(s, a);
  }
}

template void tail_cycle<double>(hipStream_t, int, TailArgs<double>);
template void tail_cycle<float>(hipStream_t, int, TailArgs<float>);

}  // namespace mgk
