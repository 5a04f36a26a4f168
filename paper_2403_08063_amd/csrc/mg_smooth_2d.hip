// Temporally blocked red-black Gauss-Seidel for 2D levels on gfx950.
//
// One launch performs S (1 or 2) red-black sweeps, out of place, with what stands before and
// after them in the V-cycle taken in: IN = kInRead, kInZero (a zero guess, not read) or
// kInProlong (u + P e); OUT = 0, kOutRestrict (the residual of the result and its full
// weighting, as the pre-smoothing needs it) or kOutNorm (the squared norm of that residual, as
// the stopping test needs it).  The per-colour kernels read and write the level once per
// half-sweep -- ten passes or, on a small level, ten launches of 3-5 us per smoothing step.
//
// Decomposition: a wave owns a strip of 128 columns (two per lane) of a chunk of rows and
// marches along y, alone: x-neighbours come from the adjacent lanes by DPP, y-neighbours are a
// queue of rows in registers, so there is no LDS and no barrier.  The 2S half-sweeps run as a
// wavefront in y: half-sweep j updates row yl - 1 - j when row yl enters.  In every row one of a
// lane's two columns has the colour of the half-sweep, the same for all half-sweeps of a step.
// Half-sweep j is exact j + 1 columns inside the strip (and rows inside the chunk): strips
// overlap by 2 H columns, H = 2S, and by 4 more where residuals are formed.  Rows are loaded
// kPre steps ahead.  Strip origins and chunk starts are odd, so parities are compile-time.
//
// Every node takes the per-colour kernels' operations in their order (mg_stencil.h): bitwise
// equal results.
#include "mg_buffer.h"
#include "mg_kernels.h"
#include "mg_lanes.h"
#include "mg_stencil.h"

#include <type_traits>
#include <utility>

namespace mgk {
namespace {

template <int V>
using IC = std::integral_constant<int, V>;

enum { kInRead = 0, kInZero = 1, kInProlong = 2 };
enum { kOutRestrict = 1, kOutNorm = 2 };

constexpr int imod(int a, int m) { return ((a % m) + m) % m; }

constexpr int kPre = 4;     // rows in flight
constexpr int kWaves = 4;   // strips or chunks per workgroup

template <typename T>
struct Args2 {
  const T *u, *f, *k, *ec;
  T *out, *fc;
  double* partial;
  int n, strips, ylen, chunks;
  T h2, ih2;
};

template <typename T, bool VAR, int S, int IN, int OUT>
struct Strip {
  static constexpr int H = 2 * S;
  static constexpr bool RES = OUT == kOutRestrict, NORM = OUT == kOutNorm;
  static constexpr int XR = RES ? 4 : NORM ? 2 : 0;  // columns by which residuals narrow a strip
  static constexpr int YR = RES ? 2 : NORM ? 1 : 0;  // final rows beyond a chunk's ends
  static constexpr int TX = 128 - 2 * H - XR;        // output columns
  static constexpr int Q = H + 4;                    // rows queued (even, multiple of kPre or not)
  static_assert(Q % 2 == 0 && TX % 2 == 0, "parities");

  __device__ __forceinline__ static double run(const Args2<T>& a, int ox, int y0, int y1)
  {
    const int n = a.n, lane = threadIdx.x & 63;
    const int gx = ox - H + 2 * lane;  // odd
    const uint32_t rowb = (uint32_t)n * (uint32_t)sizeof(T);
    uint32_t cb[2], sb[2];
    bool in[2], own[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int x = gx + o, px = 2 * lane + o;
      in[o] = x >= 1 && x <= n - 2;
      // residual strips: final columns are stored from H on, as many as the strip's stride
      own[o] = in[o] && px >= H && px < H + TX;
      cb[o] = (uint32_t)min(max(x, 0), n - 1) * (uint32_t)sizeof(T);
      sb[o] = own[o] ? cb[o] : 0x80000000u;
    }
    // residual sums: the columns whose residual this strip owns lie one further inside
    const int nlo = ox == 1 ? 1 : ox + 1, nhi = min(ox + 1 + TX, n - 1);
    const int xlo = ox == 1 ? 2 : ox + 2;
    const int gxc = gx + 1;  // even column 2X of the lane's coarse column
    const bool cown = gxc >= xlo && gxc < ox + 2 + TX && gxc <= n - 3;

    T U[Q][2], F[Q][2], K[Q][2];
    T PU[kPre][2], PF[kPre][2], PK[kPre][2];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int o = 0; o < 2; ++o) U[q][o] = F[q][o] = K[q][o] = T(0);
#pragma unroll
    for (int q = 0; q < kPre; ++q)
#pragma unroll
      for (int o = 0; o < 2; ++o) PU[q][o] = PF[q][o] = PK[q][o] = T(0);
    static_assert(kPre % 2 == 0, "a buffer keeps its row parity");

    const int nc = (n - 1) / 2 + 1;
    const uint32_t crowb = (uint32_t)nc * (uint32_t)sizeof(T);
    uint32_t ccb[2] = {0, 0};
    T CA[kPre][2], CB[kPre][2];  // coarse rows floor(y/2) and (odd rows) floor(y/2) + 1
    if constexpr (IN == kInProlong) {
      const int cx = (gx - 1) >> 1;
      ccb[0] = (uint32_t)min(max(cx, 0), nc - 1) * (uint32_t)sizeof(T);
      ccb[1] = (uint32_t)min(max(cx + 1, 0), nc - 1) * (uint32_t)sizeof(T);
    }
    auto load = [&](int y, auto BC, auto YPC) {
      constexpr int b = decltype(BC)::value, ypar = decltype(YPC)::value;  // ypar: parity of y
      const size_t yb = (size_t)min(max(y, 0), n - 1) * rowb;
      const PlaneBuf bu = plane_buf(a.u, yb, rowb), bf = plane_buf(a.f, yb, rowb);
      const PlaneBuf bk = plane_buf(VAR ? a.k : a.f, yb, rowb);
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        if constexpr (IN != kInZero) PU[b][o] = buf_load<T>(bu, cb[o], 0u);
        PF[b][o] = buf_load<T>(bf, cb[o], 0u);
        if constexpr (VAR) PK[b][o] = buf_load<T>(bk, cb[o], 0u);
      }
      if constexpr (IN == kInProlong) {
        const int Y = y >> 1;
        const PlaneBuf ca = plane_buf(a.ec, (size_t)min(max(Y, 0), nc - 1) * crowb, crowb);
        const PlaneBuf cc = plane_buf(a.ec, (size_t)min(max(Y + 1, 0), nc - 1) * crowb, crowb);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          CA[b][c] = buf_load<T>(ca, ccb[c], 0u);
          if constexpr (ypar == 1) CB[b][c] = buf_load<T>(cc, ccb[c], 0u);
        }
      }
    };

    const int ybeg = y0 - H - YR, yend = y1 + H + YR;
    int yl = ybeg;
    T acc = T(0);        // RES: the coarse node's sum so far
    T R[3] = {T(0), T(0), T(0)};  // RES: residuals of the previous step's row at 2X-1, 2X, 2X+1
    double sumsq = 0.0;
    auto preload = [&]<int... Ps>(std::integer_sequence<int, Ps...>) {
      (load(yl + Ps, IC<Ps>{}, IC<(1 + H + YR + Ps) & 1>{}), ...);  // at least kPre rows
    };
    preload(std::make_integer_sequence<int, kPre>{});

    // one step, phase P = (yl - ybeg) mod L: row yl - d in slot (P - d) mod Q
    auto body = [&](auto PC) -> bool {
      constexpr int P = decltype(PC)::value;
      constexpr int ypar = (1 + H + YR + P) & 1;  // parity of yl (y0 odd)
      constexpr int s0 = P % Q, b = P % kPre;
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        T v = IN == kInZero ? T(0) : PU[b][o];
        if constexpr (IN == kInProlong) {
          // coarse columns cx, cx + 1 for the odd column, cx + 1 for the even one; terms in the
          // order y, x
          constexpr T wy = ypar ? T(0.5) : T(1);
          T e = T(0);
#pragma unroll
          for (int q = 0; q < 1 + ypar; ++q) {
            const T c0 = q ? CB[b][0] : CA[b][0], c1 = q ? CB[b][1] : CA[b][1];
            if (o == 0) e = e + (wy * T(0.5)) * c0;
            e = e + (wy * (o == 0 ? T(0.5) : T(1))) * c1;
          }
          if (in[o] && yl >= 1 && yl <= n - 2) v = v + e;
        }
        U[s0][o] = v;
        F[s0][o] = PF[b][o];
        if constexpr (VAR) K[s0][o] = PK[b][o];
      }
      if (yl + kPre < yend) load(yl + kPre, IC<b>{}, IC<ypar>{});  // kPre is even
      constexpr int o = ypar;  // the column updated in this step
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const int p = yl - 1 - j;
        if (p < 1 || p > n - 2) continue;
        const int c = imod(P - 1 - j, Q), m = imod(P - 2 - j, Q), pl = imod(P - j, Q);
        T xm, xp, kxm = T(0), kxp = T(0);
        if (o == 0) {
          xm = from_lane_below(U[c][1]);
          xp = U[c][1];
          if constexpr (VAR) { kxm = from_lane_below(K[c][1]); kxp = K[c][1]; }
        } else {
          xm = U[c][0];
          xp = from_lane_above(U[c][0]);
          if constexpr (VAR) { kxm = K[c][0]; kxp = from_lane_above(K[c][0]); }
        }
        T ym = U[m][o], yp = U[pl][o];
        if (IN == kInZero && j == 0) xm = xp = ym = yp = T(0);  // the other colour is still 0
        const T h2f = a.h2 * F[c][o];
        T v;
        if constexpr (!VAR) v = gs_const<T, 2>(h2f, xm, xp, ym, yp, T(0), T(0));
        else v = gs_var<T, 2>(h2f, K[c][o], xm, kxm, xp, kxp, ym, K[m][o], yp, K[pl][o], T(0), T(0), T(0), T(0));
        U[c][o] = in[o] ? v : U[c][o];
      }
      // row yl - H is final
      {
        const int p = yl - H;
        if (p >= y0 && p < y1) {
          constexpr int c = imod(P - H, Q);
          const PlaneBuf bo = plane_buf(a.out, (size_t)p * rowb, rowb);
#pragma unroll
          for (int q = 0; q < 2; ++q) buf_store(U[c][q], bo, sb[q], 0u);
        }
      }
      if constexpr (RES || NORM) {
        const int q = yl - H - 1;  // its neighbours q - 1, q + 1 are final
        constexpr int c = imod(P - H - 1, Q), m = imod(P - H - 2, Q), pl = imod(P - H, Q);
        constexpr int qpar = (ypar + H + 1) & 1;
        if (RES ? (q >= y0 - 1 && q <= y1) : (q >= y0 && q < y1)) {
          const bool qin = q >= 1 && q <= n - 2;
          const T l1 = from_lane_below(U[c][1]), r0 = from_lane_above(U[c][0]);
          T kl1 = T(0), kr0 = T(0);
          if constexpr (VAR) { kl1 = from_lane_below(K[c][1]); kr0 = from_lane_above(K[c][0]); }
          T r[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const T xm = i ? U[c][0] : l1, xp = i ? r0 : U[c][1];
            T au;
            if constexpr (!VAR) au = au_const<T, 2>(a.ih2, U[c][i], xm, xp, U[m][i], U[pl][i], T(0), T(0));
            else au = au_var<T, 2>(a.ih2, U[c][i], K[c][i], xm, i ? K[c][0] : kl1, xp, i ? kr0 : K[c][1],
                                   U[m][i], K[m][i], U[pl][i], K[pl][i], T(0), T(0), T(0), T(0));
            r[i] = qin && in[i] ? F[c][i] - au : T(0);
            if constexpr (NORM) {
              const int x = gx + i;
              if (x >= nlo && x < nhi) sumsq += (double)r[i] * (double)r[i];
            }
          }
          if constexpr (RES) {
            R[0] = r[0];
            R[1] = r[1];
            R[2] = from_lane_above(r[0]);
            // the nine terms of coarse row Y in the order y, x: rows 2Y-1, 2Y, 2Y+1
            constexpr T w[3] = {T(0.25), T(0.5), T(0.25)};
            T next = T(0);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
              if (qpar == 1) {
                acc = acc + (w[i] * w[2]) * R[i];     // completes row (q - 1) / 2
                next = next + (w[i] * w[0]) * R[i];   // starts row (q + 1) / 2
              } else {
                acc = acc + (w[i] * w[1]) * R[i];
              }
            }
            if (qpar == 1) {
              const int Y = (q - 1) >> 1;
              if (cown && 2 * Y >= y0 && 2 * Y < y1 && Y >= 1 && Y <= nc - 2)
                a.fc[(size_t)Y * nc + (size_t)(gxc >> 1)] = acc;
              acc = next;
            }
          }
        }
      }
      ++yl;
      return yl < yend;
    };
    constexpr int L = Q % kPre == 0 ? Q : 2 * Q;  // phases until the queue and the loads repeat
    static_assert(L % kPre == 0, "phases");
    auto round = [&]<int... Ps>(std::integer_sequence<int, Ps...>) {
      bool go = true;
      ((go = go && body(IC<Ps>{})), ...);
      return go;
    };
    while (round(std::make_integer_sequence<int, L>{})) {
    }
    return sumsq;
  }
};

template <typename T, bool VAR, int S, int IN, int OUT>
__global__ void __launch_bounds__(64 * kWaves) k_rbgs_strips(Args2<T> a)
{
  using C = Strip<T, VAR, S, IN, OUT>;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.x * kWaves + w;
  double sumsq = 0.0;
  if (t < a.strips * a.chunks) {
    const int ox = 1 + (t % a.strips) * C::TX, y0 = 1 + (t / a.strips) * a.ylen;
    sumsq = C::run(a, ox, y0, min(y0 + a.ylen, a.n - 1));
  }
  if constexpr (OUT == kOutNorm) {
    __shared__ double part[kWaves];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sumsq += __shfl_xor(sumsq, o, 64);
    if ((threadIdx.x & 63) == 0) part[w] = sumsq;
    __syncthreads();
    if (threadIdx.x == 0) a.partial[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
  }
}

__global__ void __launch_bounds__(256)
    k_sum_2d(const double* __restrict__ partial, int count, double* __restrict__ out)
{
  __shared__ double part[4];
  double acc = 0.0;
  for (int i = threadIdx.x; i < count; i += blockDim.x) acc += partial[i];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = (part[0] + part[1]) + (part[2] + part[3]);
}

// Rows per chunk: a chunk of ylen rows takes ylen + warm steps.  While the waves are fewer than
// the device runs at once (kTarget) a shorter chunk shortens the launch; beyond that it only adds
// warm-up work, so chunks stay long enough for kTarget waves.
constexpr int kTarget = 2048;

template <typename T, bool VAR, int S, int IN, int OUT>
void launch(hipStream_t s, int n, double h, const T* k, const T* f, const T* u, T* out, const T* ec,
            T* fc, double* partial, double* norm2, int* count)
{
  using C = Strip<T, VAR, S, IN, OUT>;
  Args2<T> a{u, f, k, ec, out, fc, partial, n, 0, 0, 0, (T)(h * h), (T)(1.0 / (h * h))};
  const int m = n - 2;
  a.strips = (m + C::TX - 1) / C::TX;
  int chunks = (kTarget + a.strips - 1) / a.strips;
  a.ylen = (m + chunks - 1) / chunks;
  a.ylen += a.ylen & 1;  // chunks start on odd rows
  if (a.ylen < 4) a.ylen = 4;
  a.chunks = (m + a.ylen - 1) / a.ylen;
  const int blocks = (a.strips * a.chunks + kWaves - 1) / kWaves;
  k_rbgs_strips<T, VAR, S, IN, OUT><<<blocks, 64 * kWaves, 0, s>>>(a);
  if (OUT == kOutNorm && count) *count = blocks;
  else if (OUT == kOutNorm) k_sum_2d<<<1, 256, 0, s>>>(partial, blocks, norm2);
}

template <typename T, bool VAR, int S>
void launch_s(hipStream_t s, int n, double h, const T* k, const T* f, const T* u, T* out, bool zero,
              const T* ec, T* fc, double* partial, double* norm2, int* count)
{
  if (ec && norm2) {
    if constexpr (sizeof(T) == 8) launch<T, VAR, S, kInProlong, kOutNorm>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
  } else if (norm2) {
    if constexpr (sizeof(T) == 8) launch<T, VAR, S, kInRead, kOutNorm>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
  } else if (ec) {
    launch<T, VAR, S, kInProlong, 0>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
  } else if (fc) {
    if (zero) launch<T, VAR, S, kInZero, kOutRestrict>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
    else launch<T, VAR, S, kInRead, kOutRestrict>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
  } else {
    if (zero) launch<T, VAR, S, kInZero, 0>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
    else launch<T, VAR, S, kInRead, 0>(s, n, h, k, f, u, out, ec, fc, partial, norm2, count);
  }
}

}  // namespace

template <typename T>
void rbgs_strips(hipStream_t s, int n, double h, const T* k, const T* f, const T* u, T* out,
                 int sweeps, bool zero, const T* ec, T* fc, double* partial, double* norm2, int* count)
{
  auto go = [&](auto vc, auto sc) {
    launch_s<T, decltype(vc)::value, decltype(sc)::value>(s, n, h, k, f, u, out, zero, ec, fc, partial, norm2, count);
  };
  if (k && sweeps == 2) go(std::true_type{}, IC<2>{});
  else if (k) go(std::true_type{}, IC<1>{});
  else if (sweeps == 2) go(std::false_type{}, IC<2>{});
  else go(std::false_type{}, IC<1>{});
}

template void rbgs_strips<double>(hipStream_t, int, double, const double*, const double*, const double*,
                                  double*, int, bool, const double*, double*, double*, double*, int*);
template void rbgs_strips<float>(hipStream_t, int, double, const float*, const float*, const float*, float*,
                                 int, bool, const float*, float*, double*, double*, int*);

}  // namespace mgk
