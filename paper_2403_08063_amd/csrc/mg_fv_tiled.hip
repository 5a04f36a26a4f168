// Temporally blocked damped-Jacobi passes of the cell-centred finite-volume scheme on gfx950.
//
// One launch performs S sweeps of u + omega h^2/6 (f - A u), out of place, with what stands
// before and after them in the V-cycle taken in:
//   IN    kRead: from u;  kZero: from an identically zero u (not read);  kProlong: from
//         u + P e, the coarse-grid correction interpolated as each plane arrives;
//   RES   the residual of the result and its restriction (mean of the 8 children);
//   NORM  the squared norm of the residual of the *input*, which the first sweep forms anyway.
// A sweep alone moves 24 bytes per cell and is bound by memory (fv_jacobi_tiled, 5.2 TB/s), so
// the sweeps of a smoothing step share one pass: about 24 bytes and a halo for all of them.
//
// Decomposition (as the fused red-black smoother's): a workgroup owns a tile of 64 columns x
// 2 W RPW rows of a z-chunk and streams through its planes.  A wave holds two row groups of 32
// lanes, a lane two adjacent columns of RPW rows.  Sweep j updates plane zl - j when plane zl
// arrives: its z-neighbours are planes zl - j - 1 and zl - j + 1 of sweep j - 1, the latter
// formed earlier in the same step.  x-neighbours come from the adjacent lane by DPP, y-neighbours
// from the lane's rows or, between row groups, from LDS edge rows (double-buffered by step
// parity: one barrier per plane).  Sweep j is exact j cells inside the loaded tile; values nearer
// its edge are read only by such values and never stored.  The tile overlaps its neighbours by
// H cells: 3, or 4 where the residual is formed (which also makes tile origins odd, so that a
// lane's column pair and row pairs are the children of one coarse cell; with H = 3 origins are
// even and a pair lies between the same two coarse cells, which halves the coarse loads).
//
// Tiles that touch no domain face run without the ghost and Dirichlet selects (EDGE = false).
// Every cell takes the single passes' operations in their order: results are bitwise equal.
//
// A pass has two waves per SIMD, which keep neither the VALU (about 300 instructions per wave and
// plane, 240 of them FP64: 50 % busy at 512^3) nor memory (4.1 and 4.6 TB/s) full; a wave waits for
// memory or the barrier a third of its time.  What is not arithmetic counts: cells of a plane in one block without
// branches, the planes next to a domain face in a copy of their own, and edge rows as 16-byte
// pairs took the 512^3 passes from 1.40 and 1.07 ms (pre- and post-smoothing) to 1.14 and 0.94,
// loads and stores of a lane's columns as one access in all tiles to 1.13 and 0.91; 35 V(3,3)
// cycles 105.9 -> 87 to 88 ms.
#include "mg_buffer.h"
#include "mg_kernels.h"
#include "mg_lanes.h"

#include <type_traits>
#include <utility>

namespace mgk {
namespace {

template <int V>
using IC = std::integral_constant<int, V>;

enum { kRead = 0, kZero = 1, kProlong = 2 };

constexpr int imod(int a, int m) { return ((a % m) + m) % m; }

struct FvArgs {
  const double* u;
  const double* f;
  const double* ec;  // kProlong: coarse correction, (N/2 + 2)^3 values, ghost layer not read
  double* out;
  double* fc;        // RES: coarse right-hand side, cells only
  double* partial;   // NORM: per-workgroup sums
  int N, tiles_x, tiles_y, zlen;
  double ih2, coef;
};

template <int S, int IN, bool RES, bool NORM, int W, int RPW>
struct FvPass {
  static_assert(RPW % 2 == 0, "row pairs");
  static_assert(!NORM || IN == kRead, "the norm is that of the stored input");
  static constexpr int LW = 32, VW = 2 * W;  // lanes per row, row groups per tile
  static constexpr int BX = 2 * LW, BY = VW * RPW;
  static constexpr int H = RES ? 4 : 3;
  static constexpr int TX = BX - 2 * H, TY = BY - 2 * H;
  static constexpr int HZ = S + (RES ? 1 : 0);  // planes loaded before and after a z-chunk
  static constexpr int NL = S + (RES ? 1 : 0);  // fields whose edge rows are exchanged
  static_assert(S >= 1 && S <= 3 && TY > 0, "halo of the tile");

  struct Shared {
    double2 e[2][NL][VW][2][LW];  // [parity][field][row group][first, last row][lane]: two columns
    double red[NORM ? W : 1];
  };

  template <bool EDGE>
  __device__ __forceinline__ static void run(const FvArgs& a, Shared& sh, int ox, int oy, int z0, int z1)
  {
    const int N = a.N, m = N + 2;
    const int lane = threadIdx.x & (LW - 1), w = (int)(threadIdx.x >> 5);
    const int gx = ox - H + 2 * lane, gy = oy - H + w * RPW;  // first column and row
    const int wm = w > 0 ? w - 1 : 0, wp = w < VW - 1 ? w + 1 : VW - 1;
    const uint32_t planeb = (uint32_t)((size_t)m * (size_t)m * 8u);

    // bit 2 i + o: a cell; a cell this tile stores
    unsigned cell = 0, own = 0;
    uint32_t rowb[RPW];
    // a lane's two columns are one access, not clamped: columns outside the ghost layer take
    // values of an adjacent row or 0, which no cell reads
    const uint32_t colb = (uint32_t)(gx * 8);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int x = gx + o, px = 2 * lane + o;
      const bool xin = x >= 1 && x <= N, xown = xin && px >= H && px < H + TX;
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const int y = gy + i, py = w * RPW + i;
        const bool yin = y >= 1 && y <= N, yown = yin && py >= H && py < H + TY;
        cell |= (xin && yin) ? 1u << (2 * i + o) : 0u;
        own |= (xown && yown) ? 1u << (2 * i + o) : 0u;
      }
    }
#pragma unroll
    for (int i = 0; i < RPW; ++i)
      rowb[i] = (uint32_t)((EDGE ? min(max(gy + i, 0), N + 1) : gy + i) * m) * 8u;
    // domain faces: the columns and rows next to them have fixed parities (see H)
    constexpr int XLO = RES ? 0 : 1, XHI = 1 - XLO;
    const bool fx0 = EDGE && gx + XLO == 1, fx1 = EDGE && gx + XHI == N;

    // field j: the iterate after j sweeps, planes by phase mod 3; f by phase mod 6
    double U[S + 1][3][RPW][2], F[6][RPW][2], PU[RPW][2], PF[RPW][2];
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        PU[i][o] = 0.0;
#pragma unroll
        for (int j = 0; j <= S; ++j)
#pragma unroll
          for (int q = 0; q < 3; ++q) U[j][q][i][o] = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) F[q][i][o] = 0.0;
      }

    // u of plane z, f of plane z - 1: of each plane when it is first needed
    auto load = [&](int z) {
      const size_t zb = (size_t)min(max(z, 0), N + 1) * planeb;
      const size_t fb = (size_t)min(max(z - 1, 0), N + 1) * planeb;
      const PlaneBuf bu = plane_buf(a.u, zb, planeb), bf = plane_buf(a.f, fb, planeb);
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        if constexpr (IN != kZero) buf_load2(bu, colb + rowb[i], 0u, PU[i][0], PU[i][1]);
        buf_load2(bf, colb + rowb[i], 0u, PF[i][0], PF[i][1]);
      }
    };

    // Prolongation: the lane's columns 2X, 2X+1 lie between coarse columns X and X+1 (weight
    // 3/4 for the nearer), its rows likewise between coarse rows Y.. ; CA and CB hold the two
    // coarse planes around the current fine plane, CE the one in flight.  Outside the domain
    // the correction is extended by minus the adjacent cell (a sign per axis).
    constexpr int CR = RPW / 2 + 1;
    const int Nc = N / 2, mc = Nc + 2;
    const uint32_t cplaneb = (uint32_t)((size_t)mc * (size_t)mc * 8u);
    uint32_t ccb[2] = {0, 0}, crb[CR] = {};
    unsigned csign = 0;  // bit 2 r + c: outside the domain in x or y, not both
    double CA[CR][2], CB[CR][2], CE[CR][2];
    uint32_t cneg = 0;   // sign of a coarse plane outside the domain
    if constexpr (IN == kProlong) {
      const int X = gx >> 1, Y = gy >> 1;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        ccb[c] = (uint32_t)(EDGE ? min(max(X + c, 1), Nc) : X + c) * 8u;
      }
#pragma unroll
      for (int r = 0; r < CR; ++r) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
          csign |= ((X + c <= 0 || X + c > Nc) != (Y + r <= 0 || Y + r > Nc)) ? 1u << (2 * r + c) : 0u;
        crb[r] = (uint32_t)((EDGE ? min(max(Y + r, 1), Nc) : Y + r) * mc) * 8u;
      }
    }
    auto cload = [&](int Z) {
      cneg = Z <= 0 || Z > Nc ? 0x80000000u : 0u;
      const PlaneBuf be = plane_buf(a.ec, (size_t)min(max(Z, 1), Nc) * cplaneb, cplaneb);
#pragma unroll
      for (int r = 0; r < CR; ++r) {
        if constexpr (EDGE) {
#pragma unroll
          for (int c = 0; c < 2; ++c) CE[r][c] = buf_load<double>(be, ccb[c] + crb[r], 0u);
        } else {
          buf_load2(be, ccb[0] + crb[r], 0u, CE[r][0], CE[r][1]);
        }
      }
    };
    auto ctake = [&](double (&C)[CR][2]) {
#pragma unroll
      for (int r = 0; r < CR; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          uint32_t flip = cneg;
          if constexpr (EDGE) flip ^= ((csign >> (2 * r + c)) & 1u) << 31;
          C[r][c] = __hiloint2double((int)((uint32_t)__double2hiint(CE[r][c]) ^ flip), __double2loint(CE[r][c]));
        }
    };
    // P e at (i, o) between the planes p (the parent) and q: 8 terms in the order z, y, x, the
    // parent first, with the weights of fv_jacobi_prolong_tiled
    auto interpolate = [&](const double (&p)[CR][2], const double (&q)[CR][2], int i, int o) -> double {
      const int rp = i % 2 ? i / 2 + 1 : i / 2, rn = i % 2 ? i / 2 : i / 2 + 1;
      double e = 0.0 + 0.421875 * p[rp][o];
      e = e + 0.140625 * p[rp][1 - o];
      e = e + 0.140625 * p[rn][o];
      e = e + 0.046875 * p[rn][1 - o];
      e = e + 0.140625 * q[rp][o];
      e = e + 0.046875 * q[rp][1 - o];
      e = e + 0.046875 * q[rn][o];
      e = e + 0.015625 * q[rn][1 - o];
      return e;
    };

    // finished plane p, queue slot SO of field S, stored behind the next step's barrier
    auto store = [&](int p, auto SOC) {
      constexpr int so = decltype(SOC)::value;
      if (p < z0 || p >= z1) return;
      const PlaneBuf bo = plane_buf(a.out, (size_t)p * planeb, planeb);
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const unsigned m2 = (own >> (2 * i)) & 3u;
        if constexpr (RES) {
          // pairs are wholly inside or outside the stored columns
          buf_store2(U[S][so][i][0], U[S][so][i][1], bo, (m2 & 1u) ? colb + rowb[i] : 0x80000000u, 0u);
        } else {
          // whole pairs, and the single columns at the tile's two ends
          const bool second = m2 == 2u, single = second || m2 == 1u;
          buf_store2(U[S][so][i][0], U[S][so][i][1], bo, m2 == 3u ? colb + rowb[i] : 0x80000000u, 0u);
          buf_store(second ? U[S][so][i][1] : U[S][so][i][0], bo,
                    single ? colb + rowb[i] + (second ? 8u : 0u) : 0x80000000u, 0u);
        }
      }
    };

    double RA[RPW / 2];  // RES: sums over the children of a plane pair
#pragma unroll
    for (int i = 0; i < RPW / 2; ++i) RA[i] = 0.0;
    double sumsq[RPW][2] = {};  // of every cell; those that the tile does not own drop out at the end

    const int zbeg = z0 - HZ, zend = z1 + HZ;
    int zl = zbeg;
    // zl = zbeg + step; z0 is odd, so plane zl of phase P has parity (1 + HZ + P) & 1
    if constexpr (IN == kProlong) {
      // the first plane's coarse planes: odd 2Z-1: Z-1 (CA), Z (CB); even 2Z: Z (CA), Z+1 (CB)
      cload(zl >> 1);
      ctake(CA);
      cload((zl >> 1) + 1);
      ctake(CB);
    }
    load(zl);

    auto body = [&](auto PC) -> bool {
      constexpr int P = decltype(PC)::value;
      constexpr int zpar = (1 + HZ + P) & 1;  // parity of zl
      constexpr int rb = (P + 1) & 1, wb = P & 1;
      // plane zl enters
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          double v = IN == kZero ? 0.0 : PU[i][o];
          if constexpr (IN == kProlong) {
            // odd planes 2Z-1 have the parent Z (CB), even planes 2Z the parent Z (CA)
            const double e = zpar ? interpolate(CB, CA, i, o) : interpolate(CA, CB, i, o);
            const bool in = zl >= 1 && zl <= N && (!EDGE || ((cell >> (2 * i + o)) & 1u));
            v = in ? v + e : v;
          }
          U[0][P % 3][i][o] = v;
          F[imod(P - 1, 6)][i][o] = PF[i][o];
        }
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int o = 0; o < 2; ++o) asm volatile("" : "+v"(U[0][P % 3][i][o]));
      __syncthreads();
      store(zl - 1 - S, IC<imod(P - 1 - S, 3)>{});
      if (zl + 1 < zend) {
        if constexpr (IN == kProlong && zpar == 1) cload(((zl + 1) >> 1) + 1);
        load(zl + 1);
      }
      // (A u) at (i, o) of field j's centre plane p; ZF: p lies next to a domain face (the planes
      // that do take a copy of the code, so that the others' cells stay in one block)
      auto apply = [&](auto JC, auto QC, auto ZF, double2 em, double2 ep, int p, int i, int o) -> double {
        constexpr int j = decltype(JC)::value, d = decltype(QC)::value;  // plane p = zl - d
        constexpr int c = imod(P - d, 3), lo = imod(P - d - 1, 3), hi = imod(P - d + 1, 3);
        const double ui = U[j][c][i][o];
        double xm = o ? U[j][c][i][0] : from_lane_below(U[j][c][i][1]);
        double xp = o ? from_lane_above(U[j][c][i][0]) : U[j][c][i][1];
        double ym = i > 0 ? U[j][c][i - 1][o] : o ? em.y : em.x;
        double yp = i < RPW - 1 ? U[j][c][i + 1][o] : o ? ep.y : ep.x;
        double zm = U[j][lo][i][o], zp = U[j][hi][i][o];
        if constexpr (EDGE) {
          // a ghost neighbour enters as 2 g - u_i
          if (o == XLO) xm = fx0 ? 2.0 * xm - ui : xm;
          if (o == XHI) xp = fx1 ? 2.0 * xp - ui : xp;
          if (i % 2 == XLO) ym = gy + i == 1 ? 2.0 * ym - ui : ym;
          if (i % 2 == XHI) yp = gy + i == N ? 2.0 * yp - ui : yp;
        }
        if constexpr (decltype(ZF)::value) {
          if (p == 1) zm = 2.0 * zm - ui;
          if (p == N) zp = 2.0 * zp - ui;
        }
        double s = ui - xm;
        s = s + (ui - xp);
        s = s + (ui - ym);
        s = s + (ui - yp);
        s = s + (ui - zm);
        s = s + (ui - zp);
        return s * a.ih2;
      };
      auto sweep = [&](auto JC) {
        constexpr int j = decltype(JC)::value;  // sweep j + 1: field j -> j + 1, plane zl - 1 - j
        constexpr int c = imod(P - 1 - j, 3), fs = imod(P - 1 - j, 6);
        const int p = zl - 1 - j;
        if (p < 1 || p > N) {
#pragma unroll
          for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o) U[j + 1][c][i][o] = U[j][c][i][o];
          return;
        }
        constexpr bool zero = IN == kZero && j == 0;
        [[maybe_unused]] double R[RPW][2];
        double2 em{}, ep{};  // the adjacent row groups' edge rows
        if constexpr (!zero) {
          em = sh.e[rb][j][wm][1][lane];
          ep = sh.e[rb][j][wp][0][lane];
        }
        auto cells = [&](auto ZF) {
#pragma unroll
          for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o) {
              const double ui = U[j][c][i][o];
              double r;
              if constexpr (zero) r = F[fs][i][o] - 0.0;
              else r = F[fs][i][o] - apply(IC<j>{}, IC<1 + j>{}, ZF, em, ep, p, i, o);
              const double v = ui + a.coef * r;
              U[j + 1][c][i][o] = EDGE && !((cell >> (2 * i + o)) & 1u) ? ui : v;
              if constexpr (NORM && j == 0) R[i][o] = r;
            }
        };
        if (!zero && (p == 1 || p == N)) cells(IC<1>{});
        else cells(IC<0>{});
        if constexpr (NORM && j == 0) {
          if (p >= z0 && p < z1) {
#pragma unroll
            for (int i = 0; i < RPW; ++i)
#pragma unroll
              for (int o = 0; o < 2; ++o) sumsq[i][o] += R[i][o] * R[i][o];
          }
        }
      };
      sweep(IC<0>{});
      if constexpr (S >= 2) sweep(IC<1>{});
      if constexpr (S >= 3) sweep(IC<2>{});
      if constexpr (RES) {
        constexpr int fs = imod(P - 1 - S, 6);
        constexpr int qpar = (zpar + 1 + S) & 1;
        const int q = zl - 1 - S;
        if (q >= z0 && q < z1) {
          const double2 em = sh.e[rb][S][wm][1][lane], ep = sh.e[rb][S][wp][0][lane];
          auto cells = [&](auto ZF) {
#pragma unroll
            for (int i = 0; i < RPW; ++i)
#pragma unroll
              for (int o = 0; o < 2; ++o) {
                const double r = F[fs][i][o] - apply(IC<S>{}, IC<1 + S>{}, ZF, em, ep, q, i, o);
                if (qpar == 1 && i % 2 == 0 && o == 0) RA[i / 2] = 0.0;
                RA[i / 2] = RA[i / 2] + r;
              }
          };
          if (q == 1 || q == N) cells(IC<1>{});
          else cells(IC<0>{});
          if constexpr (qpar == 0) {
            const PlaneBuf bc = plane_buf(a.fc, (size_t)(q >> 1) * cplaneb, cplaneb);
#pragma unroll
            for (int i = 0; i < RPW; i += 2) {
              const uint32_t at = (uint32_t)(((gy + i + 1) >> 1) * mc + ((gx + 1) >> 1)) * 8u;
              buf_store(RA[i / 2] / 8.0, bc, ((own >> (2 * i)) & 1u) ? at : 0x80000000u, 0u);
            }
          }
        }
      }
      // edge rows of the planes that are centres in the next step: plane zl - j of field j
      auto edges = [&](auto JC) {
        constexpr int j = decltype(JC)::value;
        if constexpr (IN == kZero && j == 0) return;  // the sweep from zero reads no neighbours
        constexpr int c = imod(P - j, 3);
        sh.e[wb][j][w][0][lane] = make_double2(U[j][c][0][0], U[j][c][0][1]);
        sh.e[wb][j][w][1][lane] = make_double2(U[j][c][RPW - 1][0], U[j][c][RPW - 1][1]);
      };
      edges(IC<0>{});
      if constexpr (NL >= 2) edges(IC<1>{});
      if constexpr (NL >= 3) edges(IC<2>{});
      if constexpr (NL >= 4) edges(IC<3>{});
      if constexpr (IN == kProlong && zpar == 1) {
        // the next plane is even, 2Z: Z moves to CA, Z + 1 is the new CB
        if (zl + 1 < zend) {
#pragma unroll
          for (int r = 0; r < CR; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) CA[r][c] = CB[r][c];
          ctake(CB);
        }
      }
      ++zl;
      // the last step stores its own finished plane
      if (zl == zend) store(zl - 1 - S, IC<imod(P - S, 3)>{});
      return zl < zend;
    };
    auto round = [&]<int... Ps>(std::integer_sequence<int, Ps...>) {
      bool go = true;
      ((go = go && body(IC<Ps>{})), ...);
      return go;
    };
    while (round(std::make_integer_sequence<int, 6>{})) {
    }
    if constexpr (NORM) {
      double sum = 0.0;
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int o = 0; o < 2; ++o) sum += ((own >> (2 * i + o)) & 1u) ? sumsq[i][o] : 0.0;
#pragma unroll
      for (int o2 = 32; o2 >= 1; o2 >>= 1) sum += __shfl_xor(sum, o2, 64);
      if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = sum;
      __syncthreads();
      if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int v = 0; v < W; ++v) tot += sh.red[v];
        a.partial[blockIdx.x] = tot;
      }
    }
  }
};

template <int S, int IN, bool RES, bool NORM, int W, int RPW>
__global__ void __launch_bounds__(64 * W) k_fv_sweeps(FvArgs a)
{
  using C = FvPass<S, IN, RES, NORM, W, RPW>;
  __shared__ typename C::Shared sh;
  // XCD-aware tile index: workgroup b runs on XCD b % 8, which gets a contiguous tile range
  const int b = blockIdx.x, nb = gridDim.x;
  const int xcd = b & 7, jb = b >> 3, q = nb >> 3, rem = nb & 7;
  const int t = (xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q) + jb;
  const int tx = t % a.tiles_x, ty = (t / a.tiles_x) % a.tiles_y, tz = t / (a.tiles_x * a.tiles_y);
  const int ox = 1 + tx * C::TX, oy = 1 + ty * C::TY;
  const int z0 = 1 + tz * a.zlen, z1 = min(z0 + a.zlen, a.N + 1);
  const bool edge = tx == 0 || ty == 0 || ox - C::H + C::BX > a.N + 1 || oy - C::H + C::BY > a.N + 1;
  if (edge) C::template run<true>(a, sh, ox, oy, z0, z1);
  else C::template run<false>(a, sh, ox, oy, z0, z1);
}

__global__ void __launch_bounds__(256)
    k_fv_sum_partials(const double* __restrict__ partial, int count, double* __restrict__ out)
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

// Workgroups of the kernel that a device holds at once.
template <typename Kernel>
int resident(Kernel kernel, int block)
{
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess || per_cu <= 0) per_cu = 1;
  return cus * per_cu;
}

#ifndef MG_FVS_W
#define MG_FVS_W 8
#endif
#ifndef MG_FVS_RPW
#define MG_FVS_RPW 2
#endif

template <int S, int IN, bool RES, bool NORM>
void launch(hipStream_t s, int N, double h, double omega, const double* u, const double* f,
            const double* ec, double* out, double* fc, double* partial, double* norm2,
            int* count)
{
  constexpr int W = MG_FVS_W, RPW = MG_FVS_RPW;
  using C = FvPass<S, IN, RES, NORM, W, RPW>;
  auto kern = k_fv_sweeps<S, IN, RES, NORM, W, RPW>;
  static const int capacity = resident(kern, 64 * W);
  FvArgs a{u, f, ec, out, fc, partial, N, (N + C::TX - 1) / C::TX, (N + C::TY - 1) / C::TY, N,
           1.0 / (h * h), omega * (h * h / 6.0)};
  // z-chunks of even length (they start on odd planes), as many as keep the critical path --
  // rounds of resident workgroups x planes per workgroup -- shortest
  const int per = a.tiles_x * a.tiles_y;
  long long best = -1;
  for (int zlen = 2; zlen <= N; zlen += 2) {
    const long long blocks = (long long)per * ((N + zlen - 1) / zlen);
    if (NORM && blocks > kStreamPartials) continue;
    const long long cost = (blocks + capacity - 1) / capacity * (zlen + 2 * C::HZ);
    if (best < 0 || cost <= best) {
      best = cost;
      a.zlen = zlen;
    }
  }
  const int blocks = per * ((N + a.zlen - 1) / a.zlen);
  kern<<<blocks, 64 * W, 0, s>>>(a);
  if (NORM && count) *count = blocks;
  else if (NORM) k_fv_sum_partials<<<1, 256, 0, s>>>(partial, blocks, norm2);
}

template <int S>
void launch_s(hipStream_t s, int N, double h, double omega, const double* u, const double* f,
              const double* ec, double* out, double* fc, double* partial, double* norm2,
            int* count)
{
  if (ec) launch<S, kProlong, false, false>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
  else if (!u && fc) launch<S, kZero, true, false>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
  else if (!u) launch<S, kZero, false, false>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
  else if (fc && norm2) launch<S, kRead, true, true>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
  else if (fc) launch<S, kRead, true, false>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
  else launch<S, kRead, false, false>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
}

}  // namespace

void fv_sweeps(hipStream_t s, int N, double h, double omega, int sweeps, const double* u,
               const double* f, const double* ec, double* out, double* fc, double* partial,
               double* norm2, int* count)
{
  if (fv_cube_supported(N)) {
    const int blocks = fv_cube_sweeps(s, N, h, omega, sweeps, u, f, ec, out, fc, partial, norm2 != nullptr);
    if (norm2 && count) *count = blocks;
    else if (norm2) k_fv_sum_partials<<<1, 256, 0, s>>>(partial, blocks, norm2);
    return;
  }
  if (sweeps == 3) launch_s<3>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
  else launch_s<2>(s, N, h, omega, u, f, ec, out, fc, partial, norm2, count);
}

}  // namespace mgk
