// Two damped-Jacobi sweeps of the 2:1 refined layout in one pass over memory, for blocks of 64 to
// 128 cells a side on gfx950.
//
// A sweep moves 24 bytes per cell and is bound by memory (4.2 TB/s at 128^3 cells per block), so
// two sweeps share one pass.  The second sweep needs the first one's values at the block's ghosts,
// which depend on other blocks: they are formed beforehand from the cells next to the faces
// (k_blk_shell, k_blk_fill_planes) in an array g of ghost planes, so that every block is swept by
// itself.
//
// Decomposition: a workgroup owns all columns of a block x TY rows x a z-chunk and streams through
// the planes.  A row group of LW lanes holds a row, two adjacent columns per lane (LW = 64; 32 for
// B = 64, two row groups per wave), so x needs no halo: the first and last lane take the ghosts of
// their rows.  When plane zl arrives, the first sweep updates plane zl - 1 and the second plane
// zl - 2; x-neighbours come from the adjacent lane by DPP, y-neighbours from the lane's rows or,
// between row groups, from LDS edge rows (double-buffered by step parity: one barrier per plane).
// Tiles overlap by two rows on each side; rows 0 and B + 1 and planes 0 and B + 1 are ghosts, whose
// first-sweep values are read from g in place of f.
//
// Every cell takes the operations of the single sweep in its order: results are bitwise equal.
//
// Measured, one pass (two sweeps) against single sweeps with the fill between them: 1.41 ms against
// 1.44 + 0.17 + 1.44 at 128^3 cells per block, 0.19 against 0.18 + 0.04 + 0.18 at 64^3; the ghost
// planes before it take 0.34 and 0.09 ms.  A V(3,3) cycle at 128^3 with the norm riding on its
// first pass: 16.8 -> 11.9 ms.  The last of an odd number of pre-smoothing sweeps takes the
// restriction in (kRestrict): 1.51 ms, and 0.38 for its ghost planes, where the sweep, a fill and
// the restriction took 1.44 + 0.17 + 0.93; the cycle 11.9 -> 11.2 ms.
// 12 waves of 2 rows (141-168 registers, 3 waves per SIMD); 8 x 3
// takes 0.4 % longer per solve, 12 x 3, 16 x 2 and 8 x 4 spill.  Blocks of less than 64 cells a
// side are bound by launches, which this adds to (32^3: 25 us a sweep); more than 128 columns do
// not fit the lanes of a row.
// Storing the cells next to same-level faces into the neighbours' ghosts as well, here and in the
// other sweeps, costs more than the fills that it replaces (243.8 ms against 238.7 for 20 cycles).
#include "mg_blocks_layout.h"
#include "mg_kernels.h"
#include "mg_lanes.h"

#include <utility>

namespace mgk {
namespace {

template <int V>
using IC = std::integral_constant<int, V>;

constexpr int imod(int a, int m) { return ((a % m) + m) % m; }

// two adjacent columns, 8-byte aligned
typedef double Pair __attribute__((ext_vector_type(2), aligned(8)));

struct PairArgs {
  const double* u;
  const double* f;
  const double* g;
  const double* hs;
  const int* faces;
  double* out;
  double* fc;       // kRestrict: coarse right-hand side, (B / 2 + 2)^3 values per block
  double* partial;  // kNorm
  double omega;
  int B, tiles_y, chunks, zlen, zero;
};

// What a pass is: two sweeps; two sweeps and the squared norm of the input's residual; one sweep
// and the restricted residual of its result (mean of the 8 children; a lane's columns, its rows and
// a plane pair are one coarse cell's children).
enum { kSweeps = 0, kNorm = 1, kRestrict = 2 };

template <int LW, int W, int RPW, bool COARSE, int OUT_>
struct PairPass {
  static constexpr bool NORM = OUT_ == kNorm, RES = OUT_ == kRestrict;
  static_assert(!RES || RPW == 2, "a row group is one coarse row");
  static constexpr int G = 64 / LW, VW = W * G, BY = VW * RPW;
  static constexpr int H = 2, TY = BY - 2 * H;

  struct Shared {
    double2 e[2][2][VW][2][LW];  // [parity][field][row group][first, last row][lane]: two columns
    double red[W];
  };

  __device__ __forceinline__ static void run(const PairArgs& a, Shared& sh, int b, int oy, int z0, int z1)
  {
    const int B = a.B, m = B + 2;
    const int lane = threadIdx.x & (LW - 1);
    const int w = LW == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : (int)(threadIdx.x >> 5);
    const int wm = w > 0 ? w - 1 : 0, wp = w < VW - 1 ? w + 1 : VW - 1;
    const int gy = oy - H + w * RPW;
    const bool active = 2 * lane < B, first = lane == 0, last = 2 * lane + 2 == B;
    const int gx = active ? 1 + 2 * lane : 1;
    const size_t sz = (size_t)m * m, blk = sz * m, BB = (size_t)B * B;
    const int* fb = a.faces + (size_t)b * 6 * kFaceInts;
    const double h = a.hs[b];
    const double ih2 = 1.0 / (h * h), coef = a.omega * (h * h / 6.0);
    auto bound = [&](int face) { return COARSE && fb[face * kFaceInts] == kFaceBoundary; };
    const bool bx0 = first && bound(0), bx1 = last && bound(1);
    const bool by0 = bound(2), by1 = bound(3), bz0 = bound(4), bz1 = bound(5);

    const double* ub = a.u + (size_t)b * blk;
    const double* fbk = a.f + (size_t)b * blk;
    const double* gb = a.g + (size_t)b * 6 * BB;
    double* ob = a.out + (size_t)b * blk;
    // per row: offset in a plane, row of the z faces, and whether it is a y ghost or an output row
    unsigned ghost = 0, own = 0;
    uint32_t ro[RPW], zo[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const int y = gy + i, py = w * RPW + i;
      ro[i] = (uint32_t)min(max(y, 0), B + 1) * (uint32_t)m;
      zo[i] = (uint32_t)(min(max(y, 1), B) - 1) * (uint32_t)B;
      ghost |= (y == 0 || y == B + 1) ? 1u << i : 0u;
      own |= (y >= 1 && y <= B && py >= H && py < H + TY) ? 1u << i : 0u;
    }

    // field 0: u, field 1: after the first sweep, planes by phase mod 3; F: f (or the first
    // sweep's ghosts) of the planes zl - 1 and zl - 2; X0, X1: x ghosts of the two fields
    double U[2][3][RPW][2], F[2][RPW][2], PU[RPW][2], PF[RPW][2];
    double X0[RPW], X1[RPW], PX0[RPW], PX1[RPW], OUT[RPW][2];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      X0[i] = X1[i] = PX0[i] = PX1[i] = 0.0;
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        PU[i][o] = PF[i][o] = OUT[i][o] = F[0][i][o] = F[1][i][o] = 0.0;
#pragma unroll
        for (int q = 0; q < 3; ++q) U[0][q][i][o] = U[1][q][i][o] = 0.0;
      }
    }

    // u of plane z, f and x ghosts of field 0 of plane z - 1, x ghosts of field 1 of plane z - 2
    auto load = [&](int z) {
      const double* up = ub + (size_t)min(max(z, 0), B + 1) * sz;
      const int q = z - 1, qc = min(max(q, 1), B);
      const double* qp = ub + (size_t)qc * sz;
      const double* fp = fbk + (size_t)qc * sz;
      const bool zghost = q < 1 || q > B;
      const double* gz = gb + (q < 1 ? 4 : 5) * BB;
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        if (!a.zero) {
          const Pair v = *reinterpret_cast<const Pair*>(up + ro[i] + gx);
          PU[i][0] = v.x;
          PU[i][1] = v.y;
        }
        const double* p = zghost ? gz + zo[i] + (gx - 1)
                          : ((ghost >> i) & 1u) ? gb + (gy + i == 0 ? 2 : 3) * BB + (size_t)(qc - 1) * B + (gx - 1)
                                                : fp + ro[i] + gx;
        const Pair v = *reinterpret_cast<const Pair*>(p);
        PF[i][0] = v.x;
        PF[i][1] = v.y;
      }
      if (first || last) {
        const double* g1 = gb + (first ? 0 : 1) * BB + (size_t)(min(max(z - 2, 1), B) - 1) * B;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
          if (!a.zero) PX0[i] = qp[ro[i] + (first ? 0 : B + 1)];
          PX1[i] = g1[min(max(gy + i, 1), B) - 1];
        }
      }
    };

    auto store = [&](int p) {
      if (p < z0 || p >= z1) return;
      double* op = ob + (size_t)p * sz;
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        if (!(active && ((own >> i) & 1u))) continue;
        *reinterpret_cast<Pair*>(op + ro[i] + gx) = Pair{OUT[i][0], OUT[i][1]};
      }
    };

    double sumsq = 0.0, RA = 0.0;  // kNorm; kRestrict: sum over the children so far
    const int Bc = B / 2, mc = Bc + 2;
    const int zend = z1 + H;
    int zl = max(z0 - H, 0);
    load(zl);
    auto body = [&](auto PC) -> bool {
      constexpr int P = decltype(PC)::value;
      constexpr int rb = (P + 1) & 1, wb = P & 1;
      constexpr int s0 = P % 3, s1 = imod(P - 1, 3), s2 = imod(P - 2, 3);  // planes zl, zl-1, zl-2
      constexpr int f1 = P & 1, f2 = (P + 1) & 1;                          // f of zl-1, zl-2
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        X0[i] = PX0[i];
        X1[i] = PX1[i];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          U[0][s0][i][o] = PU[i][o];
          F[f1][i][o] = PF[i][o];
          asm volatile("" : "+v"(U[0][s0][i][o]));
        }
      }
      __syncthreads();
      store(zl - 3);
      if (zl + 1 < zend) load(zl + 1);

      // residual at (i, o) of field j's centre plane, phase c (lo, hi: its z-neighbours; em, ep: the
      // adjacent row groups' edge rows)
      auto resid = [&](auto JC, auto CC, auto LC, auto HC, const double (&X)[RPW], double2 em, double2 ep,
                       double fv, int p, int i, int o) -> double {
        constexpr int j = decltype(JC)::value, c = decltype(CC)::value, lo = decltype(LC)::value,
                      hi = decltype(HC)::value;
        const double ui = U[j][c][i][o];
        const double below = from_lane_below(U[j][c][i][1]), above = from_lane_above(U[j][c][i][0]);
        double xm = o ? U[j][c][i][0] : first ? X[i] : below;
        double xp = o ? (last ? X[i] : above) : U[j][c][i][1];
        double ym = i > 0 ? U[j][c][i - 1][o] : (o ? em.y : em.x);
        double yp = i < RPW - 1 ? U[j][c][i + 1][o] : (o ? ep.y : ep.x);
        double zm = U[j][lo][i][o], zp = U[j][hi][i][o];
        if constexpr (COARSE) {
          // a domain-boundary ghost holds the face value: it enters as 2 g - u_i
          if (o == 0) xm = bx0 ? 2.0 * xm - ui : xm;
          if (o == 1) xp = bx1 ? 2.0 * xp - ui : xp;
          ym = by0 && gy + i == 1 ? 2.0 * ym - ui : ym;
          yp = by1 && gy + i == B ? 2.0 * yp - ui : yp;
          zm = bz0 && p == 1 ? 2.0 * zm - ui : zm;
          zp = bz1 && p == B ? 2.0 * zp - ui : zp;
        }
        double s = ui - xm;
        s = s + (ui - xp);
        s = s + (ui - ym);
        s = s + (ui - yp);
        s = s + (ui - zm);
        s = s + (ui - zp);
        return fv - s * ih2;
      };
      {
        const int p = zl - 1;
        const bool zghost = p < 1 || p > B;
        const double2 em = sh.e[rb][0][wm][1][lane], ep = sh.e[rb][0][wp][0][lane];
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
          for (int o = 0; o < 2; ++o) {
            const double fv = F[f1][i][o];
            const double r = resid(IC<0>{}, IC<s1>{}, IC<s2>{}, IC<s0>{}, X0, em, ep, fv, p, i, o);
            const double v = U[0][s1][i][o] + coef * r;
            U[1][s1][i][o] = zghost || ((ghost >> i) & 1u) ? fv : v;
            if constexpr (NORM) {
              const bool mine = active && ((own >> i) & 1u) && p >= z0 && p < z1;
              const double rr = mine ? r : 0.0;
              sumsq += rr * rr;
            }
          }
      }
      {
        const int p = zl - 2;
        const double2 em = sh.e[rb][1][wm][1][lane], ep = sh.e[rb][1][wp][0][lane];
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
          for (int o = 0; o < 2; ++o) {
            // field 1: planes zl-2 (centre), zl-3 and zl-1
            const double r = resid(IC<1>{}, IC<s2>{}, IC<s0>{}, IC<s1>{}, X1, em, ep, F[f2][i][o], p, i, o);
            if constexpr (RES) {
              RA = i == 0 && o == 0 && (p & 1) ? r : RA + r;
              OUT[i][o] = U[1][s2][i][o];
            } else {
              OUT[i][o] = U[1][s2][i][o] + coef * r;
            }
          }
        if constexpr (RES) {
          if (p >= z0 && p < z1 && !(p & 1) && active && (own & 1u))
            a.fc[(((size_t)b * mc + (p >> 1)) * mc + ((gy + 1) >> 1)) * mc + ((gx + 1) >> 1)] = 0.125 * RA;
        }
      }
      // edge rows of the next step's centres: plane zl of field 0, zl - 1 of field 1
      sh.e[wb][0][w][0][lane] = make_double2(U[0][s0][0][0], U[0][s0][0][1]);
      sh.e[wb][0][w][1][lane] = make_double2(U[0][s0][RPW - 1][0], U[0][s0][RPW - 1][1]);
      sh.e[wb][1][w][0][lane] = make_double2(U[1][s1][0][0], U[1][s1][0][1]);
      sh.e[wb][1][w][1][lane] = make_double2(U[1][s1][RPW - 1][0], U[1][s1][RPW - 1][1]);
      ++zl;
      return zl < zend;
    };
    auto round = [&]<int... Ps>(std::integer_sequence<int, Ps...>) {
      bool go = true;
      ((go = go && body(IC<Ps>{})), ...);
      return go;
    };
    while (round(std::make_integer_sequence<int, 6>{})) {
    }
    store(zl - 3);
    if constexpr (NORM) {
#pragma unroll
      for (int o2 = 32; o2 >= 1; o2 >>= 1) sumsq += __shfl_xor(sumsq, o2, 64);
      if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = sumsq;
      __syncthreads();
      if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int v = 0; v < W; ++v) tot += sh.red[v];
        a.partial[blockIdx.x] = tot;
      }
    }
  }
};

template <int LW, int W, int RPW, bool COARSE, int OUT_>
__global__ void __launch_bounds__(64 * W) k_blk_pair(PairArgs a)
{
  using C = PairPass<LW, W, RPW, COARSE, OUT_>;
  __shared__ typename C::Shared sh;
  // XCD-aware tile index: workgroup b runs on XCD b % 8, which gets a contiguous tile range
  const int n = blockIdx.x, nb = gridDim.x;
  const int xcd = n & 7, jb = n >> 3, q = nb >> 3, rem = nb & 7;
  const int t = (xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q) + jb;
  const int ty = t % a.tiles_y, tz = (t / a.tiles_y) % a.chunks, b = t / (a.tiles_y * a.chunks);
  const int z0 = 1 + tz * a.zlen;
  C::run(a, sh, b, 1 + ty * C::TY, z0, min(z0 + a.zlen, a.B + 1));
}

__global__ void __launch_bounds__(256)
    k_blk_pair_sum(const double* __restrict__ partial, int count, double* __restrict__ out)
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

#ifndef MG_BLKP_W
#define MG_BLKP_W 12
#endif
#ifndef MG_BLKP_RPW
#define MG_BLKP_RPW 2
#endif

template <int LW, bool COARSE, int OUT_>
void launch(hipStream_t s, PairArgs a, double* norm2)
{
  constexpr int W = MG_BLKP_W, RPW = MG_BLKP_RPW;
  using C = PairPass<LW, W, RPW, COARSE, OUT_>;
  a.tiles_y = (a.B + C::TY - 1) / C::TY;
  // z-chunks: as many as keep the critical path -- rounds of workgroups, one per compute unit, x
  // planes per workgroup -- shortest; of even length (plane pairs)
  const int per = kBlocks * a.tiles_y;
  long long best = -1;
  for (int zlen = 4; zlen <= a.B; zlen += 2) {
    const long long blocks = (long long)per * ((a.B + zlen - 1) / zlen);
    if (blocks > kBlkPartials) continue;
    const long long cost = (blocks + 255) / 256 * (zlen + 2 * C::H);
    if (best < 0 || cost <= best) {
      best = cost;
      a.zlen = zlen;
    }
  }
  a.chunks = (a.B + a.zlen - 1) / a.zlen;
  const int blocks = per * a.chunks;
  k_blk_pair<LW, W, RPW, COARSE, OUT_><<<blocks, 64 * W, 0, s>>>(a);
  if (OUT_ == kNorm) k_blk_pair_sum<<<1, 256, 0, s>>>(a.partial, blocks, norm2);
}

}  // namespace

bool blk_pair_supported(int B) { return B >= 64 && B <= 128; }

void blk_pair(hipStream_t s, int B, double omega, const int* faces, const double* hs, const double* f,
              const double* u, const double* g, double* out, double* fc, bool coarse, bool zero,
              double* partial, double* norm2)
{
  const PairArgs a{u, f, g, hs, faces, out, fc, partial, omega, B, 0, 0, B, zero};
  if (B == 64) {
    if (coarse && fc) launch<32, true, kRestrict>(s, a, nullptr);
    else if (coarse) launch<32, true, kSweeps>(s, a, nullptr);
    else if (fc) launch<32, false, kRestrict>(s, a, nullptr);
    else if (norm2) launch<32, false, kNorm>(s, a, norm2);
    else launch<32, false, kSweeps>(s, a, nullptr);
  } else {
    if (coarse && fc) launch<64, true, kRestrict>(s, a, nullptr);
    else if (coarse) launch<64, true, kSweeps>(s, a, nullptr);
    else if (fc) launch<64, false, kRestrict>(s, a, nullptr);
    else if (norm2) launch<64, false, kNorm>(s, a, norm2);
    else launch<64, false, kSweeps>(s, a, nullptr);
  }
}

}  // namespace mgk
