// MI355X (gfx950) implementation of the DDF-QE DVBM hot path and its C ABI.
//
// Kernels:
//   k_collide_advect*  one full time step of Eq. (finalDiscretePDE): moments,
//                     (quasi-)equilibria, two-time relaxation and NND flux
//                     divergence of every population, fused: the column sweep
//                     (_sweep) on large grids, plane groups (_planes) on
//                     smaller ones and with walls, one thread per cell with
//                     the stencils through the caches or, in _lds, LDS tiles.
//   k_adjoint*        one reverse step: one sweep over plane groups, or for
//                     deviation storage a relaxation part and a flux sweep.
//   k_init            equilibrium populations of macroscopic fields (Sec. III A 3).
//   k_moments         rho, u, T fields and per-block float64 conservation sums.
//   k_speed           per-block extrema of the initial fields (time step, checks).
//   k_reduce_*        deterministic final reductions of the per-block partials.
//   k_encode/k_decode dense float64 populations <-> storage format.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>

#include "../../include/dvbm.h"
#include "lattice.h"
#include "node.h"
#include "step.h"
#include "planes.h"
#include "sweep.h"
#include "adjoint.h"
#include "adjoint_planes.h"

namespace dvbm {

constexpr int RED_BLOCKS = 1024;
constexpr int RED_THREADS = 256;
// most blocks of a launch of the adjoint kernels that sum parameter
// derivatives (4 partial sums each, in the workspace)
constexpr int ADJ_BLOCKS = 1024;
static_assert(ADJ_BLOCKS <= RED_BLOCKS, "adjoint partials exceed the workspace");
// workspace layout (doubles): [0, 4 RED_BLOCKS) block partials, then the
// final reductions, then (at WS_TICKET) the adjoint's block counter
constexpr int WS_TICKET = 4 * RED_BLOCKS + 32;
// then, with walls in y, the 4 ghost rows of every population plane
constexpr int WS_GHOST = 4 * RED_BLOCKS + 64;
#ifndef DVBM_CELL_TX
#define DVBM_CELL_TX 64
#endif
#ifndef DVBM_CELL_TY
#define DVBM_CELL_TY 4
#endif
#ifndef DVBM_TILE_TX
#define DVBM_TILE_TX 64
#endif
#ifndef DVBM_TILE_TY
#define DVBM_TILE_TY 4
#endif
#ifndef DVBM_ORDER
#define DVBM_ORDER 0
#endif
constexpr int CELL_TX = DVBM_CELL_TX, CELL_TY = DVBM_CELL_TY;  // per-cell kernel workgroup tile
constexpr int TILE_TX = DVBM_TILE_TX, TILE_TY = DVBM_TILE_TY;  // LDS kernel tile

// Tile (bx, by) of linear workgroup w.  Consecutive workgroups are dealt
// round-robin to the 8 XCDs, each with its own L2.  ORDER 0 keeps the plain
// row-major order; ORDER 2 gives every XCD one contiguous range of tiles in
// column-major order, so that the tiles above and below a tile (which read
// its rows as ghost layers) run on the same XCD right after it.
__device__ inline void tile_of_block(int w, int nbx, int nby, int& bx, int& by) {
  if (DVBM_ORDER == 0) {
    bx = w % nbx;
    by = w / nbx;
    return;
  }
  const int total = nbx * nby;
  const int xcd = w % 8, k = w / 8, base = total / 8, rem = total % 8;
  const int t = xcd < rem ? xcd * (base + 1) + k : rem * (base + 1) + (xcd - rem) * base + k;
  bx = t / nby;
  by = t % nby;
}

// ------------------------------------------------------------ fused step
// At most two waves per SIMD: the cell's stencil loads (about 290) are then
// all issued ahead of their uses.  Left to aim at a higher occupancy, the
// compiler issues them a few at a time and waits for each group (measured 2.5x
// slower on 256^2 with the deviation formats).
template <int SPLIT, class S, int BCX, int BCY, int PRM>
__global__ __launch_bounds__(CELL_TX* CELL_TY) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_collide_advect(
    const typename S::T* __restrict__ src,
                                                                     typename S::T* __restrict__ dst, KParams kp,
                                                                     const typename S::T* __restrict__ ghost) {
  int bx, by;
  tile_of_block(blockIdx.x, (kp.nx + CELL_TX - 1) / CELL_TX, (kp.ny + CELL_TY - 1) / CELL_TY, bx, by);
  const int x = bx * CELL_TX + threadIdx.x;
  const int y = by * CELL_TY + threadIdx.y;
  if (x >= kp.nx || y >= kp.ny) return;
  cell_update<SPLIT, S, BCX, BCY, PRM>(src, dst, kp, x, y, ghost);
}

template <int SPLIT, class S, int BCX, int BCY, int PRM>
__global__ __launch_bounds__(TILE_TX* TILE_TY) void k_collide_advect_lds(const typename S::T* __restrict__ src,
                                                                         typename S::T* __restrict__ dst,
                                                                         KParams kp) {
  __shared__ PlaneTile<typename S::C, TILE_TX, TILE_TY, Set<SPLIT>::N1> lds;
  int bx, by;
  tile_of_block(blockIdx.x, (kp.nx + TILE_TX - 1) / TILE_TX, (kp.ny + TILE_TY - 1) / TILE_TY, bx, by);
  tile_update<SPLIT, S, BCX, BCY, PRM, TILE_TX, TILE_TY>(src, dst, kp, bx, by, lds);
}

// Plane-group kernel: workgroup b is logical (strip, row range) L, strips
// fastest, dealt so that every XCD gets one contiguous range of L (neighbouring
// ranges read each other's edge rows from the XCD's L2).  Two workgroups fit a
// CU in 32/16-bit storage with the registers capped at 80, a few of them spilled
// (f32_dev, uncapped at 88 registers and one workgroup / capped: 256^2 9.46 /
// 9.43 us, 512^2 24.2 / 23.6, but 800^2 49.1 / 53.3); float64 needs 153 registers and
// runs one.
template <class S>
constexpr int planes_wpe() {
  return sizeof(typename S::T) == 8 ? 3 : 6;
}
template <int SPLIT>
constexpr int planes_threads() {
  return 128 * (Set<SPLIT>::N1 + 1);
}
__device__ inline void strip_range(int ny, int nstrips, int nranges, int blk, int& strip, int& ya, int& yb) {
  const int nb = nstrips * nranges;
  const int xcd = blk % 8, k = blk / 8, base = nb / 8, rem = nb % 8;
  const int L = xcd < rem ? xcd * (base + 1) + k : rem * (base + 1) + (xcd - rem) * base + k;
  const int j = int(unsigned(L) / unsigned(nstrips));
  strip = L - j * nstrips;
  // nranges ranges of ny / nranges rows, the first ny % nranges of them one longer
  const int rows = int(unsigned(ny) / unsigned(nranges)), longer = ny - rows * nranges;
  ya = j * rows + (j < longer ? j : longer);
  yb = ya + rows + (j < longer ? 1 : 0);
}
// Role of a wave: plane waves of f (a), of g (N1 + a), then the two coefficient
// waves.  With N1 = 5 the waves of one SIMD (every fourth) get f 0, g 0, f 2;
// f 1, g 1, g 2; f 3, g 3 and the second coefficient wave; f 4, g 4 and the
// first: with the planes of xi = 0 (no x flux) and the coefficients spread, the four
// carry within 6 % of the mean; in plain order one carries 20 % more.
template <int N1>
__device__ inline int wave_role() {
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / 64);
  return N1 == 5 ? int(0xAB7298654310ull >> (4 * w)) & 15 : w;
}
// f(integral_constant PRM) for a Prandtl mode known at run time: only the
// coefficient waves depend on it, so the kernel is not instantiated per mode.
template <class F>
__host__ __device__ inline void with_pr_mode(int prm, F&& f) {
  if (prm == PR_UNIT) f(std::integral_constant<int, PR_UNIT>());
  else if (prm == PR_LOW) f(std::integral_constant<int, PR_LOW>());
  else f(std::integral_constant<int, PR_HIGH>());
}
template <int SPLIT, class S, int BCX, int BCY>
__global__ __launch_bounds__(planes_threads<SPLIT>()) __attribute__((amdgpu_waves_per_eu(planes_wpe<S>()))) void
k_collide_advect_planes(const typename S::T* __restrict__ src, typename S::T* __restrict__ dst, KParams kp,
                        int nstrips, int nranges, int prm) {
  constexpr int N1 = Set<SPLIT>::N1;
  __shared__ PlanesShared<SPLIT, typename S::C, BCY == BC_WALL> sh;
  int strip, ya, yb;
  strip_range(kp.ny, nstrips, nranges, int(blockIdx.x), strip, ya, yb);
  const int x0 = strip * SWEEP_OWN;
  const int w = wave_role<N1>();
  const auto coeffs = [&](auto d) {
    constexpr int D = decltype(d)::value;
    if constexpr (BCY == BC_WALL) {  // the ghost rows that this range reads
      if (ya < 2) wall_coeffs<SPLIT, S, D>(kp, 0, sh);
      if (yb > kp.ny - 2) wall_coeffs<SPLIT, S, D>(kp, 1, sh);
    }
    with_pr_mode(prm, [&](auto m) { planes_coeffs<SPLIT, S, decltype(m)::value, D>(kp, yb - ya, sh); });
  };
  if (w < N1)
    planes_walk<SPLIT, S, BCX, BCY, 0>(src, dst, kp, w, x0, ya, yb, sh);
  else if (w < 2 * N1)
    planes_walk<SPLIT, S, BCX, BCY, 1>(src, dst, kp, w - N1, x0, ya, yb, sh);
  else if (w == 2 * N1)
    coeffs(std::integral_constant<int, 0>());
  else
    coeffs(std::integral_constant<int, 1>());
}

// Row range j of kseg in a column of ny rows for the column sweep: ranges of
// u m rows (m >= 1, u m <= ny; u is the ring size of the sweep) from the
// top; the last one is moved up so that it ends at row ny and may overlap its
// predecessor (rows computed by both ranges get identical values).
// Requires ny >= u and kseg = the count sweep_ranges returns.
__host__ __device__ inline int sweep_len(int ny, int want, int u) {
  int len = u * ((ny + u * want - 1) / (u * want));
  const int cap = u * (ny / u);
  return len < cap ? len : cap;
}
__device__ inline void sweep_range(int ny, int kseg, int j, int u, int& ya, int& yb) {
  const int len = sweep_len(ny, kseg, u);
  ya = j * len;
  if (ya > ny - len) ya = ny - len;
  yb = ya + len;
}

// Column sweep: workgroups of 2 K waves, wave w advancing distribution
// w / K (0: f, 1: g) of strip sg * K + w % K; workgroup b is logical (strip
// group, row range) L, dealt so that every XCD gets one contiguous range of
// L; L = j * ngroups + sg covers strip group sg, row range j.  K is 4 for
// 32/16-bit storage (two waves per SIMD).  Float64 windows need about 370
// registers, so float64 storage runs one wave per SIMD and K = 2: the same
// bytes in flight per CU.
#ifndef DVBM_SWEEP_WPE
#define DVBM_SWEEP_WPE 2
#endif
// Below this many cells a grid has too few strip groups x row ranges to
// occupy the device with the column sweep, and the plane-group kernel is
// faster.  us per step, planes / sweep:
//   25 populations  float64 900^2 155 / 162, 1024^2 197 / 197, 3001 x 1499 821 / 795;
//                   32-bit 900^2 83.7 / 85.8, 1024^2 115 / 100, 4096^2 1590 / 1446;
//                   16-bit 1024^2 64.6 / 70.4, 1500 x 1100 117 / 115
//   16 populations  float64 1024^2 119 / 122, 2048^2 472 / 498, 4096^2 1757 / 1943 (two workgroups per CU fit);
//                   32-bit 1500 x 1000 99.6 / 104, 2048 x 1024 137 / 124;
//                   16-bit 2048 x 1024 87 / 97, 2048^2 181 / 183
// Grids whose strips fill the sweep's groups of four leave the planes of 32-bit
// storage earlier, narrow ones (at most 12 strips) most:
//   25 populations  235 x 3702 104 / 92.3, 715 x 1216 95.7 / 85.7, 2160 x 402 89.9 / 86.0 (1000 x 900, 17 strips, 98.3 / 103);
//   16 populations  deviations 480 x 2145 74.8 / 67.2, 1440 x 1041 97.6 / 90.6; values 480 x 2145 75.1 / 70.2,
//                   1440 x 1041 97.1 / 96.0, 2160 x 694 97.6 / 102 (1500 x 1000, 25 strips, 98.7 / 105)
template <int SPLIT>
__host__ constexpr int64_t sweep_min_cells(int storage, int nstrips) {
  const bool full = nstrips % SWEEP_K == 0, narrow = full && nstrips <= 12;
  if (storage == DVBM_F64) return SPLIT == 2 ? 15 << 16 : INT64_MAX;
  if (storage == DVBM_BF16_DEV || storage == DVBM_FP16_DEV) return SPLIT == 2 ? 9 << 17 : 1 << 22;
  return SPLIT == 2 ? (narrow ? 6 << 17 : full ? 13 << 16 : 7 << 17)
                    : (narrow ? 31 << 15 : full && storage == DVBM_F32_DEV ? 43 << 15 : 3 << 19);
}
// 61 to 64 columns take the plane groups two strips, the second nearly empty;
// the per-cell kernel runs them one wave a row, its workgroups of four rows two
// per CU: 2048 rows at a time.  It is the faster one just below that and, with
// many rows, in 16 bits.  us per step of 64 columns, planes / cells:
//   25 populations  16 bits 1400 rows 13.4 / 14.9, 2048 16.9 / 14.8, 2200 17.8 / 20.8, 3000 22.1 / 21.6, 4096 28.5 / 26.5,
//                   11000 71.1 / 64.4; 32 bits 1000 12.1 / 11.1, 1100 12.3 / 14.2, 2048 17.4 / 16.5, 2200 18.9 / 22.3,
//                   4096 29.6 / 29.4, 8192 53.3 / 55.7, 11000 85.6 / 76.2
//   16 populations  16 bits 2048 13.2 / 13.2, 2200 14.2 / 17.4, 3000 17.5 / 16.6, 4096 22.3 / 20.2, 11000 52.5 / 48.1;
//                   32 bits 2000 13.8 / 12.8, 2200 14.2 / 17.2, 4096 21.2 / 22.0, 11000 49.8 / 51.2
// Float64 favours the planes.
template <int SPLIT>
__host__ constexpr bool cells_for_64_columns(int bytes, int ny) {
  if (bytes == 8) return false;
  if (bytes == 2) return ny >= 3000 || (SPLIT == 2 && ny > 1800 && ny <= 2048);
  return (ny > 1800 && ny <= 2048) || (SPLIT == 2 && ((ny > 900 && ny <= 1024) || ny >= 10000));
}
#ifndef DVBM_SWEEP_K64
#define DVBM_SWEEP_K64 2  // strips per workgroup, float64 storage
#endif
#ifndef DVBM_SWEEP_WPE64
#define DVBM_SWEEP_WPE64 1
#endif
template <class S>
constexpr int sweep_k() {
  return sizeof(typename S::T) == 8 ? DVBM_SWEEP_K64 : SWEEP_K;
}
template <class S>
constexpr int sweep_wpe() {
  return sizeof(typename S::T) == 8 ? DVBM_SWEEP_WPE64 : DVBM_SWEEP_WPE;
}
#ifndef DVBM_SWEEP_RING64
#define DVBM_SWEEP_RING64 DVBM_SWEEP_RING
#endif
// rows per plane in the sweep's register ring (the row ranges are multiples of it)
template <class S>
constexpr int sweep_ring() {
  return sizeof(typename S::T) == 8 ? DVBM_SWEEP_RING64 : DVBM_SWEEP_RING;
}
template <int SPLIT, class S, int BCX, int BCY, int PRM>
__global__ __launch_bounds__(128 * sweep_k<S>()) __attribute__((amdgpu_waves_per_eu(sweep_wpe<S>()))) void
k_collide_advect_sweep(const typename S::T* __restrict__ src, typename S::T* __restrict__ dst, KParams kp,
                       int ngroups, int kseg) {
  constexpr int SWEEP_K = sweep_k<S>();
  constexpr int RING = sweep_ring<S>();
  __shared__ SweepShared sh[SWEEP_K];
  const int total = ngroups * kseg;
  const int per = (total + 7) / 8;
  const int L = int(blockIdx.x % 8) * per + int(blockIdx.x / 8);
  if (L >= total) return;
  const int j = L / ngroups, sg = L % ngroups;
  int ya, yb;
  sweep_range(kp.ny, kseg, j, RING, ya, yb);
  const int w = int(threadIdx.x) / 64, k = w % SWEEP_K;
  const int x0 = (sg * SWEEP_K + k) * SWEEP_OWN;  // may lie beyond nx: then the wave stores nothing
  if (w < SWEEP_K)
    sweep_update<SPLIT, S, BCX, BCY, PRM, 0, RING>(src, dst, kp, x0, ya, yb, sh[k]);
  else
    sweep_update<SPLIT, S, BCX, BCY, PRM, 1, RING>(src, dst, kp, x0, ya, yb, sh[k]);
}

// ------------------------------------------------------------ equilibrium initialisation
template <int SPLIT, class S>
__global__ __launch_bounds__(256) void k_init(const double* __restrict__ rho, const double* __restrict__ ux,
                                              const double* __restrict__ uy, const double* __restrict__ T,
                                              typename S::T* __restrict__ dst, KParams kp) {
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  const int64_t n = int64_t(kp.nx) * kp.ny;
  for (int64_t c = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; c < n; c += int64_t(gridDim.x) * blockDim.x) {
    const int y = int(c / kp.nx), x = int(c % kp.nx);
    const double r = rho[c], t = T[c];
    const double isc = 1.0 / sqrt(kp.c2);
    const double vx = ux[c] * isc, vy = uy[c] * isc;  // normalised velocity
    const double RT = kp.R * t, th = RT / kp.c2, p = r * RT;
    const double E = r * kp.Cv * t + 0.5 * r * kp.c2 * (vx * vx + vy * vy);
    double mx[5], my[5];
    gauss_hermite_moments(vx, th - 1.0, mx);
    gauss_hermite_moments(vy, th - 1.0, my);
    double bf[5][5], bg[3][3];
    constexpr int NF = Set<SPLIT>::NF;
    for (int a = 0; a <= NF; ++a)
      for (int b = 0; a + b <= NF; ++b) bf[a][b] = r * mx[a] * my[b];
    if (SPLIT == 2) {
      const double e = r * (kp.Cv - kp.R) * t;
      for (int a = 0; a <= 2; ++a)
        for (int b = 0; a + b <= 2; ++b) bg[a][b] = e * mx[a] * my[b];
    } else {
      const double diag = (E + p) * th - E;
      bg[0][0] = E;
      bg[1][0] = vx * (E + p);
      bg[0][1] = vy * (E + p);
      bg[2][0] = (E + 2.0 * p) * vx * vx + diag;
      bg[1][1] = (E + 2.0 * p) * vx * vy;
      bg[0][2] = (E + 2.0 * p) * vy * vy + diag;
    }
    double f[Q], g[Q];
    for (int i = 0; i < Q; ++i) f[i] = g[i] = 0.0;
    expand_add<N1, NF>(bf, f);
    expand_add<N1, 2>(bg, g);
    for (int i = 0; i < Q; ++i) {
      const double w = weight<SPLIT>(i);
      using C = typename S::C;
      dst[sidx(kp, 0, i, y, x)] = S::enc64(f[i], w, 1.0);
      dst[sidx(kp, 1, i, y, x)] = S::enc64(g[i], w, g_ref_over_w<SPLIT>(kp, i));
    }
  }
}

// ------------------------------------------------------------ dense <-> storage
template <int SPLIT, class S>
__device__ inline double decode_one(const typename S::T v, int d, int i, const KParams& kp) {
  if (!S::dev) return double(S::raw(v));
  const double w = weight<SPLIT>(i);
  const double r = d == 0 ? 1.0 : g_ref_over_w<SPLIT>(kp, i);
  return w * (r + double(S::raw(v)));
}

// ------------------------------------------------------------ no-slip walls
// Ghost rows of the walls below row 0 and above row ny-1 (thermal Couette
// flow, Sec. IV): the ghost row k = 1, 2 rows away from a wall takes the
// fields of interior row k reflected through the wall values (rho_G = rho_B,
// u_G = 2 u_W - u_B, T_G = 2 T_W - T_B) and the populations
// X^eq(G) + (X_B - X^eq(B)), encoded in the storage format.
// ghost[(d Q + i) 4 + r][x] (row stride pitch), r = 0..3 for the rows -2, -1,
// ny, ny+1; one thread per (x, r).  For the per-cell kernel; the plane-group
// kernel forms its ghost rows itself.
template <int SPLIT, class S>
__global__ __launch_bounds__(256) void k_wall_ghosts(const typename S::T* __restrict__ src,
                                                     typename S::T* __restrict__ ghost, KParams kp) {
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  using C = typename S::C;
  const int t = int(blockIdx.x * blockDim.x + threadIdx.x);
  if (t >= 4 * kp.nx) return;
  const int r = t / kp.nx, x = t - r * kp.nx;
  const int yb = r == 0 ? 1 : (r == 1 ? 0 : (r == 2 ? kp.ny - 1 : kp.ny - 2));
  const int wall = r < 2 ? 0 : 1;
  double f[Q], g[Q];
  for (int i = 0; i < Q; ++i) {
    f[i] = decode_one<SPLIT, S>(src[sidx(kp, 0, i, yb, x)], 0, i, kp);
    g[i] = decode_one<SPLIT, S>(src[sidx(kp, 1, i, yb, x)], 1, i, kp);
  }
  // the boundary cell's rho, u, T (Eqs. eq_quadratur1-3 and eq:Total_energy_MB)
  const NodeMoments m = node_moments<N1>(f, g);
  const double c = sqrt(kp.c2);
  const double rho = m.rho, ux = c * m.jx / rho, uy = c * m.jy / rho;
  const double E = SPLIT == 2 ? m.g0 + 0.5 * kp.c2 * (m.pxx + m.pyy) : m.g0;
  const double T = (E / rho - 0.5 * (ux * ux + uy * uy)) * kp.inv_Cv;
  double feqB[Q], geqB[Q], feqG[Q], geqG[Q];
  equilibrium_cell<SPLIT, double>(rho, ux, uy, T, kp, feqB, geqB);
  equilibrium_cell<SPLIT, double>(rho, 2.0 * kp.wall_ux[wall] - ux, -uy, 2.0 * kp.wall_T[wall] - T, kp, feqG, geqG);
  for (int i = 0; i < Q; ++i) {
    const double w = weight<SPLIT>(i);
    ghost[(int64_t(i) * 4 + r) * kp.pitch + x] = S::enc64(feqG[i] + (f[i] - feqB[i]), w, 1.0);
    ghost[(int64_t(Q + i) * 4 + r) * kp.pitch + x] =
        S::enc64(geqG[i] + (g[i] - geqB[i]), w, g_ref_over_w<SPLIT>(kp, i));
  }
}

template <int SPLIT, class S>
__global__ __launch_bounds__(256) void k_decode(const typename S::T* __restrict__ src, double* __restrict__ X,
                                                KParams kp) {
  constexpr int Q = Set<SPLIT>::Q;
  const int64_t cells = int64_t(kp.nx) * kp.ny, n = 2 * Q * cells;
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const int di = int(k / cells);
    const int64_t c = k % cells;
    const int y = int(c / kp.nx), x = int(c % kp.nx);
    X[k] = decode_one<SPLIT, S>(src[sidx(kp, di / Q, di % Q, y, x)], di / Q, di % Q, kp);
  }
}

template <int SPLIT, class S>
__global__ __launch_bounds__(256) void k_encode(const double* __restrict__ X, typename S::T* __restrict__ dst,
                                                KParams kp) {
  constexpr int Q = Set<SPLIT>::Q;
  using C = typename S::C;
  const int64_t cells = int64_t(kp.nx) * kp.ny, n = 2 * Q * cells;
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const int di = int(k / cells), d = di / Q, i = di % Q;
    const int64_t c = k % cells;
    const int y = int(c / kp.nx), x = int(c % kp.nx);
    const double w = weight<SPLIT>(i);
    const double r = d == 0 ? 1.0 : g_ref_over_w<SPLIT>(kp, i);
    dst[sidx(kp, d, i, y, x)] = S::enc64(X[k], w, r);
  }
}

// ------------------------------------------------------------ diagnostics
// Block tree reduction of 4 doubles (sum or max/min per lane of `mode`).
__device__ inline void block_reduce4(double (&v)[4], const int (&mode)[4], double* out) {
  __shared__ double sh[4][RED_THREADS];
  const int t = threadIdx.x;
  for (int k = 0; k < 4; ++k) sh[k][t] = v[k];
  __syncthreads();
  for (int s = RED_THREADS / 2; s > 0; s >>= 1) {
    if (t < s) {
      for (int k = 0; k < 4; ++k) {
        const double a = sh[k][t], b = sh[k][t + s];
        sh[k][t] = mode[k] == 0 ? a + b : (mode[k] > 0 ? fmax(a, b) : fmin(a, b));
      }
    }
    __syncthreads();
  }
  if (t == 0)
    for (int k = 0; k < 4; ++k) out[k] = sh[k][0];
}

template <int SPLIT, class S>
__global__ __launch_bounds__(RED_THREADS) void k_moments(const typename S::T* __restrict__ src, KParams kp,
                                                         double* rho_o, double* ux_o, double* uy_o, double* T_o,
                                                         double* partials) {
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  const int64_t n = int64_t(kp.nx) * kp.ny;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const double c = sqrt(kp.c2);
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const int y = int(k / kp.nx), x = int(k % kp.nx);
    double f[Q], g[Q];
    for (int i = 0; i < Q; ++i) {
      f[i] = decode_one<SPLIT, S>(src[sidx(kp, 0, i, y, x)], 0, i, kp);
      g[i] = decode_one<SPLIT, S>(src[sidx(kp, 1, i, y, x)], 1, i, kp);
    }
    const NodeMoments m = node_moments<N1>(f, g);
    const double rho = m.rho, jx = c * m.jx, jy = c * m.jy;
    const double E = SPLIT == 2 ? m.g0 + 0.5 * kp.c2 * (m.pxx + m.pyy) : m.g0;
    const double ux = jx / rho, uy = jy / rho;
    const double T = (E / rho - 0.5 * (ux * ux + uy * uy)) * kp.inv_Cv;
    if (rho_o) rho_o[k] = rho;
    if (ux_o) ux_o[k] = ux;
    if (uy_o) uy_o[k] = uy;
    if (T_o) T_o[k] = T;
    acc[0] += rho;
    acc[1] += jx;
    acc[2] += jy;
    acc[3] += E;
  }
  const int mode[4] = {0, 0, 0, 0};
  block_reduce4(acc, mode, partials + 4 * blockIdx.x);
}

#ifndef DVBM_PART  // non-template kernel: main unit only
__global__ __launch_bounds__(RED_THREADS) void k_speed(const double* __restrict__ rho, const double* __restrict__ ux,
                                                       const double* __restrict__ uy, const double* __restrict__ T,
                                                       int64_t n, double gR, double R, double* partials) {
  // lanes: max(|u| + c_s), max(p), -min(rho), -min(T); non-finite input poisons the lane with NaN->+inf
  double v[4] = {0.0, 0.0, -INFINITY, -INFINITY};
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const double r = rho[k], t = T[k], a = ux[k], b = uy[k];
    double s = sqrt(a * a + b * b) + sqrt(gR * fmax(t, 0.0));
    double p = r * R * t;
    if (!(s == s) || !(p == p) || !isfinite(s) || !isfinite(p)) s = p = INFINITY;
    v[0] = fmax(v[0], s);
    v[1] = fmax(v[1], p);
    v[2] = fmax(v[2], (r == r) ? -r : INFINITY);
    v[3] = fmax(v[3], (t == t) ? -t : INFINITY);
  }
  const int mode[4] = {1, 1, 1, 1};
  block_reduce4(v, mode, partials + 4 * blockIdx.x);
}
#endif

#ifndef DVBM_PART  // non-template kernel: main unit only
__global__ __launch_bounds__(RED_THREADS) void k_reduce(const double* __restrict__ partials, int nblocks, int modesel,
                                                        double* out) {
  double v[4];
  int mode[4];
  for (int k = 0; k < 4; ++k) {
    mode[k] = modesel;
    v[k] = modesel == 0 ? 0.0 : -INFINITY;
  }
  for (int b = threadIdx.x; b < nblocks; b += blockDim.x)
    for (int k = 0; k < 4; ++k) v[k] = modesel == 0 ? v[k] + partials[4 * b + k] : fmax(v[k], partials[4 * b + k]);
  block_reduce4(v, mode, out);
}
#endif

// ------------------------------------------------------------ adjoint
// Adds n waves' per-lane sums of (d/dtau_ref, d/dPr) to dparams (nothing when it
// is NULL): wave `slot` of a launch leaves its sum in partials[2 slot], and the
// last one to finish (counted in *ticket, which it resets) adds them in that
// order.
__device__ inline void add_params(double (&acc)[2], int slot, int n, double* partials, unsigned* ticket, double* dparams) {
  if (!dparams) return;
  const int lane = int(threadIdx.x & 63);
  auto wave_sum = [&](double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
  };
  acc[0] = wave_sum(acc[0]);
  acc[1] = wave_sum(acc[1]);
  // The sums are stored and read at device scope, so the count needs only
  // their completion before it; a __threadfence would write every dirty line
  // of the L2 back first (256^2: 45 us with it, 28 us without).
  unsigned before = 0;
  if (lane == 0) {
    __hip_atomic_store(partials + 2 * slot, acc[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(partials + 2 * slot + 1, acc[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    before = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__builtin_amdgcn_readfirstlane(int(before)) != n - 1) return;
  asm volatile("" ::: "memory");
  const double d0 = dparams[0], d1 = dparams[1];
  double v[2] = {0.0, 0.0};
  for (int b0 = lane; b0 < n; b0 += 64 * 8) {  // eight loads in flight at a time
    double t[8][2];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      for (int j = 0; j < 2; ++j) {
        const int b = b0 + 64 * u;
        t[u][j] = __hip_atomic_load(partials + 2 * (b < n ? b : n - 1) + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      for (int j = 0; j < 2; ++j) v[j] += b0 + 64 * u < n ? t[u][j] : 0.0;
  }
  v[0] = wave_sum(v[0]);
  v[1] = wave_sum(v[1]);
  if (lane == 0) {
    dparams[0] = d0 + v[0];
    dparams[1] = d1 + v[1];
    *ticket = 0u;
  }
}

// Adjoint step, flux part: four waves per workgroup; workgroups are dealt
// so that every XCD gets one contiguous range of waves.  Wave w takes the
// plane group w % (2 N1) (distribution d, abscissa xi_a), the strip
// (w / 2 N1) % nstrips and the row range ch * (w / (2 N1 nstrips)), so the
// 2 N1 groups of the same cells share the work rows in one L2.
#ifndef DVBM_ADJ_WAVES
#define DVBM_ADJ_WAVES 4096  // waves the flux-adjoint launch aims for
#endif
#ifndef DVBM_ADJ_CH_MIN
#define DVBM_ADJ_CH_MIN 8  // fewest rows per wave (each range walks two rows more)
#endif
template <int SPLIT, class S, int BCX, int BCY, class LT>
__global__ __launch_bounds__(256) void k_adjoint_flux(const typename S::T* __restrict__ state,
                                                      const LT* __restrict__ lam1,
                                                      const double* __restrict__ work, LT* __restrict__ lam0,
                                                      KParams kp, int nstrips, int ch, int nchunks) {
  constexpr int N1 = Set<SPLIT>::N1;
  const int nb = int(gridDim.x), blk = int(blockIdx.x);
  const int xcd = blk % 8, k = blk / 8, base = nb / 8, rem = nb % 8;
  const int lb = xcd < rem ? xcd * (base + 1) + k : rem * (base + 1) + (xcd - rem) * base + k;
  const int w = lb * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) / 64);
  const int g = w % (2 * N1), rest = w / (2 * N1);
  const int strip = rest % nstrips, chunk = rest / nstrips;
  if (chunk >= nchunks) return;
  const int ya = chunk * ch, yb = ya + ch < kp.ny ? ya + ch : kp.ny;
  if (g < N1)
    sweep_adjoint_flux<SPLIT, S, BCX, BCY, 0, LT>(state, lam1, work, lam0, kp, g, strip * ADJ_STRIP, ya, yb);
  else
    sweep_adjoint_flux<SPLIT, S, BCX, BCY, 1, LT>(state, lam1, work, lam0, kp, g - N1, strip * ADJ_STRIP, ya, yb);
}

// Adjoint step in one sweep: workgroup b is logical (strip, row range) first + b, dealt as
// in the plane-group step kernel, with the same roles of the waves.  When
// dparams != NULL the two coefficient waves of every workgroup leave their
// sums of (d/dtau_ref, d/dPr) in partials[2 (2 b + k)], and the last wave to
// finish (counted in *ticket, which it resets) adds them, in that order, to
// dparams.
// Against the two kernels it replaces (a relaxation kernel per cell that wrote
// the moment cotangents to memory, and a flux sweep that read X, lam' and
// them again: 2570 bytes per cell in float64), X and lam' are read and lam is written
// once: 1200 bytes per cell plus the ranges' edge rows.  us per step, before /
// after: float64 64^2 26.7 / 13.0, 256^2 46.2 / 29.6, 1024^2 639 / 284
// (4.8 TB/s with the edges, of 5.7 for a copy); 16 populations 1024^2
// 465 / 190; float32, float32 cotangents 2048^2 1596 / 848.
// At 256^2 the edges count: 9 rows are read for 5 written.
template <int SPLIT, class S, int BCX, int BCY, class LT>
__global__ __launch_bounds__(planes_threads<SPLIT>()) __attribute__((amdgpu_waves_per_eu(3))) void k_adjoint(
    const typename S::T* __restrict__ state, const LT* __restrict__ lam1, LT* __restrict__ lam0, KParams kp,
    int nstrips, int nranges, int first, int prm, double tau_ref, double* partials,
    unsigned* ticket, double* dparams) {
  constexpr int N1 = Set<SPLIT>::N1;
  __shared__ AdjointShared<SPLIT> sh;
  int strip, ya, yb;
  strip_range(kp.ny, nstrips, nranges, first + int(blockIdx.x), strip, ya, yb);
  const int x0 = strip * SWEEP_OWN, w = wave_role<N1>();
  const auto walk = [&](auto d, int a) {
    constexpr int D = decltype(d)::value;
    if (N1 == 4 || a != N1 / 2) adjoint_walk<SPLIT, S, BCX, BCY, D, true, LT>(state, lam1, lam0, kp, a, x0, ya, yb, sh);
    else adjoint_walk<SPLIT, S, BCX, BCY, D, false, LT>(state, lam1, lam0, kp, a, x0, ya, yb, sh);
  };
  if (w < N1) {
    walk(std::integral_constant<int, 0>(), w);
  } else if (w < 2 * N1) {
    walk(std::integral_constant<int, 1>(), w - N1);
  } else {
    const int k = w - 2 * N1, lane = int(threadIdx.x & 63);
    double acc[2] = {0.0, 0.0};
    __builtin_amdgcn_s_setprio(2);
    const bool mine = lane >= 2 && lane < 62 && x0 - 2 + lane < kp.nx;
    auto own = [&](int) { return mine; };
    auto out = [&](int, const double* mbar, double keep) {
#pragma unroll
      for (int j = 0; j < N_MOMENTS; ++j) sh.res[k][j][lane] = mbar[j];
      sh.res[k][N_MOMENTS][lane] = keep;
    };
    with_pr_mode(prm, [&](auto m) {
      adjoint_coeffs<SPLIT, decltype(m)::value>(kp, k, yb - ya, tau_ref, sh, acc[0], acc[1], own, out);
    });
    add_params(acc, 2 * int(blockIdx.x) + k, 2 * int(gridDim.x), partials, ticket, dparams);
  }
}

// Relaxation part of the deviation storage on small grids: workgroup b takes
// the cells 64 b .. 64 b + 63, with the roles of the one-sweep kernel; the first
// coefficient wave writes their work rows.  Bound by the chain of one cell, which
// by one thread runs 1300 to 1500 vector instructions behind 100 loads.
template <int SPLIT, class S, class LT>
__global__ __launch_bounds__(planes_threads<SPLIT>()) __attribute__((amdgpu_waves_per_eu(3))) void k_adjoint_relax(
    const typename S::T* __restrict__ state, const LT* __restrict__ lam1, double* __restrict__ work, KParams kp,
    int prm, double tau_ref, double* partials, unsigned* ticket, double* dparams) {
  constexpr int N1 = Set<SPLIT>::N1;
  __shared__ AdjointShares<SPLIT> sh;
  const int cells = kp.nx * kp.ny, c0 = 64 * int(blockIdx.x), w = wave_role<N1>();
  if (w < N1) {
    relax_walk<SPLIT, S, 0, LT>(state, lam1, kp, w, c0, sh);
  } else if (w < 2 * N1) {
    relax_walk<SPLIT, S, 1, LT>(state, lam1, kp, w - N1, c0, sh);
  } else {
    const int k = w - 2 * N1, lane = int(threadIdx.x & 63);
    double acc[2] = {0.0, 0.0};
    auto own = [&](int) { return c0 + lane < cells; };
    auto out = [&](int, const double* mbar, double keep) {
      if (c0 + lane >= cells) return;
#pragma unroll
      for (int j = 0; j < N_MOMENTS; ++j) work[int64_t(j) * cells + c0 + lane] = mbar[j];
      work[int64_t(N_MOMENTS) * cells + c0 + lane] = keep;
    };
    with_pr_mode(prm, [&](auto m) {
      adjoint_coeffs<SPLIT, decltype(m)::value>(kp, k, 1, tau_ref, sh, acc[0], acc[1], own, out);
    });
    if (k == 0) add_params(acc, int(blockIdx.x), int(gridDim.x), partials, ticket, dparams);
  }
}

// The same by one thread per cell (grid-stride), for all other grids: beyond one
// workgroup of the plane waves per CU it keeps more loads in flight.  Adjoint step
// of float32 deviations with float32 lam', us per step, plane waves / cells: 64^2
// 22.2 / 23.8, 100^2 23.7 / 24.1, 128^2 25.0 / 24.5, 150 x 128 27.9 / 24.8, 256^2 43.5 / 34.9
// (two and more cells to a lane in turn: 333 x 250 42.3 / 38.2, 1024^2 413 / 387, 2048^2
// 1673 / 1558); without parameter sums 128^2 20.9 / 22.5, 150 x 128 23.7 / 22.9.
constexpr int ADJ_RELAX_CELLS = 16384;  // most cells of the plane waves' kernel
template <int SPLIT, class S, int PRM, class LT>
__global__ __launch_bounds__(RED_THREADS) void k_adjoint_relax_cells(const typename S::T* __restrict__ state,
                                                                     const LT* __restrict__ lam1,
                                                                     double* __restrict__ work, KParams kp,
                                                                     double tau_ref, double* partials,
                                                                     unsigned* ticket, double* dparams) {
  const int cells = kp.nx * kp.ny;
  double acc[2] = {0.0, 0.0};
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < cells; c += gridDim.x * blockDim.x)
    cell_adjoint_relax<SPLIT, S, PRM, LT>(state, lam1, work, kp, c, tau_ref, acc[0], acc[1]);
  if (!dparams) return;
  __shared__ double sums[2][RED_THREADS];
  const int t = int(threadIdx.x);
  sums[0][t] = acc[0];
  sums[1][t] = acc[1];
  __syncthreads();
  if (t >= 64) return;
  for (int j = 0; j < 2; ++j) acc[j] = (sums[j][t] + sums[j][t + 64]) + (sums[j][t + 128] + sums[j][t + 192]);
  static_assert(RED_THREADS == 256, "four waves");
  add_params(acc, int(blockIdx.x), int(gridDim.x), partials, ticket, dparams);
}

template <int SPLIT, class S>
__global__ __launch_bounds__(256) void k_adjoint_readout(const typename S::T* __restrict__ state,
                                                         const double* rb, const double* uxb, const double* uyb,
                                                         const double* Tb, double* __restrict__ lam, KParams kp) {
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  const int64_t n = int64_t(kp.nx) * kp.ny;
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const int y = int(k / kp.nx), x = int(k % kp.nx);
    double f[Q], g[Q], lf[Q], lg[Q];
    for (int i = 0; i < Q; ++i) {
      f[i] = decode_one<SPLIT, S>(state[sidx(kp, 0, i, y, x)], 0, i, kp);
      g[i] = decode_one<SPLIT, S>(state[sidx(kp, 1, i, y, x)], 1, i, kp);
    }
    const NodeMoments m = node_moments<N1>(f, g);
    readout_adjoint_cell<SPLIT>(m, kp, rb ? rb[k] : 0.0, uxb ? uxb[k] : 0.0, uyb ? uyb[k] : 0.0, Tb ? Tb[k] : 0.0,
                                lf, lg);
    for (int i = 0; i < Q; ++i) {
      lam[int64_t(i) * n + k] = lf[i];
      lam[int64_t(Q + i) * n + k] = lg[i];
    }
  }
}

template <int SPLIT>
__global__ __launch_bounds__(256) void k_adjoint_init(const double* __restrict__ lam, const double* __restrict__ rho,
                                                      const double* __restrict__ ux, const double* __restrict__ uy,
                                                      const double* __restrict__ T, double* d_rho, double* d_ux,
                                                      double* d_uy, double* d_T, KParams kp) {
  constexpr int Q = Set<SPLIT>::Q;
  const int64_t n = int64_t(kp.nx) * kp.ny;
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const double in[4] = {rho[k], ux[k], uy[k], T[k]};
    double* outs[4] = {d_rho, d_ux, d_uy, d_T};
    for (int r = 0; r < 4; ++r) {
      if (!outs[r]) continue;
      D1 v[4];
      for (int j = 0; j < 4; ++j) v[j] = D1(in[j], j == r ? 1.0 : 0.0);
      D1 f[Q], g[Q];
      equilibrium_cell<SPLIT, D1>(v[0], v[1], v[2], v[3], kp, f, g);
      double acc = 0.0;
      for (int i = 0; i < Q; ++i) acc += lam[int64_t(i) * n + k] * f[i].d + lam[int64_t(Q + i) * n + k] * g[i].d;
      outs[r][k] = acc;
    }
  }
}

// ------------------------------------------------------------ limiter branches (derivative checks)
// SplitMix64 output function (Steele, Lea & Flood, OOPSLA 2014): a bijective
// 64-bit mix, so distinct (face, branch) keys give independent-looking terms.
__device__ inline unsigned long long mix64(unsigned long long z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Branch of the limiter function phi(r) = max(0, min(beta r, (1 + r)/2, beta))
// (Sec. III A 2) in L(a, b) = (b/2) phi(a/b): 0 when r <= 0 (a b <= 0),
// 1 for beta r, 2 for (1 + r)/2, 3 for beta, the smallest of the three
// taken in that order on ties.
__device__ inline int limiter_branch(double a, double b, double beta) {
  if (!(a * b > 0.0)) return 0;
  const double A = beta * fabs(a), M = 0.5 * fabs(a + b), B = beta * fabs(b);
  return (A <= M && A <= B) ? 1 : (M <= B ? 2 : 3);
}

// Signature of the limiter branches of one step from float64 populations X
// (a population buffer in float64 storage): for every population plane with a
// non-zero velocity component along an axis, the face above each cell along
// that axis is reconstructed from its upwind side (v > 0: cells c-1, c, c+1;
// v < 0: c, c+1, c+2), and sig receives the sum, over those faces, of
// mix64(4 face + branch).  Steps that take the same branch at every face
// give equal sums; a step with any face on another branch gives a different
// sum unless the 64-bit sums collide.
template <int SPLIT, int BCX, int BCY>
__global__ __launch_bounds__(256) void k_limiter_signature(const double* __restrict__ X, KParams kp,
                                                           unsigned long long* sig) {
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  using L = GH<N1>;
  const int64_t n = int64_t(kp.nx) * kp.ny;
  const double beta = 0.5 * kp.beta2;
  unsigned long long acc = 0ull;
  for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < n; k += int64_t(gridDim.x) * blockDim.x) {
    const int y = int(k / kp.nx), x = int(k % kp.nx);
    for (int pl = 0; pl < 2 * Q; ++pl) {
      const int i = pl % Q;
      for (int ax = 0; ax < 2; ++ax) {
        const double v = ax == 0 ? L::xi(i / N1) : L::xi(i % N1);
        if (v == 0.0) continue;
        auto at = [&](int d) -> double {
          if (ax == 0) return X[sidx(kp, pl / Q, i, y, wrap_any<BCX>(x + d, kp.nx))];
          return X[sidx(kp, pl / Q, i, wrap_any<BCY>(y + d, kp.ny), x)];
        };
        const double a = v > 0.0 ? at(0) - at(-1) : at(1) - at(2);
        const double b = v > 0.0 ? at(1) - at(0) : at(0) - at(1);
        const unsigned long long face = (unsigned long long)((int64_t(ax) * 2 * Q + pl) * n + k);
        acc += mix64(4ull * face + unsigned(limiter_branch(a, b, beta)));
      }
    }
  }
  __shared__ unsigned long long sh[256];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (int(threadIdx.x) < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(sig, sh[0]);  // a sum modulo 2^64: order-independent
}

// ------------------------------------------------------------ streaming probe
// Plain grid-stride streams over n elements of V (16 bytes: four uint32, or
// 4 bytes: one uint32): mode 0 copies src to dst, 1 reads src (the xor of what
// a thread read is stored only if it equals a value no input here holds, so
// the loads stay), 2 writes dst; NT marks the accesses non-temporal.  They
// bound the HBM bandwidth a kernel reaches on this GPU with accesses of that
// width.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ inline bool is_marker(u32x4 a) { return a.x == 0x9e3779b9u && a.y == 0x7f4a7c15u && a.z == 1u && a.w == 2u; }
__device__ inline bool is_marker(uint32_t a) { return a == 0x9e3779b9u; }
template <class V, bool NT>
__device__ inline V ld_stream(const V* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <class V, bool NT>
__device__ inline void st_stream(V* p, V v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <class V, bool NT>
__global__ __launch_bounds__(256) void k_stream(const V* __restrict__ src, V* __restrict__ dst, int64_t n, int mode) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (mode == 0) {
#pragma unroll 4
    for (; i < n; i += stride) st_stream<V, NT>(dst + i, ld_stream<V, NT>(src + i));
  } else if (mode == 1) {
    V acc = V(0u);
#pragma unroll 4
    for (; i < n; i += stride) acc ^= ld_stream<V, NT>(src + i);
    if (is_marker(acc)) dst[0] = acc;
  } else {
    const V v = V(0u);
#pragma unroll 4
    for (; i < n; i += stride) st_stream<V, NT>(dst + i, v);
  }
}

}  // namespace dvbm

// =================================================================== C ABI
using namespace dvbm;

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(DVBM_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(expr)                                   \
  do {                                                  \
    hipError_t _e = (expr);                             \
    if (_e != hipSuccess) return hip_fail(_e, #expr);   \
  } while (0)

int storage_bytes(int s) { return s == DVBM_F64 ? 8 : (s == DVBM_F32 || s == DVBM_F32_DEV) ? 4 : 2; }

std::string check_params(const dvbm_params* p) {
  if (!p) return "params is NULL";
  if (p->nx < 4 || p->ny < 4) return "nx and ny must be >= 4";
  if (p->split != 1 && p->split != 2) return "split must be 1 or 2";
  if (p->storage < DVBM_F64 || p->storage > DVBM_F32_DEV) return "unknown storage";
  if ((p->bc_x != DVBM_PERIODIC && p->bc_x != DVBM_ZERO_GRADIENT) ||
      (p->bc_y != DVBM_PERIODIC && p->bc_y != DVBM_ZERO_GRADIENT && p->bc_y != DVBM_WALL))
    return "unknown boundary condition (walls are supported in y only)";
  if (p->bc_y == DVBM_WALL) {
    if (!(p->wall_T[0] > 0) || !(p->wall_T[1] > 0)) return "wall temperatures must be > 0";
    if (!std::isfinite(p->wall_ux[0]) || !std::isfinite(p->wall_ux[1])) return "wall velocities must be finite";
    if (p->kernel == DVBM_KERNEL_SWEEP || p->kernel == DVBM_KERNEL_TILE)
      return "walls run on the plane-group and the per-cell kernel only (kernel AUTO or CELL)";
  }
  if (p->visc_mode != DVBM_CONST_MU && p->visc_mode != DVBM_CONST_TAU) return "unknown visc_mode";
  if (p->kernel < DVBM_KERNEL_AUTO || p->kernel > DVBM_KERNEL_TILE) return "unknown kernel";
  if (!(p->dx > 0) || !(p->dy > 0)) return "dx, dy must be > 0";
  if (!(p->R > 0)) return "R must be > 0";
  if (!(p->gamma > 1.0) || !(p->gamma <= 2.0)) return "gamma must lie in (1, 2] (Cv >= D R / 2)";
  if (!(p->Pr > 0)) return "Pr must be > 0";
  if (!(p->tau_ref > 0) || !(p->p_ref > 0) || !(p->T_ref > 0)) return "tau_ref, p_ref, T_ref must be > 0";
  if (!(p->beta >= 1.0) || !(p->beta <= 2.0)) return "beta must lie in [1, 2]";
  if (!(p->dt > 0) && !(p->cfl > 0)) return "cfl must be > 0 when dt <= 0";
  if (!std::isfinite(p->dt)) return "dt must be finite";
  const double nmax = 2147483647.0;
  if (double(p->nx) * double(p->ny) > nmax) return "nx * ny too large";
  const double pitch = double((int64_t(p->nx) + 63) / 64 * 64);
  const double dist = pitch * double(p->ny) * storage_bytes(p->storage) * (p->split == 1 ? 16 : 25);
  if (dist > 4294967295.0) return "one distribution (Q * ny * pitch elements) must be smaller than 4 GiB";
  if (p->kernel == DVBM_KERNEL_SWEEP && p->storage != DVBM_F64 && dist > 2147483648.0)
    return "the column-sweep kernel needs a distribution of at most 2 GiB for 32/16-bit storage";
  return "";
}

int pr_mode(double Pr) { return Pr == 1.0 ? PR_UNIT : (Pr < 1.0 ? PR_LOW : PR_HIGH); }

}  // namespace

struct dvbm_handle {
  dvbm_params p;
  KParams kp;
  int Q;
  void* buf[2];
  int cur;
  double* ws;
  hipStream_t stream;
  double dt;
  mutable int step_ranges;  // row ranges per strip (group) of the plane-group or the column-sweep kernel (0: not
                            // chosen yet; the first step asks the runtime what the kernel's code leaves room for)
  int adjoint_ranges;       // and of the one-sweep adjoint, chosen by dvbm_init
  double* scratch;         // device address of the fixed scratch array on the handle's device (NULL: lookup failed)
  std::string scratch_err; // why the lookup failed
};

namespace {

KParams make_kparams(const dvbm_params& p, double dt) {
  KParams k;
  k.nx = p.nx;
  k.ny = p.ny;
  k.pitch = dvbm_pitch(&p);
  k.srow = k.pitch * (p.split == 1 ? 16 : 25);
  k.sdist = k.srow * p.ny;
  k.c2 = p.R * p.T_ref;
  k.R = p.R;
  k.Cv = p.R / (p.gamma - 1.0);
  k.inv_Cv = 1.0 / k.Cv;
  const double c = std::sqrt(k.c2);
  k.kx = dt * c / p.dx;
  k.ky = dt * c / p.dy;
  k.const_mu = p.visc_mode == DVBM_CONST_MU;
  k.om_scale = k.const_mu ? dt / (p.tau_ref * p.p_ref) : dt / p.tau_ref;
  k.Pr = p.Pr;
  k.beta2 = 2.0 * p.beta;
  if (p.split == 2) {
    k.gr0 = (k.Cv - p.R) * p.T_ref;
    k.gr1 = 0.0;
  } else {
    k.gr0 = k.Cv * p.T_ref;
    k.gr1 = 0.5 * k.c2;
  }
  for (int w = 0; w < 2; ++w) {
    k.wall_T[w] = p.wall_T[w];
    k.wall_ux[w] = p.wall_ux[w];
  }
  return k;
}

#ifndef DVBM_SWEEP_ROUNDS64
#define DVBM_SWEEP_ROUNDS64 6
#endif
#ifndef DVBM_SWEEP_ROUNDS32
#define DVBM_SWEEP_ROUNDS32 4
#endif
#ifndef DVBM_SWEEP_ROUNDS16
#define DVBM_SWEEP_ROUNDS16 1
#endif
// Compute units of the current device (256 where the runtime does not say).
int device_cus() {
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0) {
    (void)hipGetLastError();
    return 256;
  }
  return ncu;
}
// The same, and the workgroups of `kern` each of them holds at a time (1 where
// the runtime does not say).
void device_slots(const void* kern, int block, int& ncu, int& per_cu) {
  ncu = device_cus();
  per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, block, 0) != hipSuccess || per_cu <= 0) {
    (void)hipGetLastError();
    per_cu = 1;
  }
}

// Row ranges per strip of the plane-group kernel.  A range costs about three
// row steps before its first row is stored, and a second round of workgroups
// costs them again, so all workgroups run at once: one per CU, or two where
// they fit and leave ranges of at least 4 rows (f32_dev, 256^2: 8.95 us with
// 255 ranges of 5 rows, 9.55 us with 510 of 2.5; 512^2: 22.8 us with 252,
// 21.8 us with 504; three per CU, D2Q16 bf16: 13.5 us against 12.3 at 509 x 383).
// Ranges that would be longer than 32 rows are cut to 16 or less, in as many
// full rounds: neighbouring workgroups then stay close in memory (float64
// 1024^2: 206 us in one round of 68 rows, 192 us in seven of 9; f32 4096^2:
// 1590 us at 8 to 16 rows, 1790 us at 32).  That counts for less where the two
// buffers stay in the 256 MiB last-level cache (about 300 MB still do), and for
// nothing where each strip is one range; up to 48 rows one full round, which has
// fewer row steps than three, is then faster (D2Q16 f32 1024^2 48.5 us in one,
// 54.8 us in three; bf16 64 x 11000 52.5 / 57.8; float64 30000 x 33 110 / 120; but
// f32 1024^2 between walls, 18 strips and 420 MB, 134 / 120).
int planes_ranges(const void* kern, int block, int nstrips, int ny, int64_t buffer_bytes) {
  int ncu, per_cu;
  device_slots(kern, block, ncu, per_cu);
  const bool two = per_cu >= 2;
  const int at_once = two ? 2 * ncu : ncu;
  int n = at_once / nstrips;
  if (n < 1 || ny / n < 4) n = ncu / nstrips;
  const bool full = int64_t(nstrips) * n * 10 >= int64_t(at_once) * 9;
  if (n < 1 || ny / n > (full && (n == 1 || 2 * buffer_bytes <= 300000000) ? 48 : 32)) {
    const int64_t slots = int64_t(ncu) * per_cu, rounds = (int64_t(nstrips) * ny + 16 * slots - 1) / (16 * slots);
    n = int(rounds * slots / nstrips);
  } else if (n <= 4 && !full) {
    // few ranges of many strips can leave much of the device idle: then the
    // number with the least time, in row steps of a full round; a range costs
    // about 5 steps besides its rows, 3 where two workgroups share a CU, and a
    // last round of one workgroup per CU runs in 0.6 of the time of two (257
    // strips of 16 rows, bf16: 20.9 us in one range, 17.9 in two; 134 strips of
    // 32 rows, float64: 48.2 in one, 44.1 in three; 16 rows: 27.2 / 28.6)
    const auto time = [&](int m) {
      const int rounds = nstrips * m / at_once, rest = nstrips * m % at_once;
      return ((ny + m - 1) / m + (two ? 3 : 5)) * (rounds + (rest == 0 ? 0.0 : two && rest <= ncu ? 0.6 : 1.0));
    };
    for (int m = n + 1, most = 4 * n + 1; m <= most && ny / m >= 4; ++m)
      if (time(m) < 0.97 * time(n)) n = m;
  }
  return n < 1 ? 1 : (n > ny ? ny : n);
}

// Row ranges per strip of the adjoint kernel: the number of rounds of
// workgroups (1 to 4) with the least rows in sequence, a range costing about
// five row steps besides its own rows.  One round is best where the strips
// divide the device well (float64 1024^2, 18 strips: 284 us in one round of
// 14 ranges, 325 us in two), several where they don't (4096^2, 69 strips:
// three ranges fill 207 of 256 CUs, eleven 253 of them three times).
// A CU holds one workgroup, whose LDS leaves no room for a second.
static_assert(2 * sizeof(AdjointShared<1>) > 160 * 1024 && 2 * sizeof(AdjointShared<2>) > 160 * 1024, "one workgroup per CU");
int adjoint_ranges(int nstrips, int ny) {
  const int ncu = device_cus();
  int best = 1;
  int64_t least = INT64_MAX;
  for (int rounds = 1; rounds <= 4; ++rounds) {
    int n = rounds * ncu / nstrips;
    n = n < 1 ? 1 : (n > ny ? ny : n);
    const int64_t rows = int64_t(rounds) * ((ny + n - 1) / n + 5);
    if (rows < least) {
      least = rows;
      best = n;
    }
  }
  return best;
}

// Row ranges per strip group for the column sweep.  One workgroup fits a
// CU at a time, so one round of ranges (as many workgroups as the device
// holds) ends with its slowest CU; `rounds` rounds of shorter ranges let the
// faster CUs take more of them.  Ranges keep at least 48 rows (the 4
// stencil rows read beyond a range stay under 10 %), and never fewer ranges than one
// round nor ranges shorter than 9 rows.  Measured on the 4096^2 thermal
// wave: float64 storage gains 15 % at 6 rounds, float32 4.5 % at 4 rounds,
// the 16-bit formats nothing.
int sweep_ranges(const void* kern, int block, int ngroups, int ny, int rounds, int unit) {
  int ncu, per_cu;
  device_slots(kern, block, ncu, per_cu);
  const int one = ncu * per_cu / ngroups;  // ranges per strip group in one round
  int want = rounds * one < ny / 48 ? rounds * one : ny / 48;
  if (want < one) want = one;
  if (want > ny / (3 * unit)) want = ny / (3 * unit);
  if (want < 1) want = 1;
  // the number of ranges of sweep_len rows that cover the column; fewer, longer
  // ones where the last round would leave more than a tenth of the slots idle
  // (float64 3001 x 1499, 26 groups on 256 CUs: 30 ranges take four rounds,
  // the last nearly empty, 967 us; 28 take three, 812 us)
  const int slots = ncu * per_cu;
  int best = 0;
  double full = 0.0;
  for (int w = want; w >= 1 && 2 * w >= want; --w) {
    const int len = sweep_len(ny, w, unit), n = (ny + len - 1) / len;
    const int64_t groups = int64_t(n) * ngroups, rounds_up = (groups + slots - 1) / slots;
    const double f = double(groups) / double(rounds_up * slots);
    if (f > full + 1e-9) {
      full = f;
      best = n;
    }
    if (full >= 0.9) break;
  }
  return best;
}

}  // namespace

// Step and adjoint launchers: defined here for every translation unit, each
// split x storage instantiated in one kernel unit (compiled with DVBM_PART,
// in parallel with the others) and declared extern in the main unit.
namespace dvbm_launch {

// The kernel a handle's steps use (the AUTO rule of dvbm_kernel).
constexpr int KERNEL_PLANES = -1;  // the plane-group kernel: chosen by AUTO only
template <int SPLIT>
int step_kernel(const dvbm_handle* h) {
  if (h->p.kernel != DVBM_KERNEL_AUTO) return h->p.kernel;
  if (h->p.bc_y == DVBM_WALL) return KERNEL_PLANES;
  const int bytes = storage_bytes(h->p.storage), nx = h->p.nx, ny = h->p.ny;
  if (nx > SWEEP_OWN && nx <= 64 && cells_for_64_columns<SPLIT>(bytes, ny)) return DVBM_KERNEL_CELL;
  if (int64_t(nx) * ny < sweep_min_cells<SPLIT>(h->p.storage, (nx + SWEEP_OWN - 1) / SWEEP_OWN)) return KERNEL_PLANES;
  if (h->p.storage == DVBM_F64) return DVBM_KERNEL_SWEEP;
  // above 2 GiB the sweep's 32-bit offsets end (the plane groups' rows have bases
  // of their own and would reach: 6528^2 f32 4346 us against 5057)
  const uint64_t dist = uint64_t(h->kp.sdist) * uint64_t(storage_bytes(h->p.storage));
  return dist <= (uint64_t(1) << 31) ? DVBM_KERNEL_SWEEP : DVBM_KERNEL_CELL;
}

template <int SPLIT, class S, int BCX, int BCY, int PRM>
void launch_step_pr(const dvbm_handle* h, const void* src, void* dst) {
  using T = typename S::T;
  const T* s = static_cast<const T*>(src);
  T* d = static_cast<T*>(dst);
  const int kern_id = step_kernel<SPLIT>(h);
  if constexpr (BCY == BC_WALL) {
    const dim3 grid(((h->p.nx + CELL_TX - 1) / CELL_TX) * ((h->p.ny + CELL_TY - 1) / CELL_TY));
    hipLaunchKernelGGL((k_collide_advect<SPLIT, S, BCX, BCY, PRM>), grid, dim3(CELL_TX, CELL_TY), 0, h->stream, s, d,
                       h->kp, reinterpret_cast<const T*>(h->ws + WS_GHOST));
    return;
  } else {
  if (kern_id == DVBM_KERNEL_TILE) {
    const dim3 grid(((h->p.nx + TILE_TX - 1) / TILE_TX) * ((h->p.ny + TILE_TY - 1) / TILE_TY));
    hipLaunchKernelGGL((k_collide_advect_lds<SPLIT, S, BCX, BCY, PRM>), grid, dim3(TILE_TX, TILE_TY), 0, h->stream,
                       s, d, h->kp);
    return;
  }
  {
    constexpr int SWEEP_K = sweep_k<S>();
    if (kern_id == DVBM_KERNEL_SWEEP) {
      const auto kern = k_collide_advect_sweep<SPLIT, S, BCX, BCY, PRM>;
      const int nstrips = (h->p.nx + SWEEP_OWN - 1) / SWEEP_OWN;
      const int ngroups = (nstrips + SWEEP_K - 1) / SWEEP_K;
      if (h->step_ranges == 0)
        h->step_ranges = sweep_ranges(reinterpret_cast<const void*>(kern), 128 * SWEEP_K, ngroups, h->p.ny,
                                      sizeof(T) == 8 ? DVBM_SWEEP_ROUNDS64
                                                     : (sizeof(T) == 4 ? DVBM_SWEEP_ROUNDS32 : DVBM_SWEEP_ROUNDS16),
                                      sweep_ring<S>());
      const int total = ngroups * h->step_ranges;
      const dim3 grid(8 * ((total + 7) / 8));
      hipLaunchKernelGGL(kern, grid, dim3(128 * SWEEP_K), 0, h->stream, s, d, h->kp, ngroups, h->step_ranges);
      return;
    }
  }
  const dim3 grid(((h->p.nx + CELL_TX - 1) / CELL_TX) * ((h->p.ny + CELL_TY - 1) / CELL_TY));
  hipLaunchKernelGGL((k_collide_advect<SPLIT, S, BCX, BCY, PRM>), grid, dim3(CELL_TX, CELL_TY), 0, h->stream, s, d,
                     h->kp, static_cast<const T*>(nullptr));
  }
}

template <int SPLIT, class S, int BCX, int BCY>
void launch_step_bc(const dvbm_handle* h, const void* src, void* dst) {
  using T = typename S::T;
  const int prm = pr_mode(h->p.Pr);
  if (step_kernel<SPLIT>(h) == KERNEL_PLANES) {
    const auto kern = k_collide_advect_planes<SPLIT, S, BCX, BCY>;
    const int nstrips = (h->p.nx + SWEEP_OWN - 1) / SWEEP_OWN;
    if (h->step_ranges == 0)
      h->step_ranges = planes_ranges(reinterpret_cast<const void*>(kern), planes_threads<SPLIT>(), nstrips, h->p.ny,
                                     2 * h->kp.sdist * int64_t(sizeof(T)));
    hipLaunchKernelGGL(kern, dim3(unsigned(nstrips) * unsigned(h->step_ranges)), dim3(planes_threads<SPLIT>()), 0,
                       h->stream, static_cast<const T*>(src), static_cast<T*>(dst), h->kp, nstrips, h->step_ranges, prm);
    return;
  }
  if constexpr (BCY == BC_WALL)
    hipLaunchKernelGGL((k_wall_ghosts<SPLIT, S>), dim3((4 * h->p.nx + 255) / 256), dim3(256), 0, h->stream,
                       static_cast<const T*>(src), reinterpret_cast<T*>(h->ws + WS_GHOST), h->kp);
  with_pr_mode(prm, [&](auto m) { launch_step_pr<SPLIT, S, BCX, BCY, decltype(m)::value>(h, src, dst); });
}

// f(integral_constant BCX, integral_constant BCY) for the boundary rules of a
// handle without walls, and with walls in y too.
template <class F>
void with_open_bcs(const dvbm_params& p, F&& f) {
  using Periodic = std::integral_constant<int, BC_PERIODIC>;
  using Open = std::integral_constant<int, BC_ZERO_GRADIENT>;
  if (p.bc_x == DVBM_PERIODIC) {
    if (p.bc_y == DVBM_PERIODIC) f(Periodic(), Periodic());
    else f(Periodic(), Open());
  } else {
    if (p.bc_y == DVBM_PERIODIC) f(Open(), Periodic());
    else f(Open(), Open());
  }
}
template <class F>
void with_bcs(const dvbm_params& p, F&& f) {
  using Wall = std::integral_constant<int, BC_WALL>;
  if (p.bc_y != DVBM_WALL) with_open_bcs(p, f);
  else if (p.bc_x == DVBM_PERIODIC) f(std::integral_constant<int, BC_PERIODIC>(), Wall());
  else f(std::integral_constant<int, BC_ZERO_GRADIENT>(), Wall());
}

template <int SPLIT, class S>
void step(const dvbm_handle* h, const void* src, void* dst) {
  with_bcs(h->p, [&](auto bx, auto by) { launch_step_bc<SPLIT, S, decltype(bx)::value, decltype(by)::value>(h, src, dst); });
}

template <int SPLIT, class S, int BCX, int BCY, class LT>
void adjoint_bc(const dvbm_handle* h, const void* state, const LT* lam1, LT* lam0, double* dparams, double* work, double* ws);

// Cotangents lam1, lam0 stored as LT (double or float); the arithmetic and the
// work array (of the deviation storage) are float64.  ws: the reduction area (block partials of
// d/dtau_ref, d/dPr from offset 0, the block counter at WS_TICKET doubles).
template <int SPLIT, class S, class LT>
void adjoint(const dvbm_handle* h, const void* state, const LT* lam1, LT* lam0, double* dparams, double* work, double* ws) {
  with_open_bcs(h->p, [&](auto bx, auto by) {
    adjoint_bc<SPLIT, S, decltype(bx)::value, decltype(by)::value, LT>(h, state, lam1, lam0, dparams, work, ws);
  });
}

template <int SPLIT, class S, int BCX, int BCY, class LT>
void adjoint_bc(const dvbm_handle* h, const void* state, const LT* lam1, LT* lam0, double* dparams, double* work, double* ws) {
  if constexpr (!S::dev) {
    const auto kern = k_adjoint<SPLIT, S, BCX, BCY, LT>;
    const int nstrips = (h->p.nx + SWEEP_OWN - 1) / SWEEP_OWN;
    const int nr = h->adjoint_ranges, total = nstrips * nr;
    // more strips than the workspace has partials for: in turns
    for (int first = 0; first < total; first += ADJ_BLOCKS)
      hipLaunchKernelGGL(kern, dim3(unsigned(total - first < ADJ_BLOCKS ? total - first : ADJ_BLOCKS)),
                         dim3(planes_threads<SPLIT>()), 0, h->stream, static_cast<const typename S::T*>(state), lam1,
                         lam0, h->kp, nstrips, nr, first, pr_mode(h->p.Pr), h->p.tau_ref, ws,
                         reinterpret_cast<unsigned*>(ws + WS_TICKET), dparams);
  } else {
    using T = typename S::T;
    const T* s = static_cast<const T*>(state);
    unsigned* ticket = reinterpret_cast<unsigned*>(ws + WS_TICKET);
    const int64_t cells = int64_t(h->p.nx) * h->p.ny;
    if (cells <= ADJ_RELAX_CELLS) {
      hipLaunchKernelGGL((k_adjoint_relax<SPLIT, S, LT>), dim3(unsigned((cells + 63) / 64)), dim3(planes_threads<SPLIT>()),
                         0, h->stream, s, lam1, work, h->kp, pr_mode(h->p.Pr), h->p.tau_ref, ws, ticket, dparams);
    } else {
      const int64_t nb = (cells + RED_THREADS - 1) / RED_THREADS;
      with_pr_mode(pr_mode(h->p.Pr), [&](auto m) {
        hipLaunchKernelGGL((k_adjoint_relax_cells<SPLIT, S, decltype(m)::value, LT>),
                           dim3(unsigned(nb < ADJ_BLOCKS ? nb : ADJ_BLOCKS)), dim3(RED_THREADS), 0, h->stream, s, lam1,
                           work, h->kp, h->p.tau_ref, ws, ticket, dparams);
      });
    }
    const int64_t groups = 2 * Set<SPLIT>::N1, nstrips = (h->p.nx + ADJ_STRIP - 1) / ADJ_STRIP;
    int64_t ch = (int64_t(h->p.ny) * groups * nstrips + DVBM_ADJ_WAVES - 1) / DVBM_ADJ_WAVES;
    ch = ch < DVBM_ADJ_CH_MIN ? DVBM_ADJ_CH_MIN : (ch > h->p.ny ? h->p.ny : ch);
    const int64_t nchunks = (h->p.ny + ch - 1) / ch, waves = groups * nstrips * nchunks;
    hipLaunchKernelGGL((k_adjoint_flux<SPLIT, S, BCX, BCY, LT>), dim3(unsigned((waves + 3) / 4)), dim3(256), 0, h->stream,
                       s, lam1, work, lam0, h->kp, int(nstrips), int(ch), int(nchunks));
  }
}

}  // namespace dvbm_launch

#if defined(DVBM_PART)
// kernel unit DVBM_PART = 5 (split - 1) + storage + 1; the adjoint takes the
// float64, float32 and float32-deviation storages (storage 0, 1, 4)
template void dvbm_launch::step<(DVBM_PART - 1) / 5 + 1, DVBM_PART_STORE>(const dvbm_handle*, const void*, void*);
#if (DVBM_PART - 1) % 5 < 2 || (DVBM_PART - 1) % 5 == 4
template void dvbm_launch::adjoint<(DVBM_PART - 1) / 5 + 1, DVBM_PART_STORE, double>(
    const dvbm_handle*, const void*, const double*, double*, double*, double*, double*);
template void dvbm_launch::adjoint<(DVBM_PART - 1) / 5 + 1, DVBM_PART_STORE, float>(
    const dvbm_handle*, const void*, const float*, float*, double*, double*, double*);
#endif
#else
#define DVBM_EXTERN_STEP(SPLIT, S) \
  extern template void dvbm_launch::step<SPLIT, S>(const dvbm_handle*, const void*, void*);
#define DVBM_EXTERN_ADJ(SPLIT, S)                                                                           \
  extern template void dvbm_launch::adjoint<SPLIT, S, double>(const dvbm_handle*, const void*, const double*, \
                                                              double*, double*, double*, double*);          \
  extern template void dvbm_launch::adjoint<SPLIT, S, float>(const dvbm_handle*, const void*, const float*,   \
                                                             float*, double*, double*, double*);
DVBM_EXTERN_STEP(1, StoreF64)
DVBM_EXTERN_STEP(1, StoreF32)
DVBM_EXTERN_STEP(1, StoreBF16)
DVBM_EXTERN_STEP(1, StoreF16)
DVBM_EXTERN_STEP(1, StoreF32Dev)
DVBM_EXTERN_STEP(2, StoreF64)
DVBM_EXTERN_STEP(2, StoreF32)
DVBM_EXTERN_STEP(2, StoreBF16)
DVBM_EXTERN_STEP(2, StoreF16)
DVBM_EXTERN_STEP(2, StoreF32Dev)
DVBM_EXTERN_ADJ(1, StoreF64)
DVBM_EXTERN_ADJ(1, StoreF32)
DVBM_EXTERN_ADJ(1, StoreF32Dev)
DVBM_EXTERN_ADJ(2, StoreF64)
DVBM_EXTERN_ADJ(2, StoreF32)
DVBM_EXTERN_ADJ(2, StoreF32Dev)

// ------------------------------------------------------------ fixed scratch
// Device memory of dvbm_adjoint_step_noalloc, for callers that cannot
// allocate: the reduction area (block partials and block counter, laid out as
// in the workspace) in the first SCRATCH_WORK_OFFSET bytes, the adjoint work
// rows after it.  Each device holds its own copy until the process ends.  In
// host code `scratch` names a host-side stand-in, not device memory: kernels
// get the device address that hipGetSymbolAddress returns for the device.
constexpr size_t SCRATCH_BYTES = size_t(16) << 20;
constexpr size_t SCRATCH_WORK_OFFSET = size_t(64) << 10;
static_assert(size_t(WS_TICKET + 1) * sizeof(double) <= SCRATCH_WORK_OFFSET, "reduction area exceeds its slot");
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

__global__ void k_clear_counter(unsigned* counter) {
  if (threadIdx.x == 0) counter[0] = 0u;
}

namespace {

constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[SCRATCH_MAX_DEVICES] = {};

// Device address of `scratch` on the current device, looked up once per device.
hipError_t scratch_address(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// Calls F<SPLIT, Store>::run(args...) for the handle's split and storage.
template <template <int, class> class F, class... A>
void dispatch(const dvbm_params& p, A&&... args) {
  if (p.split == 2) {
    switch (p.storage) {
      case DVBM_F64: F<2, StoreF64>::run(args...); break;
      case DVBM_F32: F<2, StoreF32>::run(args...); break;
      case DVBM_BF16_DEV: F<2, StoreBF16>::run(args...); break;
      case DVBM_F32_DEV: F<2, StoreF32Dev>::run(args...); break;
      default: F<2, StoreF16>::run(args...); break;
    }
  } else {
    switch (p.storage) {
      case DVBM_F64: F<1, StoreF64>::run(args...); break;
      case DVBM_F32: F<1, StoreF32>::run(args...); break;
      case DVBM_BF16_DEV: F<1, StoreBF16>::run(args...); break;
      case DVBM_F32_DEV: F<1, StoreF32Dev>::run(args...); break;
      default: F<1, StoreF16>::run(args...); break;
    }
  }
}

template <int SPLIT, class S>
struct StepOp {
  static void run(const dvbm_handle* h, const void* src, void* dst) { dvbm_launch::step<SPLIT, S>(h, src, dst); }
};

template <int SPLIT, class S>
struct InitOp {
  static void run(const dvbm_handle* h, const double* rho, const double* ux, const double* uy, const double* T,
                  void* dst) {
    using Tt = typename S::T;
    hipLaunchKernelGGL((k_init<SPLIT, S>), dim3(RED_BLOCKS * 4), dim3(256), 0, h->stream, rho, ux, uy, T,
                       static_cast<Tt*>(dst), h->kp);
  }
};

template <int SPLIT, class S>
struct MomentsOp {
  static void run(const dvbm_handle* h, const void* src, double* rho, double* ux, double* uy, double* T,
                  double* partials) {
    using Tt = typename S::T;
    hipLaunchKernelGGL((k_moments<SPLIT, S>), dim3(RED_BLOCKS), dim3(RED_THREADS), 0, h->stream,
                       static_cast<const Tt*>(src), h->kp, rho, ux, uy, T, partials);
  }
};

template <int SPLIT, class S>
struct DecodeOp {
  static void run(const dvbm_handle* h, const void* src, double* X) {
    using Tt = typename S::T;
    hipLaunchKernelGGL((k_decode<SPLIT, S>), dim3(RED_BLOCKS * 4), dim3(256), 0, h->stream,
                       static_cast<const Tt*>(src), X, h->kp);
  }
};

template <int SPLIT, class S>
struct EncodeOp {
  static void run(const dvbm_handle* h, const double* X, void* dst) {
    using Tt = typename S::T;
    hipLaunchKernelGGL((k_encode<SPLIT, S>), dim3(RED_BLOCKS * 4), dim3(256), 0, h->stream, X,
                       static_cast<Tt*>(dst), h->kp);
  }
};

template <int SPLIT, class S>
struct AdjointOp {
  template <class LT>
  static void run(const dvbm_handle* h, const void* state, const LT* lam1, LT* lam0, double* dparams, double* work, double* ws) {
    dvbm_launch::adjoint<SPLIT, S, LT>(h, state, lam1, lam0, dparams, work, ws);
  }
};

template <int SPLIT, class S>
struct ReadoutAdjointOp {
  static void run(const dvbm_handle* h, const void* state, const double* rb, const double* uxb, const double* uyb,
                  const double* Tb, double* lam) {
    using Tt = typename S::T;
    hipLaunchKernelGGL((k_adjoint_readout<SPLIT, S>), dim3(RED_BLOCKS), dim3(256), 0, h->stream,
                       static_cast<const Tt*>(state), rb, uxb, uyb, Tb, lam, h->kp);
  }
};

// The adjoint entry points support the float64, float32 and float32-deviation
// storages (adjoint_storage_ok rejects the others before dispatch).
template <template <int, class> class F, class... A>
void dispatch_adjoint(const dvbm_params& p, A&&... args) {
  if (p.split == 2) {
    if (p.storage == DVBM_F64)
      F<2, StoreF64>::run(args...);
    else if (p.storage == DVBM_F32_DEV)
      F<2, StoreF32Dev>::run(args...);
    else
      F<2, StoreF32>::run(args...);
  } else {
    if (p.storage == DVBM_F64)
      F<1, StoreF64>::run(args...);
    else if (p.storage == DVBM_F32_DEV)
      F<1, StoreF32Dev>::run(args...);
    else
      F<1, StoreF32>::run(args...);
  }
}

}  // namespace

extern "C" {

void dvbm_params_default(dvbm_params* p) {
  if (!p) return;
  std::memset(p, 0, sizeof(*p));
  p->split = 2;
  p->storage = DVBM_F32;
  p->bc_x = p->bc_y = DVBM_PERIODIC;
  p->visc_mode = DVBM_CONST_MU;
  p->dx = p->dy = 1.0;
  p->R = 1.0;
  p->gamma = 1.4;
  p->Pr = 0.71;
  p->tau_ref = 5e-5;
  p->p_ref = 1.0;
  p->T_ref = 1.0;
  p->beta = 1.2;
  p->cfl = 0.01;
  p->dt = 0.0;
  p->wall_T[0] = p->wall_T[1] = 1.0;
  p->wall_ux[0] = p->wall_ux[1] = 0.0;
}

int dvbm_num_populations(int32_t split) {
  if (split == 1) return 16;
  if (split == 2) return 25;
  return fail(DVBM_EINVAL, "split must be 1 or 2");
}

int dvbm_velocity_set(int32_t split, double R, double T_ref, double* v, double* w) {
  if ((split != 1 && split != 2) || !v || !w || !(R > 0) || !(T_ref > 0))
    return fail(DVBM_EINVAL, "dvbm_velocity_set: bad argument");
  const double c = std::sqrt(R * T_ref);
  const int n1 = split == 1 ? 4 : 5;
  for (int a = 0; a < n1; ++a)
    for (int b = 0; b < n1; ++b) {
      const int i = a * n1 + b;
      const double xa = split == 1 ? GH<4>::xi(a) : GH<5>::xi(a);
      const double xb = split == 1 ? GH<4>::xi(b) : GH<5>::xi(b);
      const double wa = split == 1 ? GH<4>::w(a) : GH<5>::w(a);
      const double wb = split == 1 ? GH<4>::w(b) : GH<5>::w(b);
      v[2 * i] = c * xa;
      v[2 * i + 1] = c * xb;
      w[i] = wa * wb;
    }
  return n1 * n1;
}

int64_t dvbm_pitch(const dvbm_params* p) {
  if (!p || p->nx <= 0) return 0;
  return (int64_t(p->nx) + 63) / 64 * 64;
}

size_t dvbm_buffer_bytes(const dvbm_params* p) {
  if (!check_params(p).empty()) return 0;
  const int Q = p->split == 1 ? 16 : 25;
  return size_t(2) * Q * size_t(p->ny) * size_t(dvbm_pitch(p)) * storage_bytes(p->storage);
}

size_t dvbm_workspace_bytes(const dvbm_params* p) {
  size_t n = size_t(WS_GHOST) * sizeof(double);
  if (p && p->bc_y == DVBM_WALL && check_params(p).empty())  // 4 ghost rows of each of the 2Q planes
    n += size_t(2) * (p->split == 1 ? 16 : 25) * 4 * size_t(dvbm_pitch(p)) * storage_bytes(p->storage);
  return n;
}

int dvbm_init(const dvbm_params* p, const double* rho, const double* ux, const double* uy, const double* T,
              void* buf0, void* buf1, void* workspace, void* stream, dvbm_handle** out) {
  g_last_error.clear();
  const std::string err = check_params(p);
  if (!err.empty()) return fail(DVBM_EINVAL, "dvbm_init: " + err);
  if (!rho || !ux || !uy || !T || !buf0 || !buf1 || !workspace || !out)
    return fail(DVBM_EINVAL, "dvbm_init: NULL pointer argument");
  if ((reinterpret_cast<uintptr_t>(buf0) | reinterpret_cast<uintptr_t>(buf1)) & 255u)
    return fail(DVBM_EINVAL, "dvbm_init: population buffers must be 256-byte aligned");
  if (buf0 == buf1) return fail(DVBM_EINVAL, "dvbm_init: buf0 and buf1 must differ");
  *out = nullptr;
  hipStream_t s = static_cast<hipStream_t>(stream);
  double* ws = static_cast<double*>(workspace);
  const int64_t n = int64_t(p->nx) * p->ny;

  // extrema of the initial fields: time step (Sec. III A 3) and validity
  hipLaunchKernelGGL(k_speed, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, s, rho, ux, uy, T, n, p->gamma * p->R, p->R,
                     ws);
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(RED_THREADS), 0, s, ws, RED_BLOCKS, 1, ws + 4 * RED_BLOCKS);
  HIP_TRY(hipGetLastError());
  double ext[4];
  HIP_TRY(hipMemcpyAsync(ext, ws + 4 * RED_BLOCKS, sizeof(ext), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  const double smax = ext[0], pmax = ext[1], rmin = -ext[2], tmin = -ext[3];
  if (!std::isfinite(smax) || !std::isfinite(pmax) || !(rmin > 0) || !(tmin > 0))
    return fail(DVBM_ENAN, "dvbm_init: initial fields must be finite with rho > 0 and T > 0");
  const double dt = p->dt > 0 ? p->dt : p->cfl * std::fmin(p->dx, p->dy) / smax;

  // stiffness: omega_1 = dt / tau_1 must stay <= 2 (explicit Euler relaxation)
  const double om_nu = p->visc_mode == DVBM_CONST_MU ? dt * pmax / (p->tau_ref * p->p_ref) : dt / p->tau_ref;
  const double om1 = p->Pr > 1.0 ? om_nu * p->Pr : om_nu;
  if (om1 > 2.0)
    return fail(DVBM_ESTIFF, "dvbm_init: dt / tau_1 = " + std::to_string(om1) + " > 2 for the initial state");

  dvbm_handle* h = new dvbm_handle;
  h->p = *p;
  h->dt = dt;
  h->kp = make_kparams(*p, dt);
  h->Q = p->split == 1 ? 16 : 25;
  h->buf[0] = buf0;
  h->buf[1] = buf1;
  h->cur = 0;
  h->ws = ws;
  h->stream = s;
  h->step_ranges = 0;
  h->adjoint_ranges = adjoint_ranges((h->p.nx + SWEEP_OWN - 1) / SWEEP_OWN, h->p.ny);
  // the fixed scratch of dvbm_adjoint_step_noalloc on this device (set-up only:
  // that entry point then makes no runtime call besides its launches)
  h->scratch = nullptr;
  if (hipError_t es = scratch_address(&h->scratch); es != hipSuccess) {
    h->scratch = nullptr;
    h->scratch_err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(es);
    (void)hipGetLastError();
  }
  hipError_t e = hipMemsetAsync(ws + WS_TICKET, 0, sizeof(double), s);  // the adjoint's block counter
  if (e != hipSuccess) {
    delete h;
    return hip_fail(e, "dvbm_init: workspace");
  }
  dispatch<InitOp>(h->p, h, rho, ux, uy, T, buf0);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    delete h;
    return hip_fail(e, "dvbm_init: equilibrium initialisation");
  }
  *out = h;
  return DVBM_OK;
}

int dvbm_step(dvbm_handle* h, int64_t nsteps) {
  if (!h) return fail(DVBM_EINVAL, "dvbm_step: NULL handle");
  if (nsteps < 0) return fail(DVBM_EINVAL, "dvbm_step: nsteps < 0");
  for (int64_t k = 0; k < nsteps; ++k) {
    dispatch<StepOp>(h->p, h, h->buf[h->cur], h->buf[1 - h->cur]);
    h->cur ^= 1;
  }
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_step_from(dvbm_handle* h, const void* src, void* dst) {
  if (!h || !src || !dst) return fail(DVBM_EINVAL, "dvbm_step_from: NULL argument");
  if (src == dst) return fail(DVBM_EINVAL, "dvbm_step_from: src and dst must differ");
  dispatch<StepOp>(h->p, h, src, dst);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_moments(dvbm_handle* h, double* rho, double* ux, double* uy, double* T, double* sums_host) {
  if (!h) return fail(DVBM_EINVAL, "dvbm_moments: NULL handle");
  dispatch<MomentsOp>(h->p, h, h->buf[h->cur], rho, ux, uy, T, h->ws);
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(RED_THREADS), 0, h->stream, h->ws, RED_BLOCKS, 0,
                     h->ws + 4 * RED_BLOCKS);
  HIP_TRY(hipGetLastError());
  if (sums_host) {
    HIP_TRY(hipMemcpyAsync(sums_host, h->ws + 4 * RED_BLOCKS, 4 * sizeof(double), hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    for (int k = 0; k < 4; ++k)
      if (!std::isfinite(sums_host[k])) return fail(DVBM_ENAN, "dvbm_moments: non-finite conservation sum");
  }
  return DVBM_OK;
}

int dvbm_load_populations(dvbm_handle* h, const double* X) {
  if (!h || !X) return fail(DVBM_EINVAL, "dvbm_load_populations: NULL argument");
  dispatch<EncodeOp>(h->p, h, X, h->buf[h->cur]);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_store_populations(dvbm_handle* h, double* X) {
  if (!h || !X) return fail(DVBM_EINVAL, "dvbm_store_populations: NULL argument");
  dispatch<DecodeOp>(h->p, h, h->buf[h->cur], X);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

double dvbm_get_dt(const dvbm_handle* h) { return h ? h->dt : 0.0; }

void* dvbm_state(const dvbm_handle* h) { return h ? h->buf[h->cur] : nullptr; }

int dvbm_state_index(const dvbm_handle* h) { return h ? h->cur : fail(DVBM_EINVAL, "NULL handle"); }

int dvbm_set_state_index(dvbm_handle* h, int index) {
  if (!h || (index != 0 && index != 1)) return fail(DVBM_EINVAL, "dvbm_set_state_index: bad argument");
  h->cur = index;
  return DVBM_OK;
}

void dvbm_destroy(dvbm_handle* h) { delete h; }

const char* dvbm_last_error(void) { return g_last_error.c_str(); }

size_t dvbm_adjoint_bytes(const dvbm_params* p) {
  if (!check_params(p).empty()) return 0;
  const int Q = p->split == 1 ? 16 : 25;
  return size_t(2) * Q * size_t(p->ny) * size_t(p->nx) * sizeof(double);
}

static int adjoint_storage_ok(const dvbm_handle* h, const char* who) {
  if (h->p.storage != DVBM_F64 && h->p.storage != DVBM_F32 && h->p.storage != DVBM_F32_DEV)
    return fail(DVBM_EINVAL, std::string(who) + ": the adjoint supports f64, f32 and f32_dev storage");
  if (h->p.bc_y == DVBM_WALL) return fail(DVBM_EINVAL, std::string(who) + ": the adjoint does not support walls");
  // the adjoint addresses a cotangent plane, or a row of N1 planes, through one
  // buffer resource with 32-bit offsets and discards stores at offset 2^31
  // (the distribution limit keeps N1 float64 planes below that)
  if (int64_t(h->p.nx) * h->p.ny * int64_t(sizeof(double)) >= (int64_t(1) << 31))
    return fail(DVBM_EINVAL, std::string(who) + ": a cotangent plane must stay below 2 GiB");
  return DVBM_OK;
}

size_t dvbm_adjoint_work_bytes(const dvbm_params* p) {
  if (!check_params(p).empty()) return 0;
  return size_t(ADJ_WORK_ROWS) * size_t(p->nx) * size_t(p->ny) * sizeof(double);
}

int dvbm_adjoint_step(dvbm_handle* h, const void* state_n, const double* lam_np1, double* lam_n, double* dparams,
                      void* work) {
  if (!h || !state_n || !lam_np1 || !lam_n || !work) return fail(DVBM_EINVAL, "dvbm_adjoint_step: NULL argument");
  if (lam_np1 == lam_n) return fail(DVBM_EINVAL, "dvbm_adjoint_step: lam_np1 and lam_n must differ");
  if (int rc = adjoint_storage_ok(h, "dvbm_adjoint_step")) return rc;
  dispatch_adjoint<AdjointOp>(h->p, h, state_n, lam_np1, lam_n, dparams, static_cast<double*>(work), h->ws);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_adjoint_step_f32(dvbm_handle* h, const void* state_n, const float* lam_np1, float* lam_n,
                          double* dparams, void* work) {
  if (!h || !state_n || !lam_np1 || !lam_n || !work)
    return fail(DVBM_EINVAL, "dvbm_adjoint_step_f32: NULL argument");
  if (lam_np1 == lam_n) return fail(DVBM_EINVAL, "dvbm_adjoint_step_f32: lam_np1 and lam_n must differ");
  if (int rc = adjoint_storage_ok(h, "dvbm_adjoint_step_f32")) return rc;
  dispatch_adjoint<AdjointOp>(h->p, h, state_n, lam_np1, lam_n, dparams, static_cast<double*>(work), h->ws);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_adjoint_step_noalloc(dvbm_handle* h, const void* state_n, const double* lam_np1, double* lam_n,
                              double* dparams) {
  if (!h || !state_n || !lam_np1 || !lam_n) return fail(DVBM_EINVAL, "dvbm_adjoint_step_noalloc: NULL argument");
  if (lam_np1 == lam_n) return fail(DVBM_EINVAL, "dvbm_adjoint_step_noalloc: lam_np1 and lam_n must differ");
  if (int rc = adjoint_storage_ok(h, "dvbm_adjoint_step_noalloc")) return rc;
  const size_t need = dvbm_adjoint_work_bytes(&h->p);
  if (need > SCRATCH_BYTES - SCRATCH_WORK_OFFSET)
    return fail(DVBM_EINVAL, "dvbm_adjoint_step_noalloc: the grid needs " + std::to_string(need) +
                                 " bytes of work rows, more than the " +
                                 std::to_string(SCRATCH_BYTES - SCRATCH_WORK_OFFSET) +
                                 " bytes the fixed scratch holds (at most " +
                                 std::to_string((SCRATCH_BYTES - SCRATCH_WORK_OFFSET) / (ADJ_WORK_ROWS * 8)) +
                                 " cells); use dvbm_adjoint_step with a caller work array");
  if (!h->scratch) return fail(DVBM_EHIP, "dvbm_adjoint_step_noalloc: " + h->scratch_err);
  double* red = h->scratch;
  double* work = h->scratch + SCRATCH_WORK_OFFSET / sizeof(double);
  // the block counter must start at zero (the last block of each call resets it)
  hipLaunchKernelGGL(k_clear_counter, dim3(1), dim3(64), 0, h->stream, reinterpret_cast<unsigned*>(red + WS_TICKET));
  dispatch_adjoint<AdjointOp>(h->p, h, state_n, lam_np1, lam_n, dparams, work, red);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_adjoint_moments(dvbm_handle* h, const void* state, const double* d_rho, const double* d_ux,
                         const double* d_uy, const double* d_T, double* lam) {
  if (!h || !state || !lam) return fail(DVBM_EINVAL, "dvbm_adjoint_moments: NULL argument");
  if (int rc = adjoint_storage_ok(h, "dvbm_adjoint_moments")) return rc;
  dispatch_adjoint<ReadoutAdjointOp>(h->p, h, state, d_rho, d_ux, d_uy, d_T, lam);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_stream_probe(const void* src, void* dst, size_t bytes, int32_t mode, int32_t width, void* stream) {
  const int m = mode & 3;
  const bool nt = (mode & 4) != 0;
  if (mode < 0 || mode > 6 || m > 2 || (width != 16 && width != 4) || bytes < size_t(width) ||
      bytes % size_t(width))
    return fail(DVBM_EINVAL,
                "dvbm_stream_probe: mode 0..2 (+4 non-temporal), width 16 or 4, bytes a positive multiple of width");
  if ((m != 2 && !src) || !dst) return fail(DVBM_EINVAL, "dvbm_stream_probe: NULL buffer");
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % size_t(width))
    return fail(DVBM_EINVAL, "dvbm_stream_probe: buffers must be aligned to width");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t n = int64_t(bytes / size_t(width));
  // about four elements per thread (measured fastest for 4 GiB; fewer, longer-running blocks lose up to 20 %)
  const int64_t want = (n + 4 * 256 - 1) / (4 * 256);
  const dim3 grid(unsigned(want < (int64_t(1) << 20) ? want : (int64_t(1) << 20))), block(256);
  auto launch = [&](auto kern, auto* sp, auto* dp) { hipLaunchKernelGGL(kern, grid, block, 0, s, sp, dp, n, m); };
  if (width == 16) {
    const auto* sp = static_cast<const u32x4*>(src);
    auto* dp = static_cast<u32x4*>(dst);
    if (nt) launch(k_stream<u32x4, true>, sp, dp);
    else launch(k_stream<u32x4, false>, sp, dp);
  } else {
    const auto* sp = static_cast<const uint32_t*>(src);
    auto* dp = static_cast<uint32_t*>(dst);
    if (nt) launch(k_stream<uint32_t, true>, sp, dp);
    else launch(k_stream<uint32_t, false>, sp, dp);
  }
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_limiter_signature(dvbm_handle* h, const void* state, uint64_t* sig) {
  if (!h || !state || !sig) return fail(DVBM_EINVAL, "dvbm_limiter_signature: NULL argument");
  if (h->p.storage != DVBM_F64) return fail(DVBM_EINVAL, "dvbm_limiter_signature: float64 storage only");
  if (h->p.bc_y == DVBM_WALL) return fail(DVBM_EINVAL, "dvbm_limiter_signature: walls are not supported");
  const double* X = static_cast<const double*>(state);
  auto* out = reinterpret_cast<unsigned long long*>(sig);
  const bool px = h->p.bc_x == DVBM_PERIODIC, py = h->p.bc_y == DVBM_PERIODIC;
  const dim3 grid(RED_BLOCKS), block(256);
  auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, h->stream, X, h->kp, out); };
  if (h->p.split == 2) {
    if (px && py) launch(k_limiter_signature<2, BC_PERIODIC, BC_PERIODIC>);
    else if (py) launch(k_limiter_signature<2, BC_ZERO_GRADIENT, BC_PERIODIC>);
    else if (px) launch(k_limiter_signature<2, BC_PERIODIC, BC_ZERO_GRADIENT>);
    else launch(k_limiter_signature<2, BC_ZERO_GRADIENT, BC_ZERO_GRADIENT>);
  } else {
    if (px && py) launch(k_limiter_signature<1, BC_PERIODIC, BC_PERIODIC>);
    else if (py) launch(k_limiter_signature<1, BC_ZERO_GRADIENT, BC_PERIODIC>);
    else if (px) launch(k_limiter_signature<1, BC_PERIODIC, BC_ZERO_GRADIENT>);
    else launch(k_limiter_signature<1, BC_ZERO_GRADIENT, BC_ZERO_GRADIENT>);
  }
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

int dvbm_adjoint_init(dvbm_handle* h, const double* lam0, const double* rho, const double* ux, const double* uy,
                      const double* T, double* d_rho, double* d_ux, double* d_uy, double* d_T) {
  if (!h || !lam0 || !rho || !ux || !uy || !T) return fail(DVBM_EINVAL, "dvbm_adjoint_init: NULL argument");
  if (h->p.split == 2)
    hipLaunchKernelGGL(k_adjoint_init<2>, dim3(RED_BLOCKS), dim3(256), 0, h->stream, lam0, rho, ux, uy, T, d_rho,
                       d_ux, d_uy, d_T, h->kp);
  else
    hipLaunchKernelGGL(k_adjoint_init<1>, dim3(RED_BLOCKS), dim3(256), 0, h->stream, lam0, rho, ux, uy, T, d_rho,
                       d_ux, d_uy, d_T, h->kp);
  HIP_TRY(hipGetLastError());
  return DVBM_OK;
}

}  // extern "C"

#endif  // DVBM_PART
