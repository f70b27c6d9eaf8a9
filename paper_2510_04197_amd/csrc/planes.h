// Plane-group form of the fused DDF-QE DVBM step: the kernel of grids too
// small to fill the device with the column sweep, and of walls in y.
//
// A workgroup advances a strip of SWEEP_OWN columns over a range of rows with
// 2 N1 + 2 waves.  Wave (d, a) walks the N1 planes (a, b), b = 0 .. N1-1, of
// distribution d up the rows; as in the column sweep the x neighbours come
// from the adjacent lanes, the rows of the y stencil stay in registers and
// every face value is formed once.  A plane wave leaves its planes' share of
// the next row's float64 moments in LDS; the last two waves, one per
// distribution, turn the shares of a row into its collision coefficients
// while the plane waves advect the row before it, so a row costs one barrier.
//
// On such grids the length of one thread's chain bounds the step: one thread
// per cell runs 2000 to 3300 vector instructions behind 290 loads with at
// most one wave per SIMD to hide them.  Here a wave runs a tenth of that per
// row, and a CU holds 12 waves (float64: 153 registers, one workgroup) or 24.
// Measured, us per step, against the one-thread-per-cell kernels (float64:
// with LDS tiles; other storages: all stencils through the caches):
//   float64  64^2 6.0 (19.3), 256^2 15.0 (23.9), 512^2 39 (58)
//   float64, 16 populations, 512 x 4  4.9 (13.6)
//   float32 deviations  64^2 4.4 (9.3), 256^2 9.0 (11.8), 512^2 21.8 (30.5)
//   float16 deviations, 16 populations, 509 x 383  12.1 (17.1)
//   thermal Couette flow between walls, float64, 4 x 128  9.1 (38.6)
// No-slip walls: a range next to a wall forms the ghost rows it reads itself,
// by the same exchange (shares of the two mirrored rows, the difference of the
// two equilibria's coefficients, expansion), two barriers per wall; a
// kernel of its own for them took 4.6 us of the 13.4 us a step then took.
#pragma once

#include "step.h"
#include "sweep.h"

namespace dvbm {

// Coefficients a_(p,q), p + q <= N, of one Grad expansion.
constexpr int n_coeffs(int N) { return (N + 1) * (N + 2) / 2; }

// With walls: by distance k from the wall, the ghost row's equilibrium
// coefficients less those of the row it mirrors.
template <int SPLIT, bool WALL>
struct PlanesWall {};
template <int SPLIT>
struct PlanesWall<SPLIT, true> {
  double wf[2][n_coeffs(Set<SPLIT>::NF)][64];
  double wg[2][n_coeffs(Set<SPLIT>::NG)][64];
};

// Double-buffered by row parity.
template <int SPLIT, class R, bool WALL>
struct PlanesShared : PlanesWall<SPLIT, WALL> {
  static constexpr int N1 = Set<SPLIT>::N1;
  double fsum[2][N1][4][64];                      // sums over b of xi_b^k f, k = 0..3, per column a
  double gsum[2][N1][2][64];                      // of xi_b^k g, k = 0, 1
  R cf[2][n_coeffs(Set<SPLIT>::NF) + 1][64];      // f: coefficients, then om1
  R cg[2][n_coeffs(Set<SPLIT>::NG) + 1][64];      // g
};

// A value that is the same in every lane, kept in scalar registers.
__device__ inline float uniform(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ inline double uniform(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(int(uint32_t(b)));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(int(uint32_t(b >> 32)));
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// Keeps the value's computation at this place: values carried from row to row
// would otherwise be sunk into the next row step, with everything they are
// computed from.
template <class R>
__device__ inline void here(R& v) { asm volatile("" : "+v"(v)); }
// An LDS address that the accesses at constant offsets share (beyond the first
// 64 KiB of a block each access gets an address register of its own otherwise).
template <class P>
__device__ inline P* lds_base(P* p) {
  using Q = __attribute__((address_space(3))) P*;
  Q q = (Q)p;
  asm volatile("" : "+v"(q));
  return (P*)q;
}

// Moments of one cell (lane) from the columns' sums.
template <int SPLIT, class S>
__device__ inline NodeMoments lane_moments(const KParams& kp, const double (*fsum)[4][64], const double (*gsum)[2][64],
                                           int lane) {
  constexpr int N1 = Set<SPLIT>::N1;
  double mf[10], mg[3];
  fold_columns<0, N1, S::dev>(
      [&](int k, double& s0, double& s1, double& s2, double& s3) {
        s0 = fsum[k][0][lane];
        s1 = fsum[k][1][lane];
        s2 = fsum[k][2][lane];
        s3 = fsum[k][3][lane];
      },
      mf);
  fold_columns<1, N1, S::dev>(
      [&](int k, double& s0, double& s1, double& s2, double& s3) {
        s0 = gsum[k][0][lane];
        s1 = gsum[k][1][lane];
        s2 = s3 = 0.0;
      },
      mg);
  return S::dev ? add_rest_moments(mf, mg, kp) : as_moments(mf, mg);
}

// The collision coefficients of distribution D in the order p, q, then om1.
template <int SPLIT, class S, int PRM, int D>
__device__ inline void node_coeffs(const KParams& kp, const double (*fsum)[4][64], const double (*gsum)[2][64],
                                   typename S::C (*out)[64], int lane) {
  using R = typename S::C;
  constexpr int N = D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG;
  const NodeMoments m = lane_moments<SPLIT, S>(kp, fsum, gsum, lane);
  R bf[5][5], bg[3][3], om1;
  collision_coeffs<SPLIT, PRM, R>(m, kp, kp.om_scale, kp.Pr, bf, bg, om1);
  if constexpr (S::dev) subtract_rest<SPLIT>(bf, bg, om1, kp);
  int k = 0;
#pragma unroll
  for (int p = 0; p <= N; ++p)
#pragma unroll
    for (int q = 0; p + q <= N; ++q, ++k) out[k][lane] = D == 0 ? bf[p][q] : bg[p][q];
  out[k][lane] = om1;
}

// Equilibrium coefficients of distribution D (order p, q) added to out with a
// sign: rho, the normalised velocity and T (Sec. II D 2, Apps. A and D).
template <int SPLIT, int D>
__device__ inline void add_equilibrium_coeffs(double sign, double rho, double ux, double uy, double T,
                                              const KParams& kp, double* out) {
  constexpr int N = D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG;
  const double RT = kp.R * T, th = RT / kp.c2, p = rho * RT;
  double mx[5], my[5];
  gauss_hermite_moments(ux, th - 1.0, mx);
  gauss_hermite_moments(uy, th - 1.0, my);
  if (D == 0 || SPLIT == 2) {
    const double w = sign * (D == 0 ? rho : rho * (kp.Cv - kp.R) * T);
    int k = 0;
#pragma unroll
    for (int a = 0; a <= N; ++a)
#pragma unroll
      for (int b = 0; a + b <= N; ++b, ++k) out[k] += w * mx[a] * my[b];
  } else {  // order (0,0) (0,1) (0,2) (1,0) (1,1) (2,0)
    const double E = rho * kp.Cv * T + 0.5 * rho * kp.c2 * (ux * ux + uy * uy);
    const double Ep = E + p, E2p = E + 2.0 * p, diag = Ep * th - E;
    out[0] += sign * E;
    out[1] += sign * uy * Ep;
    out[2] += sign * (E2p * uy * uy + diag);
    out[3] += sign * ux * Ep;
    out[4] += sign * E2p * ux * uy;
    out[5] += sign * (E2p * ux * ux + diag);
  }
}

// No-slip wall w (0: below row 0, 1: above row ny - 1): from the shares of the
// two rows next to it (slot k: k rows away), the coefficients X^eq(G) - X^eq(B)
// of distribution D, with the ghost fields rho_G = rho_B, u_G = 2 u_W - u_B,
// T_G = 2 T_W - T_B.
template <int SPLIT, class S, int D, class SH>
__device__ inline void wall_coeffs(const KParams& kp, int w, SH& sh) {
  constexpr int M = n_coeffs(D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG);
  const int lane = threadIdx.x & 63;
  __syncthreads();
  for (int k = 0; k < 2; ++k) {
    const NodeMoments m = lane_moments<SPLIT, S>(kp, sh.fsum[k], sh.gsum[k], lane);
    const double irho = 1.0 / m.rho, ux = m.jx * irho, uy = m.jy * irho;
    const double E = SPLIT == 2 ? m.g0 + 0.5 * kp.c2 * (m.pxx + m.pyy) : m.g0;
    const double T = (E * irho - 0.5 * kp.c2 * (ux * ux + uy * uy)) * kp.inv_Cv;
    double d[M];
#pragma unroll
    for (int j = 0; j < M; ++j) d[j] = 0.0;
    add_equilibrium_coeffs<SPLIT, D>(1.0, m.rho, 2.0 * kp.wall_ux[w] / sqrt(kp.c2) - ux, -uy, 2.0 * kp.wall_T[w] - T,
                                     kp, d);
    add_equilibrium_coeffs<SPLIT, D>(-1.0, m.rho, ux, uy, T, kp, d);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      if constexpr (D == 0) sh.wf[k][j][lane] = d[j];
      else sh.wg[k][j][lane] = d[j];
    }
  }
  __syncthreads();
}

// Rows held per plane: the rows y-1 .. y+2 (xi_b > 0) or y .. y+3, the last one
// or two in flight.  The moments of row y + 1 are summed at the start of row
// step y, so a ring of three would leave a row of xi_b > 0 less than one
// row step to arrive.
constexpr int PLANES_RING = 4;

// Rows [ya, yb) of the planes (a, .) of distribution D in the strip whose first
// owned column is x0.  Waves of xi_a < 0 hold the columns in reverse, so that
// the upwind neighbour is the lane before for every wave: mirrored, the face
// formulas of both directions are the same, with the speed's magnitude.
// Lanes 2 .. 61 own their cells, as in the column sweep.
// Window of plane (a, b): ring row r holds row y - 1 + r when xi_b > 0, y + r
// otherwise; at phase P = (y - ya) % ring it is in register (P + r) % ring.
// A row is requested when the window drops one, and decoded at its first use.
// (Inlined by force: with several callers it would become a call, whose
// registers go through scratch.)
template <int SPLIT, class S, int BCX, int BCY, int D>
__device__ __attribute__((always_inline)) inline void planes_walk(
    const typename S::T* __restrict__ src, typename S::T* __restrict__ dst, const KParams& kp, int a, int x0, int ya,
    int yb, PlanesShared<SPLIT, typename S::C, BCY == BC_WALL>& sh) {
  using R = typename S::C;
  using T = typename S::T;
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int N = D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG;
  constexpr uint32_t SZ = sizeof(T);
  constexpr int RG = PLANES_RING;
  using L = GH<N1>;

  const int lane = threadIdx.x & 63;
  const double xa = L::xi(a);
  const int col = xa < 0.0 ? 63 - lane : lane;
  const int x = x0 - 2 + col;
  const bool own = col >= 2 && col < 62 && x < kp.nx;
  // (x < nx + 62: on grids of at least a strip one wrap suffices)
  const uint32_t vo = uint32_t(kp.nx >= 64 ? wrap<BCX>(x, kp.nx) : wrap_any<BCX>(x, kp.nx)) * SZ;
  const uint32_t vo_st = own ? vo : 0x80000000u;
  const uint32_t row_bytes = uint32_t(kp.srow) * SZ;
  const uint32_t plane_bytes = uint32_t(kp.pitch) * SZ;
  const uint32_t dist_bytes = uint32_t(kp.sdist) * SZ;
  const int ny = kp.ny;
  const uint32_t pl0 = uint32_t(a * N1);
  const R beta2 = uniform(R(kp.beta2));
  const R kvx = uniform(R(kp.kx) * R(xa < 0.0 ? -xa : xa));
  R kvy[N1];
#pragma unroll
  for (int b = 0; b < N1; ++b) kvy[b] = uniform(R(kp.ky) * R(L::xi(b)));
  const double wa = S::dev ? 1.0 : L::w(a);
  R hp[N + 1];
#pragma unroll
  for (int p = 0; p <= N; ++p) hp[p] = uniform(R(wa * hn(p, xa)));

  // (with walls, rows outside the domain read the edge row and are replaced)
  auto row = [&](int yy) -> rsrc_t { return row_rsrc(src, D, dist_bytes, wrap<BCY>(yy, ny), row_bytes); };
  auto load = [&](rsrc_t r, int b, uint32_t lo) -> R {
    return Bits<T>::keep(Buf<T>::ld(r, (pl0 + uint32_t(b)) * plane_bytes, lo));
  };
  auto face = [&](R u, R c, R n) -> R {
    if constexpr (sizeof(T) == 2) return add_quarter(c, lim4_walk16(c - u, n - c, beta2));
    else return add_quarter(c, lim4_walk(c - u, n - c, beta2));
  };

  auto coeff = [&](int par, int k) -> R {
    if constexpr (D == 0) return sh.cf[par][k][col];
    else return sh.cg[par][k][col];
  };
  auto share = [&](const R* v, int s) {
    double s0, s1, s2, s3;
    if constexpr (S::dev) weighted_pair_sums<N1>(v, s0, s1, s2, s3);
    else pair_sums<N1>(v, s0, s1, s2, s3);
    if (D == 0) {
      sh.fsum[s][a][0][col] = s0;
      sh.fsum[s][a][1][col] = s1;
      sh.fsum[s][a][2][col] = s2;
      sh.fsum[s][a][3][col] = s3;
    } else {
      sh.gsum[s][a][0][col] = s0;
      sh.gsum[s][a][1][col] = s1;
    }
  };
  R win[N1][RG], fbelow[N1];
  R above[2][N1];  // with a wall above the range: its ghost rows
  {
    R extra[N1];
#pragma unroll
    for (int dy = -2; dy <= RG - 1; ++dy) {
      const rsrc_t r = row(ya + dy);
      static_for<N1>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        constexpr double xb = L::xi(b);
        if (xb > 0.0) {
          if (dy == -2) extra[b] = load(r, b, vo);
          else if (dy <= RG - 2) win[b][dy + 1] = load(r, b, vo);
        } else if (xb < 0.0) {
          if (dy == -1) extra[b] = load(r, b, vo);
          else if (dy >= 0) win[b][dy] = load(r, b, vo);
        } else if (dy >= 0) {
          win[b][dy] = load(r, b, vo);
        }
      });
    }
    if constexpr (BCY == BC_WALL) {
      // populations of the wall's ghost row k (as stored): X^eq(G) + (X_B - X^eq(B))
      auto ghosts = [&](int w, R (&out)[2][N1]) {
        R vb[2][N1];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const rsrc_t r = row(w == 0 ? k : ny - 1 - k);
#pragma unroll
          for (int b = 0; b < N1; ++b) vb[k][b] = load(r, b, vo);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
          for (int b = 0; b < N1; ++b) vb[k][b] = Bits<T>::decode(vb[k][b]);
          share(vb[k], k);
        }
        __syncthreads();
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          double e[N + 1];
#pragma unroll
          for (int q = 0; q <= N; ++q) e[q] = 0.0;
          int j = 0;
#pragma unroll
          for (int p = 0; p <= N; ++p)
#pragma unroll
            for (int q = 0; p + q <= N; ++q, ++j) {
              const double h = wa * hn(p, xa);
              if constexpr (D == 0) e[q] += h * sh.wf[k][j][col];
              else e[q] += h * sh.wg[k][j][col];
            }
#pragma unroll
          for (int b = 0; b < N1; ++b) {
            double v = double(vb[k][b]);
#pragma unroll
            for (int q = 0; q <= N; ++q) v += (S::dev ? 1.0 : L::w(b)) * hn(q, L::xi(b)) * e[q];
            out[k][b] = Bits<T>::keep(S::enc64(v, 1.0, 0.0));
          }
        }
      };
      if (ya < 2) {
        R g[2][N1];
        ghosts(0, g);
#pragma unroll
        for (int b = 0; b < N1; ++b) {
          if (L::xi(b) > 0.0) {
            extra[b] = g[1 - ya][b];
            if (ya == 0) win[b][0] = g[0][b];
          } else if (L::xi(b) < 0.0 && ya == 0) {
            extra[b] = g[0][b];
          }
        }
      }
      if (yb > ny - 2) {
        ghosts(1, above);
#pragma unroll
        for (int dy = 0; dy <= RG - 1; ++dy) {
          const int k = ya + dy - ny;
          if (k < 0) continue;
#pragma unroll
          for (int b = 0; b < N1; ++b) {
            const R v = k == 0 ? above[0][b] : above[1][b];
            if (L::xi(b) > 0.0 && dy <= RG - 2) win[b][dy + 1] = v;
            if (L::xi(b) < 0.0) win[b][dy] = v;
          }
        }
      }
    }
    static_for<N1>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      constexpr double xb = L::xi(b);
      win[b][0] = Bits<T>::decode(win[b][0]);
      if (xb != 0.0) {
        win[b][1] = Bits<T>::decode(win[b][1]);
        const R e = Bits<T>::decode(extra[b]);
        fbelow[b] = xb > 0.0 ? face(e, win[b][0], win[b][1]) : face(win[b][1], win[b][0], e);
      }
    });
  }
  {
    R v[N1];
#pragma unroll
    for (int b = 0; b < N1; ++b) v[b] = L::xi(b) > 0.0 ? win[b][1] : win[b][0];
    share(v, 0);
  }
  __syncthreads();

  auto row_step = [&](auto phc, auto movc, int y) {
    constexpr int P = decltype(phc)::value;
    constexpr bool MOV = decltype(movc)::value;  // xi_a != 0
    const int par = (y - ya) & 1;
    // row y + 1: decoded where this is its first use, its share of the moments
    {
      R v[N1];
      static_for<N1>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        constexpr double xb = L::xi(b);
        constexpr int s = xb > 0.0 ? (P + 2) % RG : (P + 1) % RG;
        if (xb >= 0.0) win[b][s] = Bits<T>::decode(win[b][s]);
        v[b] = win[b][s];
      });
      if (y + 1 < yb) share(v, par ^ 1);
    }
    __syncthreads();
    R e[N + 1];
#pragma unroll
    for (int q = 0; q <= N; ++q) e[q] = R(0);
    {
      int k = 0;
#pragma unroll
      for (int p = 0; p <= N; ++p)
#pragma unroll
        for (int q = 0; p + q <= N; ++q, ++k) e[q] += hp[p] * coeff(par, k);
    }
    const R om1 = coeff(par, n_coeffs(N));
    const rsrc_t rp = row(y + RG - 1), rn = row(y + RG);
    const uint32_t vo_pos = y + RG - 1 <= yb ? vo : 0x80000000u;
    const uint32_t vo_neg = y + RG <= yb + 1 ? vo : 0x80000000u;
    const uint32_t vo_own = y + RG < yb ? vo : 0x80000000u;
    const rsrc_t rd = row_rsrc(dst, D, dist_bytes, y, row_bytes);
    static_for<N1>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      constexpr double xb = L::xi(b);
      R* wn = win[b];
      const R c0 = xb > 0.0 ? wn[(P + 1) % RG] : wn[P];
      R xn = -om1 * c0;
#pragma unroll
      for (int q = 0; q <= N; ++q) {
        const double h = (S::dev ? 1.0 : L::w(b)) * hn(q, xb);
        if (h != 0.0) xn += R(h) * e[q];
      }
      if constexpr (MOV) {
        const R d = c0 - lane_prev(c0);
        const R fr = add_quarter(c0, lim4_walk(d, lane_next(d), beta2));  // face downwind
        xn -= kvx * (fr - lane_prev(fr));
      }
      if (xb != 0.0) {
        if (xb < 0.0) wn[(P + 2) % RG] = Bits<T>::decode(wn[(P + 2) % RG]);
        const R r0 = wn[P], r1 = wn[(P + 1) % RG], r2 = wn[(P + 2) % RG];
        const R fa = xb > 0.0 ? face(r0, r1, r2) : face(r2, r1, r0);
        xn -= kvy[b] * (fa - fbelow[b]);
        fbelow[b] = fa;
      }
      const R xnew = c0 + xn;
      T out;
      if constexpr (S::dev) out = S::enc_dev(xnew);
      else out = S::enc(xnew, R(1), R(0));
      Buf<T>::st(rd, (pl0 + b) * plane_bytes, vo_st, out);
      const int k = xb > 0.0 ? y + RG - 1 - ny : y + RG - ny;
      if (BCY == BC_WALL && xb != 0.0 && k >= 0)
        wn[P] = k == 0 ? above[0][b] : above[1][b];
      else
        wn[P] = load(xb > 0.0 ? rp : rn, b, xb > 0.0 ? vo_pos : (xb < 0.0 ? vo_neg : vo_own));
    });
  };
  auto walk = [&](auto mov) {
    int y = ya;
    for (;;) {
      row_step(std::integral_constant<int, 0>(), mov, y);
      if (++y >= yb) break;
      row_step(std::integral_constant<int, 1>(), mov, y);
      if (++y >= yb) break;
      row_step(std::integral_constant<int, 2>(), mov, y);
      if (++y >= yb) break;
      row_step(std::integral_constant<int, 3>(), mov, y);
      if (++y >= yb) break;
    }
  };
  if (xa != 0.0) walk(std::true_type());
  else walk(std::false_type());
}

template <int SPLIT, class S, int PRM, int D, class SH>
__device__ __attribute__((always_inline)) inline void planes_coeffs(const KParams& kp, int n, SH& sh) {
  const int lane = threadIdx.x & 63;
  for (int k = 0; k < n; ++k) {
    __syncthreads();
    node_coeffs<SPLIT, S, PRM, D>(kp, sh.fsum[k & 1], sh.gsum[k & 1], D == 0 ? sh.cf[k & 1] : sh.cg[k & 1], lane);
  }
  __syncthreads();
}

}  // namespace dvbm
