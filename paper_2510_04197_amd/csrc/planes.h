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
//   float16 deviations, 16 populations, 509 x 383  12.2 (17.1)
#pragma once

#include "step.h"
#include "sweep.h"

namespace dvbm {

// Coefficients a_(p,q), p + q <= N, of one Grad expansion.
constexpr int n_coeffs(int N) { return (N + 1) * (N + 2) / 2; }

// Double-buffered by row parity.
template <int SPLIT, class R>
struct PlanesShared {
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

// Moments of one cell (lane) from the columns' sums, and the collision
// coefficients of distribution D, in the order p, q, then om1.
template <int SPLIT, class S, int PRM, int D>
__device__ inline void node_coeffs(const KParams& kp, const double (*fsum)[4][64], const double (*gsum)[2][64],
                                   typename S::C (*out)[64], int lane) {
  using R = typename S::C;
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int N = D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG;
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
  const NodeMoments m = S::dev ? add_rest_moments(mf, mg, kp) : as_moments(mf, mg);
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
template <int SPLIT, class S, int BCX, int BCY, int D>
__device__ __attribute__((always_inline)) inline void planes_walk(const typename S::T* __restrict__ src, typename S::T* __restrict__ dst,
                                   const KParams& kp, int a, int x0, int ya, int yb,
                                   const typename S::T* __restrict__ ghost,
                                   PlanesShared<SPLIT, typename S::C>& sh) {
  using R = typename S::C;
  using T = typename S::T;
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
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

  struct Row { rsrc_t r; uint32_t so, stride; };
  auto row = [&](int yy) -> Row {
    if constexpr (BCY == BC_WALL) {
      if (yy < 0 || yy >= ny) {
        const int g = yy < 0 ? yy + 2 : (yy - ny < 2 ? yy - ny + 2 : 3);
        const char* p = reinterpret_cast<const char*>(ghost) + size_t(D * Q) * 4 * plane_bytes;
        const rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0, Q * 4 * plane_bytes, RSRC_WORD3);
        return Row{r, uint32_t(g) * plane_bytes + pl0 * 4 * plane_bytes, 4 * plane_bytes};
      }
      return Row{row_rsrc(src, D, dist_bytes, yy, row_bytes), pl0 * plane_bytes, plane_bytes};
    } else {
      return Row{row_rsrc(src, D, dist_bytes, wrap<BCY>(yy, ny), row_bytes), pl0 * plane_bytes, plane_bytes};
    }
  };
  auto load = [&](const Row& r, int b, uint32_t lo) -> R {
    return Bits<T>::keep(Buf<T>::ld(r.r, r.so + uint32_t(b) * r.stride, lo));
  };
  auto face = [&](R u, R c, R n) -> R { return add_quarter(c, lim4_walk(c - u, n - c, beta2)); };

  R win[N1][RG], fbelow[N1];
  {
    R extra[N1];
#pragma unroll
    for (int dy = -2; dy <= RG - 1; ++dy) {
      const Row r = row(ya + dy);
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
        for (int q = 0; p + q <= N; ++q, ++k) e[q] += hp[p] * (D == 0 ? sh.cf[par][k][col] : sh.cg[par][k][col]);
    }
    const R om1 = D == 0 ? sh.cf[par][n_coeffs(N)][col] : sh.cg[par][n_coeffs(N)][col];
    const Row rp = row(y + RG - 1), rn = row(y + RG);
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

template <int SPLIT, class S, int PRM, int D>
__device__ __attribute__((always_inline)) inline void planes_coeffs(const KParams& kp, int n, PlanesShared<SPLIT, typename S::C>& sh) {
  const int lane = threadIdx.x & 63;
  for (int k = 0; k < n; ++k) {
    __syncthreads();
    node_coeffs<SPLIT, S, PRM, D>(kp, sh.fsum[k & 1], sh.gsum[k & 1], D == 0 ? sh.cf[k & 1] : sh.cg[k & 1], lane);
  }
  __syncthreads();
}

}  // namespace dvbm
