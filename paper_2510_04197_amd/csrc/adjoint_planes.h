// Discrete adjoint step over plane groups.  The value formats (float64,
// float32) take it in one sweep.  The float32 deviations keep the flux sweep,
// and share the relaxation part on small grids.  Their neighbours are often stored
// equal, exactly on the limiter's kink, where the flux sweep follows the rounding
// of the decoded difference; branches taken from the stored deviations, as one
// sweep would, give the derivative zero there and so other results (333 x 250,
// relative L2 1.7e-5 of lam; both as far from those of unrounded populations,
// 3.5e-5 and 3.7e-5).
#pragma once

#include "adjoint.h"
#include "planes.h"

namespace dvbm {

// (g dL/da, g dL/db) of L(a, b) = (b/2) phi(a, b) = 1/2 minmod(beta a, (a+b)/2, beta b)
// on the branch the forward evaluation takes: the smallest of beta |a|,
// |a + b| / 2 and beta |b|, the first in this order on ties, 0 unless a b > 0.
// With |a| <= |b| the second wins when 2 beta |a| > |a + b|, otherwise when
// 2 beta |b| >= |a + b|; both derivatives are then 1/4, else the smaller
// argument's is beta / 2.
__device__ inline void lim_pullback(double a, double b, double beta2, double g, double& ga, double& gb) {
  const double s = fabs(a + b), m = beta2 * fmin(fabs(a), fabs(b));
  const bool act = a * b > 0.0, ale = fabs(a) <= fabs(b);
  const bool mid = (m > s) | ((m >= s) & !ale);
  const double ug = (mid ? 0.25 : 0.25 * beta2) * g;
  ga = (act & (mid | ale)) ? ug : 0.0;
  gb = (act & (mid | !ale)) ? ug : 0.0;
}

// ------------------------------------------------------------ adjoint step, row sweep
// The step adjoint of the value formats as one sweep, with the plane groups of the step kernel of
// small grids: a workgroup takes a strip of SWEEP_OWN columns and a range of
// rows with 2 N1 + 2 waves.  Wave (d, a) walks the N1 planes (a, b) of
// distribution d upwards and assembles, row after row,
//   lam(c) = (1 - om1) lam'(c) + sum_r mbar_r dm_r/dX + flux cotangent.
// The moment cotangents mbar of a row need all 2Q planes: each plane wave
// leaves its planes' share of the row's moments and of the lam'-weighted
// Hermite projections in LDS two rows ahead, and the last two waves take the
// reverse pass coeffs_vjp of alternate rows, each over two row steps, while the
// plane waves work on the rows before.  One barrier per row; X and lam' are
// read once and lam written once.

template <int SPLIT>
struct AdjointShares {
  static constexpr int N1 = Set<SPLIT>::N1, NF = Set<SPLIT>::NF;
  // shares by row parity and column a: sums over b of xi_b^k X (f: k = 0..3,
  // g: 0, 1), of lam' w_b He_q(xi_b)/q! (q = 0..NF, 0..2), and of lam' X
  double fsh[2][N1][4 + NF + 1 + 1][64];
  double gsh[2][N1][2 + 3 + 1][64];
};
// (res first: within 64 KiB of the block's base an access needs no address of
// its own)
template <int SPLIT>
struct AdjointResults {
  double res[2][ADJ_WORK_ROWS][64];  // mbar, then 1 - om1
};
template <int SPLIT>
struct AdjointShared : AdjointResults<SPLIT>, AdjointShares<SPLIT> {
  static constexpr int N1 = Set<SPLIT>::N1;
  double lam[2 * N1][2][N1][64];  // lam' of the last two rows of every wave, by row parity
};

// One wave's share of a cell: from its planes' X and lam', to out[64 j].
template <int SPLIT, int D>
__device__ inline void adjoint_share(const double* v, const double* l, double* out) {
  constexpr int N1 = Set<SPLIT>::N1, N = D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG, K = D == 0 ? 4 : 2;
  using L = GH<N1>;
  double t[N + 1], s = 0.0, m0, m1, m2, m3;
  pair_sums<N1>(v, m0, m1, m2, m3);
#pragma unroll
  for (int q = 0; q <= N; ++q) t[q] = 0.0;
#pragma unroll
  for (int b = 0; b < N1; ++b) {
#pragma unroll
    for (int q = 0; q <= N; ++q) {
      const double h = L::w(b) * hn(q, L::xi(b));
      if (h != 0.0) t[q] += l[b] * h;
    }
    s += l[b] * v[b];
  }
  double* o = lds_base(out);
  o[0] = m0;
  o[64] = m1;
  if (D == 0) {
    o[2 * 64] = m2;
    o[3 * 64] = m3;
  }
#pragma unroll
  for (int q = 0; q <= N; ++q) o[(K + q) * 64] = t[q];
  o[(K + N + 1) * 64] = s;
}

// Along x, lane l forms the face between its column and the one before (waves
// of xi_a < 0 hold the columns in reverse, so the lane before is upwind for
// every wave), and the face's three partials reach their cells through lane
// shifts.  Under the zero-gradient rule columns outside the domain are copies
// of the edge column and carry no lam'; they hand their share to it.
// Along y every face is formed once.  With row r = c + 2 the wave forms face r
// (xi_b > 0) or face r-1 (xi_b < 0); in both cases its three inputs are the
// rows r-2, r-1, r and its three partials belong to them, so the sums of the
// rows r-1 and r (with their own x shares) are carried on (p1, p2) and row
// c = r-2 is finished.  The walk starts two rows early, at c = ya - 2, to
// collect the shares of the faces below ya.  Under the zero-gradient rule the
// rows outside the domain are copies of the edge rows and carry no lam':
// their shares (the rows -2, -1 and ny, ny+1) go to the edge rows.
// Registers bound the occupancy (12 waves, 168 each): of X and lam' the rows
// r-1 and r and one in flight are kept, with the last differences; lam' of row c
// waits in LDS.  MOV: xi_a != 0 (a function each: the registers fit).
template <int SPLIT, class S, int BCX, int BCY, int D, bool MOV, class LT>
__device__ __attribute__((always_inline)) inline void adjoint_walk(const typename S::T* __restrict__ state, const LT* __restrict__ lam1,
                                    LT* __restrict__ lam0, const KParams& kp, int a, int x0, int ya, int yb,
                                    AdjointShared<SPLIT>& sh) {
  static_assert(!S::dev, "value formats");
  using T = typename S::T;
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  constexpr int N = D == 0 ? Set<SPLIT>::NF : Set<SPLIT>::NG;
  constexpr bool ZGY = BCY != BC_PERIODIC;
  constexpr bool XF64 = sizeof(T) == 8, LF64 = sizeof(LT) == 8;
  using L = GH<N1>;
  const int ny = kp.ny;
  const int lane = threadIdx.x & 63;
  const double xa = L::xi(a);
  const bool mirror = xa < 0.0;
  const int col = mirror ? 63 - lane : lane;
  const int x = x0 - 2 + col;
  const bool own = col >= 2 && col < 62 && x < kp.nx;
  const int gx = kp.nx >= 64 ? wrap<BCX>(x, kp.nx) : wrap_any<BCX>(x, kp.nx);
  const bool inx = BCX == BC_PERIODIC || (x >= 0 && x < kp.nx);
  const double beta2 = uniform(kp.beta2);
  const double kvx = uniform(kp.kx * (mirror ? -xa : xa));
  const uint32_t vo = uint32_t(gx) * uint32_t(sizeof(T));
  const uint32_t row_bytes = uint32_t(kp.srow) * uint32_t(sizeof(T));
  const uint32_t plane_bytes = uint32_t(kp.pitch) * uint32_t(sizeof(T));
  const uint32_t dist_bytes = uint32_t(kp.sdist) * uint32_t(sizeof(T));
  const uint32_t pl0 = uint32_t(a * N1);
  // cotangents: dense rows of nx values; one buffer resource per row covers the
  // row's N1 planes (below 2^31 bytes: a distribution of 4-byte values or
  // wider stays below 4 GiB).  The lanes that own no cell store to offset 2^31,
  // which the bounds check discards, so no branch guards the stores
  const uint32_t lrow_bytes = uint32_t(kp.nx) * uint32_t(sizeof(LT));
  const uint32_t lplane_bytes = lrow_bytes * uint32_t(ny);
  const size_t lbase = size_t(D * Q + a * N1) * size_t(lplane_bytes);
  auto lrow = [&](const LT* p, int yy) -> rsrc_t {
    const char* q = reinterpret_cast<const char*>(p) + lbase + size_t(yy) * lrow_bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(q), 0, (N1 - 1) * lplane_bytes + lrow_bytes, RSRC_WORD3);
  };
  const uint32_t lvo = uint32_t(gx) * uint32_t(sizeof(LT));
  const uint32_t lvo_st = own ? lvo : 0x80000000u;
  double kvy[N1];
#pragma unroll
  for (int b = 0; b < N1; ++b) kvy[b] = uniform(kp.ky * (L::xi(b) > 0.0 ? L::xi(b) : -L::xi(b)));  // one per +-xi_b
  const double xa2 = uniform(xa * xa), xa3 = uniform(xa * xa * xa), xau = uniform(xa);

  double X[N1][3], Lm[N1][3];              // rows r - 1, r and the one in flight
  double dp[N1], dlp[N1], p1[N1], p2[N1];  // differences of the rows r - 1 and r - 2; carried sums
  double gs[N1];
  T xin[N1];  // the row in flight, where it is not float64
  LT lin[N1];
  double zf[3];  // 1 inside the domain, 0 for the rows outside (zero-gradient)
#pragma unroll
  for (int b = 0; b < N1; ++b) p1[b] = p2[b] = gs[b] = 0.0;

  // request row r into ring slot s, by way of (xi, li) where it is not float64;
  // rows past the last needed one (yb + 1) read nothing (offset 2^31)
  auto request = [&](auto slot, int r, T* xi, LT* li) {
    constexpr int s = decltype(slot)::value;
    const int ry = wrap<BCY>(r, ny);
    zf[s] = (!ZGY || (r >= 0 && r < ny)) ? 1.0 : 0.0;
    const rsrc_t rx = row_rsrc(state, D, dist_bytes, ry, row_bytes), rl = lrow(lam1, ry);
    const uint32_t ox = r <= yb + 1 ? vo : 0x80000000u, ol = r <= yb + 1 ? lvo : 0x80000000u;
#pragma unroll
    for (int b = 0; b < N1; ++b) {
      const T v = Buf<T>::ld(rx, (pl0 + b) * plane_bytes, ox);
      if constexpr (XF64) X[b][s] = v;
      else xi[b] = v;
      const LT l = Buf<LT>::ld(rl, b * lplane_bytes, ol);
      if constexpr (LF64) Lm[b][s] = l;
      else li[b] = l;
    }
  };
  auto arrive = [&](auto slot, const T* xi, const LT* li) {
    constexpr int s = decltype(slot)::value;
#pragma unroll
    for (int b = 0; b < N1; ++b) {
      if constexpr (!XF64) X[b][s] = double(S::raw(xi[b]));
      if constexpr (!LF64) Lm[b][s] = double(li[b]);
    }
  };

  auto step = [&](auto phase, auto outc, int c) {
    constexpr int P = decltype(phase)::value;
    constexpr bool OUT = decltype(outc)::value;  // c >= ya: the row is the range's own
    constexpr int s1 = (P + 1) % 3, s2 = (P + 2) % 3, s3 = P;
    const int par = (c - ya) & 1;
    // row r = c + 2 has arrived; row c + 3 is requested
    arrive(std::integral_constant<int, s2>(), xin, lin);
    request(std::integral_constant<int, s3>(), c + 3, xin, lin);
    if (c + 2 < yb) {
      double v[N1], l[N1];
#pragma unroll
      for (int b = 0; b < N1; ++b) {
        v[b] = X[b][s2];
        l[b] = Lm[b][s2];
      }
      adjoint_share<SPLIT, D>(v, l, D == 0 ? &sh.fsh[par][a][0][col] : &sh.gsh[par][a][0][col]);
    }
    __syncthreads();
    const bool last = ZGY && c == ny - 1;
    const double* w = lds_base(&sh.res[par][0][col]);
    const rsrc_t ro = lrow(lam0, OUT ? c : ya);
    double* lc0 = lds_base(&sh.lam[D * N1 + a][par][0][lane]);
    // relaxation: with xi_a fixed the Hermite polynomial of the moment
    // cotangents is a cubic (f) or linear (g) polynomial in xi_b
    double A0, A1, A2, A3, keep;
    if constexpr (OUT) {
      keep = w[N_MOMENTS * 64];
      if constexpr (D == 0) {
        A0 = w[0 * 64] + w[1 * 64] * xau + w[3 * 64] * xa2 + w[6 * 64] * xa3;
        A1 = w[2 * 64] + w[4 * 64] * xau + w[7 * 64] * xa2;
        A2 = w[5 * 64] + w[8 * 64] * xau;
        A3 = w[9 * 64];
      } else {
        A0 = w[10 * 64] + w[11 * 64] * xau;
        A1 = w[12 * 64];
      }
    }
#pragma unroll
    for (int b = 0; b < N1; ++b) {
      const double xb = L::xi(b);
      __builtin_amdgcn_sched_barrier(0);
      // x of row r: inputs l-2, l-1, l of the face; cell l takes slot 2 of face l, 1 of l+1, 0 of l+2
      double sx = 0.0;
      if constexpr (MOV) {
        const double lc = (BCX == BC_PERIODIC || inx) ? (ZGY ? zf[s2] * Lm[b][s2] : Lm[b][s2]) : 0.0;
        const double d = X[b][s2] - lane_prev(X[b][s2]);
        const double g = kvx * (lc - lane_prev(lc));
        double ga, gb;  // the face's partials: -ga, g + ga - gb, gb
        lim_pullback(lane_prev(d), d, beta2, g, ga, gb);
        sx = gb + lane_next((g - gb) + (ga - lane_next(ga)));
        if (BCX != BC_PERIODIC) {
          const double a1 = lane_prev(sx), a2 = lane_prev(a1), b1 = lane_next(sx), b2 = lane_next(b1);
          if (x == (mirror ? kp.nx - 1 : 0)) sx += a1 + a2;
          if (x == (mirror ? 0 : kp.nx - 1)) sx += b1 + b2;
        }
      }
      // y: the face of this row and the carried sums
      double out = p1[b];
      if (xb != 0.0) {
        const double dn = X[b][s2] - X[b][s1];
        const double dl = ZGY ? zf[s2] * Lm[b][s2] - zf[s1] * Lm[b][s1] : Lm[b][s2] - Lm[b][s1];
        double ga, gb;
        if (xb > 0.0) {  // face r: dL/dface = kv (lam'(r) - lam'(r-1))
          const double g = kvy[b] * dl;
          lim_pullback(dp[b], dn, beta2, g, ga, gb);
          out -= ga;
          p1[b] = p2[b] + (g + (ga - gb));
          p2[b] = sx + gb;
        } else {  // face r-1: dL/dface = kv (lam'(r-1) - lam'(r-2)), kv < 0
          const double g = -kvy[b] * dlp[b];
          lim_pullback(dn, dp[b], beta2, g, ga, gb);
          out += gb;
          p1[b] = p2[b] + (g + (ga - gb));
          p2[b] = sx - ga;
          dlp[b] = dl;
        }
        dp[b] = dn;
        if (last) out += p1[b] + p2[b];  // shares of the rows ny, ny+1
      } else {
        p1[b] = p2[b];
        p2[b] = sx;
      }
      here(p1[b]);
      here(p2[b]);
      if constexpr (!OUT) {
        if (ZGY) gs[b] += out;  // shares of the rows -2, -1 (used when ya == 0)
      } else {
        if (ZGY && c == 0) out += gs[b];
        if constexpr (D == 0) out += A0 + xb * (A1 + xb * (A2 + xb * A3)) + keep * lc0[b * 64];
        else out += A0 + xb * A1 + keep * lc0[b * 64];
        Buf<LT>::st(ro, b * lplane_bytes, lvo_st, LT(out));
      }
      lc0[b * 64] = Lm[b][s2];  // row r takes the place of row r - 2
    }
  };

  int c = ya - 2;
  {
    T x0[N1], x1[N1];
    LT l0[N1], l1[N1];
    request(std::integral_constant<int, 0>(), c, x0, l0);
    request(std::integral_constant<int, 1>(), c + 1, x1, l1);
    request(std::integral_constant<int, 2>(), c + 2, xin, lin);
    arrive(std::integral_constant<int, 0>(), x0, l0);
    arrive(std::integral_constant<int, 1>(), x1, l1);
  }
#pragma unroll
  for (int b = 0; b < N1; ++b) {
    dp[b] = X[b][1] - X[b][0];
    dlp[b] = ZGY ? zf[1] * Lm[b][1] - zf[0] * Lm[b][0] : Lm[b][1] - Lm[b][0];
  }
  const auto out = std::true_type();
  step(std::integral_constant<int, 0>(), std::false_type(), c);
  step(std::integral_constant<int, 1>(), std::false_type(), c + 1);
  c += 2;
  for (;;) {
    step(std::integral_constant<int, 2>(), out, c);
    if (++c >= yb) break;
    step(std::integral_constant<int, 0>(), out, c);
    if (++c >= yb) break;
    step(std::integral_constant<int, 1>(), out, c);
    if (++c >= yb) break;
  }
}

// The reverse pass of the rows k, k + 2, ... of n (k = 0, 1): row r's shares
// are complete at the barrier before its step, its result is there two
// barriers later.  out(r, mbar, 1 - om1) takes it; where own(r), the cell's
// shares of d/dtau_ref and d/dPr are added to g_tau, g_pr.
template <int SPLIT, int PRM, class OWN, class OUT>
__device__ __attribute__((always_inline)) inline void adjoint_coeffs(const KParams& kp, int k, int n, double tau_ref,
                                                                     const AdjointShares<SPLIT>& sh, double& g_tau,
                                                                     double& g_pr, OWN&& own, OUT&& out) {
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int NF = Set<SPLIT>::NF;
  using L = GH<N1>;
  const int lane = threadIdx.x & 63;
  const double tau_factor = uniform(-kp.om_scale / tau_ref);  // d om_scale / d tau_ref
  int left = n + 2;                                           // barriers of the plane waves
  if (k == 1) {
    __syncthreads();
    --left;
  }
  for (int r = k; r < n; r += 2) {
    __syncthreads();
    const double(*fs)[4 + NF + 2][64] = sh.fsh[k];
    const double(*gp)[6][64] = sh.gsh[k];
    double mf[10], mg[3];
    fold_columns<0, N1, false>(
        [&](int j, double& s0, double& s1, double& s2, double& s3) {
          s0 = fs[j][0][lane];
          s1 = fs[j][1][lane];
          s2 = fs[j][2][lane];
          s3 = fs[j][3][lane];
        },
        mf);
    fold_columns<1, N1, false>(
        [&](int j, double& s0, double& s1, double& s2, double& s3) {
          s0 = gp[j][0][lane];
          s1 = gp[j][1][lane];
          s2 = s3 = 0.0;
        },
        mg);
    const NodeMoments m = as_moments(mf, mg);
    // mu[p][q] = sum_a w_a He_p(xi_a)/p! (sum_b lam'_(a,b) w_b He_q(xi_b)/q!)
    double mu_f[5][5], mu_g[3][3], s = 0.0;
#pragma unroll
    for (int p = 0; p < 5; ++p)
#pragma unroll
      for (int q = 0; q < 5; ++q) mu_f[p][q] = 0.0;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int q = 0; q < 3; ++q) mu_g[p][q] = 0.0;
#pragma unroll
    for (int j = 0; j < N1; ++j) {
#pragma unroll
      for (int q = 0; q <= NF; ++q) {
        const double t = fs[j][4 + q][lane];
#pragma unroll
        for (int p = 0; p + q <= NF; ++p) {
          const double h = L::w(j) * hn(p, L::xi(j));
          if (h != 0.0) mu_f[p][q] += h * t;
        }
      }
#pragma unroll
      for (int q = 0; q <= 2; ++q) {
        const double t = gp[j][2 + q][lane];
#pragma unroll
        for (int p = 0; p + q <= 2; ++p) {
          const double h = L::w(j) * hn(p, L::xi(j));
          if (h != 0.0) mu_g[p][q] += h * t;
        }
      }
      s += fs[j][4 + NF + 1][lane] + gp[j][5][lane];
    }
    __syncthreads();
    left -= 2;
    double mbar[N_MOMENTS], d_oms, d_pr, om1;
    coeffs_vjp<SPLIT, PRM>(m, kp, kp.om_scale, kp.Pr, mu_f, mu_g, s, mbar, d_oms, d_pr, om1);
    out(r, mbar, 1.0 - om1);
    if (own(r)) {
      g_tau += d_oms * tau_factor;  // om_scale = dt / tau_ref [/ p_ref]
      g_pr += d_pr;
    }
  }
  for (; left > 0; --left) __syncthreads();
}

// ------------------------------------------------------------ relaxation part alone
// The moment cotangents and 1 - om1 of 64 consecutive cells from cell c0 on,
// into the work array (deviation storage): the plane waves' side.
template <int SPLIT, class S, int D, class LT>
__device__ __attribute__((always_inline)) inline void relax_walk(const typename S::T* __restrict__ state,
                                                                 const LT* __restrict__ lam1, const KParams& kp, int a,
                                                                 int c0, AdjointShares<SPLIT>& sh) {
  static_assert(S::dev, "deviation formats");
  constexpr int N1 = Set<SPLIT>::N1;
  constexpr int Q = Set<SPLIT>::Q;
  using L = GH<N1>;
  const int lane = threadIdx.x & 63, cells = kp.nx * kp.ny;
  const int c = c0 + lane < cells ? c0 + lane : cells - 1, y = c / kp.nx, x = c - y * kp.nx;
  const double xa = L::xi(a);
  double v[N1], l[N1];
#pragma unroll
  for (int b = 0; b < N1; ++b) {
    const double xb = L::xi(b), r = D == 0 ? 1.0 : (SPLIT == 2 ? kp.gr0 : kp.gr0 + kp.gr1 * (xa * xa + xb * xb - 2.0));
    v[b] = L::w(a) * L::w(b) * (r + double(S::raw(state[sidx(kp, D, a * N1 + b, y, x)])));
    l[b] = double(lam1[int64_t(D * Q + a * N1 + b) * cells + c]);
  }
  adjoint_share<SPLIT, D>(v, l, D == 0 ? &sh.fsh[0][a][0][lane] : &sh.gsh[0][a][0][lane]);
  for (int k = 0; k < 3; ++k) __syncthreads();  // (as many as the coefficient waves of one row)
}

}  // namespace dvbm
