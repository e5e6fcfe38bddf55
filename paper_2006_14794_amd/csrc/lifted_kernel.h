// Forward sweep of the signature kernel of lifted paths (the static-kernel
// lift of eq. (PDE_lifted)) with the Gaussian static kernel
//     kappa(a, b) = exp(-|a - b|^2 / (2 sigma^2)).
// By the finite-difference form that follows eq. (PDE_lifted), the coarse
// coefficient of the cell between nodes p, p+1 of x and q, q+1 of y is the
// second difference
//     G[p][q] = kappa(x_{p+1}, y_{q+1}) - kappa(x_p, y_{q+1})
//               - kappa(x_{p+1}, y_q) + kappa(x_p, y_q)
// (the printed second term has x_t where the pairing needs y_t), in place of
// <dx_p, dy_q>; the scheme on P_lambda is otherwise the plain one.
//
// Mapping: the lane strips, DPP exchange, runs of pairs and cell update of
// the plain sweep (sweep_fwd_kernel.h).  What changes is the coefficient:
//   * lane l keeps the x NODES of its coarse rows, x_{p0+1} .. x_{p0+CR}
//     (in double, the exact values, where the registers allow: a difference
//     is then one instruction; nodes above the grid repeat x_0, which makes
//     their coefficients exactly 0);
//   * the wave streams y node rows; at node y_t a lane evaluates
//     kappa(x_{p0+c}, y_t) for its nodes c = 1 .. CR in double, the squared
//     distances from the lane's first node's where they are near it (below);
//     with at least
//     2^lambda rows per lane its node 0 is lane l-1's node CR, which that
//     lane evaluated at the previous step (one column ahead) with the same
//     inputs and instructions, and arrives by DPP (with fewer rows, lanes
//     share coarse rows and node 0 is evaluated too); then the row differences
//     d_t[c] = kappa(x_{p0+c+1}, y_t) - kappa(x_{p0+c}, y_t) and
//     G[p0+c][t-1] = d_t[c] - d_{t-1}[c];
//   * each pair's stream starts with its node y_0, a priming step that only
//     records d_0 (so a run of n_b-increment pairs takes sum (n_b + 1) steps).
// The coefficient is a second difference of values near 1; forming it in
// double keeps its relative error near 2^-50 |kappa| / |G| rather than the
// 2^-24 |kappa| / |G| of float.
//
// Bound: the issue of double operations (about 4.8 cycles each per wave), mostly
// distances and exponentials.  128 x 128 Gram of 256-point paths, d = 9, order 1
// (four nodes per lane and step): 2.10 ms with the nodes converted in every step
// and the library's exponential, 2.00 with nodes in double and exp2_nonpositive,
// 1.69 with the distances of near nodes.  Short paths run four runs side by side
// in a wave, as in the plain sweep: 100 x 100 of 30 points, d = 3, order 0 33 us
// against 68 with one run per wave; symmetric 150 of 60 points, d = 4, order 1 88
// against 137.
#pragma once
#include <math.h>

#include <type_traits>

#include "sweep_fwd_kernel.h"

namespace sk {
namespace lift {

using fwd::cell_block;
using fwd::first_row;
using fwd::group_prev;
using fwd::implicit_factors;
using fwd::load_row;
using fwd::n_inc;
using fwd::store_out;
using fwd::wave_run;

// First node row of path k in a dense node buffer: paths are consecutive,
// each with n_k + 1 rows (uniform: len rows).
__device__ __forceinline__ int64_t first_node(const int64_t* start, int32_t len, int64_t k) {
  return start ? start[k] + k : k * (int64_t)len;
}

// v[i] = 2^(v[i] - SHIFT) for v[i] <= 0 (or its rounding; a NaN stays one):
// v = k + f, |f| <= 1/2, and 2^f by the polynomial of degree 11 that interpolates it at the Chebyshev nodes
// (relative error 2.0e-17 in exact arithmetic; 2^0 is exactly 1).  v below kExpLow
// must be clamped to it first (the result is 0 either way).  All N side by side:
// each is one chain of dependent operations, which two waves per SIMD do not hide.
constexpr double kExpLow = -1100.0;
template <int N, int SHIFT>
__device__ __forceinline__ void exp2_nonpositive(double (&v)[N]) {
  constexpr double kRound = 0x1.8p52 - SHIFT;  // v + kRound holds k - SHIFT in its low bits
  constexpr double kC[12] = {1.0,
                             0x1.62e42fefa39efp-1,
                             0x1.ebfbdff82c5aep-3,
                             0x1.c6b08d704a0c6p-5,
                             0x1.3b2ab6fb9f1a5p-7,
                             0x1.5d87fe78a3f9cp-10,
                             0x1.430913112c61bp-13,
                             0x1.ffcbfc6da6ed1p-17,
                             0x1.62bfc2c86d700p-20,
                             0x1.b524ebd13a55fp-24,
                             0x1.e6228acd1c6e5p-28,
                             0x1.e9ec1fcb69a7fp-32};
  double f[N], p[N];
  int k[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double t = v[i] + kRound;
    k[i] = (int)(unsigned)(unsigned long long)__double_as_longlong(t);
    f[i] = v[i] - (t - kRound);
    p[i] = kC[11];
  }
#pragma unroll
  for (int j = 10; j >= 0; --j)
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = __builtin_fma(p[i], f[i], kC[j]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = __builtin_ldexp(p[i], k[i]);
}

// NG > 1: several runs side by side, as in sweep_fwd_kernel.h.
template <int R, int LAM, int D, int NG>
__global__ __launch_bounds__(256) void lifted_sweep_kernel(const SweepArgs a) {
  constexpr int GL = 64 / NG;
  constexpr int DP = (D + 3) & ~3;
  constexpr int S = 1 << LAM;
  constexpr int CR = (R >> LAM) > 0 ? (R >> LAM) : 1;
  // the nodes in double up to the registers of two waves per SIMD
  using Node = typename std::conditional<CR * D <= 40, double, float>::type;

  const int lane = threadIdx.x & (GL - 1);  // of the group
  const int gid = NG == 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))
                          : (int)(threadIdx.x / GL);
  const int64_t w = a.wave0 + (int64_t)blockIdx.x * (blockDim.x / GL) + gid;
  if (w >= a.wave0 + a.n_waves) return;  // uniform per group

  int64_t ia, b0, b1, total;
  int32_t m;
  if (!wave_run(a, w, lane, GL * R, LAM, ia, b0, b1, m, total, GL)) return;
  const int M = m << LAM;

  // strips aligned to the bottom of the grid, as in the plain sweep
  const int off = GL * R - M;  // virtual rows above row 0 (uniform)
  const int row0 = lane * R - off;
  const int p0 = row0 >> LAM;
  const int64_t xnode = first_node(a.x_start, a.x_len, ia);
  Node xn[CR][D];  // nodes p0 + 1 .. p0 + CR
#pragma unroll
  for (int c = 0; c < CR; ++c) {
    const int p = p0 + 1 + c < 0 ? 0 : p0 + 1 + c;  // p0 + CR <= m always
    float t[DP];
    load_row<DP>(a.incx + (xnode + p) * DP, t);
#pragma unroll
    for (int k = 0; k < D; ++k) xn[c][k] = (Node)t[k];
  }
  const double z_per = a.lift_log2;  // -log2(e) / (2 sigma^2)
  // Near nodes: with e = x_c - x_1 (x_1 the lane's first node) the distances
  // |x_c - y|^2 = |x_1 - y|^2 + 2 e (x_1 - y) + |e|^2 take one multiply-add per
  // channel instead of two operations.  They round by a few 2^-53 (r + |e|^2), so
  // the exponents by a few 2^-53 (kNearest + |exponent|), where -|exponent| is the
  // rounding of the plain form; a wave that holds a longer jump (or a node that is
  // not finite) keeps the nodes themselves.
  constexpr bool kNear = sizeof(Node) == 8 && CR > 1;
  constexpr double kNearest = 16.0;
  bool near = false;
  double ee[CR];  // |e|^2
  if constexpr (kNear) {
    bool ok = true;
    ee[0] = 0.0;
#pragma unroll
    for (int c = 1; c < CR; ++c) {
      ee[c] = 0.0;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const double e = xn[c][k] - xn[0][k];
        ee[c] = __builtin_fma(e, e, ee[c]);
      }
      ok = ok && -z_per * ee[c] <= kNearest;
    }
    near = __builtin_amdgcn_ballot_w64(!ok) == 0;
    if (near) {
#pragma unroll
      for (int c = 1; c < CR; ++c)
#pragma unroll
        for (int k = 0; k < D; ++k) xn[c][k] = 2.0 * (xn[c][k] - xn[0][k]);
    }
  }
  // node p0 where the lane evaluates it itself: lanes that share coarse rows,
  // and lane 0 of a strip that starts at the grid's first row (then x_0, the
  // same for all of a wave's lanes that use it)
  float xf[D];
  {
    const int p = R >= S ? 0 : (p0 < 0 ? 0 : p0);
    float t[DP];
    load_row<DP>(a.incx + (xnode + p) * DP, t);
#pragma unroll
    for (int k = 0; k < D; ++k)
      xf[k] = R >= S && NG == 1
                  ? __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(t[k])))
                  : t[k];
  }

  // y stream: stream row g of the run is node row first_node(b0) + g; every
  // pair of a run has cn increments, so cn + 1 rows
  const int32_t cn = n_inc(a.y_n, a.y_len, b0);
  const int32_t rows32 = (int32_t)(total + total / cn);
  int32_t g = -lane;
  const float* __restrict__ yp = a.incy + (first_node(a.y_start, a.y_len, b0) + g) * DP;
  int32_t q = -1;  // column of the current pair; -1: its priming node

  double u[R];
#pragma unroll
  for (int r = 0; r < R; ++r) u[r] = 1.0;
  double pub[S], up[S];
#pragma unroll
  for (int cc = 0; cc < S; ++cc) {
    pub[cc] = 1.0;
    up[cc] = 1.0;
  }
  double up_last = 1.0;
  double dprev[CR];
#pragma unroll
  for (int c = 0; c < CR; ++c) dprev[c] = 0.0;
  // this lane's node-CR kernel value at the previous step, for lane l+1
  // (R >= 2^lambda: lane l's first coarse row is lane l-1's last plus one)
  double kpub = 0.0;
  // A group's first lane has no lane above: when its strip starts above the grid
  // (off > 0) its nodes 0 and 1 are both x_0 and node 1's value serves; when the
  // grid fills the lanes exactly, node 0 is evaluated as well (a uniform branch).
  const bool own_top = off == 0;

  float yA[DP], yB[DP], yC[DP];
  load_row<DP>(yp, yA);
  load_row<DP>(yp + DP, yB);
  const int32_t nsteps = (int32_t)sweep_steps(rows32, GL);

  // kernel values carry the coefficient's fine-cell factor 2^-(2 lambda + 1)
  constexpr int kShift = 2 * LAM + 1;
  auto step = [&](auto nearby, float (&yn)[DP], float (&refill)[DP])
                  __attribute__((always_inline)) {
    load_row<DP>(yp + 2 * DP, refill);
    double yd[D];
#pragma unroll
    for (int k = 0; k < D; ++k) yd[k] = (double)yn[k];
    // the lane's nodes: log2 of their kernel values, channel by channel over all
    // of them, then the values
    double kv[CR];
    if constexpr (decltype(nearby)::value) {
      double t[D];
#pragma unroll
      for (int k = 0; k < D; ++k) t[k] = (double)xn[0][k] - yd[k];
#pragma unroll
      for (int c = 0; c < CR; ++c) kv[c] = ee[c];
#pragma unroll
      for (int k = 0; k < D; ++k) {
        kv[0] = __builtin_fma(t[k], t[k], kv[0]);
#pragma unroll
        for (int c = 1; c < CR; ++c) kv[c] = __builtin_fma((double)xn[c][k], t[k], kv[c]);
      }
      // (r >= 0 but for its rounding)
#pragma unroll
      for (int c = 1; c < CR; ++c) kv[c] += kv[0];
    } else {
#pragma unroll
      for (int c = 0; c < CR; ++c) kv[c] = 0.0;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        double t[CR];
#pragma unroll
        for (int c = 0; c < CR; ++c) t[c] = (double)xn[c][k] - yd[k];
#pragma unroll
        for (int c = 0; c < CR; ++c) kv[c] = __builtin_fma(t[c], t[c], kv[c]);
      }
    }
    bool low = false;
#pragma unroll
    for (int c = 0; c < CR; ++c) {
      kv[c] *= z_per;
      low = low || kv[c] < kExpLow;
    }
    if (__builtin_amdgcn_ballot_w64(low)) {  // rare: values that underflow to 0
      if constexpr (decltype(nearby)::value) {
        // (an infinite y is infinitely far from all of them)
#pragma unroll
        for (int c = 1; c < CR; ++c) kv[c] = kv[0] == -HUGE_VAL ? kv[0] : kv[c];
      }
#pragma unroll
      for (int c = 0; c < CR; ++c) kv[c] = kv[c] < kExpLow ? kExpLow : kv[c];
    }
    exp2_nonpositive<CR, kShift>(kv);
    // (all of them here: sunk into the blocks that use them, they would run one
    // after another)
#pragma unroll
    for (int c = 0; c < CR; ++c) asm volatile("" : "+v"(kv[c]));
    auto own_node = [&]() __attribute__((always_inline)) {
      double z[1] = {0.0};
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const double t = (double)xf[k] - yd[k];
        z[0] = __builtin_fma(t, t, z[0]);
      }
      z[0] *= z_per;
      z[0] = z[0] < kExpLow ? kExpLow : z[0];
      exp2_nonpositive<1, kShift>(z);
      return z[0];
    };
    double kap[CR + 1];
#pragma unroll
    for (int c = 0; c < CR; ++c) kap[c + 1] = kv[c];
    if constexpr (R >= S) {
      double keep0 = kap[1];
      if (own_top) keep0 = own_node();
      kap[0] = group_prev<NG>(kpub, keep0, lane == 0);
      kpub = kap[CR];
    } else {
      kap[0] = own_node();  // lanes share coarse rows: no lane above holds node 0
    }

#pragma unroll
    for (int cc = 0; cc < S; ++cc) up[cc] = group_prev<NG>(pub[cc], up[cc], lane == 0);

    if ((uint32_t)g < (uint32_t)rows32) {
      double dn[CR];
#pragma unroll
      for (int c = 0; c < CR; ++c) dn[c] = kap[c + 1] - kap[c];
      if (q < 0) {
        q = 0;
      } else {
        double gk[CR], h[CR];
#pragma unroll
        for (int c = 0; c < CR; ++c) h[c] = dn[c] - dprev[c];
        if (a.implicit) {
          implicit_factors<CR>(h, gk);
        } else {
#pragma unroll
          for (int c = 0; c < CR; ++c) gk[c] = 1.0 + h[c];
        }
        double v[R][S];
        float sv[1];
        cell_block<R, LAM, CR, false>(v, sv, u, up, up_last, gk);
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = v[r][S - 1];
#pragma unroll
        for (int cc = 0; cc < S; ++cc) pub[cc] = v[R - 1][cc];
        up_last = up[S - 1];
        if (++q == cn) {
          if (lane == GL - 1) {
            const int64_t cb = b0 + g / (cn + 1);
            store_out(a, ia, cb,
                      (a.mode == 2 && a.no_diag && cb == ia) ? 0.0f : (float)u[R - 1]);
          }
#pragma unroll
          for (int r = 0; r < R; ++r) u[r] = 1.0;
          up_last = 1.0;
          q = -1;
        }
      }
#pragma unroll
      for (int c = 0; c < CR; ++c) dprev[c] = dn[c];
    }
    ++g;
    yp += DP;
  };

  auto steps = [&](auto nearby) __attribute__((always_inline)) {
    for (int32_t t = 0; t < nsteps; t += 3) {
      step(nearby, yA, yC);
      step(nearby, yB, yA);
      step(nearby, yC, yB);
    }
  };
  if constexpr (kNear) {
    if (near) {
      steps(std::true_type{});
      return;
    }
  }
  steps(std::false_type{});
}

}  // namespace lift
}  // namespace sk
