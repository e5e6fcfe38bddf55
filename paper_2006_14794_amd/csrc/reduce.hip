// Moments-matching reduction of a discrete measure on paths (Section
// "Moments-matching reduction algorithm for the support of a discrete measure
// on paths"): for weights alpha and the signature-kernel Gram K of the
// support, the proximal-gradient iteration of eq. (fixed_point) for eq.
// (min_lasso),
//     beta <- A_t(beta - gamma grad L(beta)),  grad L(beta) = 2 K (beta - alpha),
// with A_t soft-thresholding at t = gamma lam (the proximal map of
// gamma lam |.|_1).
//
// The whole iteration runs in one launch, and its iterations depend on one
// another: what counts is the time of one matrix-vector product and what it
// takes to hand its result to the next (see the three kernels below).
#include <math.h>

#include "internal.h"

namespace sk {
namespace {

__device__ __forceinline__ double soft(double v, double t) {
  return v > t ? v - t : (v < -t ? v + t : 0.0);
}

__device__ __forceinline__ double bits_to_double(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Lanes 16-31 and 48-63 of `a` trade places with lanes 0-15 and 32-47 of `b`.
__device__ __forceinline__ void swap16(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi =
      __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = bits_to_double(lo[0], hi[0]);
  b = bits_to_double(lo[1], hi[1]);
}
// Lanes 32-63 of `a` trade places with lanes 0-31 of `b`.
__device__ __forceinline__ void swap32(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi =
      __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = bits_to_double(lo[0], hi[0]);
  b = bits_to_double(lo[1], hi[1]);
}

// acc[q mod 4] += k[q] x_{B + q}, q < 8, x_j the value of lane j of each lane's
// row of 16 (row_newbcast, the one DPP control of double instructions, fused into
// the multiply-add; two wait states between a VALU write of x and a DPP read).
template <int B>
__device__ __forceinline__ void dot8(const double* k, double x, double (&acc)[4]) {
#define SK_F(a, q, j) \
  "v_fmac_f64_dpp %" #a ", %4, %" #q " row_newbcast:%" #j " row_mask:0xf bank_mask:0xf\n\t"
  asm volatile("s_nop 1\n\t" SK_F(0, 5, 13) SK_F(1, 6, 14) SK_F(2, 7, 15) SK_F(3, 8, 16) SK_F(0, 9, 17)
      SK_F(1, 10, 18) SK_F(2, 11, 19) SK_F(3, 12, 20)
      : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
      : "v"(x), "v"(k[0]), "v"(k[1]), "v"(k[2]), "v"(k[3]), "v"(k[4]), "v"(k[5]), "v"(k[6]),
        "v"(k[7]), "n"(B), "n"(B + 1), "n"(B + 2), "n"(B + 3), "n"(B + 4), "n"(B + 5),
        "n"(B + 6), "n"(B + 7));
#undef SK_F
}
__device__ __forceinline__ void dot16(const double (&k)[16], double x, double (&acc)[4]) {
  dot8<0>(&k[0], x, acc);
  dot8<8>(&k[8], x, acc);
}

// Sums and maxima over the lanes: within rows of 16 by DPP rotations, across
// them by lane swaps; every lane receives the total.
template <int ROR>
__device__ __forceinline__ double row_ror(double v) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, 0x120 + ROR, 0xF, 0xF, true);
  const int hi =
      __builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), 0x120 + ROR, 0xF, 0xF, true);
  return bits_to_double((unsigned)lo, (unsigned)hi);
}
__device__ __forceinline__ double row_sum(double v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  return v + row_ror<1>(v);
}
__device__ __forceinline__ double across_rows(double v) {  // the sum of the four rows' values
  double w = v;
  swap16(v, w);
  v += w;
  w = v;
  swap32(v, w);
  return v + w;
}
__device__ __forceinline__ double wave_sum(double v) { return across_rows(row_sum(v)); }
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Common driver: every lane that owns a component i (own) holds alpha_i and
// beta_i.  P provides
//   matvec(v)      (K v)_i for the owners, v_i held by them
//   sum(v), max(v) totals over the owners' values (0 from the others)
//   loss(it, v)    records the total of v as loss[it] (may lag behind)
//   leader()       one thread of the launch
// and may put barriers inside any of them: all threads make the same calls.
template <class P>
__device__ __forceinline__ void reduce_driver(const ReduceArgs& a, P& p, bool own, int i,
                                              double alpha) {
  double beta = alpha;
  auto ista = [&](double lam, double step, int iters, bool record) {
    const double t = step * lam, s2 = step * 2.0;
    for (int it = 0; it <= iters; ++it) {
      const double d = beta - alpha;
      const double g = p.matvec(d);
      if (record) p.loss(it, own ? d * g + lam * fabs(beta) : 0.0);
      if (it == iters) break;
      if (own) beta = soft(beta - s2 * g, t);
    }
  };

  // step: the caller's, else 1 / (2 lambda_max(K)) from power iteration
  // (|lambda| of largest modulus), with a 5% margin
  double step = a.step;
  if (!(step > 0.0)) {
    double d = own ? 1.0 + 1e-3 * (double)(i % 7) : 0.0;
    double rho = 0.0;
    for (int it = 0; it < 200; ++it) {
      const double g = p.matvec(d);
      const double nrm = sqrt(p.sum(own ? g * g : 0.0));
      rho = nrm;  // |K v| with |v| = 1 after the first iteration
      d = own ? (nrm > 0.0 ? g / nrm : 0.0) : 0.0;
    }
    step = rho > 0.0 ? 1.0 / (2.0 * 1.05 * rho) : 1.0;
  }
  if (p.leader() && a.step_out) a.step_out[0] = step;

  if (a.support <= 0) {
    ista(a.lam, step, a.iters, a.loss != nullptr);
  } else {
    // bisection on the penalty over [0, lambda_max], lambda_max = 2 max |(K alpha)_i|
    const double g = p.matvec(alpha);
    double lo = 0.0, hi = p.max(own ? fabs(2.0 * g) : 0.0);
    bool found = false;
    double lam = hi;
    for (int r = 0; r < a.rounds; ++r) {
      lam = 0.5 * (lo + hi);
      ista(lam, step, a.iters, false);  // from the previous round's beta
      const int nnz = (int)p.sum(own && beta != 0.0 ? 1.0 : 0.0);
      if (nnz == a.support) {
        if (own) a.beta[i] = beta;
        if (p.leader()) a.lam_out[0] = lam;
        found = true;
      }
      if (nnz > a.support)
        lo = lam;
      else
        hi = lam;
    }
    if (found) return;
    if (p.leader()) a.lam_out[0] = lam;
  }
  if (own) a.beta[i] = beta;
}

// K[i][j], 0 beyond n (a clamped load and a select: branches around a hundred
// loads would keep as many masks)
__device__ __forceinline__ float entry(const ReduceArgs& a, int i, int j) {
  const int ic = i < a.n ? i : a.n - 1, jc = j < a.n ? j : a.n - 1;
  const float v = a.K[(int64_t)ic * a.ld + jc];
  return i < a.n && j < a.n ? v : 0.0f;
}

// Up to 64 atoms: one wave, no LDS and no barrier.  K sits in registers (double)
// and the vector is broadcast within rows of 16 lanes inside the multiply-adds.
// n <= 32: lane 16 r + c owns component 16 (r / 2) + c and forms its sum over
// the column half r mod 2; n <= 64: lane i owns component i and takes the four
// blocks of the vector one after another.  An iteration is 16 (64) multiply-adds
// in four chains, the exchange between the lane rows, and the threshold.
template <int NB>
struct WaveSolver {
  static constexpr int Q = NB == 32 ? 1 : 4;  // blocks of 16 columns per lane
  const ReduceArgs& a;
  double k[Q][16];
  int r;
  __device__ __forceinline__ WaveSolver(const ReduceArgs& a_, int lane, int i) : a(a_) {
    r = lane >> 4;
    const int c0 = NB == 32 ? 16 * (r & 1) : 0;
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int j = 0; j < 16; ++j) k[q][j] = (double)entry(a, i, c0 + 16 * q + j);
  }
  __device__ __forceinline__ double matvec(double v) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    double lo = v, hi = v;
    swap32(lo, hi);  // rows 0, 1 of v in both halves of lo; rows 2, 3 in hi
    if constexpr (NB == 32) {
      // both rows of a half hold the same 16 components: lo those below 16, hi
      // the others
      dot16(k[0], (r & 1) ? hi : lo, acc);
      double g = (acc[0] + acc[1]) + (acc[2] + acc[3]), h = g;
      swap16(g, h);  // the other column half's sum
      return g + h;
    } else {
      double lo2 = lo, hi2 = hi;
      swap16(lo, lo2);  // row 0 of v in every row of lo, row 1 in lo2
      swap16(hi, hi2);  // rows 2 and 3
      dot16(k[0], lo, acc);
      dot16(k[Q > 1 ? 1 : 0], lo2, acc);
      dot16(k[Q > 2 ? 2 : 0], hi, acc);
      dot16(k[Q > 3 ? 3 : 0], hi2, acc);
      return (acc[0] + acc[1]) + (acc[2] + acc[3]);
    }
  }
  __device__ __forceinline__ double sum(double v) { return wave_sum(once(v)); }
  __device__ __forceinline__ double max(double v) { return wave_max(v); }
  __device__ __forceinline__ void loss(int it, double v) {
    const double f = wave_sum(once(v));
    if (leader()) a.loss[it] = f;
  }
  __device__ __forceinline__ bool leader() const { return threadIdx.x == 0; }
  // n <= 32: a component's two owners count once
  __device__ __forceinline__ double once(double v) const {
    return NB == 32 && (r & 1) ? 0.0 : v;
  }
};

template <int NB>
__global__ __launch_bounds__(64) void reduce_wave_kernel(const ReduceArgs a) {
  const int lane = threadIdx.x;
  const int i = NB == 32 ? 16 * (lane >> 5) + (lane & 15) : lane;
  const bool own = i < a.n;
  WaveSolver<NB> p(a, lane, i);
  reduce_driver(a, p, own, i, own ? (double)a.alpha[i] : 0.0);
}

// Up to 256 atoms: one workgroup, K in registers.  A wave holds 16 P rows: lane
// 16 r + c the rows c, c + 16, ... of them over the quarter r of the columns, and
// the four quarters' sums meet by lane swaps.  P = 1 in double up to 192 atoms; at
// 256 K takes half the register file as floats, so P = 2 on eight waves of twice
// the registers, converted in every product (hoisted out of the iterations the
// conversions would need those registers again).  The vector crosses the waves
// through LDS, double-buffered, so that an iteration has one barrier; recorded
// losses are summed a product later, after that barrier.
template <int NP, class TK, int P>
struct BlockSolver {
  static constexpr int W = NP / (16 * P);  // waves
  static constexpr int Q = NP / 64;        // blocks of 16 columns per lane
  struct Shared {
    double x[2][NP];
    double part[2][W];
    double red[2][W];
  };
  // the component of a lane: with P = 2 the upper two lane rows own the upper
  // 16 rows of the wave
  static __device__ __forceinline__ int component() {
    const int lane = threadIdx.x & 63;
    return 16 * P * (threadIdx.x >> 6) + (P == 2 ? 16 * (lane >> 5) : 0) + (lane & 15);
  }
  const ReduceArgs& a;
  Shared& s;
  TK k[P][Q][16];
  int r, c, w, buf = 0, rbuf = 0, pending = -1;
  __device__ __forceinline__ BlockSolver(const ReduceArgs& a_, Shared& s_) : a(a_), s(s_) {
    const int lane = threadIdx.x & 63;
    w = threadIdx.x >> 6;
    r = lane >> 4;
    c = lane & 15;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          k[p][q][j] = (TK)entry(a, 16 * (P * w + p) + c, r * (NP / 4) + 16 * q + j);
  }
  __device__ __forceinline__ double matvec(double v) {
    if (r == 0 || (P == 2 && r == 2)) s.x[buf][component()] = v;
    __syncthreads();
    if (pending >= 0) {
      if (threadIdx.x == 0) {
        double f = 0.0;
        for (int j = 0; j < W; ++j) f += s.part[pending & 1][j];
        a.loss[pending] = f;
      }
      pending = -1;
    }
    double g[P];
    double acc[P][4] = {};
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const double x = s.x[buf][r * (NP / 4) + 16 * q + c];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if constexpr (sizeof(TK) == 8) {
          dot16(k[p][q], x, acc[p]);
        } else {
#pragma unroll
          for (int h = 0; h < 16; h += 8) {
            double kd[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              // (double)k, as an instruction that stays in the loop
              asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(kd[j]) : "v"(k[p][q][h + j]));
            }
            if (h == 0)
              dot8<0>(kd, x, acc[p]);
            else
              dot8<8>(kd, x, acc[p]);
          }
        }
      }
    }
    buf ^= 1;
#pragma unroll
    for (int p = 0; p < P; ++p)
      g[p] = across_rows((acc[p][0] + acc[p][1]) + (acc[p][2] + acc[p][3]));
    return P == 2 && r >= 2 ? g[P - 1] : g[0];
  }
  // the total of a wave's components (in its first lane)
  static __device__ __forceinline__ double over_wave(double v) {
    v = row_sum(v);
    if constexpr (P == 2) {
      double w2 = v;
      swap32(v, w2);
      v += w2;
    }
    return v;
  }
  // (two buffers: a wave is at most one call ahead of the others)
  template <class F>
  __device__ __forceinline__ double combine(double v, F f) {
    if ((threadIdx.x & 63) == 0) s.red[rbuf][w] = v;
    __syncthreads();
    double t = s.red[rbuf][0];
    for (int j = 1; j < W; ++j) t = f(t, s.red[rbuf][j]);
    rbuf ^= 1;
    return t;
  }
  __device__ __forceinline__ double sum(double v) {
    return combine(over_wave(v), [](double x, double y) { return x + y; });
  }
  __device__ __forceinline__ double max(double v) {
    return combine(wave_max(v), [](double x, double y) { return fmax(x, y); });
  }
  __device__ __forceinline__ void loss(int it, double v) {
    const double f = over_wave(v);
    if ((threadIdx.x & 63) == 0) s.part[it & 1][w] = f;
    if (it == a.iters) {  // no product follows
      __syncthreads();
      if (threadIdx.x == 0) {
        double t = 0.0;
        for (int j = 0; j < W; ++j) t += s.part[it & 1][j];
        a.loss[it] = t;
      }
    } else {
      pending = it;
    }
  }
  __device__ __forceinline__ bool leader() const { return threadIdx.x == 0; }
};

template <int NP, class TK, int P>
__global__ __launch_bounds__(4 * NP / P) void reduce_block_kernel(const ReduceArgs a) {
  using Solver = BlockSolver<NP, TK, P>;
  __shared__ typename Solver::Shared s;
  // the lanes of a component carry it alike; beyond n they hold zeros
  const int i = Solver::component();
  const bool own = i < a.n;
  Solver p(a, s);
  reduce_driver(a, p, own, i, own ? (double)a.alpha[i] : 0.0);
}

// Beyond 256 atoms: one workgroup of 16 waves reading K from L2, whole lines of
// a row by consecutive lanes, eight rows at a time per wave (a lane reading a
// row of its own touched a line per lane and load); the eight sums are folded
// over the lanes together.  The vectors sit in LDS.
template <int T, int NMAX>
struct Shared {
  double beta[NMAX];
  double d[NMAX];
  double g[NMAX];
  double alpha[NMAX];
  double red[T / 64];
};

template <int T, class S>
__device__ double block_sum(double v, S& s) {
  v = wave_sum(v);
  const int wid = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) s.red[wid] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < T / 64; ++w) t += s.red[w];
  return t;
}

template <int T, class S>
__device__ double block_max(double v, S& s) {
  v = wave_max(v);
  const int wid = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) s.red[wid] = v;
  __syncthreads();
  double t = s.red[0];
  for (int w = 1; w < T / 64; ++w) t = fmax(t, s.red[w]);
  return t;
}

// out[i] = sum_j K[i][j] x[j]
template <int T>
__device__ void matvec(const ReduceArgs& a, const double* x, double* out) {
  const int n = a.n, lane = threadIdx.x & 63;
  for (int i0 = 8 * (threadIdx.x >> 6); i0 < n; i0 += 8 * (T / 64)) {
    const float* __restrict__ row[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) row[r] = a.K + (int64_t)(i0 + r < n ? i0 + r : n - 1) * a.ld;
    double acc[8] = {};
    // sixteen loads in flight per lane: alone on its CU, the workgroup waits on
    // L2's latency once per turn
    int j = lane;
    for (; j + 64 < n; j += 128) {
      float ka[8], kb[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        ka[r] = row[r][j];
        kb[r] = row[r][j + 64];
      }
      const double xa = x[j], xb = x[j + 64];
#pragma unroll
      for (int r = 0; r < 8; ++r) acc[r] = fma((double)kb[r], xb, fma((double)ka[r], xa, acc[r]));
    }
    if (j < n) {
      const double xj = x[j];
#pragma unroll
      for (int r = 0; r < 8; ++r) acc[r] = fma((double)row[r][j], xj, acc[r]);
    }
    // after the swaps lane row q holds the sums of rows 2 q (v0) and 2 q + 1 (v1)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      swap32(acc[r], acc[r + 4]);
      acc[r] += acc[r + 4];
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      swap16(acc[r], acc[r + 2]);
      acc[r] += acc[r + 2];
    }
    const double v0 = row_sum(acc[0]), v1 = row_sum(acc[1]);
    const int c = lane & 15, i = i0 + 2 * (lane >> 4) + c;
    if (c < 2 && i < n) out[i] = c ? v1 : v0;
  }
}

// `iters` iterations from the current beta; loss (optional) receives the
// objective before each iteration and after the last.
template <int T, class S>
__device__ void ista_run(const ReduceArgs& a, S& s, double lam, double step, int iters,
                         double* loss) {
  const int n = a.n;
  for (int it = 0; it <= iters; ++it) {
    for (int i = threadIdx.x; i < n; i += T) s.d[i] = s.beta[i] - s.alpha[i];
    __syncthreads();
    matvec<T>(a, s.d, s.g);  // g = K d
    __syncthreads();
    if (loss) {
      double part = 0.0;
      for (int i = threadIdx.x; i < n; i += T) part += s.d[i] * s.g[i] + lam * fabs(s.beta[i]);
      const double f = block_sum<T>(part, s);
      if (threadIdx.x == 0) loss[it] = f;
    }
    if (it == iters) break;
    for (int i = threadIdx.x; i < n; i += T)
      s.beta[i] = soft(s.beta[i] - step * 2.0 * s.g[i], step * lam);
    __syncthreads();
  }
}

template <int T, int NMAX>
__global__ __launch_bounds__(T) void reduce_kernel(const ReduceArgs a) {
  __shared__ Shared<T, NMAX> s;
  const int n = a.n;
  for (int i = threadIdx.x; i < n; i += T) {
    s.alpha[i] = (double)a.alpha[i];
    s.beta[i] = s.alpha[i];
  }
  __syncthreads();

  // step: the caller's, else 1 / (2 lambda_max(K)) from power iteration
  // (|lambda| of largest modulus), with a 5% margin
  double step = a.step;
  if (!(step > 0.0)) {
    for (int i = threadIdx.x; i < n; i += T) s.d[i] = 1.0 + 1e-3 * (double)(i % 7);
    __syncthreads();
    double rho = 0.0;
    for (int it = 0; it < 200; ++it) {
      matvec<T>(a, s.d, s.g);
      __syncthreads();
      double part = 0.0;
      for (int i = threadIdx.x; i < n; i += T) part += s.g[i] * s.g[i];
      const double nrm = sqrt(block_sum<T>(part, s));
      rho = nrm;  // |K v| with |v| = 1 after the first iteration
      for (int i = threadIdx.x; i < n; i += T) s.d[i] = nrm > 0.0 ? s.g[i] / nrm : 0.0;
      __syncthreads();
    }
    step = rho > 0.0 ? 1.0 / (2.0 * 1.05 * rho) : 1.0;
  }
  if (threadIdx.x == 0 && a.step_out) a.step_out[0] = step;

  if (a.support <= 0) {
    ista_run<T>(a, s, a.lam, step, a.iters, a.loss);
  } else {
    // bisection on the penalty over [0, lambda_max], lambda_max = 2 max |(K alpha)_i|
    matvec<T>(a, s.alpha, s.g);
    __syncthreads();
    double part = 0.0;
    for (int i = threadIdx.x; i < n; i += T) part = fmax(part, fabs(2.0 * s.g[i]));
    double lo = 0.0, hi = block_max<T>(part, s);
    bool found = false;
    double lam = hi;
    for (int r = 0; r < a.rounds; ++r) {
      lam = 0.5 * (lo + hi);
      ista_run<T>(a, s, lam, step, a.iters, nullptr);
      double cnt = 0.0;
      for (int i = threadIdx.x; i < n; i += T) cnt += s.beta[i] != 0.0 ? 1.0 : 0.0;
      const int nnz = (int)block_sum<T>(cnt, s);
      if (nnz == a.support) {
        for (int i = threadIdx.x; i < n; i += T) a.beta[i] = s.beta[i];
        if (threadIdx.x == 0) a.lam_out[0] = lam;
        found = true;
      }
      if (nnz > a.support)
        lo = lam;
      else
        hi = lam;
      __syncthreads();
    }
    if (found) return;
    if (threadIdx.x == 0) a.lam_out[0] = lam;
  }
  for (int i = threadIdx.x; i < n; i += T) a.beta[i] = s.beta[i];
}

}  // namespace

// Microseconds per iteration (without recorded losses 0.12 at n = 30), before:
// one wave with the vector broadcast through scalar registers up to 64 atoms,
// one workgroup whose lanes each read a row of K from L2 beyond.
//   n          30    64   100   192    256   300   400  1500
//   now      0.24  0.35  0.56  0.85   1.55   7.2  10.9   117
//   before   0.57  0.86   9.4    20     33    38    69  1380
// The lines lie where K no longer fits the registers: 64 doubles a lane of one
// wave; 96 of 12 waves; 128 floats of 8 waves.
hipError_t launch_reduce(const ReduceArgs& a, hipStream_t stream) {
  if (a.n <= 0 || a.n > kMaxReduceN) return hipErrorInvalidValue;
  if (a.n <= 32)
    hipLaunchKernelGGL(reduce_wave_kernel<32>, dim3(1), dim3(64), 0, stream, a);
  else if (a.n <= 64)
    hipLaunchKernelGGL(reduce_wave_kernel<64>, dim3(1), dim3(64), 0, stream, a);
  else if (a.n <= 128)
    hipLaunchKernelGGL((reduce_block_kernel<128, double, 1>), dim3(1), dim3(512), 0, stream, a);
  else if (a.n <= 192)
    hipLaunchKernelGGL((reduce_block_kernel<192, double, 1>), dim3(1), dim3(768), 0, stream, a);
  else if (a.n <= 256)
    hipLaunchKernelGGL((reduce_block_kernel<256, float, 2>), dim3(1), dim3(512), 0, stream, a);
  else
    hipLaunchKernelGGL((reduce_kernel<1024, kMaxReduceN>), dim3(1), dim3(1024), 0, stream, a);
  return hipGetLastError();
}

}  // namespace sk
