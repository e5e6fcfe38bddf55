// Independent pairs (x_k, y_k) of uneven lengths: the explicit scheme of
// Section 3.1, eq. (explicit_finite_diff), on P_lambda, one pair at a time per
// wavefront, with a persistent grid that takes pairs from a length-sorted
// device queue (longest first).
//
// Per pair the shorter path is put on the rows (the scheme is symmetric in
// its two arguments), so the wave streams the longer path's columns.  When
// the rows exceed one wave's strips (64 lanes x R), the grid is processed in
// row bands from the top: lane 63 of band b writes its bottom row (one
// double per fine column) to a per-wave buffer, and lane 0 of band b+1
// reads it as its upper neighbour instead of the boundary value 1.  Within a
// band the mapping is the forward sweep's: lane strips, one coarse column per
// step, DPP wave_shr:1 between lanes, coarse coefficients on the fly.
#pragma once
#include <math.h>

#include <type_traits>

#include "internal.h"
#include "sweep_fwd_kernel.h"

namespace sk {
namespace pairk {

using fwd::first_row;
using fwd::from_prev_lane;
using fwd::load_row;
using fwd::n_inc;

template <int R, int LAM, int D>
__global__ __launch_bounds__(256) void pair_kernel(const PairArgs a) {
  constexpr int DP = (D + 3) & ~3;
  constexpr int S = 1 << LAM;
  constexpr int CR = (R >> LAM) > 0 ? (R >> LAM) : 1;

  const int lane = threadIdx.x & 63;
  const int64_t slot = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  double* __restrict__ bb = a.bandbuf + slot * a.band_stride;
  const int32_t count = a.count ? *a.count : a.n_pairs;
  const int32_t* __restrict__ order = a.order;
  if (order && a.order_base) order += *a.order_base;

  // A wave's first pair is its place's, so that as many pairs as SIMDs or fewer run
  // on as many SIMDs and not where a wave happened to reach the queue first (the
  // corrector's 1045 order-3 pairs of 256 points on 2048 waves: predict 1.36 ms, 1.50
  // with every claim from the queue).  Places go round the compute units, as the
  // workgroups do, then round each one's waves: few pairs have a compute unit each
  // (42 order-3 pairs of 128 points, d = 12, on 260 waves: 169 us, 188 four to a
  // unit; 503 of 257 points, d = 2, on 600: 396 and 466).  Then one vector atomic
  // per pair.
  const uint32_t layer = blockIdx.x / a.units, in = blockIdx.x - layer * a.units;
  const uint32_t left = gridDim.x - layer * a.units;
  const uint32_t place = layer * a.units * (blockDim.x >> 6) +
                         (threadIdx.x >> 6) * (left < a.units ? left : a.units) + in;
  auto claim = [&]() __attribute__((always_inline)) {
    int32_t k = 0;
    if (lane == 0) k = atomicAdd(a.counter, 1);
    // scalar: the task loop's control flow is uniform
    return (int32_t)(gridDim.x * (blockDim.x >> 6)) + __builtin_amdgcn_readlane(k, 0);
  };
  for (int32_t k = __builtin_amdgcn_readfirstlane((int32_t)place); k < count; k = claim()) {
    const int32_t pid = order ? order[k] : k;
    const int64_t ix = a.gram_ny ? pid / a.gram_ny : pid;
    const int64_t iy = a.gram_ny ? pid - ix * a.gram_ny : pid;
    const int32_t mx = n_inc(a.x_n, a.x_len, ix), my = n_inc(a.y_n, a.y_len, iy);
    if (mx < 0 || my < 0 || mx == 0 || my == 0) {
      // every lane stores the same value: no lane-dependent branch may precede
      // a back-edge of this loop.  With a lane-0-only store here the compiler
      // sent lanes 1..63 straight from that store back to the queue-index
      // broadcast with the atomic skipped (they cannot be lane 0), so they ran
      // a second loop header without lane 0 and read lane 0's stale index:
      // part of the wave swept the previous task again.
      a.out[pid] = (mx < 0 || my < 0) ? __builtin_nanf("") : 1.0f;
      continue;
    }
    const bool swap = mx > my;
    const int32_t m = swap ? my : mx, n = swap ? mx : my;
    const float* __restrict__ rinc =
        swap ? a.incy + first_row(a.y_start, a.y_len, iy) * DP
             : a.incx + first_row(a.x_start, a.x_len, ix) * DP;
    const float* __restrict__ cinc =
        swap ? a.incx + first_row(a.x_start, a.x_len, ix) * DP
             : a.incy + first_row(a.y_start, a.y_len, iy) * DP;
    const int M = m << LAM;
    const int nb = (M + 64 * R - 1) / (64 * R);
    const int off = nb * 64 * R - M;  // virtual rows above row 0, in the top band
    const int32_t nsteps = (int32_t)sweep_steps(n);
    double result = 1.0;

    for (int band = 0; band < nb; ++band) {
      // the previous band's bottom row (written by lane 63) must be visible
      if (band > 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const bool top = (band == 0), last = (band == nb - 1);
      const int row0 = (band * 64 + lane) * R - off;
      const int p0 = row0 >> LAM;
      float dx[CR][D];
#pragma unroll
      for (int c = 0; c < CR; ++c) {
        float t[DP];
        if (p0 + c >= 0 && p0 + c < m) {
          load_row<DP>(rinc + (int64_t)(p0 + c) * DP, t);
        } else {
#pragma unroll
          for (int q = 0; q < DP; ++q) t[q] = 0.0f;
        }
#pragma unroll
        for (int q = 0; q < D; ++q) dx[c][q] = t[q];
      }

      double u[R];
#pragma unroll
      for (int r = 0; r < R; ++r) u[r] = 1.0;
      double pub[S];
#pragma unroll
      for (int cc = 0; cc < S; ++cc) pub[cc] = 1.0;
      double up_last = 1.0;
      // The top band's first off / R lanes hold only virtual rows: zero
      // increments and the boundary value 1 whatever the step, so the band
      // starts at the first real lane's first column (lane l at column
      // t0 - l), saving those steps of pipeline fill.
      const int32_t t0 = top ? off / R : 0;
      int32_t g = t0 - lane;
      const float* __restrict__ yp = cinc + (int64_t)g * DP;
      // upper neighbours of lane 0: the boundary (top band) or the band above
      auto bnd_load = [&](int32_t t, double (&v)[S]) {
#pragma unroll
        for (int cc = 0; cc < S; ++cc) v[cc] = top ? 1.0 : bb[(int64_t)t * S + cc];
      };

      float dyA[DP], dyB[DP], dyC[DP];
      double bA[S], bB[S], bC[S];
      load_row<DP>(yp, dyA);
      load_row<DP>(yp + DP, dyB);
      bnd_load(0, bA);
      bnd_load(1, bB);

      auto step = [&](int32_t t, float (&dy)[DP], float (&refill)[DP], double (&bv)[S],
                      double (&brefill)[S]) {
        load_row<DP>(yp + 2 * DP, refill);
        bnd_load(t + 2, brefill);
        float h32[CR];
#pragma unroll
        for (int c = 0; c < CR; ++c) {
          float s = 0.0f;
#pragma unroll
          for (int q = 0; q < D; ++q) s = __builtin_fmaf(dx[c][q], dy[q], s);
          h32[c] = s;
        }
        double up[S];
#pragma unroll
        for (int cc = 0; cc < S; ++cc) up[cc] = from_prev_lane(pub[cc], bv[cc]);

        if ((uint32_t)g < (uint32_t)n) {
          double gk[CR];
          if (a.implicit) {
            double h[CR];
#pragma unroll
            for (int c = 0; c < CR; ++c) h[c] = (double)h32[c] * a.scale;  // exact: 2^-k
            fwd::implicit_factors<CR>(h, gk);
          } else {
#pragma unroll
            for (int c = 0; c < CR; ++c) gk[c] = __builtin_fma((double)h32[c], a.scale, 1.0);
          }
          double v[R][S];
#pragma unroll
          for (int dgl = 0; dgl < R + S - 1; ++dgl) {
#pragma unroll
            for (int cc = 0; cc < S; ++cc) {
              const int r = dgl - cc;
              if (r < 0 || r >= R) continue;
              const double A = (cc == 0) ? u[r] : v[r][cc - 1];
              const double B = (r == 0) ? up[cc] : v[r - 1][cc];
              const double C = (r == 0) ? ((cc == 0) ? up_last : up[cc - 1])
                                        : ((cc == 0) ? u[r - 1] : v[r - 1][cc - 1]);
              v[r][cc] = __builtin_fma(gk[(R >= S) ? (r >> LAM) : 0], A + B, -C);
            }
          }
#pragma unroll
          for (int r = 0; r < R; ++r) u[r] = v[r][S - 1];
#pragma unroll
          for (int cc = 0; cc < S; ++cc) pub[cc] = v[R - 1][cc];
          up_last = up[S - 1];
          if (lane == 63) {
            if (!last) {
#pragma unroll
              for (int cc = 0; cc < S; ++cc) bb[(int64_t)g * S + cc] = pub[cc];
            } else if (g == n - 1) {
              result = u[R - 1];
            }
          }
        }
        ++g;
        yp += DP;
      };

      // (from t0 the last iteration may run up to two steps past nsteps:
      // inactive for every lane, rows within the stream padding)
      for (int32_t t = t0; t < nsteps; t += 3) {
        step(t, dyA, dyC, bA, bC);
        step(t + 1, dyB, dyA, bB, bA);
        step(t + 2, dyC, dyB, bC, bB);
      }
      if (!last) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    }
    // lane 63 holds the value; every lane stores it (no lane-dependent branch
    // before the back-edge, see above)
    a.out[pid] = (float)fwd::lane_value(result, 63);
  }
}

// Pipelined row bands.  The queue holds band tasks in
// pair order, band by band (task_base[k] = first task of the k-th pair of the
// class); a wave takes one task, i.e. one band of one pair, so all bands of a
// pair are swept at the same time, each one lagging the band above by a
// little over one wave's pipeline fill.
//   * Band b writes its bottom row (one double per fine column) into the
//     task's own slot buffer with agent-scope atomic stores, once per value.
//   * The slot buffers are filled with a signalling-NaN sentinel beforehand
//     (arithmetic never produces it), so a value is ready when it differs from
//     the sentinel: band b+1 polls the slots of task tau - 1 with agent-scope
//     atomic loads, kChunk coarse columns at a time, one chunk ahead, staging
//     them in LDS for lane 0.
//   * A task only waits on the task taken just before it (same pair), whose
//     wave is running, so the chain always advances; the wait is bounded all
//     the same, and on expiry the missing values become NaN, which flows to
//     the pair's output and releases the bands below.
constexpr int kChunk = 16;          // coarse columns staged per chunk
constexpr int kSpinMax = 1 << 18;  // polls per value before giving up
constexpr int kYRing = 128;        // y rows held in LDS: at least 64 + kChunk, a power of two

__device__ __forceinline__ bool is_sentinel(double v) {
  return (uint64_t)__double_as_longlong(v) == kBandSlotSentinel;
}

// LDS of one wave of the pipelined band kernel.
template <int LAM, int D>
struct BandStage {
  static constexpr int DP = (D + 3) & ~3;
  // floats per y row: 16-byte reads of consecutive rows by consecutive lanes
  // then touch every bank
  static constexpr int YS = DP == 4 ? 4 : DP + 4;
  float y[kYRing * YS];            // y rows, by column mod kYRing
  double up[2][kChunk << LAM];     // upper neighbours of lane 0, two chunks
  double low[kChunk << LAM];       // lane 63's bottom row, by column mod kChunk
};

// One band task: the band's lanes hold RT fine rows each, lane l's first row
// being row0 (rows above row 0 are virtual: zero increments, value 1).  top:
// the band's upper neighbours are the boundary; last: it ends the pair and
// lane 63 writes the pair's value.
//
// A few long pairs leave each wave alone on its SIMD, and then a step costs
// its latencies.  A step that loads a y row and stores lane 63's bottom row
// waits, every step, for memory operations issued two steps earlier (on gfx950
// loads and stores share one counter, and the stores are acknowledged across
// the XCDs): about 1000 cycles a step whatever the rows.  So every memory
// operation happens once per chunk of kChunk steps, a whole chunk ahead of its
// use: the chunk's y rows, the upper neighbours and the bottom row pass through
// LDS, and a step reads LDS one step ahead.  Five pairs of 2000 points, d = 2,
// order 4 (32 000 x 32 000 fine cells each): see pair_layout's model.
//
// LONE: step loops of their own for either scheme and for the steps in which
// every lane is inside the pair's columns, so that a step has no branch but
// lane 63's store: alone on its SIMD a wave pays each taken branch in full
// (3.88 ms against 4.63 on the five pairs above).  With several waves per SIMD
// and three band heights in one kernel the extra bodies cost more than they
// save (4096 ragged pairs: 3.30 ms against 2.90), so the fitted kernel has one.
template <int RT, int LAM, int D, bool LONE>
__device__ __forceinline__ void band_sweep(const PairArgs& a, BandStage<LAM, D>& st, int lane,
                                           int32_t tau, bool top, bool last, int row0,
                                           int32_t pid, int32_t m, int32_t n,
                                           const float* __restrict__ rinc,
                                           const float* __restrict__ cinc) {
  constexpr int DP = (D + 3) & ~3;
  constexpr int YS = BandStage<LAM, D>::YS;
  constexpr int S = 1 << LAM;
  constexpr int CR = (RT >> LAM) > 0 ? (RT >> LAM) : 1;
  constexpr int CHS = kChunk * S;        // doubles per chunk
  constexpr int PER = (CHS + 63) / 64;   // doubles per lane per chunk
  static_assert(kChunk * DP / 4 <= 64 && kYRing >= 64 + kChunk, "one float4 per lane and chunk");
  double* __restrict__ own = a.tbuf + (int64_t)tau * a.tstride;
  const double* __restrict__ above = a.tbuf + (int64_t)(tau - 1) * a.tstride;

  const int p0 = row0 >> LAM;
  float dx[CR][D];
#pragma unroll
  for (int c = 0; c < CR; ++c) {
    float t[DP];
    if (p0 + c >= 0 && p0 + c < m) {
      load_row<DP>(rinc + (int64_t)(p0 + c) * DP, t);
    } else {
#pragma unroll
      for (int q = 0; q < DP; ++q) t[q] = 0.0f;
    }
#pragma unroll
    for (int q = 0; q < D; ++q) dx[c][q] = t[q];
  }

  // a chunk's y rows and upper neighbours of lane 0, in registers until the
  // chunk begins
  bool failed = false;  // wave-uniform
  double pf[PER];
  float4 py;
  auto fetch = [&](int32_t chunk) {  // issue the loads of a chunk
    py = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int32_t yc = chunk * kChunk + lane / (DP / 4);
    if (lane < kChunk * (DP / 4) && yc < n)
      py = reinterpret_cast<const float4*>(cinc)[(int64_t)yc * (DP / 4) + lane % (DP / 4)];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane + 64 * i;
      const int32_t col = chunk * kChunk + e / S;
      pf[i] = 0.0;
      if (!top && e < CHS && col < n)
        pf[i] = __hip_atomic_load(above + (int64_t)col * S + (e % S), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto commit = [&](int32_t chunk) {  // wait for a chunk's values, then stage them
    if (lane < kChunk * (DP / 4))
      *reinterpret_cast<float4*>(
          &st.y[((chunk * kChunk + lane / (DP / 4)) & (kYRing - 1)) * YS + 4 * (lane % (DP / 4))]) =
          py;
    bool missing = false;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane + 64 * i;
      const int32_t col = chunk * kChunk + e / S;
      double v = pf[i];
      if (!top && e < CHS && col < n) {
        int spins = 0;
        while (!failed && is_sentinel(v) && spins < kSpinMax) {
          ++spins;
          __builtin_amdgcn_s_sleep(2);
          v = __hip_atomic_load(above + (int64_t)col * S + (e % S), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
        }
        if (is_sentinel(v)) {
          v = __builtin_nan("");
          missing = true;
        }
      }
      if (e < CHS) st.up[chunk & 1][e] = top ? 1.0 : v;
    }
    // a value that never came poisons the rest of this band (no more waits)
    failed = failed || __ballot(missing) != 0;
  };
  auto flush = [&](int32_t c0) {  // the bottom row at columns c0 .. c0 + kChunk - 1
    if (last) return;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane + 64 * i;
      const int32_t col = c0 + e / S;
      if (e < CHS && (uint32_t)col < (uint32_t)n)
        __hip_atomic_store(own + (int64_t)col * S + (e % S), st.low[e], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  };

  double u[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) u[r] = 1.0;
  double pub[S];
#pragma unroll
  for (int cc = 0; cc < S; ++cc) pub[cc] = 1.0;
  double up_last = 1.0;
  struct In {
    float dy[DP];
    double up[S];
  };
  auto read_in = [&](int32_t t, In& in) {  // inputs of step t (t >= 0)
    const float4* r = reinterpret_cast<const float4*>(&st.y[((t - lane) & (kYRing - 1)) * YS]);
#pragma unroll
    for (int c = 0; c < DP / 4; ++c) {
      const float4 f = r[c];
      in.dy[4 * c + 0] = f.x;
      in.dy[4 * c + 1] = f.y;
      in.dy[4 * c + 2] = f.z;
      in.dy[4 * c + 3] = f.w;
    }
#pragma unroll
    for (int cc = 0; cc < S; ++cc) in.up[cc] = st.up[(t / kChunk) & 1][(t % kChunk) * S + cc];
  };
  // impl: 1 the implicit scheme's cell factor, 0 the explicit one, -1 as
  // a.implicit says.  full: every lane is inside the pair's columns.
  auto step = [&](auto impl, auto full, int32_t t, const In& in) {
    constexpr int kImpl = decltype(impl)::value;
    const int32_t g = t - lane;
    float h32[CR];
#pragma unroll
    for (int c = 0; c < CR; ++c) {
      float s = 0.0f;
#pragma unroll
      for (int q = 0; q < D; ++q) s = __builtin_fmaf(dx[c][q], in.dy[q], s);
      h32[c] = s;
    }
    double up[S];
#pragma unroll
    for (int cc = 0; cc < S; ++cc) up[cc] = from_prev_lane(pub[cc], in.up[cc]);

    if (decltype(full)::value || (uint32_t)g < (uint32_t)n) {
      double gk[CR];
      if (kImpl == 1 || (kImpl < 0 && a.implicit)) {
        double h[CR];
#pragma unroll
        for (int c = 0; c < CR; ++c) h[c] = (double)h32[c] * a.scale;  // exact: 2^-k
        fwd::implicit_factors<CR>(h, gk);
      } else {
#pragma unroll
        for (int c = 0; c < CR; ++c) gk[c] = __builtin_fma((double)h32[c], a.scale, 1.0);
      }
      double v[RT][S];
      float sv[1];
      fwd::cell_block<RT, LAM, CR, false>(v, sv, u, up, up_last, gk);
#pragma unroll
      for (int r = 0; r < RT; ++r) u[r] = v[r][S - 1];
#pragma unroll
      for (int cc = 0; cc < S; ++cc) pub[cc] = v[RT - 1][cc];
      up_last = up[S - 1];
      if (lane == 63) {
#pragma unroll
        for (int cc = 0; cc < S; ++cc) st.low[(g & (kChunk - 1)) * S + cc] = pub[cc];
      }
    }
  };

  // Iteration k runs the steps kChunk k - 1 .. kChunk (k + 1) - 2, so that the
  // last column of a chunk of lane 63's bottom row (63 steps behind) ends with
  // an iteration.
  constexpr int kLag = 64 / kChunk + 1;  // chunks lane 63 is behind
  const int32_t iters = (n + 63) / kChunk + 1;
  fetch(0);
  In ia, ib;
#pragma unroll
  for (int q = 0; q < DP; ++q) ia.dy[q] = 0.0f;
#pragma unroll
  for (int cc = 0; cc < S; ++cc) ia.up[cc] = 1.0;  // step -1: no lane is active
  auto steps = [&](auto impl, auto full, int32_t t0) {
#pragma unroll 1
    for (int32_t j = 0; j < kChunk; j += 2) {
      read_in(t0 + j + 1, ib);
      step(impl, full, t0 + j, ia);
      // (the read past the iteration's last step is its successor's first, in
      // this chunk)
      read_in(t0 + j + 2, ia);
      step(impl, full, t0 + j + 1, ib);
    }
  };
  for (int32_t k = 0; k < iters; ++k) {
    commit(k);
    flush(kChunk * (k - kLag));  // stores and loads stay in flight for the whole iteration
    fetch(k + 1);
    const int32_t t0 = kChunk * k - 1;
    if constexpr (!LONE)
      steps(std::integral_constant<int, -1>{}, std::false_type{}, t0);
    else if (a.implicit)
      steps(std::integral_constant<int, 1>{}, std::false_type{}, t0);
    else if (t0 >= 63 && t0 + kChunk <= n)
      steps(std::integral_constant<int, 0>{}, std::true_type{}, t0);
    else
      steps(std::integral_constant<int, 0>{}, std::false_type{}, t0);
  }
  flush(kChunk * (iters - kLag));
  // lane 63 holds the value (its rows keep it after the last column); every
  // lane stores it (see pair_kernel)
  const double result = fwd::lane_value(u[RT - 1], 63);
  if (last) a.out[pid] = (float)result;
}

// Full bands hold R fine rows per lane (64 R rows).  The pair's rows are cut
// from the bottom, so only the top band is partial.  FIT_TOP: the top band
// takes the smallest of R/4, R/2 and R rows per lane that covers its rows,
// which saves the issue slots of lanes that would only hold virtual rows; the
// band plan counts the bands at R rows per lane, which this split keeps.
// Without FIT_TOP every band has R rows per lane: the kernel holds one sweep
// body, which the compiler schedules a little better (about 4% on a chain of
// bands), for batches whose top bands need all R rows anyway.
template <int R, int LAM, int D, bool FIT_TOP>
__global__ __launch_bounds__(256) void pair_band_kernel(const PairArgs a) {
  constexpr int DP = (D + 3) & ~3;
  __shared__ BandStage<LAM, D> stage[4];

  const int lane = threadIdx.x & 63;
  const int wl = threadIdx.x >> 6;
  const int32_t count = *a.count;
  if (count == 0) return;
  const int32_t* __restrict__ order = a.order;
  const int32_t total_tasks = a.task_base[count];

  for (;;) {
    int32_t tau = 0;
    if (lane == 0) tau = atomicAdd(a.task_counter, 1);
    tau = __builtin_amdgcn_readlane(tau, 0);  // scalar (see pair_kernel)
    if (tau >= total_tasks) break;
    // the pair of this task: the last k with task_base[k] <= tau
    int32_t lo = 0, hi = count - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (a.task_base[mid] <= tau) lo = mid; else hi = mid - 1;
    }
    const int32_t band = tau - a.task_base[lo];
    const int32_t pid = order[lo];
    const int64_t ix = a.gram_ny ? pid / a.gram_ny : pid;
    const int64_t iy = a.gram_ny ? pid - ix * a.gram_ny : pid;
    const int32_t mx = n_inc(a.x_n, a.x_len, ix), my = n_inc(a.y_n, a.y_len, iy);
    if (mx <= 0 || my <= 0) {  // one task for such a pair
      // every lane stores the same value (see pair_kernel)
      a.out[pid] = (mx < 0 || my < 0) ? __builtin_nanf("") : 1.0f;
      continue;
    }
    const bool swap = mx > my;
    const int32_t m = swap ? my : mx, n = swap ? mx : my;
    const float* __restrict__ rinc =
        swap ? a.incy + first_row(a.y_start, a.y_len, iy) * DP
             : a.incx + first_row(a.x_start, a.x_len, ix) * DP;
    const float* __restrict__ cinc =
        swap ? a.incx + first_row(a.x_start, a.x_len, ix) * DP
             : a.incy + first_row(a.y_start, a.y_len, iy) * DP;
    const int M = m << LAM;
    const int nb = (M + 64 * R - 1) / (64 * R);
    const int top_rows = M - (nb - 1) * 64 * R;  // 1 .. 64 R
    const bool last = band == nb - 1;
    // rows per lane of this band: R / 4, R / 2 or R (one if-else chain, no
    // continue after a sweep)
    const int quarter = R >= 4 ? R / 4 : R, half = R >= 2 ? R / 2 : R;
    const int rt = (!FIT_TOP || band > 0)      ? R
                   : 64 * quarter >= top_rows ? quarter
                   : 64 * half >= top_rows    ? half
                                              : R;
    if (rt == R) {
      const int row0 = band > 0 ? top_rows + ((band - 1) * 64 + lane) * R
                                : lane * R - (64 * R - top_rows);
      band_sweep<R, LAM, D, !FIT_TOP>(a, stage[wl], lane, tau, band == 0, last, row0, pid, m, n, rinc,
                            cinc);
    } else if (rt == half) {
      band_sweep<(R >= 2 ? R / 2 : R), LAM, D, !FIT_TOP>(a, stage[wl], lane, tau, true, last,
                                               lane * half - (64 * half - top_rows), pid, m,
                                               n, rinc, cinc);
    } else {
      band_sweep<(R >= 4 ? R / 4 : R), LAM, D, !FIT_TOP>(a, stage[wl], lane, tau, true, last,
                                               lane * quarter - (64 * quarter - top_rows),
                                               pid, m, n, rinc, cinc);
    }
  }
}

}  // namespace pairk
}  // namespace sk
