// Gradient of a weighted sum of Gram entries, two sweeps per cell: the
// discrete adjoint of grad_kernel.h (same recurrences, same mapping of lanes,
// bands and segments) with the forward values of the reverse pass obtained by
// running the scheme itself backwards.
//
// The cell recurrence K[i+1][j+1] = g (K[i+1][j] + K[i][j+1]) - K[i][j] solves
// for its oldest corner with the same operations,
//     K[i][j] = g (K[i+1][j] + K[i][j+1]) - K[i+1][j+1],
// so the reverse wavefront, which meets the cells from the terminal corner on,
// rebuilds the forward nodes as it goes: each reverse step forms the cell sum
// A + B (one add), the older node (one FMA), the adjoint value (two FMAs) and
// the coefficient gradient (one FMA, the cell sum in double).  Nothing is
// recomputed from the left and no cell sums are stored.  grad_kernel.h runs
// the forward steps a second time from checkpoints instead: about 196 VALU
// instructions per 8 fine cells against 150 here at four rows per lane and 120
// at eight.  Bound: instruction issue (about 80 % of it at two waves per
// SIMD).  Measured, 64 x 64 pairs of 512 points, d = 4, order 1, x side only:
// 2.07 ms against 4.05; both sides of the 2016 pairs of a symmetric Gram:
// 1.24 against 2.67; 48 x 40 pairs of 100 points, d = 5, both sides: 0.169
// against 0.354.  Steps of the first: 3.0 ms with four rows per lane; 2.35
// with eight, the checkpoints read without prefetch (their registers) and
// only every fourth segment; 2.26 with the y-side sums in LDS, pair ends by
// step index and the cell factor handed over instead of the coefficient; 2.04
// to 2.15 with those sums laid out by channel.
//
// What the reverse pass needs of the forward one:
//  * the nodes right of its first column: each lane's state after every
//    ck_every-th segment of C steps (`ckpt`) and at the last column of every
//    pair (`pend`: the strip's R + 1 nodes);
//  * the nodes below a band: the band's bottom row (`hand_f`); below a lane's
//    strip they are the top nodes of the lane beneath, handed up by DPP as
//    the adjoint values are.
//
// Rounding.  Backwards the scheme amplifies rounding errors like the
// Riemann function of the region it crosses, which is a pair's columns or those
// between two checkpoints (at most four segments apart, whatever the pairs of
// the run) and for paths with huge kernels not bounded by a constant.  So the
// error is measured wherever a stretch of rebuilt nodes ends: at a checkpoint
// against the forward nodes that replace them, and at the first column of every
// pair of the run against the boundary value 1 (within a run by the sum over each
// lane's strip).  A task in which any differs by
// more than kRevTol relative to max(1, |K|) is appended to a list that
// grad_kernel.h works off afterwards, overwriting the task's results.
// kRevTol is a sixteenth of the rounding of the float cell sums there.
//
// Short paths.  NG > 1 packs NG pairs side by side in a wave, each on 64 / NG
// lanes (x paths of at most 64 R / NG fine rows, one band): the lanes of a
// 64-lane strip beyond the path's rows would otherwise sweep virtual rows,
// and the wavefront's fill takes 64 / NG - 1 steps instead of 63.
#pragma once
#include "grad_kernel.h"

namespace sk {
namespace grad {

using fwd::group_prev;

// Largest accepted difference between a rebuilt node and the forward one.
constexpr double kRevTol = 1.0 / (1 << 28);
__device__ __forceinline__ bool drifted(double rebuilt, double forward) {
  return !(fabs(rebuilt - forward) <= kRevTol * fmax(1.0, fabs(forward)));
}

// Lane l receives lane l+1's value within its group of 64 / NG lanes; a group's
// last lane keeps `keep`.
template <int NG, class T>
__device__ __forceinline__ T group_next(T v, T keep, bool last) {
  if constexpr (NG == 1) {
    return from_next_lane(v, keep);
  } else if constexpr (NG == 4) {  // row_shl:1
    if constexpr (sizeof(T) == 4) {
      return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(keep), __float_as_int(v),
                                                        0x101, 0xF, 0xF, false));
    } else {
      const unsigned long long bv = (unsigned long long)__double_as_longlong(v);
      const unsigned long long bk = (unsigned long long)__double_as_longlong(keep);
      const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)bk, (int)(unsigned)bv, 0x101, 0xF,
                                                 0xF, false);
      const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(bk >> 32),
                                                 (int)(unsigned)(bv >> 32), 0x101, 0xF, 0xF, false);
      return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                              (unsigned long long)(unsigned)lo));
    }
  } else {
    const T t = from_next_lane(v, keep);
    return last ? keep : t;
  }
}

template <int R, int LAM, int D, int C, int NG, bool YS>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(grad_rev_waves(R, LAM, D), 2))) void grad_rev_kernel(
    const GradArgs a) {
  constexpr int GL = 64 / NG;             // lanes per pair
  constexpr int DP = (D + 3) & ~3;
  constexpr int S = 1 << LAM;
  constexpr int CR = (R >> LAM) > 0 ? (R >> LAM) : 1;
  constexpr int KS = R + S + 1;           // checkpoint doubles per lane
  constexpr int YR = C + GL - 1;          // y rows of a segment, per group
  constexpr int Y4 = NG * YR * DP / 4;    // float4s of a segment's y rows
  constexpr int PY = (Y4 + 63) / 64;      // ... per lane
  constexpr int YQ = DP / 4 | 1;          // float4s from one y row in LDS to the next: odd, since
                                          // neighbouring lanes read neighbouring rows
  constexpr int NB = C * S;               // lane 0's upper neighbours per segment (NG == 1)
  constexpr int PB = (NB + 63) / 64;
  constexpr int NK = NG * C * S;          // the last lanes' bottom nodes per segment
  constexpr int PK = (NK + 63) / 64;
  constexpr int LW = S + 1;               // a band's hand-over per column: S a values and
                                          // the first coarse row's cell factor
  constexpr int NL = C * LW;              // ... per segment (NG == 1)
  constexpr int PL = (NL + 63) / 64;
  constexpr int NW = NG == 1 && NL > NK ? NL : NK;
  constexpr int YW = NG == 1 ? 128 : 64;  // columns of the y-side ring: at least C + GL - 1
  constexpr int YL = YW + 1;              // ... and doubles from one channel to the next
  constexpr int NY = NG * C * D;          // y-side sums completed by a segment
  constexpr int PO = (NY + 63) / 64;
  static_assert(YW >= C + GL - 1, "y-side ring");
  static_assert(C % 2 == 0 && C <= 32 && KS == grad_rev_state_doubles(R, LAM), "scratch geometry");
  __shared__ float4 sy[NG * YR * YQ];  // the segment's y rows, zero outside the task
  __shared__ double sb[NG == 1 ? NB : 1];  // [step][fine column]: lane 0's upper neighbours
  __shared__ double skn[NK];   // [group][step][fine column]: bottom nodes of the last lane's strip
  __shared__ double sl[NG == 1 ? NL : 1];  // [step][LW]: lane 63's lower neighbours
  __shared__ double sw[NW];    // outputs of the segment
  __shared__ double spe[(R + 1) * 64];  // [node][lane]: the strips' nodes at a pair's last column
  __shared__ double ring[YS ? NG * D * YL : 1];  // [group][channel][column mod YW]: y-side sums

  const int lane = threadIdx.x;
  const int lg = lane & (GL - 1), grp = lane / GL;
  const bool first = lg == 0, lastl = lg == GL - 1;
  const GradRevSlot L =
      grad_rev_slot_layout(R, LAM, a.nb_max, a.nck_max, a.cols_max, NG == 1 ? a.run : 1);
  double* __restrict__ scr = a.scratch + (int64_t)blockIdx.x * a.slot_stride;
  double* __restrict__ ckpt = scr + L.ckpt;
  double* __restrict__ hand_f = scr + L.hand_f;
  double* __restrict__ hand_a = scr + L.hand_a;
  double* __restrict__ pend = scr + L.pend;
  const int64_t ck_band = (int64_t)a.nck_max * KS * 64;
  const int64_t hf_band = a.cols_max * S;
  const int64_t ha_buf = (a.cols_max + 1) * (S + 1);
  const int64_t pe_band = (int64_t)(NG == 1 ? a.run : 1) * (R + 1) * 64;

  for (;;) {
    int32_t task = 0;
    if (lane == 0) task = atomicAdd(a.counter, 1);
    task = __builtin_amdgcn_readlane(task, 0);  // scalar: uniform loop control
    if (task >= a.n_tasks) break;
    int64_t ia, b0, b1, jslot;
    if (NG == 1 && a.order) {
      const int64_t pid = a.order[task];
      ia = pid / a.ny;
      b0 = pid - ia * a.ny;
      b1 = b0 + 1;
      jslot = b0;
    } else {
      ia = task / a.runs_per_row;
      jslot = task - ia * a.runs_per_row;
      b0 = jslot * a.run;
      b1 = b0 + a.run < a.ny ? b0 + a.run : a.ny;
    }
    const int32_t m = n_inc(a.x_n, a.x_len, ia);
    double* __restrict__ px = a.part_x + ((int64_t)ia * a.runs_per_row + jslot) * a.mrows * D;
    // below the diagonal of a symmetric Gram there is nothing to do (NG > 1:
    // the groups of such pairs stay idle)
    if (NG == 1 && a.mode == 2 && b0 < ia) b0 = ia;
    if (a.mode == 2 && a.no_diag && b0 <= ia && ia < b1) {
      // the diagonal of a symmetric Gram without it: the constant 0, no
      // gradient (every lane stores the same values)
      if (YS)
        fill_rows(a.part_y + ((int64_t)ia * a.ny + ia) * a.nrows * D, (int64_t)a.nrows * D,
                  m < 0 ? __builtin_nan("") : 0.0, lane);
      if (a.K) a.K[ia * a.ny + ia] = 0.0f;
      if (NG == 1) ++b0;
    }
    const int32_t n = b0 < b1 ? n_inc(a.y_n, a.y_len, b0) : 0;
    const bool none = a.mode == 2 && b1 <= ia + (a.no_diag ? 1 : 0);  // no pair of the triangle

    if (none || !(b0 < b1 && m > 0 && n > 0)) {
      // Nothing to sweep.  Values: a broken path NaN, a one-point path 1;
      // gradients 0 (NaN for a broken pair).  Every lane stores the same values.
      const bool broken = m < 0 || (b0 < b1 && n < 0);
      fill_rows(px, (int64_t)a.mrows * D, broken ? __builtin_nan("") : 0.0, lane);
      for (int64_t b = b0; b < b1 && !none; ++b) {
        const int32_t nb_ = n_inc(a.y_n, a.y_len, b);
        const bool bad_ = m < 0 || nb_ < 0;
        if (YS)
          fill_rows(a.part_y + ((int64_t)ia * a.ny + b) * a.nrows * D, (int64_t)a.nrows * D,
                    bad_ ? __builtin_nan("") : 0.0, lane);
        if (a.K) store_value(a, ia, b, bad_ ? __builtin_nanf("") : 1.0f);
      }
      continue;
    }

    // this lane's pair: of a run (NG == 1, all lanes alike) or of its group
    const int64_t bg = NG == 1 ? b0 : b0 + grp;
    const bool live = NG == 1 || (bg < b1 && (a.mode != 2 || bg > ia || (bg == ia && !a.no_diag)));
    const int32_t total = NG == 1 ? (int32_t)((b1 - b0) * n) : (live ? n : 0);
    const int32_t span = (NG == 1 ? total : n) + GL - 1;  // steps of the wavefront
    const int32_t nseg = (span + C - 1) / C;
    const int M = m << LAM;
    const int nb = NG == 1 ? (M + 64 * R - 1) / (64 * R) : 1;
    const int off = nb * GL * R - M;  // virtual rows above row 0, in the top band
    const float* __restrict__ xinc = a.incx + first_row(a.x_start, a.x_len, ia) * DP;
    const float* __restrict__ ycol = a.incy + first_row(a.y_start, a.y_len, b0) * DP;
    double* __restrict__ pyt = YS ? a.part_y + ((int64_t)ia * a.ny + b0) * a.nrows * D : nullptr;
    bool bad = false;      // this lane met nodes that differ too much, or will
    bool give_up = false;  // (uniform) some lane did

    // columns of group q as the staging loops (any lane, any group) see them
    auto group_total = [&](int q) -> int32_t {
      if (NG == 1) return total;
      const int64_t b = b0 + q;
      return b < b1 && (a.mode != 2 || b > ia || (b == ia && !a.no_diag)) ? n : 0;
    };

    // ---- staging of a segment's inputs (registers one segment ahead, then LDS)
    auto fetch_y = [&](int32_t seg, float4 (&py)[PY]) {
      const int32_t t0 = seg * C;
#pragma unroll
      for (int i = 0; i < PY; ++i) {
        const int e = lane + 64 * i;
        py[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const int q = NG == 1 ? 0 : e / (YR * DP / 4);
        const int e1 = e - q * (YR * DP / 4);
        const int32_t g = t0 - (GL - 1) + e1 / (DP / 4);
        if (e < Y4 && (uint32_t)g < (uint32_t)group_total(q))
          py[i] = at(reinterpret_cast<const float4*>(ycol),
                     (uint32_t)((q * n + g) * (DP / 4) + e1 % (DP / 4)));
      }
    };
    auto put_y = [&](const float4 (&py)[PY]) {
#pragma unroll
      for (int i = 0; i < PY; ++i) {
        const int e = lane + 64 * i;
        if (e < Y4) sy[e / (DP / 4) * YQ + e % (DP / 4)] = py[i];
      }
    };
    // lane 0's upper neighbours at steps t0 .. t0 + C - 1 (columns t0 + j; 1
    // beyond the task, where every forward value is 1)
    auto fetch_up = [&](int32_t seg, bool top, const double* __restrict__ above,
                        double (&pb)[PB]) {
      const int32_t t0 = seg * C;
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        const int e = lane + 64 * i;
        pb[i] = 1.0;
        const int32_t col = t0 + e / S;
        if (!top && e < NB && col < total) pb[i] = at(above, (uint32_t)(col * S + e % S));
      }
    };
    auto put_up = [&](const double (&pb)[PB]) {
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        const int e = lane + 64 * i;
        if (e < NB) sb[e] = pb[i];
      }
    };
    // the y row of a lane at step t0 + j
    auto get_dy = [&](int j, float (&dy)[DP]) {
      const float4* r = &sy[(grp * YR + j - lg + GL - 1) * YQ];
#pragma unroll
      for (int c = 0; c < DP / 4; ++c) {
        const float4 f = r[c];
        dy[4 * c] = f.x;
        dy[4 * c + 1] = f.y;
        dy[4 * c + 2] = f.z;
        dy[4 * c + 3] = f.w;
      }
    };
    auto load_dx = [&](int p0, float (&dx)[CR][D]) {
#pragma unroll
      for (int c = 0; c < CR; ++c) {
        float tr[DP];
        if (p0 + c >= 0 && p0 + c < m) {
          load_row<DP>(xinc + (int64_t)(p0 + c) * DP, tr);
        } else {
#pragma unroll
          for (int k = 0; k < DP; ++k) tr[k] = 0.0f;
        }
#pragma unroll
        for (int k = 0; k < D; ++k) dx[c][k] = tr[k];
      }
    };
    // The step j < C at which a lane whose column at the segment's first step
    // is g0 is at the last column of a pair (k n - 1 for some k >= 1) of the
    // task, or -1: at most one, the host forming runs of several pairs only
    // for n >= C.
    auto pair_end = [&](int32_t g0) -> int {
      const int32_t c0 = g0 > 0 ? g0 : 0;
      const int32_t e = (c0 / n) * n + n - 1;
      return e < total && e - g0 < C ? e - g0 : -1;
    };
    struct FwdIn {
      float dy[DP];
      double up[S];
    };
    auto read_fwd = [&](int j, FwdIn& in) {
      get_dy(j, in.dy);
#pragma unroll
      for (int cc = 0; cc < S; ++cc) in.up[cc] = NG == 1 ? sb[j * S + cc] : 1.0;
    };
    auto inner = [&](const float (&dx)[CR][D], const float (&dy)[DP], float (&h32)[CR]) {
#pragma unroll
      for (int c = 0; c < CR; ++c) {
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < D; ++k) s = __builtin_fmaf(dx[c][k], dy[k], s);
        h32[c] = s;
      }
    };

    // ---------------- forward pass: bands top to bottom ----------------
    for (int band = 0; band < nb && !give_up; ++band) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");  // hand_f of the band above
      const bool top = band == 0, last = band == nb - 1;
      const int p0 = ((band * GL + lg) * R - off) >> LAM;  // floor; < 0 for virtual rows
      float dx[CR][D];
      load_dx(p0, dx);
      // the band's increments have arrived before the segment loop starts:
      // otherwise the compiler's wait for them can land at the head of a step
      // loop and cover the staging loads in flight there too (vmcnt(0))
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      const double* __restrict__ above = hand_f + (int64_t)(band > 0 ? band - 1 : 0) * hf_band;
      double* __restrict__ below = hand_f + (int64_t)band * hf_band;
      double* __restrict__ ck = ckpt + (int64_t)band * ck_band;
      double* __restrict__ pn = pend + (int64_t)band * pe_band;
      double u[R], pub[S], up_last = 1.0, bl = 1.0;
#pragma unroll
      for (int r = 0; r < R; ++r) u[r] = 1.0;
#pragma unroll
      for (int cc = 0; cc < S; ++cc) pub[cc] = 1.0;
      float4 py[PY];
      double pb[PB];
      fetch_y(0, py);
      if (NG == 1) fetch_up(0, top, above, pb);
      for (int32_t seg = 0; seg < nseg; ++seg) {
        const int32_t t0 = seg * C;
        __syncthreads();  // the previous segment's reads of the staging are done
        put_y(py);
        if (NG == 1) put_up(pb);
        __syncthreads();
        if (seg + 1 < nseg) {
          fetch_y(seg + 1, py);
          if (NG == 1) fetch_up(seg + 1, top, above, pb);
        }
        const int pe = pair_end(t0 - lg);
        auto fwd_pass_step = [&](const int j, const FwdIn& in) {
          float h32[CR];
          inner(dx, in.dy, h32);
          double up[S];
#pragma unroll
          for (int cc = 0; cc < S; ++cc) up[cc] = group_prev<NG>(pub[cc], in.up[cc], first);
          double gk[CR];
#pragma unroll
          for (int c = 0; c < CR; ++c) gk[c] = 1.0 + (double)h32[c];
          bl = u[R - 1];
          double v[R][S];
          float st[1];
          fwd::cell_block<R, LAM, CR, false>(v, st, u, up, up_last, gk);
#pragma unroll
          for (int r = 0; r < R; ++r) u[r] = v[r][S - 1];
#pragma unroll
          for (int cc = 0; cc < S; ++cc) pub[cc] = v[R - 1][cc];
          up_last = up[S - 1];
          // the last lane's bottom row: for the band below and the reverse
          // pass, and in the last band the Gram value at the last column of a
          // pair (its last entry)
          if (lastl) {
#pragma unroll
            for (int cc = 0; cc < S; ++cc) sw[(grp * C + j) * S + cc] = pub[cc];
          }
          if (pe == j) {
            // last column of a pair: the left boundary of the next pair
            spe[lane] = up_last;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              spe[(r + 1) * 64 + lane] = u[r];
              u[r] = 1.0;
            }
            up_last = 1.0;
          }
        };
        // two steps per iteration, alternating two input buffers (the read
        // past the segment's last step re-reads that step)
        FwdIn fa, fb;
        read_fwd(0, fa);
#pragma unroll 1
        for (int j = 0; j < C; j += 2) {
          __builtin_amdgcn_sched_barrier(0);
          read_fwd(j + 1, fb);
          fwd_pass_step(j, fa);
          __builtin_amdgcn_sched_barrier(0);
          read_fwd(j + 2 < C ? j + 2 : j + 1, fa);
          fwd_pass_step(j + 1, fb);
        }
        // (global stores stay out of the step loop: a loop with stores makes
        // the compiler wait for the staging loads in flight before entering it)
        __syncthreads();
        // the bottom row at columns t0 - (GL - 1) .. t0 + C - GL
        for (int e = lane; e < NK; e += 64) {
          const int q = NG == 1 ? 0 : e / (C * S);
          const int e1 = e - q * (C * S);
          const int32_t col = t0 + e1 / S - (GL - 1);
          if ((uint32_t)col < (uint32_t)group_total(q))
            at(below, (uint32_t)((q * n + col) * S + e1 % S)) = sw[e];
        }
        if (last && a.K) {  // the values of the pairs that end in this segment
          for (int e = lane; e < NG * C; e += 64) {
            const int q = NG == 1 ? 0 : e / C;
            const int32_t col = t0 + (e - q * C) - (GL - 1);
            if ((uint32_t)col < (uint32_t)group_total(q) && (col + 1) % n == 0)
              store_value(a, ia, b0 + q + col / n, (float)sw[e * S + S - 1]);
          }
        }
        if (pe >= 0) {
          const int32_t k = NG == 1 ? (t0 - lg + pe) / n : 0;
          const uint32_t c0 = (uint32_t)(k * (R + 1) * 64 + lane);
#pragma unroll
          for (int r = 0; r <= R; ++r) at(pn, c0 + r * 64) = spe[r * 64 + lane];
          bad = bad || fabs(spe[R * 64 + lane]) > a.huge;
        }
        // the state after every ck_every-th segment and the last one
        if ((seg + 1) % a.ck_every == 0 || seg + 1 == nseg) {
          if (__ballot(bad || fabs(u[R - 1]) > a.huge) != 0) {
            give_up = true;
            break;
          }
          const uint32_t c0 = (uint32_t)(seg / a.ck_every * KS * 64 + lane);
#pragma unroll
          for (int r = 0; r < R - 1; ++r) at(ck, c0 + r * 64) = u[r];
#pragma unroll
          for (int cc = 0; cc < S; ++cc) at(ck, c0 + (R - 1 + cc) * 64) = pub[cc];
          at(ck, c0 + (R - 1 + S) * 64) = up_last;
          at(ck, c0 + (R + S) * 64) = bl;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }

    // ---------------- reverse pass: bands bottom to top ----------------
    for (int band = give_up ? -1 : nb - 1; band >= 0; --band) {
      // checkpoints, hand_f, hand_a, part_y
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      const bool top = band == 0, last = band == nb - 1;
      const int row0 = (band * GL + lg) * R - off;
      const int p0 = row0 >> LAM;
      const int cb_below = ((row0 + R) >> LAM) - p0;  // coarse row of the cell row below, relative
      float dx[CR][D];
      load_dx(p0, dx);
      double dxd[CR][D];  // the same increments in double, for the y-side products
#pragma unroll
      for (int c = 0; c < CR; ++c)
#pragma unroll
        for (int k = 0; k < D; ++k) dxd[c][k] = (double)dx[c][k];
      double dxacc[CR][D];
#pragma unroll
      for (int c = 0; c < CR; ++c)
#pragma unroll
        for (int k = 0; k < D; ++k) dxacc[c][k] = 0.0;
      const double* __restrict__ hfb = hand_f + (int64_t)band * hf_band;
      const double* __restrict__ abl = hand_a + (int64_t)((band + 1) & 1) * ha_buf;
      double* __restrict__ abw = hand_a + (int64_t)(band & 1) * ha_buf;
      const double* __restrict__ ck = ckpt + (int64_t)band * ck_band;
      const double* __restrict__ pn = pend + (int64_t)band * pe_band;

      // bottom nodes of the last lane's strip at steps t0 .. t0 + C - 1: fine
      // columns 0 .. S - 1 of its coarse column (the node left of a pair's
      // first column is the boundary; outside the task everything is 1)
      auto fetch_kn = [&](int32_t seg, double (&pkn)[PK]) {
        const int32_t t0 = seg * C;
#pragma unroll
        for (int i = 0; i < PK; ++i) {
          const int e = lane + 64 * i;
          pkn[i] = 1.0;
          const int q = NG == 1 ? 0 : e / (C * S);
          const int e1 = e - q * (C * S);
          const int32_t col = t0 + e1 / S - (GL - 1);
          if (e < NK && (uint32_t)col < (uint32_t)group_total(q) &&
              (e1 % S != 0 || col % n != 0))
            pkn[i] = at(hfb, (uint32_t)((q * n + col) * S + e1 % S - 1));
        }
      };
      auto put_kn = [&](const double (&pkn)[PK]) {
#pragma unroll
        for (int i = 0; i < PK; ++i) {
          const int e = lane + 64 * i;
          if (e < NK) skn[e] = pkn[i];
        }
      };
      // lane 63's lower neighbours at steps t0 .. t0 + C - 1 (columns
      // t0 + j - 63; zero outside the task and below the last band)
      auto fetch_low = [&](int32_t seg, double (&pl)[PL]) {
        const int32_t t0 = seg * C;
#pragma unroll
        for (int i = 0; i < PL; ++i) {
          const int e = lane + 64 * i;
          pl[i] = 0.0;
          const int j = e / LW, f = e - j * LW;
          const int32_t col = t0 + j - 63;
          if (!last && e < NL && (uint32_t)col < (uint32_t)total)
            pl[i] = at(abl, (uint32_t)(col * LW + f));
        }
      };
      auto put_low = [&](const double (&pl)[PL]) {
#pragma unroll
        for (int i = 0; i < PL; ++i) {
          const int e = lane + 64 * i;
          if (e < NL) sl[e] = pl[i];
        }
      };
      double kr[R];   // the strip's nodes (rows 0 .. R - 1) right of the block
      double kc;      // ... and its bottom one
      double pubK[S]; // published top nodes at the block's fine columns
      double ar[R];   // a of the strip's cells at the first fine column of the next coarse column
      double gr[CR];  // cell factors of that column
#pragma unroll
      for (int r = 0; r < R; ++r) ar[r] = 0.0;
#pragma unroll
      for (int c = 0; c < CR; ++c) gr[c] = 1.0;
      double pubA[S];  // published top-row a
#pragma unroll
      for (int cc = 0; cc < S; ++cc) pubA[cc] = 0.0;
      double prev_ab0 = 0.0;  // lane l+1's top-row a at the next column's first fine column
      double gpub = 1.0;      // published cell factor (first coarse row)
#pragma unroll
      for (int r = 0; r < R; ++r) kr[r] = 1.0;
      kc = 1.0;
#pragma unroll
      for (int cc = 0; cc < S; ++cc) pubK[cc] = 1.0;

      // The y-side sums of a column, sum_p dG[p][q] dx_p, collect in an LDS
      // ring: each lane adds its strip's part at the step it meets the column
      // (the last lane first, so in a fixed order), and a column is complete
      // when the first lane has passed it.  Neighbouring lanes add to neighbouring
      // columns of a channel, that is to neighbouring banks (a column's channels
      // side by side put lanes on the same banks: 48 x 40 paths of 120 points, 16
      // channels, order 1 1657 us for the whole call against 524).  Passing partial sums from lane to
      // lane by DPP cost three instructions per channel and step.
      if constexpr (YS) {
        for (int e = lane; e < NG * D * YL; e += 64) ring[e] = 0.0;
      }

      float4 py[PY];
      double pkn[PK], pl[PL];
      fetch_y(nseg - 1, py);
      fetch_kn(nseg - 1, pkn);
      if (NG == 1) fetch_low(nseg - 1, pl);
      for (int32_t seg = nseg - 1; seg >= 0; --seg) {
        const int32_t t0 = seg * C;
        const int32_t g0 = t0 - lg;  // column of this lane at step t0
        __syncthreads();  // the previous segment's reads of the staging are done
        put_y(py);
        put_kn(pkn);
        if (NG == 1) put_low(pl);
        __syncthreads();
        if (seg > 0) {
          fetch_y(seg - 1, py);
          fetch_kn(seg - 1, pkn);
          if (NG == 1) fetch_low(seg - 1, pl);
        }
        // After every ck_every-th segment (and the last): the rebuilt nodes
        // against the saved ones (!(<=): a NaN counts as a difference), which
        // replace them: the nodes right of the segment, and the bottom nodes
        // of its last column, published one lane down so that the first
        // reverse step receives them like the others receive their neighbours'.
        if ((seg + 1) % a.ck_every == 0 || seg + 1 == nseg) {
          const uint32_t c0 = (uint32_t)(seg / a.ck_every * KS * 64 + lane);
          double pk[KS];
#pragma unroll
          for (int i = 0; i < KS; ++i) pk[i] = at(ck, c0 + i * 64);
          if (seg + 1 < nseg) {
#pragma unroll
            for (int r = 0; r < R; ++r) bad = bad || drifted(kr[r], pk[r == 0 ? R - 1 + S : r - 1]);
            // (or at a pair's end since the last checkpoint) the task is handed back:
            // this segment is its last (leaving the loops here costs 2 % more)
            if (__ballot(bad) != 0) seg = band = 0;
          }
          kr[0] = pk[R - 1 + S];
#pragma unroll
          for (int r = 1; r < R; ++r) kr[r] = pk[r - 1];
          kc = pk[R - 2 + S];
#pragma unroll
          for (int cc = 0; cc < S; ++cc)
            pubK[cc] = group_prev<NG>(cc == 0 ? pk[R + S] : pk[R - 2 + cc], 1.0, first);
        }
        // the nodes at the last column of the pair that ends in the segment,
        // and the terminal cell's seed: the cell (last lane of the last band,
        // last row) receives it through its below-right neighbour, a = 0 + 0 - (-w)
        const int pe = pair_end(g0);
        double seed = 0.0;
        if (pe >= 0) {
          const int32_t k = NG == 1 ? (g0 + pe) / n : 0;
          const uint32_t c0 = (uint32_t)(k * (R + 1) * 64 + lane);
#pragma unroll
          for (int r = 0; r <= R; ++r) spe[r * 64 + lane] = at(pn, c0 + r * 64);
          if (last && lastl) seed = -pair_weight(a, ia, NG == 1 ? b0 + k : bg);
        }
        // the bands below have left their part of the y-side sums in part_y
        auto y_slot = [&](int e, int32_t& col) -> uint32_t {  // of element e of NY
          const int q = NG == 1 ? 0 : e / (C * D);
          const int e1 = e - q * (C * D);
          col = t0 + e1 / D;
          if ((uint32_t)col >= (uint32_t)group_total(q)) col = -1;
          const int32_t bq = NG == 1 ? col / n : q, qq = NG == 1 ? col - bq * n : col;
          return (uint32_t)((bq * a.nrows + qq) * D + e1 % D);
        };
        double po[NG == 1 ? PO : 1];
        if constexpr (YS && NG == 1) {
#pragma unroll
          for (int i = 0; i < PO; ++i) {
            const int e = lane + 64 * i;
            int32_t col;
            const uint32_t o = y_slot(e, col);
            po[i] = 0.0;
            if (!last && e < NY && col >= 0) po[i] = at(pyt, o);
          }
        }
        struct RevIn {
          float dy[DP];
          double kl[S];
          double lo[NG == 1 ? LW : 1];
        };
        auto read_rev = [&](int j, RevIn& in) {
          get_dy(j, in.dy);
#pragma unroll
          for (int cc = 0; cc < S; ++cc) in.kl[cc] = skn[(grp * C + j) * S + cc];
          if constexpr (NG == 1) {
#pragma unroll
            for (int f = 0; f < LW; ++f) in.lo[f] = sl[j * LW + f];
          }
        };
        double edge = 0.0;
        auto rev_step = [&](const int j, const RevIn& in) {
          const float(&dy)[DP] = in.dy;
          float h32[CR];
          inner(dx, dy, h32);
          double ab[S], kb[S];  // lane l+1's top-row a and top nodes
#pragma unroll
          for (int cc = 0; cc < S; ++cc) {
            ab[cc] = group_next<NG>(pubA[cc], NG == 1 ? in.lo[NG == 1 ? cc : 0] : 0.0, lastl);
            kb[cc] = group_next<NG>(pubK[cc], in.kl[cc], lastl);
          }
          // the coarse row below the strip is lane l+1's first one (R >= S), or
          // with R < S the lane's own or the next lane's (cb_below)
          const double gb = group_next<NG>(gpub, NG == 1 ? in.lo[NG == 1 ? S : 0] : 0.0, lastl);
          if (pe == j) {  // last column of a pair: nothing to the right
            // but, inside a run, the next pair, whose rebuilt left boundary is
            // summed here and checked after the segment (edge)
            if constexpr (NG == 1) {
              double s[R];
#pragma unroll
              for (int r = 0; r < R; ++r) s[r] = kr[r];
#pragma unroll
              for (int o = R / 2; o > 0; o /= 2)
#pragma unroll
                for (int r = 0; r < o; ++r) s[r] += s[r + o];
              edge = s[0];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
              ar[r] = 0.0;
              kr[r] = spe[r * 64 + lane];
            }
            kc = spe[R * 64 + lane];
            // (their factors are the next pair's, perhaps not finite)
#pragma unroll
            for (int c = 0; c < CR; ++c) gr[c] = 1.0;
            prev_ab0 = seed;
          }
          double gk[CR];
#pragma unroll
          for (int c = 0; c < CR; ++c) gk[c] = 1.0 + (double)h32[c];
          const double gbelow = (R >= S || cb_below) ? gb : gk[0];
          double v[R][S], kn[R][S], dg[CR];
#pragma unroll
          for (int c = 0; c < CR; ++c) dg[c] = 0.0;
#pragma unroll
          for (int dgl = R + S - 2; dgl >= 0; --dgl) {
#pragma unroll
            for (int cc = S - 1; cc >= 0; --cc) {
              const int r = dgl - cc;
              if (r < 0 || r >= R) continue;
              const int cr = (R >= S) ? (r >> LAM) : 0;
              // forward nodes: left-bottom, right-top, right-bottom
              const double ka = (r == R - 1) ? kb[cc] : kn[r + 1][cc];
              const double kt = (cc == S - 1) ? kr[r] : kn[r][cc + 1];
              const double kd = (r == R - 1) ? ((cc == S - 1) ? kc : kb[cc + 1])
                                             : ((cc == S - 1) ? kr[r + 1] : kn[r + 1][cc + 1]);
              const double sum = ka + kt;
              kn[r][cc] = __builtin_fma(gk[cr], sum, -kd);
              const double right = (cc == S - 1) ? ar[r] : v[r][cc + 1];
              const double gR = (cc == S - 1) ? gr[cr] : gk[cr];
              const double belowv = (r == R - 1) ? ab[cc] : v[r + 1][cc];
              const double gB = (r == R - 1) ? gbelow : gk[(R >= S) ? ((r + 1) >> LAM) : 0];
              const double diag = (r == R - 1) ? ((cc == S - 1) ? prev_ab0 : ab[cc + 1])
                                               : ((cc == S - 1) ? ar[r + 1] : v[r + 1][cc + 1]);
              v[r][cc] = __builtin_fma(gR, right, __builtin_fma(gB, belowv, -diag));
              // coefficient gradient of the coarse cell
              dg[cr] = __builtin_fma(v[r][cc], sum, dg[cr]);
            }
          }
#pragma unroll
          for (int c = 0; c < CR; ++c)
#pragma unroll
            for (int k = 0; k < D; ++k)
              dxacc[c][k] = __builtin_fma(dg[c], (double)dy[k], dxacc[c][k]);
          if constexpr (YS) {
            double* yr = &ring[grp * D * YL + ((t0 + j - lg) & (YW - 1))];
#pragma unroll
            for (int k = 0; k < D; ++k) {
              double t = dg[0] * dxd[0][k];
#pragma unroll
              for (int c = 1; c < CR; ++c) t = __builtin_fma(dg[c], dxd[c][k], t);
              __hip_atomic_fetch_add(&yr[k * YL], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
          }
          // the first lane's outputs for the band above
          if (NG == 1 && !top && first) {
#pragma unroll
            for (int cc = 0; cc < S; ++cc) sw[j * LW + cc] = v[0][cc];
            sw[j * LW + S] = gk[0];
          }
          gpub = gk[0];
#pragma unroll
          for (int cc = 0; cc < S; ++cc) {
            pubA[cc] = v[0][cc];
            pubK[cc] = kn[0][cc];
          }
          prev_ab0 = ab[0];
          kc = kb[0];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            ar[r] = v[r][0];
            kr[r] = kn[r][0];
          }
#pragma unroll
          for (int c = 0; c < CR; ++c) gr[c] = gk[c];
        };
        // inputs read one step ahead, alternating two buffers
        RevIn ra, rb;
        read_rev(C - 1, ra);
#pragma unroll 1
        for (int j = C - 1; j >= 1; j -= 2) {
          __builtin_amdgcn_sched_barrier(0);
          read_rev(j - 1, rb);
          rev_step(j, ra);
          __builtin_amdgcn_sched_barrier(0);
          read_rev(j >= 2 ? j - 2 : 0, ra);
          rev_step(j - 1, rb);
        }
        if (seg == 0) {  // left of the first column: the boundary
#pragma unroll
          for (int r = 0; r < R; ++r) bad = bad || drifted(kr[r], 1.0);
        }
        // left of the first column of the next pair of a run: the sum of a strip's
        // nodes (their errors grow alike from the right and hardly cancel: over
        // some 900 random pairs the largest error of a node was at most 2.2 times
        // the largest sum in 99 of 100, 12 times in all; comparing each node in
        // the step cost 6 to 10 % where pairs have 40 columns)
        if (NG == 1 && pe >= 0 && g0 + pe + 1 < total)
          bad = bad || !(fabs(edge - R) <= 2.0 * kRevTol);
        // the columns t0 .. t0 + C - 1, which the first lane has passed: the
        // y-side sums of the bands so far (final for the top band), and for
        // the band above the top-row a values and cell factors
        if (YS || !top) __syncthreads();
        if constexpr (YS) {
#pragma unroll
          for (int i = 0; i < PO; ++i) {
            const int e = lane + 64 * i;
            if (e < NY) {
              int32_t col;
              const uint32_t o = y_slot(e, col);
              const int q = NG == 1 ? 0 : e / (C * D);
              const int e1 = e - q * (C * D);
              double& r = ring[(q * D + e1 % D) * YL + ((t0 + e1 / D) & (YW - 1))];
              if (col >= 0) at(pyt, o) = NG == 1 ? po[NG == 1 ? i : 0] + r : r;
              r = 0.0;
            }
          }
        }
        if (NG == 1 && !top) {
          for (int e = lane; e < NL; e += 64) {
            const int32_t col = t0 + e / LW;
            if ((uint32_t)col < (uint32_t)total) at(abw, (uint32_t)(col * LW + e % LW)) = sw[e];
          }
        }
      }

      // x-side increment gradients of the band's coarse rows
      if constexpr (R < S) {
        // S / R consecutive lanes (aligned groups) share one coarse row
        constexpr int G = S / R;
#pragma unroll
        for (int o = 1; o < G; o <<= 1)
#pragma unroll
          for (int k = 0; k < D; ++k) dxacc[0][k] += __shfl_xor(dxacc[0][k], o, 64);
      }
      if constexpr (NG > 1) {  // the pairs of a wave share their x path
#pragma unroll
        for (int o = GL; o < 64; o <<= 1)
#pragma unroll
          for (int c = 0; c < CR; ++c)
#pragma unroll
            for (int k = 0; k < D; ++k) dxacc[c][k] += __shfl_xor(dxacc[c][k], o, 64);
      }
      const bool writer =
          grp == 0 && ((R >= S) || (lane % ((R < S) ? (S / R) : 1) == 0));
#pragma unroll
      for (int c = 0; c < CR; ++c) {
        const int p = p0 + c;
        if (writer && p >= 0 && p < m) {
#pragma unroll
          for (int k = 0; k < D; ++k) px[(int64_t)p * D + k] = dxacc[c][k];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }
    if (give_up || __ballot(bad) != 0) {
      int32_t i = 0;
      if (lane == 0) i = atomicAdd(a.redo_count, 1);
      i = __builtin_amdgcn_readlane(i, 0);
      a.redo[i] = task;  // every lane stores the same value
    }
    // rows of px beyond this path's increments (ragged batches) are never read
  }
}

}  // namespace grad
}  // namespace sk
