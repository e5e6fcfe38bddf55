// Sweep of the explicit (or implicit) scheme driven by precomputed coarse
// coefficients, for any number of channels.
//
// The fused sweeps (sweep_fwd_kernel.h) keep each lane's x increments in
// registers, which bounds the channels they take.  For wider paths the
// coarse increment Gram (Section 3.1: G0[p][q] = <dx_p, dy_q>) is formed
// first, a dense contraction over the channels on the matrix cores, and
// written in the order the sweep consumes it: wave-step t = g + lane of the run's
// column stream g, slot (lane, coarse row of the strip), scaled by the fine-cell
// factor 2^-(2 lambda + 1) (times 1 / rep^2 on a refined batch).  One step of one
// wave then reads 64 x CR consecutive floats.
//   * coef_kernel<PREC, NK> computes 32 x 128 tiles with v_mfma_f32_32x32x2_f32
//     (float32 increments) or v_mfma_f32_32x32x16_{bf16,f16} (16-bit inputs,
//     float32 sums) and turns them in LDS, so that it stores whole 128-byte
//     lines.
//   * coef_refined_kernel<PREC> serves dyadic orders beyond 3 (a batch refined rep
//     times): G0 of coarse cell (p, q) fills the rep x rep refined cells
//     (p rep + i, q rep + j).
//   * coef_sweep_kernel<R, LAM, IMPL, NG> is the one-wave sweep with the
//     inner products replaced by those loads (prefetched two steps ahead).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "internal.h"
#include "sweep_fwd_kernel.h"

namespace sk {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kKC = 32;    // channels staged per step
constexpr int kCols = 128; // columns per workgroup (four 32-column tiles)

using fwd::cell_block;
using fwd::first_row;
using fwd::group_prev;
using fwd::implicit_factors;
using fwd::locate_run;
using fwd::n_inc;
using fwd::store_out;
using fwd::wave_run;

// Lane of a strip layout of `gl` lanes that owns refined coarse row p of an
// m-row grid: strips are aligned to the bottom, lane l holding rows
// [m - (gl - l) cr, m - (gl - 1 - l) cr).
__device__ __forceinline__ int strip_lane(int32_t m, int32_t p, int32_t cr, int gl) {
  return gl - (m - p + cr - 1) / cr;
}

// The slots of a launched run: runs are numbered from a.s.wave0, ng of them side
// by side in a wave, each on gl = 64 / ng lanes.
__device__ __forceinline__ float* run_slots(const CoefArgs& a, int64_t wl, int gl, int32_t cr) {
  return a.s.coef + (wl / a.ng) * a.s.coef_stride + (wl % a.ng) * gl * cr;
}

template <int PREC>  // 0: float32, 1: bf16, 2: fp16
__global__ __launch_bounds__(256) void coef_refined_kernel(const CoefArgs a) {
  __shared__ float xs[32][kKC + 1];
  __shared__ float ys[kCols][kKC + 1];
  const int64_t slot = blockIdx.x;
  const int64_t wl = slot / a.s.run;
  const int32_t j = (int32_t)(slot - wl * a.s.run);
  // the pair of this slot, enumerated as the sweep's
  int64_t ia, b0, b1;
  if (!locate_run(a.s, a.s.wave0 + wl, ia, b0, b1)) return;
  const int64_t b = b0 + j;
  if (b >= b1) return;
  const int gl = 64 / a.ng;
  // refined counts (the sweep's) and the unrefined ones of the increments
  const int32_t mr = n_inc(a.s.x_n, a.s.x_len, ia), nr = n_inc(a.s.y_n, a.s.y_len, b);
  if (mr <= 0 || nr <= 0 || ((int64_t)mr << a.lam) > gl * (int64_t)a.R) return;
  const int32_t rep = a.rep;
  const int32_t m = mr / rep, n = nr / rep;
  const int32_t p_base = blockIdx.y * 32, q_base = blockIdx.z * kCols;
  if (p_base >= m || q_base >= n) return;
  const int64_t xrow = a.s.x_start ? a.s.x_start[ia] / rep : ia * (int64_t)m;
  const int64_t yrow = a.s.y_start ? a.s.y_start[b] / rep : b * (int64_t)n;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int row = lane & 31, half = lane >> 5;

  f32x16 acc = {};
  for (int k0 = 0; k0 < a.d; k0 += kKC) {
    __syncthreads();  // the previous step's tiles are consumed
    for (int e = threadIdx.x; e < 32 * kKC; e += blockDim.x) {
      const int r = e / kKC, k = e - r * kKC;
      xs[r][k] = (p_base + r < m && k0 + k < a.d)
                     ? a.incx[(xrow + p_base + r) * a.dpad + k0 + k]
                     : 0.0f;
    }
    for (int e = threadIdx.x; e < kCols * kKC; e += blockDim.x) {
      const int c = e / kKC, k = e - c * kKC;
      ys[c][k] = (q_base + c < n && k0 + k < a.d)
                     ? a.incy[(yrow + q_base + c) * a.dpad + k0 + k]
                     : 0.0f;
    }
    __syncthreads();
    const int col = wid * 32 + row;
    if constexpr (PREC == 0) {
#pragma unroll
      for (int kk = 0; kk < kKC; kk += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[row][kk + half], ys[col][kk + half], acc,
                                                    0, 0, 0);
    } else {
#pragma unroll
      for (int kk = 0; kk < kKC; kk += 16) {
        if constexpr (PREC == 1) {
          bf16x8 A, B;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            A[t] = (__bf16)xs[row][kk + half * 8 + t];
            B[t] = (__bf16)ys[col][kk + half * 8 + t];
          }
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B, acc, 0, 0, 0);
        } else {
          f16x8 A, B;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            A[t] = (_Float16)xs[row][kk + half * 8 + t];
            B[t] = (_Float16)ys[col][kk + half * 8 + t];
          }
          acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B, acc, 0, 0, 0);
        }
      }
    }
  }

  // accumulator register r of this lane: row 8 (r / 4) + 4 half + (r mod 4),
  // column row (the MFMA output layout)
  const int32_t cr = a.R >> a.lam;
  const int32_t q = q_base + wid * 32 + row;
  if (q >= n) return;
  float* __restrict__ base = run_slots(a, wl, gl, cr);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int32_t p = p_base + 8 * (r >> 2) + 4 * half + (r & 3);
    if (p >= m) continue;
    const float v = acc[r] * a.scale;
    for (int32_t i = 0; i < rep; ++i) {
      const int32_t pr = p * rep + i;
      const int l2 = strip_lane(mr, pr, cr, gl);
      const int32_t c = pr - (mr - (gl - l2) * cr);
      for (int32_t jj = 0; jj < rep; ++jj) {
        const int64_t t = (int64_t)j * nr + (int64_t)q * rep + jj + l2;
        base[(t * 64 + l2) * cr + c] = v;
      }
    }
  }
}

// The unrefined coefficients of one x path against the column stream of its y
// paths (their increment rows are consecutive; ragged y batches: of one pair):
// one 32 x 128 tile per workgroup, whatever runs its columns belong to.
//
// A wave holds its 32 columns' increments and the tile's rows in registers (lane
// (row or column, half): channels 8 k + 4 half .. + 3 of NK groups of 8; wider
// paths in several passes), so the operands need no LDS.  The tile then goes
// through LDS: with flat row index f = lane CR + row of the strip, step t of a run's slots
// holds 32 consecutive f of a tile as one 128-byte line, each from its own column
// t - lane.  Stored from the accumulators each value went to a line of its own
// (64 x 48 pairs of 150 points, d = 40: 442 us of the call's 526).  One tile per
// workgroup: in a loop over row tiles each tile's loads waited for the previous
// one's stores (one counter), 193 us.  Tiles start at multiples of 32 in f; bound:
// the lines' stores and the MFMAs (2 d flops a value).
// Now 146 us of that call's 243; the sweep, bound by its loads, 104 (132 before)
// with six rows per lane for 298 instead of eight and idle lanes' loads held.
constexpr int kTileStride = 130;  // floats per tile row: steps' reads touch distinct banks
template <int PREC, int NK>
__global__ __launch_bounds__(256) void coef_kernel(const CoefArgs a) {
  __shared__ float tile[32 * kTileStride];
  const int gl = 64 / a.ng;
  const int32_t cr = a.R >> a.lam;
  // the row's pairs [bs, be), its first run and that run's first pair if the runs
  // were not clipped (32-bit by rows: the host bounds a row's columns)
  int64_t ia, run0;
  uint32_t bs, be, aligned;
  const uint32_t run = (uint32_t)a.s.run;
  if (a.by_row) {
    ia = a.row0 + blockIdx.x;
    const int64_t s = a.s.tri ? a.s.tri - 1 : 0;
    bs = a.s.mode == 2 ? (uint32_t)(ia + s) : 0;
    be = (uint32_t)a.s.ny;
    aligned = bs / run * run;
    run0 = a.s.mode != 2 ? ia * a.s.runs_per_row
           : a.s.tri32   ? (int64_t)tri_runs_of<uint32_t>((uint32_t)ia, (uint32_t)a.s.runs_per_row,
                                                          run, (uint32_t)s)
                         : tri_runs(ia, a.s.runs_per_row, a.s.run, s);
  } else {
    int64_t b0, b1;
    run0 = a.s.wave0 + blockIdx.x;
    if (!locate_run(a.s, run0, ia, b0, b1)) return;
    bs = (uint32_t)b0;
    be = (uint32_t)b1;
    aligned = bs;
  }
  if (bs >= be) return;
  const int32_t m = n_inc(a.s.x_n, a.s.x_len, ia);
  const int32_t n = n_inc(a.s.y_n, a.s.y_len, bs);  // of every pair of several
  if (m <= 0 || n <= 0 || ((int64_t)m << a.lam) > gl * (int64_t)a.R) return;
  const int32_t total = (int32_t)(be - bs) * n;
  const int32_t q_base = (int32_t)blockIdx.y * kCols;
  const int32_t off = gl * cr - m;  // flat index of row 0: virtual rows above it
  const int32_t f0 = (off & ~31) + 32 * (int32_t)blockIdx.z;
  if (q_base >= total || f0 >= gl * cr) return;
  const float* __restrict__ xinc = a.incx + first_row(a.s.x_start, a.s.x_len, ia) * a.dpad;
  const float* __restrict__ yinc = a.incy + first_row(a.s.y_start, a.s.y_len, bs) * a.dpad;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int row = lane & 31, half = lane >> 5;
  const uint32_t inv = (1u << 20) / (uint32_t)cr + 1;  // f / cr = f inv >> 20 for f < 2080, cr <= 32
  // the runs of the tile's columns
  const int32_t q_end = q_base + kCols < total ? q_base + kCols : total;
  const int32_t k_first = (int32_t)((bs + (uint32_t)q_base / (uint32_t)n - aligned) / run);
  const int32_t k_last = (int32_t)((bs + (uint32_t)(q_end - 1) / (uint32_t)n - aligned) / run);
  if (run0 + k_last < a.s.wave0 || run0 + k_first >= a.s.wave0 + a.s.n_waves) return;

  // NK groups of 8 channels from k0 on of one row of increments
  auto load = [&](const float* __restrict__ p, bool real, int32_t k0, float4 (&v)[NK]) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int32_t c = k0 + 8 * k + 4 * half;
      v[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (real && c < a.dpad) v[k] = *reinterpret_cast<const float4*>(p + c);
    }
  };
  auto contract = [&](const float4 (&x)[NK], const float4 (&y)[NK], int32_t groups, f32x16& acc) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      if (k >= groups) break;  // uniform
      if constexpr (PREC == 0) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[k].x, y[k].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[k].y, y[k].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[k].z, y[k].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[k].w, y[k].w, acc, 0, 0, 0);
      } else if (k % 2 == 0) {
        // two groups: a lane's eight channels of the instruction's sixteen (which
        // ones is free, the same for x and y)
        const float xv[8] = {x[k].x, x[k].y, x[k].z, x[k].w, x[k + 1].x, x[k + 1].y, x[k + 1].z,
                             x[k + 1].w};
        const float yv[8] = {y[k].x, y[k].y, y[k].z, y[k].w, y[k + 1].x, y[k + 1].y, y[k + 1].z,
                             y[k + 1].w};
        if constexpr (PREC == 1) {
          bf16x8 A, B;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            A[t] = (__bf16)xv[t];
            B[t] = (__bf16)yv[t];
          }
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B, acc, 0, 0, 0);
        } else {
          f16x8 A, B;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            A[t] = (_Float16)xv[t];
            B[t] = (_Float16)yv[t];
          }
          acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B, acc, 0, 0, 0);
        }
      }
    }
  };

  const int32_t q = q_base + wid * 32 + row;
  const float* __restrict__ yp = yinc + (int64_t)q * a.dpad;
  const float* __restrict__ xp = xinc + (int64_t)(f0 - off + row) * a.dpad;
  const bool x_real = (uint32_t)(f0 - off + row) < (uint32_t)m;
  float4 x[NK], y[NK];
  f32x16 acc = {};
  for (int32_t k0 = 0; k0 < a.dpad; k0 += 8 * NK) {
    load(xp, x_real, k0, x);
    load(yp, q < total, k0, y);
    const int32_t left = (a.dpad - k0 + 7) / 8;
    contract(x, y, left < NK ? left : NK, acc);
  }
  // accumulator register r of this lane: tile row 8 (r / 4) + 4 half + (r mod 4),
  // column `row` (the MFMA output layout)
#pragma unroll
  for (int r = 0; r < 16; ++r)
    tile[(8 * (r >> 2) + 4 * half + (r & 3)) * kTileStride + wid * 32 + row] = acc[r] * a.scale;
  __syncthreads();
  // the steps that hold the tile, run by run: thread (step, group of four rows)
  const int32_t l_first = (int32_t)((uint32_t)f0 * inv >> 20);
  const int32_t l_last = (int32_t)((uint32_t)(f0 + 31) * inv >> 20);
  const int32_t r0 = 4 * (threadIdx.x & 7);
  // row i holds column t - lag[i] of its run at step t
  int32_t lag[4];
  bool real[4], all = true;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t f = f0 + r0 + i;
    lag[i] = (int32_t)((uint32_t)f * inv >> 20);
    real[i] = (uint32_t)(f - off) < (uint32_t)m;
    all = all && real[i];
  }
  for (int32_t k = k_first; k <= k_last; ++k) {
    const int64_t wl = run0 + k - a.s.wave0;
    if (wl < 0 || wl >= a.s.n_waves) continue;  // another chunk's
    // the run's columns [c0, c1) of the row's stream, and those of the tile
    const uint32_t bk = aligned + (uint32_t)k * run;
    const int32_t c0 = (int32_t)((bk > bs ? bk : bs) - bs) * n;
    const int32_t c1 = (int32_t)((bk + run < be ? bk + run : be) - bs) * n;
    const int32_t ca = (c0 > q_base ? c0 : q_base) - c0;
    const int32_t cb = (c1 < q_end ? c1 : q_end) - c0;
    const int32_t to_tile = c0 - q_base;  // run column to tile column
    float* __restrict__ base = run_slots(a, wl, gl, cr) + f0 + r0;
    for (int32_t t = ca + l_first + (threadIdx.x >> 3); t < cb + l_last; t += 32) {
      const float* __restrict__ tp = &tile[r0 * kTileStride + t + to_tile];
      float* __restrict__ o = base + (int64_t)t * (64 * cr);
      if (all && t - lag[3] >= ca && t - lag[0] < cb) {
        *reinterpret_cast<float4*>(o) =
            make_float4(tp[-lag[0]], tp[kTileStride - lag[1]], tp[2 * kTileStride - lag[2]],
                        tp[3 * kTileStride - lag[3]]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int32_t c = t - lag[i];
          if (real[i] && c >= ca && c < cb) o[i] = tp[i * kTileStride - lag[i]];
        }
      }
    }
  }
}

// The one-wave sweep of sweep_fwd_kernel.h with the coarse coefficients read
// from the layout coef_kernel writes.  R >= 2^LAM: every coarse row belongs to
// one lane.  Rows above the grid (virtual rows of the top strip) take
// coefficient 0 without reading.
// NG > 1: several runs side by side, as in sweep_fwd_kernel.h.
template <int R, int LAM, bool IMPL, int NG>
__global__ __launch_bounds__(256) void coef_sweep_kernel(const SweepArgs a) {
  constexpr int GL = 64 / NG;
  constexpr int S = 1 << LAM;
  constexpr int CR = R >> LAM;
  static_assert(CR >= 1, "a coarse row must not span lanes");

  const int lane = threadIdx.x & (GL - 1);  // of the group
  const int gid = NG == 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))
                          : (int)(threadIdx.x / GL);
  const int64_t wl = (int64_t)blockIdx.x * (blockDim.x / GL) + gid;  // launched run
  const int64_t w = a.wave0 + wl;
  if (wl >= a.n_waves) return;
  int64_t ia, b0, b1, total;
  int32_t m;
  if (!wave_run(a, w, lane, GL * R, LAM, ia, b0, b1, m, total, GL)) return;
  const int32_t p0 = m - (GL - lane) * CR;  // negative rows are virtual
  const int32_t total32 = (int32_t)total;
  const int32_t cn = n_inc(a.y_n, a.y_len, b0);
  int32_t g = -lane;
  int32_t q = 0;
  // wave-step t of this lane's slot: cp + t 64 CR
  const float* __restrict__ cp =
      a.coef + wl / NG * a.coef_stride + (int64_t)(threadIdx.x & 63) * CR;

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
  bool real[CR];
#pragma unroll
  for (int c = 0; c < CR; ++c) real[c] = p0 + c >= 0;

  float cA[CR], cB[CR], cC[CR];
#pragma unroll
  for (int c = 0; c < CR; ++c) {
    cA[c] = cp[c];
    cB[c] = cp[64 * CR + c];
  }
  const int32_t nsteps = (int32_t)sweep_steps(total, GL);
  // lanes of virtual rows alone stay where they are (one line in the L1): the
  // sweep is bound by its loads, and a load under a condition costs more than it
  // saves (the wait for it then covers all loads in flight: 144 us against 114)
  const int32_t ahead = p0 + CR > 0 ? 64 * CR : 0;
  auto step = [&](float (&cur)[CR], float (&refill)[CR]) {
#pragma unroll
    for (int c = 0; c < CR; ++c) refill[c] = cp[2 * 64 * CR + c];
#pragma unroll
    for (int cc = 0; cc < S; ++cc) up[cc] = group_prev<NG>(pub[cc], up[cc], lane == 0);
    if ((uint32_t)g < (uint32_t)total32) {
      double gk[CR], h[CR];
#pragma unroll
      for (int c = 0; c < CR; ++c) h[c] = real[c] ? (double)cur[c] : 0.0;
      if constexpr (IMPL) {
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
          const int64_t cb = b0 + g / cn;
          store_out(a, ia, cb, (a.mode == 2 && a.no_diag && cb == ia) ? 0.0f : (float)u[R - 1]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = 1.0;
        up_last = 1.0;
        q = 0;
      }
    }
    ++g;
    cp += ahead;
  };
  for (int32_t t = 0; t < nsteps; t += 3) {
    step(cA, cC);
    step(cB, cA);
    step(cC, cB);
  }
}

using SweepFn = void (*)(const SweepArgs);

template <int R, int LAM, int NG>
SweepFn pick_impl(bool implicit) {
  if constexpr ((R >> LAM) >= 1 && R % (1 << LAM) == 0 && (NG == 1 || R <= 16))
    return implicit ? &coef_sweep_kernel<R, LAM, true, NG> : &coef_sweep_kernel<R, LAM, false, NG>;
  else
    return nullptr;
}

template <int R, int NG>
SweepFn pick_lam(int lam, bool implicit) {
  switch (lam) {
    case 0: return pick_impl<R, 0, NG>(implicit);
    case 1: return pick_impl<R, 1, NG>(implicit);
    case 2: return pick_impl<R, 2, NG>(implicit);
    case 3: return pick_impl<R, 3, NG>(implicit);
    default: return nullptr;
  }
}

template <int NG>
SweepFn pick_rows(int R, int lam, bool implicit) {
  switch (R) {
    case 1: return pick_lam<1, NG>(lam, implicit);
    case 2: return pick_lam<2, NG>(lam, implicit);
    case 3: return pick_lam<3, NG>(lam, implicit);
    case 4: return pick_lam<4, NG>(lam, implicit);
    case 5: return pick_lam<5, NG>(lam, implicit);
    case 6: return pick_lam<6, NG>(lam, implicit);
    case 8: return pick_lam<8, NG>(lam, implicit);
    case 10: return pick_lam<10, NG>(lam, implicit);
    case 12: return pick_lam<12, NG>(lam, implicit);
    case 16: return pick_lam<16, NG>(lam, implicit);
    case 20: return pick_lam<20, NG>(lam, implicit);
    case 24: return pick_lam<24, NG>(lam, implicit);
    case 32: return pick_lam<32, NG>(lam, implicit);
    default: return nullptr;
  }
}

template <int PREC>
void launch_coef_prec(const CoefArgs& a, const dim3& grid, hipStream_t stream) {
  if (a.dpad <= 32)
    hipLaunchKernelGGL((coef_kernel<PREC, 4>), grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((coef_kernel<PREC, 8>), grid, dim3(256), 0, stream, a);
}

}  // namespace

void* coef_sweep_fn(bool implicit, int lam, int R, int ng) {
  return reinterpret_cast<void*>(ng == 1   ? pick_rows<1>(R, lam, implicit)
                                 : ng == 4 ? pick_rows<4>(R, lam, implicit)
                                           : nullptr);
}

int64_t coef_wave_floats(int64_t total_cols, int R, int lam, int ng) {
  // the sweep's steps plus its two-step prefetch
  return (sweep_steps(total_cols, 64 / ng) + 2) * 64 * (int64_t)(R >> lam);
}

hipError_t launch_coef(const CoefArgs& a, int precision, int64_t max_m, int64_t max_n,
                       hipStream_t stream) {
  const int64_t runs = a.s.n_waves;
  if (runs == 0 || max_m <= 0 || max_n <= 0) return hipSuccess;
  if (a.rep == 1) {
    // columns of a row's stream (by_row) or of a run
    const int64_t cols = max_n * (a.by_row ? a.s.ny : a.s.run);
    const int64_t cb = (cols + kCols - 1) / kCols;
    const int64_t rows = a.by_row ? a.rows : runs;
    // row tiles of the tallest path, wherever its rows start in a multiple of 32
    const int64_t tiles = (max_m + 31 + 31) / 32;
    if (rows > 0x7FFFFFFF || cb > 65535 || tiles > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)rows, (unsigned)cb, (unsigned)tiles);
    if (precision == kRoundBf16)
      launch_coef_prec<1>(a, grid, stream);
    else if (precision == kRoundF16)
      launch_coef_prec<2>(a, grid, stream);
    else
      launch_coef_prec<0>(a, grid, stream);
    return hipGetLastError();
  }
  const int64_t slots = runs * a.s.run;
  const int64_t rb = (max_m + 31) / 32, cb = (max_n + kCols - 1) / kCols;
  if (slots > 0x7FFFFFFF || rb > 65535 || cb > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)slots, (unsigned)rb, (unsigned)cb);
  if (precision == kRoundBf16)
    hipLaunchKernelGGL(coef_refined_kernel<1>, grid, dim3(256), 0, stream, a);
  else if (precision == kRoundF16)
    hipLaunchKernelGGL(coef_refined_kernel<2>, grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(coef_refined_kernel<0>, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_coef_sweep(const SweepArgs& a, int lam, int R, int ng, bool implicit,
                             hipStream_t stream, int wpb) {
  const SweepFn f = reinterpret_cast<SweepFn>(coef_sweep_fn(implicit, lam, R, ng));
  if (!f) return hipErrorInvalidValue;
  if (a.n_waves == 0) return hipSuccess;
  if (wpb != 1 && wpb != 2) wpb = 4;
  const int64_t blocks = (a.n_waves + wpb * ng - 1) / (wpb * ng);
  hipLaunchKernelGGL(f, dim3((unsigned)blocks), dim3(64 * wpb), 0, stream, a);
  return hipGetLastError();
}

}  // namespace sk
