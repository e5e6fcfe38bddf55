// Argument block and scratch geometry of the Gram gradient kernel
// (grad_kernel.h), kept apart so that the kernel compiles from this file, the
// forward sweep's header and nothing else of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sk {

// Work description of one gradient launch.  A task is a run of pairs
// (x_ia, y_b), b in [b0, b1), sharing the x path (uniform y batches), or one
// pair taken from `order` (ragged batches).
struct GradArgs {
  const float* incx;        // dense x increments, pre-scaled by 2^-(2 lam + 1)
  const float* incy;        // dense y increments
  const int32_t* x_n;       // ragged plans (nullptr for a uniform batch)
  const int64_t* x_start;
  const int32_t* y_n;
  const int64_t* y_start;
  int32_t x_len, y_len;     // points per path as swept (upper bounds when ragged)
  int64_t nx, ny;
  int32_t mode;             // 1: every pair; 2: upper triangle of a symmetric Gram
  int32_t no_diag;          // mode 2: the diagonal is the constant 0 (no gradient)
  int32_t run;              // pairs per task of a uniform y batch
  int64_t runs_per_row;     // tasks per x path (ny when `order` is set)
  int32_t n_tasks;
  const int32_t* order;     // ragged: task t is pair order[t] = a ny + b; nullptr: runs
  int32_t* counter;         // queue head, zeroed before the launch
  const float* dK;          // [nx][ny] upstream weights
  float* K;                 // [nx][ny] forward values (nullptr: not written)
  double* scratch;          // per wave slot: slot_stride doubles (grad_slot_layout)
  int64_t slot_stride;
  int32_t nb_max;           // row bands of the tallest x path
  int32_t nseg_max;         // segments of the longest task
  int32_t ck_every;         // reversing kernel: segments per checkpoint,
  int32_t nck_max;          // ... and checkpoints of the longest task
  double huge;              // ... and the node value from which a task is handed back unseen
  int64_t cols_max;         // coarse columns of the longest task
  double* part_x;           // [nx][runs_per_row][mrows][dim]: x-side increment gradients
  double* part_y;           // [nx][ny][nrows][dim]: y-side increment gradients
  int32_t mrows, nrows;     // x_len - 1, y_len - 1
  // tasks whose rebuilt forward nodes differed too much (grad_rev_kernel.h):
  // that kernel appends them here, and grad_kernel.h takes its tasks from this
  // list alone (nullptr there: all n_tasks tasks, where the plan has no
  // reversing launch before it)
  int32_t* redo;
  int32_t* redo_count;      // zeroed before the launches
};

// Fine rows per lane of the gradient kernel: bands of 64 R rows.
constexpr int kGradRows = 4;

// Forward steps per segment: the adjoint recomputes a segment from its
// checkpoint and keeps the segment's R 2^lam cell sums per step on chip, the
// first grad_lds_steps steps in LDS (64 floats per lane: 16 KB per wave) and
// the rest in registers (32 floats per lane; half that at order 0, whose
// increments and gradient accumulators take more registers).
__host__ __device__ constexpr int grad_reg_steps(int lam, int d) {
  const int rs = kGradRows << lam;
  // order 0 keeps four coarse rows per lane (increments, accumulators)
  const int floats = 32 / (lam == 0 ? 2 : 1) + 0 * d;
  const int c = floats / rs;
  return c < 1 ? 1 : c;
}
__host__ __device__ constexpr int grad_lds_steps(int lam) {
  const int c = 64 / (kGradRows << lam);
  return c < 1 ? 1 : c;
}
__host__ __device__ constexpr int grad_segment(int lam, int d) {
  return grad_reg_steps(lam, d) + grad_lds_steps(lam);
}

// Doubles of the wave state saved per lane at a checkpoint: the lane's first
// R - 1 values at its last fine column, its bottom row at the 2^lam fine
// columns of its last step (whose last entry is the R-th value, unless that
// column ended a pair and the values restarted at 1), and the upper-left
// neighbour of its next block.
__host__ __device__ constexpr int grad_state_doubles(int lam) {
  return kGradRows + (1 << lam);
}

// Scratch of one wave slot, in doubles:
//   checkpoints  [nb_max][nseg_max - 1][state][64 lanes]   (segment 0 starts from the boundary)
//   hand_f       [nb_max - 1][cols_max << lam]             forward: bottom rows of the bands
//   hand_a       [2][cols_max + 1][2^lam + 1]              adjoint: a values of a band's top
//                                                         row and its first coarse row's
//                                                         coefficient, for the band above
struct GradSlot {
  int64_t ckpt, hand_f, hand_a, stride;
};
__host__ __device__ inline GradSlot grad_slot_layout(int lam, int nb_max, int nseg_max,
                                                     int64_t cols_max) {
  GradSlot s{};
  const int64_t S = int64_t(1) << lam;
  s.ckpt = 0;
  s.hand_f = (int64_t)nb_max * (nseg_max - 1) * grad_state_doubles(lam) * 64;
  s.hand_a = s.hand_f + (int64_t)(nb_max - 1) * cols_max * S;
  s.stride = s.hand_a + 2 * (cols_max + 1) * (S + 1);
  s.stride = (s.stride + 31) & ~int64_t(31);  // 256-byte aligned slots
  return s;
}

// ---- the reversing kernel (grad_rev_kernel.h) ----
// Compiled rows per lane R: 4 always, 8 where the increments and accumulators
// of the 8 / 2^lam coarse rows leave two waves per SIMD, or (more than 16 values)
// one: half as many bands or lanes make up for it where a path fills them (30 x 30
// paths of 400 points, d = 5, order 1: 929 us the call, 1293 with four rows; 64 x
// 64 of 100, d = 7, order 2: 625 against 785; 100 x 100 of 120, d = 6, order 1 the
// other way round: 953 against 860, and four rows run).
__host__ __device__ constexpr bool grad_rev_fits(int R, int lam, int d) {
  if (R == 4) return true;
  return R == 8 && lam <= 2 && (8 >> lam) * d <= 24;
}
// Steps per segment of the staging.  Even, at most 32 (the pair-end masks).
__host__ __device__ constexpr int grad_rev_segment(int lam) {
  return lam == 0 ? 32 : lam == 1 ? 24 : lam == 2 ? 16 : 8;
}
// Segments between two checkpoints (R + 2^lam + 1 doubles per lane): at most
// four, and one in tasks of fewer than 16 segments, so that the rebuilt nodes
// drift over at most an eighth of a task's columns, or one segment.
__host__ __device__ constexpr int grad_rev_ck_every(int nseg_max) {
  return nseg_max >= 32 ? 4 : nseg_max >= 16 ? nseg_max / 8 : 1;
}
// Two waves per SIMD (256 registers) where the increments and their double
// accumulators leave room for the sweep's state; else one or two, as the
// registers allow.
__host__ __device__ constexpr int grad_rev_waves(int R, int lam, int d) {
  return (R == 8 ? (8 >> lam) * d <= 16
                 : 3 * ((R >> lam) > 0 ? (R >> lam) : 1) * d + 4 * d <= 64) &&
                 lam < 3
             ? 2
             : 1;
}
__host__ __device__ constexpr int grad_rev_state_doubles(int R, int lam) {
  return R + (1 << lam) + 1;
}

// Scratch of one wave slot, in doubles:
//   ckpt    [nb_max][nck_max][state][64 lanes]    the state after every ck_every segments
//   hand_f  [nb_max][cols_max << lam]             bottom rows of the bands
//   hand_a  [2][cols_max + 1][2^lam + 1]          as in GradSlot
//   pend    [nb_max][pairs][R + 1][64 lanes]      the strips' nodes at the pairs' last columns
struct GradRevSlot {
  int64_t ckpt, hand_f, hand_a, pend, stride;
};
__host__ __device__ inline GradRevSlot grad_rev_slot_layout(int R, int lam, int nb_max,
                                                            int nck_max, int64_t cols_max,
                                                            int64_t pairs) {
  GradRevSlot s{};
  const int64_t S = int64_t(1) << lam;
  s.ckpt = 0;
  s.hand_f = (int64_t)nb_max * nck_max * grad_rev_state_doubles(R, lam) * 64;
  s.hand_a = s.hand_f + (int64_t)nb_max * cols_max * S;
  s.pend = s.hand_a + 2 * (cols_max + 1) * (S + 1);
  s.stride = s.pend + (int64_t)nb_max * pairs * (R + 1) * 64;
  s.stride = (s.stride + 31) & ~int64_t(31);
  return s;
}

}  // namespace sk
