// Launchers of the forward sweep kernels (sweep_fwd_kernel.h) and the table of
// compiled configurations (instantiated per dyadic order in sweep_lam*.hip).
#include "dispatch.h"
#include "internal.h"

namespace sk {

#define SK_DECL(k, l) void* sweep_fn_k##k##_l##l##_(int R, int d);
SK_DECL(3, 0) SK_DECL(3, 1) SK_DECL(3, 2) SK_DECL(3, 3)
SK_DECL(6, 0) SK_DECL(6, 1) SK_DECL(6, 2) SK_DECL(6, 3)
SK_DECL(7, 0) SK_DECL(7, 1) SK_DECL(7, 2) SK_DECL(7, 3)
#undef SK_DECL
#define SK_DECL(k, l) void* sweep_fn_k##k##_l##l##_g1(int R, int d); void* sweep_fn_k##k##_l##l##_g4(int R, int d);
SK_DECL(0, 0) SK_DECL(0, 1) SK_DECL(0, 2) SK_DECL(0, 3)
SK_DECL(4, 0) SK_DECL(4, 1) SK_DECL(4, 2) SK_DECL(4, 3)
SK_DECL(5, 0) SK_DECL(5, 1) SK_DECL(5, 2) SK_DECL(5, 3)
#undef SK_DECL

void* none_(int, int) { return nullptr; }  // kinds 1 and 2 are not compiled, 0, 4 and 5 by forward_fn and lifted_fn

void* sweep_fn(int kind, int lam, int R, int d) {
  using Pick = void* (*)(int, int);
  static const Pick table[8][4] = {
      {none_, none_, none_, none_},
      {none_, none_, none_, none_},
      {none_, none_, none_, none_},
      {sweep_fn_k3_l0_, sweep_fn_k3_l1_, sweep_fn_k3_l2_, sweep_fn_k3_l3_},
      {none_, none_, none_, none_},
      {none_, none_, none_, none_},
      {sweep_fn_k6_l0_, sweep_fn_k6_l1_, sweep_fn_k6_l2_, sweep_fn_k6_l3_},
      {sweep_fn_k7_l0_, sweep_fn_k7_l1_, sweep_fn_k7_l2_, sweep_fn_k7_l3_}};
  if (kind < 0 || kind > 7 || lam < 0 || lam > 3) return nullptr;
  return table[kind][lam](R, d);
}

namespace {
void* grouped_fn(int kind, int lam, int R, int ng, int d) {
  using Pick = void* (*)(int, int);
#define SK_ROW(k, l) {sweep_fn_k##k##_l##l##_g1, sweep_fn_k##k##_l##l##_g4}
#define SK_KIND_ROWS(k) {SK_ROW(k, 0), SK_ROW(k, 1), SK_ROW(k, 2), SK_ROW(k, 3)}
  static const Pick table[3][4][2] = {SK_KIND_ROWS(0), SK_KIND_ROWS(5), SK_KIND_ROWS(4)};
#undef SK_KIND_ROWS
#undef SK_ROW
  if (lam < 0 || lam > 3 || (ng != 1 && ng != 4)) return nullptr;
  return table[kind][lam][ng == 1 ? 0 : 1](R, d);
}
}  // namespace

void* forward_fn(bool implicit, int lam, int R, int ng, int d) {
  return grouped_fn(implicit ? 1 : 0, lam, R, ng, d);
}
void* lifted_fn(int lam, int R, int ng, int d) { return grouped_fn(2, lam, R, ng, d); }

bool forward_takes(int64_t fine_rows, int lam, int d) {
  return lam >= 0 && lam <= 3 && d >= 1 && d <= 16 &&
         fine_rows <= 64 * (int64_t)max_fitting_rows(lam, d);
}

bool lifted_takes(int64_t fine_rows, int lam, int d) {
  return lam >= 0 && lam <= 3 && d >= 1 && d <= 16 &&
         fine_rows <= 64 * (int64_t)max_lifted_rows(lam, d);
}

namespace {
hipError_t launch_forward(void* fn, const SweepArgs& a, int ng, hipStream_t stream, int wpb) {
  auto f = reinterpret_cast<void (*)(const SweepArgs)>(fn);
  if (!f) return hipErrorInvalidValue;
  if (a.n_waves == 0) return hipSuccess;
  if (wpb != 1 && wpb != 2) wpb = 4;  // the kernels are bounded to 256 threads
  const int64_t blocks = (a.n_waves + wpb * ng - 1) / (wpb * ng);
  hipLaunchKernelGGL(f, dim3((unsigned)blocks), dim3(64 * wpb), 0, stream, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_sweep(const SweepArgs& a, int lam, int R, int ng, int d, hipStream_t stream,
                        int waves_per_block) {
  return launch_forward(forward_fn(a.implicit != 0, lam, R, ng, d), a, ng, stream,
                        waves_per_block);
}

hipError_t launch_lifted(const SweepArgs& a, int lam, int R, int ng, int d, hipStream_t stream,
                         int waves_per_block) {
  return launch_forward(lifted_fn(lam, R, ng, d), a, ng, stream, waves_per_block);
}

}  // namespace sk
