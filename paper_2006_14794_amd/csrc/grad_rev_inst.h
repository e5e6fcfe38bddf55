// Instantiations of the reversing gradient kernel (grad_rev_kernel.h) at one
// dyadic order SK_LAM, SK_ROWS rows per lane and SK_NG pairs per wave, for 1
// to 16 channels where they are compiled.  Included by
// grad_rev_l{lam}_r{rows}_g{ng}.hip so that they compile in parallel
// translation units.
#include "dispatch.h"
#include "grad_rev_kernel.h"

#define SK_CAT2(a, b) a##b
#define SK_CAT(a, b) SK_CAT2(a, b)

namespace sk {
namespace {
template <bool YS>
struct GradRev {
  using Fn = void*;
  template <int R, int LAM, int D>
  static Fn get() {
    if constexpr (grad_rev_fits(R, LAM, D))
      return reinterpret_cast<void*>(
          &grad::grad_rev_kernel<R, LAM, D, grad_rev_segment(LAM), SK_NG, YS>);
    else
      return nullptr;
  }
};
}  // namespace

void* SK_CAT(SK_CAT(SK_CAT(SK_CAT(SK_CAT(grad_rev_fn_l, SK_LAM), _r), SK_ROWS), _g), SK_NG)(int d,
                                                                                           bool ys) {
  return ys ? pick_d<GradRev<true>, SK_ROWS, SK_LAM>(d)
            : pick_d<GradRev<false>, SK_ROWS, SK_LAM>(d);
}

}  // namespace sk
