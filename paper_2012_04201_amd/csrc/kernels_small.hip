// The LDS-resident fp32 training kernel for one small hidden layer, all variants.
#include "train_small_f32.h"

#include "kernels.h"

namespace {
template <int KT>
const void* by_outputs(int co) {
  return co == 1 ? (const void*)k_train_small<KT, 1> : (co == 2 ? (const void*)k_train_small<KT, 2> : (const void*)k_train_small<KT, 4>);
}
}  // namespace

const void* small_kernel(int kt, int co) { return kt == 1 ? by_outputs<1>(co) : (kt == 2 ? by_outputs<2>(co) : by_outputs<4>(co)); }
