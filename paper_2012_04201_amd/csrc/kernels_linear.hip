// The wavefront-per-model training kernel, all variants: padded outputs 1, 2, 4, 8, 16 by rows of W per lane 1, 2,
// 4, at most 32 parameters per lane.
#include "train_linear_f32.h"

#include "kernels.h"

namespace {
template <int CO>
const void* by_rows(int ki) {
  switch (ki) {
    case 1: return (const void*)k_train_linear<CO, 1>;
    case 2: return (const void*)k_train_linear<CO, 2>;
  }
  if constexpr (CO <= 8) return (const void*)k_train_linear<CO, 4>;
  return nullptr;
}
}  // namespace

const void* linear_kernel(int co, int ki) {
  switch (co) {
    case 1: return by_rows<1>(ki);
    case 2: return by_rows<2>(ki);
    case 4: return by_rows<4>(ki);
    case 8: return by_rows<8>(ki);
  }
  return by_rows<16>(ki);
}
