// The linear kernel with the data set in LDS, all variants: columns padded to a multiple of 8, one or two outputs, all
// columns in LDS or the first of them in global memory.
#include "train_linear_lds_f32.h"

#include "kernels.h"

namespace {
template <int CO, bool FAR>
const void* by_columns(int dd) {
  switch (dd) {
    case 8: return (const void*)k_train_linear_lds<8, CO, FAR>;
    case 16: return (const void*)k_train_linear_lds<16, CO, FAR>;
    case 24: return (const void*)k_train_linear_lds<24, CO, FAR>;
    case 32: return (const void*)k_train_linear_lds<32, CO, FAR>;
    case 40: return (const void*)k_train_linear_lds<40, CO, FAR>;
    case 48: return (const void*)k_train_linear_lds<48, CO, FAR>;
    case 56: return (const void*)k_train_linear_lds<56, CO, FAR>;
    case 64: return (const void*)k_train_linear_lds<64, CO, FAR>;
  }
  return nullptr;
}
}  // namespace

const void* linear_lds_kernel(int dd, int co, bool far) {
  if (far) return co == 1 ? by_columns<1, true>(dd) : by_columns<2, true>(dd);
  return co == 1 ? by_columns<1, false>(dd) : by_columns<2, false>(dd);
}
