// The linear kernel with the data set in LDS, all variants: columns padded to a multiple of 8, one or two outputs.
#include "train_linear_lds_f32.h"

#include "kernels.h"

namespace {
template <int CO>
const void* by_columns(int dd) {
  switch (dd) {
    case 8: return (const void*)k_train_linear_lds<8, CO>;
    case 16: return (const void*)k_train_linear_lds<16, CO>;
    case 24: return (const void*)k_train_linear_lds<24, CO>;
    case 32: return (const void*)k_train_linear_lds<32, CO>;
    case 40: return (const void*)k_train_linear_lds<40, CO>;
    case 48: return (const void*)k_train_linear_lds<48, CO>;
    case 56: return (const void*)k_train_linear_lds<56, CO>;
    case 64: return (const void*)k_train_linear_lds<64, CO>;
  }
  return nullptr;
}
}  // namespace

const void* linear_lds_kernel(int dd, int co) { return co == 1 ? by_columns<1>(dd) : by_columns<2>(dd); }
