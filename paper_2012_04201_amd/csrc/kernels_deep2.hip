// The fp32 training kernel for two hidden layers: exactly the cuts deep_cut() makes.
#include "train_deep_f32.h"

#include "kernels.h"

const void* deep_kernel2(int kt, int waves) {
  switch (kt) {
    case 1: return waves == 4 ? (const void*)k_train_deep<1, 2, 4> : (const void*)k_train_deep<1, 2, 8>;
    case 2: return waves == 4 ? (const void*)k_train_deep<2, 2, 4> : (const void*)k_train_deep<2, 2, 8>;
    case 3: return waves == 4 ? (const void*)k_train_deep<3, 2, 4> : (const void*)k_train_deep<3, 2, 8>;
    case 4: return waves == 4 ? (const void*)k_train_deep<4, 2, 4> : (const void*)k_train_deep<4, 2, 8>;
  }
  return nullptr;
}
