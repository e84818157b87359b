// The wider LDS-resident fp32 training kernel, all variants.
#include "train_mid_f32.h"

#include "kernels.h"

const void* mid_kernel(int kt) {
  switch (kt) {
    case 2: return (const void*)k_train_mid<2>;
    case 4: return (const void*)k_train_mid<4>;
    case 5: return (const void*)k_train_mid<5>;
    case 6: return (const void*)k_train_mid<6>;
    case 8: return (const void*)k_train_mid<8>;
  }
  return nullptr;
}
