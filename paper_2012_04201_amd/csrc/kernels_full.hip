// The full-batch kernel, all variants: k tiles of the input layer, unit tiles, outputs, waves.
#include "train_full_f32.h"

#include "kernels.h"

namespace {
template <int KT, int NT, int W>
const void* by_outputs(int co) {
  if constexpr (KT * NT <= 4)
    switch (co) {
      case 1: return (const void*)k_train_full<KT, NT, 1, W>;
      case 2: return (const void*)k_train_full<KT, NT, 2, W>;
      case 3: return (const void*)k_train_full<KT, NT, 3, W>;
      case 4: return (const void*)k_train_full<KT, NT, 4, W>;
    }
  return nullptr;
}
template <int KT, int W>
const void* by_tiles(int nt, int co) {
  switch (nt) {
    case 1: return by_outputs<KT, 1, W>(co);
    case 2: return by_outputs<KT, 2, W>(co);
    case 3: return by_outputs<KT, 3, W>(co);
    case 4:
      if constexpr (W == 8) return by_outputs<KT, 4, W>(co);  // (from 100 rows on: full_cut())
  }
  return nullptr;
}
}  // namespace

const void* full_kernel(int kt, int nt, int co, int waves) {
  if (waves == 4) return kt == 1 ? by_tiles<1, 4>(nt, co) : by_tiles<2, 4>(nt, co);
  return kt == 1 ? by_tiles<1, 8>(nt, co) : by_tiles<2, 8>(nt, co);
}
