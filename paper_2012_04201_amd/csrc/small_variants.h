// The register-resident fp32 training kernel for one small hidden layer: all variants of one input width.
#pragma once
#include "train_small_f32.h"

#include "kernels.h"

namespace {
template <int KT, int NT, int CO, int W>
const void* small_variant() {
  if constexpr (sm_occurs(KT, NT, CO, W)) return (const void*)k_train_small<KT, NT, CO, W>;
  return nullptr;
}
template <int KT, int NT, int W>
const void* small_by_outputs(int co) {
  return co == 1 ? small_variant<KT, NT, 1, W>() : (co == 2 ? small_variant<KT, NT, 2, W>() : small_variant<KT, NT, 4, W>());
}
template <int KT, int W>
const void* small_by_tiles(int nt, int co) {
  switch (nt) {
    case 1: return small_by_outputs<KT, 1, W>(co);
    case 2: return small_by_outputs<KT, 2, W>(co);
    case 3: return small_by_outputs<KT, 3, W>(co);
  }
  return nullptr;
}
template <int KT>
const void* small_by_cut(int nt, int waves, int co) {
  return waves == 2 ? small_by_tiles<KT, 2>(nt, co) : (waves == 4 ? small_by_tiles<KT, 4>(nt, co) : small_by_tiles<KT, 8>(nt, co));
}
}  // namespace
