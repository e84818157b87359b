// The register-resident fp32 training kernel for one small hidden layer: all variants of one input width.
#pragma once
#include "train_small_f32.h"

#include "kernels.h"

namespace {
template <int KT, int NT, int W>
const void* small_by_outputs(int co) {
  if constexpr (NT <= 2)
    if (co == 4) return (const void*)k_train_small<KT, NT, 4, W>;
  return co == 1 ? (const void*)k_train_small<KT, NT, 1, W> : (co == 2 ? (const void*)k_train_small<KT, NT, 2, W> : nullptr);
}
// exactly the cuts small_cut() makes
template <int KT>
const void* small_by_cut(int nt, int waves, int co) {
  if constexpr (KT == 1)
    if (waves == 2) return nt == 1 ? small_by_outputs<KT, 1, 2>(co) : nullptr;
  if (waves == 8) return nt == 1 ? small_by_outputs<KT, 1, 8>(co) : (nt == 2 ? small_by_outputs<KT, 2, 8>(co) : nullptr);
  if constexpr (KT <= 2)
    if (nt == 3) return small_by_outputs<KT, 3, 4>(co);
  return nt == 1 ? small_by_outputs<KT, 1, 4>(co) : (nt == 2 ? small_by_outputs<KT, 2, 4>(co) : nullptr);
}
}  // namespace
