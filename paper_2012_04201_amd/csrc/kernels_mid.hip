// The register-resident fp32 training kernel with an output layer on MFMA: exactly the cuts mid_cut() makes.
#include "train_mid_f32.h"

#include "kernels.h"

namespace {
template <int KT>
const void* mid_by_cut(int nt, int waves, bool split) {
  if (waves == 4) return nt == 1 ? (const void*)k_train_mid<KT, 1, 4> : nullptr;
  if constexpr (md_splittable(KT, 2, 8))
    if (nt == 2 && split) return (const void*)k_train_mid2_split<KT>;
  if constexpr (KT <= 6)
    if (nt == 2) return (const void*)k_train_mid<KT, 2, 8>;
  return nt == 1 ? (const void*)k_train_mid<KT, 1, 8> : nullptr;
}
}  // namespace

const void* mid_kernel(int kt, int nt, int waves, bool split) {
  switch (kt) {
    case 1: return mid_by_cut<1>(nt, waves, split);
    case 2: return mid_by_cut<2>(nt, waves, split);
    case 3: return mid_by_cut<3>(nt, waves, split);
    case 4: return mid_by_cut<4>(nt, waves, split);
    case 5: return mid_by_cut<5>(nt, waves, split);
    case 6: return mid_by_cut<6>(nt, waves, split);
    case 7: return mid_by_cut<7>(nt, waves, split);
    case 8: return mid_by_cut<8>(nt, waves, split);
  }
  return nullptr;
}
