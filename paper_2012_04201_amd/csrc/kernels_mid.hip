// The register-resident fp32 training kernel with an output layer on MFMA: exactly the cuts mid_cut() makes.
#include "train_mid_f32.h"

#include "kernels.h"

namespace {
template <int KT>
const void* mid_by_cut(int nt, int waves) {
  if (waves == 4) return nt == 1 ? (const void*)k_train_mid<KT, 1, 4> : nullptr;
  if constexpr (KT <= 6)
    if (nt == 2) return (const void*)k_train_mid<KT, 2, 8>;
  return nt == 1 ? (const void*)k_train_mid<KT, 1, 8> : nullptr;
}
}  // namespace

const void* mid_kernel(int kt, int nt, int waves) {
  switch (kt) {
    case 1: return mid_by_cut<1>(nt, waves);
    case 2: return mid_by_cut<2>(nt, waves);
    case 3: return mid_by_cut<3>(nt, waves);
    case 4: return mid_by_cut<4>(nt, waves);
    case 5: return mid_by_cut<5>(nt, waves);
    case 6: return mid_by_cut<6>(nt, waves);
    case 7: return mid_by_cut<7>(nt, waves);
    case 8: return mid_by_cut<8>(nt, waves);
  }
  return nullptr;
}
