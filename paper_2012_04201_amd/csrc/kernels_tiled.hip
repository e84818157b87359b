// The LDS-tiled bf16 training kernel.
#include "train_tiled_bf16.h"

#include "kernels.h"

namespace {

__global__ __launch_bounds__(TB_THREADS) void k_train_tiled(const TrainParams P) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_item;
  __shared__ double red[TB_THREADS / 64];
  char* slot = P.slots + (uint64_t)blockIdx.x * P.slot_bytes;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    if (item >= P.n_items) break;
    const __attribute__((address_space(4))) TItem* ti = (const __attribute__((address_space(4))) TItem*)P.items + item / P.n_folds;
    Tiled T{P, ti->d, ti->y, slot, smem, red, item % P.n_folds};
    T.run();
  }
}

}  // namespace

const void* tiled_kernel() { return (const void*)k_train_tiled; }
