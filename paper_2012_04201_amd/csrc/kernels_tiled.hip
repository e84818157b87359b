// The LDS-tiled bf16 training kernel.
#include "train_tiled_bf16.h"

#include "kernels.h"

namespace {

typedef const __attribute__((address_space(4))) TItem ConstTItem;

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
    ConstTItem* ti = (ConstTItem*)P.items + item / P.n_folds;
    Tiled<false> T{P, ti->d, ti->y, slot, smem, red, item % P.n_folds, Team{{nullptr}, {0, 1}}, nullptr};
    T.run();
  }
}

// A team of workgroups per model; team k has item k.  (A queue would hand the longest model to whoever comes to it first, also to a
// workgroup that has been left alone.)
__global__ __launch_bounds__(TB_THREADS) void k_train_tiled_team(const TrainParams P) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_met;
  __shared__ TeamPlace s_place;
  __shared__ double red[TB_THREADS / 64];
  const TeamSeat seat = team_seat(blockIdx.x, (int)(gridDim.x >> 3) / P.team_size);
  const int item = seat.team;
  if (item >= P.n_items) return;
  TeamBlock block{P.teams + item * TEAM_WORDS};
  if (threadIdx.x == 0) s_place = team_join(block, seat.member, P.team_size, __builtin_amdgcn_s_getreg(20 | (3 << 11)));  // XCC_ID
  __syncthreads();
  const Team team{block, {uniform(s_place.member), uniform(s_place.members)}};
  if (team.place.members == 0) return;
  ConstTItem* ti = (ConstTItem*)P.items + item / P.n_folds;
  Tiled<true> T{P, ti->d, ti->y, P.slots + (uint64_t)item * P.slot_bytes, smem, red, item % P.n_folds, team, &s_met};
  T.run();
}

}  // namespace

const void* tiled_kernel(bool team) { return team ? (const void*)k_train_tiled_team : (const void*)k_train_tiled; }
