// How several workgroups come to train one model together, and how they wait for each other.  Plain C++ over a control
// block `Ctl`, so that the same code runs on the GPU (TeamBlock in train_tiled_bf16.h) and on threads of the host.
//
// A team forms when its kernel starts: whoever is running puts itself on a list, the leader waits for the others for a
// bounded time (they may have no CU yet) and closes it.  A closed list is never changed again, so the word itself says who is
// in, and nobody waits for an answer.  A member that has waited twice as long for the leader takes itself off.  Whoever is not
// in has nothing to do: the leader trains the model with those who are, alone if need be.
//
// Every later wait is for a workgroup that runs, and bounded all the same.  Whoever gives one up says so in a word that is
// never cleared, and all others of the team find it at the next meeting at the latest.
#pragma once
#include <stdint.h>

#ifdef __HIP__
#define TEAM_FN __device__ inline
#else
#define TEAM_FN inline
#endif

constexpr int TEAM_MOST = 8;
constexpr int TEAM_JOIN_POLLS = 200;      // about 100 us
constexpr int TEAM_MEET_POLLS = 1 << 23;  // seconds: the members all run, so only a fault elsewhere lets a wait end here
constexpr uint64_t TEAM_CLOSED = 1ull << 63;

// Which team and which of its members a workgroup is, in a launch of rows * 8 teams: workgroups b, b + 8, .. lie on one XCD as a
// rule, so a team's do.  All leaders come first: where CUs become free one by one, because other calls hold them, each is a model's
// before any is a second one's, and who comes late finds the list closed.
struct TeamSeat {
  int team, member;
};
TEAM_FN TeamSeat team_seat(uint32_t block, int rows) {
  const int at = (int)(block >> 3), m = at / rows;
  return TeamSeat{(at - m * rows) * 8 + (int)(block & 7), m};
}

struct TeamPlace {
  int member, members;  // members == 0: not in the team
};

// Of the list: member k's four bits are 8 | the number of its XCD, or 0.
TEAM_FN TeamPlace team_place(uint64_t list, int m) {
  TeamPlace p = {0, 0};
  const uint64_t leader = list & 15;  // only its XCD's can be in: new weights pass through that one's L2
  if (((list >> (4 * m)) & 15) != leader) return p;
  for (int k = 0; k < TEAM_MOST; k++)
    if (((list >> (4 * k)) & 15) == leader) {
      p.members++;
      if (k < m) p.member++;
    }
  return p;
}

// Called by one thread of a workgroup: its place among the `size` workgroups of the block; m == 0 is the leader.
//   uint64_t list()                          the list
//   uint64_t change(uint64_t from, to)       compare and swap; what was there
//   void pause()
template <class Ctl>
TEAM_FN TeamPlace team_join(Ctl& c, int m, int size, uint32_t xcd) {
  const uint64_t me = (uint64_t)(8 | (xcd & 7)) << (4 * m);
  uint64_t all = 0;
  for (int k = 0; k < size; k++) all |= 8ull << (4 * k);
  uint64_t seen = c.list();
  auto put = [&](uint64_t clear, uint64_t set) {  // false: closed before
    while (!(seen & TEAM_CLOSED)) {
      const uint64_t was = c.change(seen, (seen & ~clear) | set);
      if (was == seen) return true;
      seen = was;
    }
    return false;
  };
  if (!put(0, me)) return TeamPlace{0, 0};
  seen = c.list();
  const int polls = m == 0 ? TEAM_JOIN_POLLS : 2 * TEAM_JOIN_POLLS;
  for (int i = 0; i < polls && !(seen & TEAM_CLOSED) && !(m == 0 && (seen & all) == all); i++) {
    c.pause();
    seen = c.list();
  }
  if (m == 0) {
    put(0, TEAM_CLOSED);
    return team_place(seen, 0);  // (as it was when it was closed)
  }
  if (put(me, 0)) return TeamPlace{0, 0};
  return team_place(seen, m);
}

// The n-th meeting: true once all members have come to it.  false: somebody has given up waiting, here or before.
//   void arrive(int member, uint32_t n)
//   int state(int members, uint32_t n)       1 all have arrived, 2 not and somebody has given up, 0 neither
//   void give_up()
template <class Ctl>
TEAM_FN bool team_meet(Ctl& c, int member, int members, uint32_t n) {
  c.arrive(member, n);
  for (int i = 0; i < TEAM_MEET_POLLS; i++) {
    const int s = c.state(members, n);
    if (s) return s == 1;
  }
  c.give_up();
  return false;
}
