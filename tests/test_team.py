"""CPU tests of how workgroups form a team and meet (csrc/team.h), on threads of the host in place of workgroups."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_04201_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not on PATH")

PRELUDE = r"""
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include "%s"

struct Block {
  std::atomic<uint64_t> word{0};
  std::atomic<uint32_t> met[TEAM_MOST] = {}, gone{0};
};
struct Ctl {
  Block& b;
  int us;  // a poll's pause
  uint64_t list() { return b.word.load(); }
  uint64_t change(uint64_t from, uint64_t to) { b.word.compare_exchange_strong(from, to); return from; }
  void pause() { if (us) std::this_thread::sleep_for(std::chrono::microseconds(us)); else std::this_thread::yield(); }
  void arrive(int m, uint32_t n) { b.met[m].store(n); }
  int state(int members, uint32_t n) {
    int there = 0;
    for (int k = 0; k < members; k++) there += b.met[k].load() >= n;
    return there == members ? 1 : b.gone.load() ? 2 : 0;
  }
  void give_up() { b.gone.store(1); }
};
#define CHECK(x) do { if (!(x)) { printf("line %%d: %%s\n", __LINE__, #x); exit(1); } } while (0)
static void nap(int ms) { std::this_thread::sleep_for(std::chrono::milliseconds(ms)); }

// Members `who`, member m on XCD xcd[m] after delay[m] ms; the places they end up with.
static std::vector<TeamPlace> join(const std::vector<int>& who, int size, const std::vector<int>& xcd, const std::vector<int>& delay, int us) {
  Block b;
  std::vector<TeamPlace> got(size, TeamPlace{0, 0});
  std::vector<std::thread> t;
  for (int m : who) t.emplace_back([&, m] { if (delay[m]) nap(delay[m]); Ctl c{b, us}; got[m] = team_join(c, m, size, xcd[m]); });
  for (auto& x : t) x.join();
  return got;
}
// One team: the leader's, of consecutive numbers in the order of the members; the others have no place.
static int agreed(const std::vector<TeamPlace>& got) {
  int in = 0;
  for (size_t m = 0; m < got.size(); m++)
    if (got[m].members) {
      CHECK(got[m].member == in && (in > 0 || m == 0));
      in++;
    }
  for (const TeamPlace& p : got) CHECK(p.members == 0 || p.members == in);
  return in;
}
static std::vector<int> all(int n) { std::vector<int> v; for (int i = 0; i < n; i++) v.push_back(i); return v; }
"""


def run(tmp_path, body):
    src, exe = tmp_path / "team.cpp", str(tmp_path / "team")
    src.write_text(PRELUDE % os.path.join(CSRC, "team.h") + "int main() {\n" + body + "\n}\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-Wall", str(src), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout


def test_all_leaders_are_launched_first_and_a_team_on_one_xcd(tmp_path):
    run(tmp_path, r"""
      for (int rows = 1; rows <= 16; rows++)
        for (int size = 1; size <= 8; size++) {
          std::vector<int> seen(rows * 8 * size, 0);
          for (int b = 0; b < rows * 8 * size; b++) {
            const TeamSeat s = team_seat(b, rows);
            CHECK(s.team >= 0 && s.team < rows * 8 && s.member >= 0 && s.member < size && s.team % 8 == b % 8);
            CHECK((s.member == 0) == (b < rows * 8));
            seen[s.team * size + s.member]++;
          }
          for (int k : seen) CHECK(k == 1);
        }
    """)


@pytest.mark.parametrize("size", [1, 2, 3, 8])
def test_everybody_on_time(tmp_path, size):
    run(tmp_path, "for (int i = 0; i < 20; i++) CHECK(agreed(join(all(%d), %d, std::vector<int>(8, i %% 8), std::vector<int>(8, 0), 1000)) == %d);"
        % (size, size, size))


@pytest.mark.parametrize("who,xcd,delay,members", [
    ("{0, 2, 3}", "{5, 5, 5, 5}", "{0, 0, 0, 0}", 3),             # one that never gets a CU
    ("{0, 1, 2, 3}", "{5, 5, 5, 5}", "{0, 0, 300, 0}", 3),        # one that comes when the list is closed
    ("{0, 1, 2, 3}", "{5, 1, 5, 6}", "{0, 0, 0, 0}", 2),          # others' XCDs
    ("{0, 1, 2, 3}", "{5, 1, 1, 1}", "{0, 0, 0, 0}", 1),          # a leader left alone
    ("{0, 1, 2, 3}", "{5, 5, 5, 5}", "{300, 0, 0, 0}", 1),        # a leader who comes when all others have gone
    ("{1, 2, 3}", "{5, 5, 5, 5}", "{0, 0, 0, 0}", 0),             # ... or never
])
def test_whoever_is_not_there_is_not_in(tmp_path, who, xcd, delay, members):
    """(200 polls of 0.2 ms are the leader's patience, 400 a member's.)"""
    run(tmp_path, "CHECK(agreed(join(%s, 4, %s, %s, 200)) == %d);" % (who, xcd, delay, members))


def test_leaving_while_the_list_is_closed(tmp_path):
    """Members without patience against a leader who closes at any moment of it: whatever comes out, they agree."""
    run(tmp_path, r"""
      int seen[9] = {};
      for (int i = 0; i < 3000; i++) {
        std::vector<int> delay(8, 0);
        seen[agreed(join(all(8), 8, std::vector<int>(8, 3), delay, 0))]++;
      }
      for (int i = 0; i < 60; i++) {
        std::vector<int> delay(8, 0);
        delay[0] = 30 + i % 20;  // about when the others go
        seen[agreed(join(all(8), 8, std::vector<int>(8, 3), delay, 50))]++;
      }
      for (int i = 0; i < 9; i++) printf("%d ", seen[i]);
    """)


def test_meetings_wait_for_everybody(tmp_path):
    run(tmp_path, r"""
      Block b;
      std::atomic<int> work{0};
      std::vector<std::thread> t;
      for (int m = 0; m < 4; m++) t.emplace_back([&, m] {
        Ctl c{b, 0};
        for (uint32_t n = 1; n <= 2000; n++) {
          work++;
          CHECK(team_meet(c, m, 4, n) && work.load() >= 4 * (int)n);
        }
      });
      for (auto& x : t) x.join();
      CHECK(b.gone.load() == 0);
    """)


@pytest.mark.parametrize("left", [0, 3])
def test_a_lost_member_costs_one_wait_and_everybody_knows(tmp_path, left):
    """A member stops coming after its tenth meeting: no other gets past the eleventh, and nobody waits a second time."""
    run(tmp_path, r"""
      Block b;
      std::atomic<int> waits{0};
      std::vector<std::thread> t;
      for (int m = 0; m < 4; m++) t.emplace_back([&, m] {
        struct Counting : Ctl { std::atomic<int>& w; Counting(Block& b, std::atomic<int>& w) : Ctl{b, 0}, w(w) {}
                                void give_up() { w++; Ctl::give_up(); } } c(b, waits);
        for (uint32_t n = 1; n <= 10; n++) CHECK(team_meet(c, m, 4, n));
        if (m == %d) return;
        CHECK(!team_meet(c, m, 4, 11));
        CHECK(!team_meet(c, m, 4, 12) && !team_meet(c, m, 4, 13));
      });
      for (auto& x : t) x.join();
      CHECK(b.gone.load() == 1 && waits.load() >= 1 && waits.load() <= 3);
    """ % left)
