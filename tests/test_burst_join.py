"""CPU checks of how blocks come together for a burst (csrc/burst_join.h): the protocol compiled for
the host over std::atomic words, its blocks run one after the other in orders a dispatcher may
choose, and as threads."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_03327_amd", "csrc")

HARNESS = r"""
#define DOBFS_DEVICE inline
#include "burst_join.h"
#include <atomic>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>
using namespace dobfs;

// `tick` runs before every access: another block's turn.
struct Words {
  std::atomic<uint32_t> joined{0};
  std::atomic<unsigned long long> members{0};
  void (*tick)(Words&) = nullptr;
  int polls = 0;
  void turn() { ++polls; if (tick) tick(*this); }
  uint32_t load_joined() { turn(); return joined.load(); }
  uint32_t or_joined(uint32_t v) { turn(); return joined.fetch_or(v); }
  uint32_t add_joined() { turn(); return joined.fetch_add(1); }
  unsigned long long load_members() { turn(); return members.load(); }
  void store_members(unsigned long long v) { members.store(v); }
};

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int no_leader() {  // candidates whose leader has not started leave, soon and without having joined
  Words w;
  for (int k = 0; k < 3; ++k) {
    unsigned long long told = 1;
    w.polls = 0;
    CHECK(burst_follow(w, &told) == -1 && told == 0);
    CHECK(w.polls < 1000);
  }
  CHECK((w.joined & kBurstCount) == 0);
  w.polls = 0;
  CHECK(burst_lead(w, 31, 0) == 0);  // and it goes on without them
  CHECK(w.polls < 100);
  return 0;
}

int few() {  // a leader with a full-size level waits for candidates that come late, not for good
  Words w;
  w.tick = [](Words& x) { if (x.polls % 10 == 0 && (x.joined & kBurstOpen)) x.joined.fetch_add(1); };
  CHECK(burst_lead(w, 31, 16) >= 16);
  Words v;
  v.tick = [](Words& x) { if (x.polls % 10 == 0 && (x.joined & kBurstOpen)) x.joined.fetch_add(1); };
  CHECK(burst_lead(v, 31, 2) < 8 && v.polls < 100);
  Words none;
  CHECK(burst_lead(none, 31, 16) == 0 && none.polls < 1000);
  return 0;
}

int too_late() {
  Words w;
  CHECK(burst_lead(w, 31, 0) == 0);
  w.store_members(1);
  unsigned long long told;
  CHECK(burst_follow(w, &told) == -1 && told == 0);
  return 0;
}

int threads(int candidates, int spread) {  // whoever joins has a place of its own and is told
  for (int round = 0; round < 200; ++round) {
    Words w;
    std::vector<int32_t> at(candidates, -2);
    std::vector<unsigned long long> told(candidates, 0);
    std::vector<std::thread> t;
    std::atomic<uint32_t> n{0};
    for (int k = 0; k < candidates; ++k) t.emplace_back([&, k] {
      for (int i = 0; i < spread * ((k * 7 + round) % 5); ++i) std::this_thread::yield();
      at[k] = burst_follow(w, &told[k]);
    });
    t.emplace_back([&] {
      for (int i = 0; i < round % 3; ++i) std::this_thread::yield();
      n = burst_lead(w, uint32_t(candidates), uint32_t(round % (candidates + 1)));
      w.store_members(n + 1);
    });
    for (auto& x : t) x.join();
    std::vector<int> place(candidates, 0);
    uint32_t joined = 0;
    for (int k = 0; k < candidates; ++k) {
      if (at[k] < 0) { CHECK(told[k] == 0); continue; }
      CHECK(told[k] == n + 1 && uint32_t(at[k]) < n && place[at[k]]++ == 0);
      ++joined;
    }
    CHECK(joined == n);
  }
  return 0;
}

int main(int, char** argv) {
  if (!std::strcmp(argv[1], "no_leader")) return no_leader();
  if (!std::strcmp(argv[1], "too_late")) return too_late();
  if (!std::strcmp(argv[1], "few")) return few();
  if (!std::strcmp(argv[1], "threads")) return threads(7, 0) || threads(7, 3);
  return 2;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("burst")
    (d / "h.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(d / "h.cpp"), "-o", str(d / "h")], check=True)
    return str(d / "h")


@pytest.mark.parametrize("case", ["no_leader", "too_late", "few", "threads"])
def test_burst_join(harness, case):
    r = subprocess.run([harness, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
