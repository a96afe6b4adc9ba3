// How blocks of one launch come together for a burst. M gives the words of the
// step's slot that they meet in: load_joined / or_joined / add_joined on the
// counter, load_members / store_members on the result (0: not yet known), all
// agent-scope atomics on the device.
//
// The leader (block 0) opens the counter once it runs, waits a little for the
// candidates and closes it; what it had counted is the team, and it tells its
// members. A candidate joins an open counter only: while it is not open it waits a
// bounded time and then leaves, as one that comes after the close does. So nobody
// waits for a block that has not started, in whatever order blocks are dispatched:
// the leader's wait is bounded, and who has joined waits for a leader that is on its
// way to tell.
#pragma once

#include <cstdint>

namespace dobfs {

constexpr uint32_t kBurstClosed = 1u << 31, kBurstOpen = 1u << 30, kBurstCount = kBurstOpen - 1u;
constexpr uint32_t kBurstJoinPolls = 16;   // the leader's wait for the candidates (about 4 us)
constexpr uint32_t kBurstWantPolls = 256;  // its wait while they are too few for the level (about 60 us)
constexpr uint32_t kBurstOpenPolls = 256;  // a candidate's wait for the leader (about 60 us)
constexpr uint32_t kBurstSpin = 1u << 22;  // bound of the waits for blocks that run (polls)

// The leader: opens, waits and closes. want: how many the first level has a round of work for (the
// blocks that stay out have left by then, so a full-size level would be left to a few: 32 rounds for
// one member). Returns how many candidates joined, at most `most`.
template <class M>
DOBFS_DEVICE uint32_t burst_lead(M& m, uint32_t most, uint32_t want) {
  m.or_joined(kBurstOpen);
  uint32_t seen = 0;
  for (uint32_t p = 0; seen < most && p < (seen < want ? kBurstWantPolls : kBurstJoinPolls); ++p)
    seen = m.load_joined() & kBurstCount;
  const uint32_t got = m.or_joined(kBurstClosed) & kBurstCount;
  return got < most ? got : most;
}

// A candidate: its place among those that joined, or -1 when it came too late or found no leader;
// *members: what the leader told (0: it never did, which is an error).
template <class M>
DOBFS_DEVICE int32_t burst_follow(M& m, unsigned long long* members) {
  *members = 0;
  uint32_t seen = m.load_joined();
  for (uint32_t p = 0; p < kBurstOpenPolls && !(seen & kBurstOpen); ++p) seen = m.load_joined();
  if (!(seen & kBurstOpen) || (seen & kBurstClosed)) return -1;
  const uint32_t at = m.add_joined();
  if (at & kBurstClosed) return -1;
  for (uint32_t p = 0; p < kBurstSpin && *members == 0; ++p) *members = m.load_members();
  return int32_t(at & kBurstCount);
}

}  // namespace dobfs
