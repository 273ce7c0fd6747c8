// meet.hpp -- how workgroups of one launch meet over flags in the workspace
// without waiting for each other: each does its share, and the one that comes
// last finishes the work of all.  The steps stand here over a policy F of the
// flags' memory, so that a host program can step the same code through every
// order of its accesses.
//
// A meeting of n workgroups has n words; a raised flag is the launch's tag.
//   F::raise(i, tag)    word i = tag
//   F::settle()         returns once that store has completed
//   F::all_up(n, tag)   reads all n words; true when each is the tag
//   F::lower(n)         word 0 is exchanged with 0, the others set to 0;
//                       returns what word 0 held
//
// Nothing sets the words ahead of the launch: they hold whatever the workspace
// held.  So a tag is a word that no data is: its upper half is a NaN as fp32, as
// a pair of bf16 and, with the lower, as fp64, and no index or count; and its
// payload of 52 bits starts from a number of the system's random source, so that
// data made to look like a tag is not one.
#pragma once

#include <sys/random.h>

#include <atomic>
#include <chrono>
#include <cstdint>

namespace lora {

using meet_word = uint64_t;

// A number of the system's random source.
inline uint64_t random_word() {
  uint64_t v = 0;
  if (getentropy(&v, sizeof v) == 0) return v;
  // (no random source: the time in ns, spread over the word by an odd factor)
  return (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull;
}

// Tags of a process's launches, never 0 and never the same twice (2^52 of them).
class MeetTags {
 public:
  MeetTags() : next_(random_word()) {}
  meet_word take() {
    uint64_t payload;
    do {
      payload = next_.fetch_add(1, std::memory_order_relaxed) & (BITS - 1);
    } while (payload == 0);  // (that word is an infinity, not a NaN)
    return 0x7FF0000000000000ull | payload;
  }

 private:
  static constexpr uint64_t BITS = uint64_t(1) << 52;
  std::atomic<uint64_t> next_;
};

// Workgroup `mine` arrives, its share complete in memory.  True when it sees
// every flag up: every workgroup's share was complete before its own flag
// rose, and of two that rise last, the later one's look follows both, so at
// least one sees all.  More than one may, each with all the shares before it.
template <class F>
constexpr bool meet_arrive(F &f, int mine, int n, meet_word tag) {
  f.raise(mine, tag);
  f.settle();
  return f.all_up(n, tag);
}

// One that saw all flags up lowers them (0 is no launch's tag), for a replay
// of the launch with the same tag, and learns whether it is the one that
// finishes: the exchange on word 0 hands the tag to one workgroup only.  The
// others must leave without a trace, above all without raising a flag of the
// next meeting: raised a second time, after that meeting has lowered its
// flags, it would stay up into the replay and stand there for a share that is
// not yet written.
template <class F>
constexpr meet_word meet_lower(F &f, int n) {
  return f.lower(n);
}

}  // namespace lora
