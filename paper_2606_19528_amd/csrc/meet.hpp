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
#pragma once

#include <cstdint>

namespace lora {

using meet_word = uint32_t;

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
