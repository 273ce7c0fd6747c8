// Host model of the few-token kernel's meetings: the steps of meet.hpp over a
// memory whose every access is one step, taken in every order that the
// workgroups of a launch allow.
//
//   meet_model <tiles> <parts> <launches> <variant> <tag>
//
// `tiles` row tiles of `parts` workgroups each: the parts of a tile meet, the one
// that finishes the tile stores the tile's share and meets the other tiles'.
// All launches carry one tag, as the replays of a graph do.  Prints the number
// of states; exits 1 when some order ends a launch with a tile not finished
// exactly once, the last meeting not finished, a share read that this launch had
// not yet written, or a flag still up.
// variant: "claim", the protocol; "all", in which every workgroup that sees all
// flags goes on and a tile may be finished twice, with the same values (a
// mistake that the model has to find: the second to finish raises the tile's
// flag again).
// tag: "taken", one of MeetTags; "counted", a small number (a mistake again).
// The flags start as the whole numbers 1, 2, 3, ..., and so do they once more as
// pairs of 32 bits.
//
//   meet_model tags <count>
//
// prints the first and exits 1 if one of `count` tags is a word that ordinary
// data holds: a half or the whole below 2^30 as an integer, or a finite fp64.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <unordered_map>
#include <unordered_set>
#include <vector>

#include "meet.hpp"

using lora::meet_word;

namespace {

using Word = uint64_t;
struct Op {
  enum Kind { READ, WRITE, SWAP, COUNT } kind;
  int at;
  Word value;
};
// Memory as one workgroup sees it: results of the accesses it has made are
// fed back from its history, the next access is thrown to the scheduler.
struct Memory {
  const std::vector<Word> &history;
  size_t made = 0;
  Word access(Op op) {
    if (made < history.size()) return history[made++];
    throw op;
  }
  Word read(int at) { return access({Op::READ, at, 0}); }
  void write(int at, Word v) { access({Op::WRITE, at, v}); }
  Word swap(int at, Word v) { return access({Op::SWAP, at, v}); }
  void count(int at) { access({Op::COUNT, at, 1}); }
};

struct Flags {
  Memory &m;
  int base;
  bool down;  // the order in which the words of one look are read
  void raise(int i, meet_word tag) { m.write(base + i, tag); }
  void settle() {}
  bool all_up(int n, meet_word tag) {
    bool all = true;
    for (int i = 0; i < n; ++i) all &= m.read(base + (down ? n - 1 - i : i)) == tag;
    return all;
  }
  meet_word lower(int n) {
    const meet_word old = (meet_word)m.swap(base, 0);
    for (int i = 1; i < n; ++i) m.write(base + i, 0);
    return old;
  }
};

int tiles, parts;
bool claim;
meet_word TAG;

// memory: flags of the tiles, flags of the last meeting, shares, counts
int at_flags(int tile) { return tile * parts; }
int at_last() { return tiles * parts; }
int at_part(int tile, int p) { return tiles * parts + tiles + tile * parts + p; }
int at_tile(int tile) { return tiles * parts * 2 + tiles + tile; }
int at_finished(int tile) { return tiles * parts * 2 + tiles * 2 + tile; }
int at_end() { return tiles * parts * 2 + tiles * 3; }
int at_stale() { return at_end() + 1; }
int words() { return at_end() + 2; }

void workgroup(Memory &m, int tile, int p, Word launch) {
  const bool down = (tile + p) & 1;
  auto share = [&](int at) {
    if (m.read(at) != launch) m.count(at_stale());
  };
  m.write(at_part(tile, p), launch);
  if (parts > 1) {
    Flags f{m, at_flags(tile), down};
    if (!lora::meet_arrive(f, p, parts, TAG)) return;
    const meet_word word0 = lora::meet_lower(f, parts);
    for (int q = 0; q < parts; ++q) share(at_part(tile, q));
    if (claim && word0 != TAG) return;
  }
  m.count(at_finished(tile));
  m.write(at_tile(tile), launch);
  if (tiles > 1) {
    Flags f{m, at_last(), down};
    if (!lora::meet_arrive(f, tile, tiles, TAG)) return;
    lora::meet_lower(f, tiles);
    for (int t = 0; t < tiles; ++t) share(at_tile(t));
  }
  m.count(at_end());
}

struct State {
  std::vector<Word> mem;
  std::vector<std::vector<Word>> history;
  std::vector<bool> done;
  std::string key() const {
    std::string k((const char *)mem.data(), mem.size() * sizeof(Word));
    for (size_t g = 0; g < history.size(); ++g) {
      k.push_back(done[g] ? 'd' : 'r');
      if (done[g]) continue;  // (what a workgroup that has left saw no longer matters)
      k.append((const char *)history[g].data(), history[g].size() * sizeof(Word));
      k.push_back('|');
    }
    return k;
  }
};

int fail(const char *what, Word launch) {
  std::printf("launch %d: %s\n", (int)launch, what);
  return 1;
}

}  // namespace

int main(int argc, char **argv) {
  lora::MeetTags tags;
  if (argc == 3 && !std::strcmp(argv[1], "tags")) {
    meet_word last = 0;
    for (int i = 0, n = std::atoi(argv[2]); i < n; ++i) {
      const meet_word t = tags.take();
      if (i == 0) std::printf("%llu\n", (unsigned long long)t);
      double d;
      std::memcpy(&d, &t, sizeof d);
      if (t >> 32 < 1u << 30 || !std::isnan(d) || t == last) return 1;
      last = t;
    }
    return 0;
  }
  if (argc != 6) return 2;
  TAG = std::strcmp(argv[5], "counted") ? tags.take() : 2;
  tiles = std::atoi(argv[1]);
  parts = std::atoi(argv[2]);
  const int launches = std::atoi(argv[3]);
  claim = std::strcmp(argv[4], "all") != 0;
  const int groups = tiles * parts;
  size_t states = 0;
  std::vector<std::vector<Word>> starts(2, std::vector<Word>(words(), 0));
  for (int w = 0; w < at_part(0, 0); ++w) {
    starts[0][w] = w + 1;
    starts[1][w] = (Word)(2 * w + 2) << 32 | (2 * w + 1);
  }
  for (Word launch = 1; launch <= (Word)launches; ++launch) {
    std::unordered_set<std::string> seen;
    std::unordered_map<std::string, std::vector<Word>> ends;
    std::vector<State> stack;
    for (auto &m : starts) stack.push_back({m, std::vector<std::vector<Word>>(groups), std::vector<bool>(groups)});
    while (!stack.empty()) {
      State s = std::move(stack.back());
      stack.pop_back();
      std::vector<State> next;
      bool any = false;
      for (int g = 0; g < groups; ++g) {
        if (s.done[g]) continue;
        any = true;
        Memory m{s.history[g]};
        State n = s;
        try {
          workgroup(m, g / parts, g % parts, launch);
          n.done[g] = true;
          n.history[g].clear();
          next.assign(1, std::move(n));  // leaving concerns nobody else
          break;
        } catch (const Op &op) {
          Word &w = n.mem[op.at];
          n.history[g].push_back(op.kind == Op::READ || op.kind == Op::SWAP ? w : 0);
          if (op.kind == Op::WRITE || op.kind == Op::SWAP) w = op.value;
          if (op.kind == Op::COUNT) w += op.value;
        }
        next.push_back(std::move(n));
      }
      if (!any) {
        if (s.mem[at_stale()]) return fail("a share was read before this launch wrote it", launch);
        for (int t = 0; t < tiles; ++t)
          if (claim ? s.mem[at_finished(t)] != 1 : s.mem[at_finished(t)] < 1)
            return fail("a tile was not finished exactly once", launch);
        if (!s.mem[at_end()]) return fail("nobody finished the last meeting", launch);
        for (int w = 0; w < at_part(0, 0); ++w)
          if (s.mem[w] == TAG) return fail("a flag is still up", launch);
        for (int w = at_finished(0); w < words(); ++w) s.mem[w] = 0;
        ends.emplace(std::string((const char *)s.mem.data(), s.mem.size() * sizeof(Word)), s.mem);
        continue;
      }
      for (State &n : next)
        if (seen.insert(n.key()).second) stack.push_back(std::move(n));
    }
    states += seen.size();
    starts.clear();
    for (auto &e : ends) starts.push_back(e.second);
  }
  std::printf("states %zu\n", states);
  return 0;
}
