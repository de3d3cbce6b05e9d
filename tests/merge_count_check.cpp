// Walks every order in which the workgroups of two launches that overlap on one workspace can meet on one counter word
// (csrc/kvq_merge_count.h), and then, from every value they can leave there, every order of a launch that follows after
// both have ended: its last workgroup, and no other, has to find out that it is the last, and a replay of it as well.
// usage: merge_count_check [one]   -- with "one" all launches carry the same number, which must go wrong.
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "kvq_merge_count.h"

using kvq::MergeWord;

struct Group {                       // one workgroup: its launch's tag and number of records, its next operation, what it has read
  MergeWord tag; int records, at; MergeWord seen; bool last;
  bool operator<(const Group& o) const {
    if (at != o.at) return at < o.at;
    if (seen != o.seen) return seen < o.seen;
    return last < o.last;
  }
};
struct State {
  MergeWord word; std::vector<Group> groups;
  bool operator<(const State& o) const { return word != o.word ? word < o.word : groups < o.groups; }
};
enum { kMark, kAdd, kSwap, kReset, kDone };

// One memory operation of a workgroup and what it does with the answer.
static void add(State& s, Group& g) {
  const MergeWord before = s.word++;
  if (kvq::merge_unmarked(before, g.tag)) { g.seen = before + 1; g.at = kSwap; return; }
  g.seen = 0; g.last = kvq::merge_last(before, g.records); g.at = g.last ? kReset : kDone;
}
static void operate(State& s, Group& g) {
  switch (g.at) {
    case kMark: if (s.word < g.tag) s.word = g.tag; g.at = kAdd; break;
    case kAdd: add(s, g); break;
    case kSwap:
      if (!kvq::merge_unmarked(g.seen, g.tag)) {
        g.seen = 0; g.last = kvq::merge_last(s.word++, g.records); g.at = g.last ? kReset : kDone;
      } else if (s.word == g.seen) {
        s.word = g.tag | 1; g.seen = 0; g.last = kvq::merge_last(g.tag, g.records); g.at = g.last ? kReset : kDone;
      } else g.seen = s.word;
      break;
    case kReset: s.word = g.tag; g.at = kDone; break;
  }
}
static int counted(const State& s) {
  int n = 0;
  for (const Group& g : s.groups) n += g.at > kSwap;
  return n;
}
// All words the groups can leave, whatever their order.  *wrong (may be null): set if a group of one launch finds itself last
// too early, or none does.
static std::set<MergeWord> walk(const State& start, bool* wrong) {
  std::set<State> known{start};
  std::vector<State> open{start};
  std::set<MergeWord> left;
  while (!open.empty()) {
    const State s = open.back();
    open.pop_back();
    bool done = true;
    for (size_t i = 0; i < s.groups.size(); ++i) {
      if (s.groups[i].at == kDone) continue;
      done = false;
      State t = s;
      operate(t, t.groups[i]);
      if (wrong && s.groups[i].at <= kSwap && t.groups[i].at > kSwap &&
          t.groups[i].last != (counted(t) == (int)t.groups.size()))
        *wrong = true;
      if (known.insert(t).second) open.push_back(t);
    }
    if (done) left.insert(s.word);
  }
  return left;
}
static void launch(State& s, MergeWord tag, int records) {
  for (int i = 0; i < records; ++i) s.groups.push_back(Group{tag, records, kMark, 0, false});
}

int main(int argc, char** argv) {
  const bool one = argc > 1 && !strcmp(argv[1], "one");
  // the launch that follows carries a greater number than both, or (a graph's replay) a smaller one, or one in between
  const MergeWord n[3][3] = {{7, 8, 9}, {8, 7, 5}, {7, 9, 8}};
  unsigned long walks = 0, bad = 0;
  for (const MergeWord* order : n) {
    const MergeWord a = kvq::merge_tag(order[0]), b = one ? a : kvq::merge_tag(order[1]), c = one ? a : kvq::merge_tag(order[2]);
    const MergeWord before[] = {0, ~0ull, kvq::merge_tag(10) | 1, a | 1};
    for (int i = 0; i < (one ? 2 : 4); ++i)
      for (int na = 2, nb = 2; nb <= 3; ++nb) {
        State two{before[i], {}};
        launch(two, a, na);
        launch(two, b, nb);
        for (MergeWord l : walk(two, nullptr))
          for (int nc = 2; nc <= 4; ++nc) {
            bool wrong = false;
            State next{l, {}};
            launch(next, c, nc);
            for (MergeWord l2 : walk(next, &wrong)) {         // ... and the same launch again, as a graph replays it
              State again{l2, {}};
              launch(again, c, nc);
              walk(again, &wrong);
            }
            ++walks;
            bad += wrong;
          }
      }
  }
  printf("walks=%lu wrong=%lu\n", walks, bad);
  return bad != 0;
}
