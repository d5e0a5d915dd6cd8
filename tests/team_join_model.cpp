// Every interleaving of the accesses that the workgroups of a launch make while they agree
// on a team: prints "ok <states>" or the first end state that breaks the agreement.
#include <array>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "team_join.h"

namespace {

struct Word {
  uint32_t x = 0;
  uint32_t add(uint32_t d) { const uint32_t o = x; x += d; return o; }
  uint32_t load() { return x; }
  uint32_t cas(uint32_t e, uint32_t v) { const uint32_t o = x; if (x == e) x = v; return o; }
};

struct State {
  Word w;
  std::vector<gr::TeamJoin> g;
  std::vector<long> key() const {
    std::vector<long> k{(long)w.x};
    for (const auto& j : g)
      for (long v : {(long)j.next, (long)j.index, (long)j.size, (long)j.called_off, (long)j.now, (long)j.polls})
        k.push_back(v);
    return k;
  }
};

int members, expected;
std::set<std::vector<long>> seen;

void bad(const State& s, const char* what) {
  std::printf("%s: word %08x", what, s.w.x);
  for (const auto& j : s.g) std::printf(" [member %d index %d size %d off %d]", j.member, j.index, j.size, j.called_off);
  std::printf("\n");
  std::exit(1);
}

void check_end(const State& s) {
  int in = 0, offs = 0;
  std::set<int> places;
  for (const auto& j : s.g) {
    offs += j.called_off;
    if (j.index < 0) continue;
    ++in;
    places.insert(j.index);
    if (!j.member) bad(s, "a workgroup of another XCD joined");
    if (j.size != members) bad(s, "a member with another team size");
    if (j.index >= members) bad(s, "a place outside the team");
  }
  if ((int)places.size() != in) bad(s, "two members with one place");
  if (in != 0 && in != members) bad(s, "only some members run");
  if (in != 0 && expected != (int)s.g.size()) bad(s, "a team of an incomplete count");
  if (members > 0 && (in == 0) != (offs == 1)) bad(s, "left without one member calling off");
}

void walk(const State& s, int depth) {
  if (depth > 10000) bad(s, "no end");
  if (!seen.insert(s.key()).second) return;
  bool any = false;
  for (size_t i = 0; i < s.g.size(); ++i) {
    if (s.g[i].next == gr::TeamJoin::kDone) continue;
    any = true;
    State t = s;
    t.g[i].step(t.w);
    walk(t, depth + 1);
  }
  if (!any) check_end(s);
}

}  // namespace

int main(int argc, char** argv) {
  const int grid = std::atoi(argv[1]), polls = std::atoi(argv[3]);
  members = std::atoi(argv[2]);
  expected = grid + std::atoi(argv[4]);
  State s;
  for (int i = 0; i < grid; ++i) s.g.emplace_back((uint32_t)expected, i < members, polls);
  walk(s, 0);
  std::printf("ok %zu\n", seen.size());
}
