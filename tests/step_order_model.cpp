// Streams and events as sets of what has happened before, and random programs of contexts on a few streams.  Every two persistent steps of a
// device must be ordered, one that leaves no room also against every small step; of the small steps no five may be unordered among each other.
// A context that shares the stream of all others must cost no event, small contexts on four streams neither, and a stream that a caller
// captures, or that has no context any more, must see none.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "../paper_2410_12513_amd/csrc/step_order.h"

namespace {
struct Event_ { std::set<int> before; bool recorded = false; };
struct Model {
  using Stream = int; using Event = Event_*; using Error = int;
  static std::vector<std::set<int>> before;      // [stream] steps that are done before what is enqueued there next
  static std::vector<bool> captured;
  static std::vector<int> contexts;              // [stream] live ones: a stream may go with its last
  static int calls, bad;
  static Error make(Event* e) { *e = new Event_(); return 0; }
  static Error record(Event e, Stream s) { ++calls; bad += captured[s] || contexts[s] == 0; e->before = before[s]; e->recorded = true; return 0; }
  static Error wait(Stream s, Event e) {
    ++calls; bad += captured[s] || !e->recorded;
    before[s].insert(e->before.begin(), e->before.end());
    return 0;
  }
  static bool capturing(Stream s) { return captured[s]; }
};
std::vector<std::set<int>> Model::before;
std::vector<bool> Model::captured;
std::vector<int> Model::contexts;
int Model::calls, Model::bad;

using first::StepKind;
struct Unordered {                               // steps just go out
  using Set = int;
  int join(StepKind, int, int, Set*) { return 0; }
  void leave(Set, int) {}
  template <typename F> int run(Set, int, F f) { return f(); }
};

struct Step { StepKind kind; int stream; };
// Five small steps of which no two are ordered?  (after[t] holds all steps before t, so one look a pair is enough.)
bool five_unordered(const std::vector<std::set<int>>& after, const std::vector<int>& small, std::vector<int>& pick, size_t from) {
  if (pick.size() == 5) return true;
  for (size_t i = from; i < small.size(); ++i) {
    bool free = true;
    for (int p : pick) free = free && !after[small[i]].count(p);
    if (!free) continue;
    pick.push_back(small[i]);
    if (five_unordered(after, small, pick, i + 1)) return true;
    pick.pop_back();
  }
  return false;
}

// mode 0: all kinds on six streams; 1: all kinds on one; 2: small ones on four.  Number of violations, -1: an error.
template <typename Orders>
int violations(unsigned seed, int mode) {
  constexpr int STREAMS = 6;
  std::mt19937 rng(seed);
  Model::before.assign(STREAMS, {}); Model::captured.assign(STREAMS, false); Model::contexts.assign(STREAMS, 0); Model::calls = Model::bad = 0;
  Orders orders;
  struct Context { StepKind kind; int stream; typename Orders::Set in; };
  std::vector<Context> contexts;
  std::vector<Step> steps;
  std::vector<std::set<int>> after;              // [step] the steps before it
  int found = 0;
  for (int op = 0; op < 120; ++op) {
    const int what = rng() % 10;
    bool any_captured = false;
    for (int s = 0; s < STREAMS; ++s) any_captured |= Model::captured[s];
    if (contexts.empty() || (what <= 1 && contexts.size() < 9 && !any_captured)) {
      const int s = mode == 1 ? 1 : rng() % (mode == 2 ? 4 : STREAMS), k = rng() % 8;
      Context c{mode == 2 || k < 5 ? StepKind::SMALL : k < 7 ? StepKind::PERSISTENT : StepKind::PERSISTENT_NO_ROOM, s, {}};
      if (orders.join(c.kind, s, 4, &c.in)) return -1;
      contexts.push_back(c);
      ++Model::contexts[s];
    } else if (what == 2 && contexts.size() > 1) {
      const size_t i = rng() % contexts.size();
      const int s = contexts[i].stream;
      if (Model::captured[s]) continue;
      for (auto& b : Model::before) b.insert(Model::before[s].begin(), Model::before[s].end());    // destroying waits for the stream
      orders.leave(contexts[i].in, s);
      contexts.erase(contexts.begin() + i);
      --Model::contexts[s];
    } else if (what == 3 && rng() % 4 == 0) {
      const int s = contexts[rng() % contexts.size()].stream;
      Model::captured[s] = !Model::captured[s];
    } else {
      const Context& c = contexts[rng() % contexts.size()];
      const int s = c.stream;
      auto launch = [&] {
        if (Model::captured[s]) return 0;        // into the caller's graph
        const int me = (int)steps.size();
        for (int t = 0; t < me; ++t)
          if (!Model::before[s].count(t)) {
            const bool both = c.kind != StepKind::SMALL && steps[t].kind != StepKind::SMALL;
            const bool no_room = c.kind == StepKind::PERSISTENT_NO_ROOM || steps[t].kind == StepKind::PERSISTENT_NO_ROOM;
            found += both || no_room;
          }
        after.push_back(Model::before[s]);
        Model::before[s].insert(me);
        steps.push_back(Step{c.kind, s});
        return 0;
      };
      if (orders.run(c.in, s, launch)) return -1;
    }
  }
  std::vector<int> small, pick;
  for (int t = 0; t < (int)steps.size(); ++t)
    if (steps[t].kind == StepKind::SMALL) small.push_back(t);
  return found + five_unordered(after, small, pick, 0);
}
}  // namespace

int main() {
  using Orders = first::StepOrders<Model>;
  long unordered = 0;
  for (unsigned seed = 0; seed < 800; ++seed) {
    if (violations<Orders>(seed, 0) != 0 || Model::bad) { std::printf("seed %u: steps not ordered, or an event on a captured or dead stream\n", seed); return 1; }
    for (int mode = 1; mode < 3; ++mode)
      if (violations<Orders>(seed, mode) != 0 || Model::calls) { std::printf("seed %u: events without need (%d)\n", seed, mode); return 1; }
    if (seed < 200) unordered += violations<Unordered>(seed, 0);
  }
  if (unordered == 0) { std::printf("the model finds nothing\n"); return 1; }
  std::printf("ok\n");
  return 0;
}
