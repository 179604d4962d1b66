// Streams and events as sets of what has happened before, and random programs of contexts on a few streams: every two steps of a
// device must be ordered, a context that shares the stream of all others must cost no event, and a stream that a caller captures must see none.
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
  static int calls, bad;
  static Error make(Event* e) { *e = new Event_(); return 0; }
  static Error record(Event e, Stream s) { ++calls; bad += captured[s]; e->before = before[s]; e->recorded = true; return 0; }
  static Error wait(Stream s, Event e) {
    ++calls; bad += captured[s] || !e->recorded;
    before[s].insert(e->before.begin(), e->before.end());
    return 0;
  }
  static bool capturing(Stream s) { return captured[s]; }
};
std::vector<std::set<int>> Model::before;
std::vector<bool> Model::captured;
int Model::calls, Model::bad;

struct Unordered {                               // steps just go out
  int join(int) { return 0; }
  void leave(int) {}
  template <typename F> int run(int, F f) { return f(); }
};

template <typename Order>
int unordered_pairs(unsigned seed, bool one_stream) {
  constexpr int STREAMS = 4;
  std::mt19937 rng(seed);
  Model::before.assign(STREAMS, {}); Model::captured.assign(STREAMS, false); Model::calls = Model::bad = 0;
  Order order;
  std::vector<int> contexts;                     // the stream of each
  std::vector<int> steps;                        // all so far
  int pairs = 0;
  for (int op = 0; op < 120; ++op) {
    const int what = rng() % 10;
    bool any_captured = false;
    for (int s = 0; s < STREAMS; ++s) any_captured |= Model::captured[s];
    if (contexts.empty() || (what == 0 && contexts.size() < 6 && !any_captured)) {
      const int s = one_stream ? 1 : rng() % STREAMS;
      if (order.join(s)) return -1;
      contexts.push_back(s);
    } else if (what == 1 && contexts.size() > 1) {
      const size_t i = rng() % contexts.size();
      const int s = contexts[i];
      if (Model::captured[s]) continue;
      for (auto& b : Model::before) b.insert(Model::before[s].begin(), Model::before[s].end());    // destroying waits for the stream
      order.leave(s);
      contexts.erase(contexts.begin() + i);
    } else if (what == 2) {
      const int s = contexts[rng() % contexts.size()];
      Model::captured[s] = !Model::captured[s];
    } else {
      const int s = contexts[rng() % contexts.size()];
      const int e = order.run(s, [&] {
        if (Model::captured[s]) return 0;        // into the caller's graph
        for (int t : steps) pairs += !Model::before[s].count(t);
        Model::before[s].insert((int)steps.size());
        steps.push_back((int)steps.size());
        return 0;
      });
      if (e) return -1;
    }
  }
  return pairs;
}
}  // namespace

int main() {
  long unordered = 0;
  for (unsigned seed = 0; seed < 3000; ++seed) {
    if (unordered_pairs<first::StepOrder<Model>>(seed, false) != 0 || Model::bad) { std::printf("seed %u: steps not ordered, or an event on a captured stream\n", seed); return 1; }
    if (unordered_pairs<first::StepOrder<Model>>(seed, true) != 0 || Model::calls) { std::printf("seed %u: events on one stream\n", seed); return 1; }
    unordered += unordered_pairs<Unordered>(seed, false);
  }
  if (unordered == 0) { std::printf("the model finds nothing\n"); return 1; }
  std::printf("ok\n");
  return 0;
}
