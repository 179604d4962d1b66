// Order of decode steps whose workgroups wait for each other and that must not be on the chip together.
//
// The persistent step kernel (step_kernel.h) needs every compute unit.  Two of them at once - contexts on streams of their own - would each
// hold compute units that the other needs until a wait gives up, so a device's steps of that kind run one after the other: a step waits
// for an event behind the latest one on another stream, and leaves an event behind itself.  As long as all such contexts of a device share one
// stream (one context: always) the stream does that, and no event is recorded or waited for.  (A step of the 1B shape, 520 us, takes 5 us longer
// with the event, 11 where two contexts take turns.)
//
// The whole-step kernel of small fp32 models (small_step.h) waits between its 64 workgroups too, but needs little: a persistent kernel on
// every compute unit leaves each of them room for one such workgroup, so four of these steps always find their places, whatever else
// runs.  They go through four lanes, in each of which steps are ordered as above; contexts are spread over the lanes by their streams, so that
// up to four streams see no event.  A persistent kernel of a geometry that takes so much LDS that no workgroup fits beside it is
// ordered against all lanes.
//
// The runtime's calls come in through Api, so that the rule can be run against a model of streams and events without a GPU.
#pragma once
#include <map>
#include <mutex>
#include <vector>

namespace first {

// Api: types Stream, Event, Error; Error{} is success.  make(Event*), record(Event, Stream), wait(Stream, Event): Error; capturing(Stream): bool.
template <typename Api>
class StepOrder {
 public:
  using Stream = typename Api::Stream;
  using Event = typename Api::Event;
  using Error = typename Api::Error;

  // A context that launches such steps works on st from now on / no longer (its steps are done).
  Error join(Stream st) {
    std::lock_guard<std::mutex> lock(mutex);
    Error e{};
    if (!made) { e = Api::make(&event); made = e == Error{}; }
    if (made && streams.size() == 1 && !streams.count(st)) e = mark_latest();      // (its steps so far left no events)
    if (e == Error{}) ++streams[st];
    return e;
  }
  void leave(Stream st) {
    std::lock_guard<std::mutex> lock(mutex);
    const auto it = streams.find(st);
    if (it == streams.end() || --it->second > 0) return;
    streams.erase(it);
    if (has_latest && latest == st) has_latest = false;
  }
  // Enqueues one step on st through launch().  While a caller captures st into a graph of their own nothing runs now, and events of
  // other streams cannot be waited for there: the launch goes into the graph as it is, and ordering its replays is up to the caller.
  template <typename F>
  Error run(Stream st, F launch) {
    std::lock_guard<std::mutex> lock(mutex);
    Error e{};
    const bool alone = streams.size() < 2;
    if (!alone && Api::capturing(st)) return launch();
    if (!alone && has_latest && latest != st) {
      e = mark_latest();
      if (e == Error{} && marked) e = Api::wait(st, event);
    }
    if (e == Error{}) e = launch();
    if (e != Error{}) return e;
    has_latest = true; latest = st; marked = false;
    return alone ? e : mark_latest();
  }
  bool has(Stream st) {
    std::lock_guard<std::mutex> lock(mutex);
    return streams.count(st) > 0;
  }
  size_t size() {
    std::lock_guard<std::mutex> lock(mutex);
    return streams.size();
  }
  // f() while no step is being enqueued and no event recorded: the context's own captures, whose stream must not see an event.
  template <typename F>
  auto hold(F f) {
    std::lock_guard<std::mutex> lock(mutex);
    return f();
  }

 private:
  // The event stands behind the latest step.
  Error mark_latest() {
    if (!has_latest || marked || Api::capturing(latest)) return Error{};
    const Error e = Api::record(event, latest);
    marked = e == Error{};
    return e;
  }
  std::mutex mutex;
  std::map<Stream, int> streams;       // of the live contexts, with their number
  Event event{};
  bool made = false, has_latest = false, marked = false;
  Stream latest{};                     // stream of the latest step
};

enum class StepKind { PERSISTENT, PERSISTENT_NO_ROOM, SMALL };
constexpr int SMALL_STEP_LANES = 4;

// The orders of one device.
template <typename Api>
class StepOrders {
 public:
  using Stream = typename Api::Stream;
  using Error = typename Api::Error;
  using Set = std::vector<StepOrder<Api>*>;           // what a context's steps go through (locks are taken in the order of the members below)

  // in: the orders of a context of this kind on st; on an error none.
  Error join(StepKind kind, Stream st, Set* in) {
    std::lock_guard<std::mutex> lock(mutex);
    Set want;
    if (kind == StepKind::SMALL) {
      StepOrder<Api>* lane = &lanes[0];
      for (auto& l : lanes)
        if (!lane->has(st) && (l.has(st) || l.size() < lane->size())) lane = &l;
      want = {lane};
    } else {
      if (kind == StepKind::PERSISTENT_NO_ROOM)
        for (auto& l : lanes) want.push_back(&l);
      want.push_back(&persistent);
    }
    for (StepOrder<Api>* o : want) {
      const Error e = o->join(st);
      if (e != Error{}) { leave(*in, st); in->clear(); return e; }
      in->push_back(o);
    }
    return Error{};
  }
  static void leave(const Set& in, Stream st) {
    for (StepOrder<Api>* o : in) o->leave(st);
  }
  template <typename F>
  static Error run(const Set& in, Stream st, F& launch, size_t i = 0) {
    if (i == in.size()) return launch();
    return in[i]->run(st, [&]() { return run(in, st, launch, i + 1); });
  }
  template <typename F>
  static auto hold(const Set& in, F& f, size_t i = 0) -> decltype(f()) {
    if (i == in.size()) return f();
    return in[i]->hold([&]() { return hold(in, f, i + 1); });
  }

 private:
  std::mutex mutex;
  StepOrder<Api> lanes[SMALL_STEP_LANES], persistent;
};

}  // namespace first
