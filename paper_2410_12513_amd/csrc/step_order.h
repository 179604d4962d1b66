// Order of decode steps whose workgroups wait for each other and that must not be on the chip together.
//
// The persistent step kernel (step_kernel.h) needs every compute unit.  Two of them at once - contexts on streams of their own - would each
// hold compute units that the other needs until a wait gives up, so a device's steps of that kind run one after the other: a step waits
// for an event behind the latest one on another stream, and leaves an event behind itself.  As long as all such contexts of a device share one
// stream (one context: always) the stream does that, and no event is recorded or waited for.  (A step of the 1B shape, 520 us, takes 5 us longer
// with the event, 11 where two contexts take turns.)
//
// The whole-step kernel of small fp32 models (small_step.h) waits between its 64 workgroups too, but needs little: a persistent kernel on
// every compute unit leaves each of them room for one such workgroup, so four of these steps always find their places on 256 compute units,
// whatever else runs.  They go through four lanes, in each of which steps are ordered as above; contexts are spread over the lanes by their streams, so that
// up to four streams see no event.  A persistent kernel of a geometry that takes so much LDS that no workgroup fits beside it, and the
// one that runs a batched step (batch_step.h), is ordered against all lanes.
//
// A context belongs to an order from its first such step on: one that does not decode costs the others nothing.
//
// The runtime's calls come in through Api, so that the rule can be run against a model of streams and events without a GPU.
#pragma once
#include <map>
#include <mutex>
#include <vector>

namespace first {

// Api: types Stream, Event, Error; Error{} is success.  make(Event*), record(Event, Stream), wait(Stream, Event): Error; capturing(Stream): bool.
// One order.  Not safe for several threads by itself: StepOrders holds its lock around every call.
template <typename Api>
class StepOrder {
 public:
  using Stream = typename Api::Stream;
  using Event = typename Api::Event;
  using Error = typename Api::Error;

  // A context that launches such steps works on st from now on / no longer (its steps are done).
  Error join(Stream st) {
    Error e{};
    if (!made) { e = Api::make(&event); made = e == Error{}; }
    if (made && streams.size() == 1 && !streams.count(st)) e = mark_latest();      // (its steps so far left no events)
    if (e == Error{}) ++streams[st];
    return e;
  }
  void leave(Stream st) {
    const auto it = streams.find(st);
    if (it == streams.end() || --it->second > 0) return;
    streams.erase(it);
    if (has_latest && latest == st) has_latest = false;
  }
  // Enqueues one step on st through launch().  While a caller captures st into a graph of their own nothing runs now, and events of
  // other streams cannot be waited for there: the launch goes into the graph as it is, and ordering its replays is up to the caller.
  template <typename F>
  Error run(Stream st, F launch) {
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
  bool has(Stream st) const { return streams.count(st) > 0; }
  size_t size() const { return streams.size(); }

 private:
  // The event stands behind the latest step.
  Error mark_latest() {
    if (!has_latest || marked || Api::capturing(latest)) return Error{};
    const Error e = Api::record(event, latest);
    marked = e == Error{};
    return e;
  }
  std::map<Stream, int> streams;       // of the contexts, with their number
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
  using Set = std::vector<StepOrder<Api>*>;           // what a context's steps go through

  // in: the orders of a context of this kind on st; on an error none.  n_lanes: small steps that find room beside a persistent one (of this
  // device: the same in every call).
  Error join(StepKind kind, Stream st, int n_lanes, Set* in) {
    std::lock_guard<std::mutex> lock(mutex);
    Set want;
    if (kind == StepKind::SMALL) {
      StepOrder<Api>* lane = &lanes[0];
      for (int i = 1; i < n_lanes; ++i)
        if (!lane->has(st) && (lanes[i].has(st) || lanes[i].size() < lane->size())) lane = &lanes[i];
      want = {lane};
    } else {
      if (kind == StepKind::PERSISTENT_NO_ROOM)
        for (auto& l : lanes) want.push_back(&l);
      want.push_back(&persistent);
    }
    for (StepOrder<Api>* o : want) {
      const Error e = o->join(st);
      if (e != Error{}) {
        for (StepOrder<Api>* joined : *in) joined->leave(st);
        in->clear();
        return e;
      }
      in->push_back(o);
    }
    return Error{};
  }
  void leave(const Set& in, Stream st) {
    std::lock_guard<std::mutex> lock(mutex);
    for (StepOrder<Api>* o : in) o->leave(st);
  }
  template <typename F>
  Error run(const Set& in, Stream st, F launch) {
    std::lock_guard<std::mutex> lock(mutex);
    return run_through(in, st, launch, 0);
  }
  // f() while no event is recorded: what captures a stream that contexts share, so that none gets into the graph.
  template <typename F>
  auto hold(F f) {
    std::lock_guard<std::mutex> lock(mutex);
    return f();
  }

 private:
  template <typename F>
  static Error run_through(const Set& in, Stream st, F& launch, size_t i) {
    if (i == in.size()) return launch();
    return in[i]->run(st, [&]() { return run_through(in, st, launch, i + 1); });
  }
  std::mutex mutex;
  StepOrder<Api> lanes[SMALL_STEP_LANES], persistent;
};

}  // namespace first
