// Order of decode steps whose workgroups wait for each other and that must not be on the chip together.
//
// The persistent step kernel (step_kernel.h) needs every compute unit.  Two of them at once - contexts on streams of their own - would each
// hold compute units that the other needs until a wait gives up, so a device's steps of that kind run one after the other: a step waits
// for an event behind the latest one on another stream, and leaves an event behind itself.  As long as all such contexts of a device share one
// stream (one context: always) the stream does that, and no event is recorded or waited for.
//
// The runtime's calls come in through Api, so that the rule can be run against a model of streams and events without a GPU.
#pragma once
#include <map>
#include <mutex>

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

}  // namespace first
