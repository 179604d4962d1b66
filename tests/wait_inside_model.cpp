// A wait inside a workgroup (csrc/wait_inside.h) beside the poll that it depends on, in simulated time: one wave polls memory for another workgroup's word, up to
// SK_SPIN_LIMIT turns, and then says in LDS that it is there or that it gave up; the other wave waits for that.
#include <cstdio>
#include <initializer_list>

#include "../paper_2410_12513_amd/csrc/wait_inside.h"

using namespace first;

namespace {
constexpr double POLL_US = 2.0, TURN_US = 0.1;         // a turn of the poll (a round trip of memory), of the wait (two of LDS and a pause)

struct End { WaitEnd end; double at; };
// The word is there `late` us after both waves began to wait; polls: how many the wait depends on, one after the other, each as late.
End wait(double late, int polls) {
  const double limit = SK_SPIN_LIMIT * POLL_US, there_at = late <= limit ? polls * late : 1e300, gives_up_at = late <= limit ? 1e300 : limit;
  double now = 0;
  const WaitEnd e = wait_inside([&] { return now >= there_at; }, [&] { return now >= gives_up_at; }, [&] { now += TURN_US; });
  return {e, now};
}
}  // namespace

int main() {
  const double limit = SK_SPIN_LIMIT * POLL_US;
  // whatever the poll still gets, the wait gets: up to three polls in a row (activations, squares, activations again)
  for (const double late : {0.0, 5.0, 1e3, 1e5, 0.2e6, 0.3e6, 1e6, 2e6, limit}) {
    const End e = wait(late, 3);
    if (e.end != WaitEnd::THERE || e.at < 3 * late) { std::printf("%.0f us late: the wait ended with %d at %.0f\n", late, (int)e.end, e.at); return 1; }
  }
  // what the poll does not get ends the wait when the poll gives up
  const End e = wait(limit + POLL_US, 1);
  if (e.end != WaitEnd::GIVEN_UP || e.at > limit + 2 * TURN_US) { std::printf("beyond the poll's limit: %d at %.0f\n", (int)e.end, e.at); return 1; }
  // and it ends by itself if neither ever happens
  unsigned turns = 0;
  if (wait_inside([] { return false; }, [] { return false; }, [&] { ++turns; }) != WaitEnd::RAN_OUT || turns != INSIDE_LIMIT) { std::printf("no end\n"); return 1; }
  std::printf("ok\n");
  return 0;
}
