// Bookkeeping of timed launches whose neighbours share an event.
#pragma once

#include <cstddef>
#include <vector>

namespace phprng {
namespace bat {

// A timed launch, from the end a of the one before it to its own end b; b
// belongs to the launch after it, unless this is the last of its chain (one
// call's launches, in order).
template <class Event>
struct Pending {
  int cls;
  Event a, b;
  bool last;
};

// Takes finished launches out of `pending`: add(p) gets each, give(e) every
// event that no launch needs any more.  finished(b) is asked in order, and
// once it says no, the rest of that chain stays without a question: a launch
// that had finished a moment later would give back the event on which the one
// before it still waits.
template <class Event, class Finished, class Add, class Give>
void take_finished(std::vector<Pending<Event>> &pending, Finished finished, Add add, Give give) {
  size_t keep = 0;
  bool held = false;  // a launch earlier in this chain stays
  for (size_t i = 0; i < pending.size(); ++i) {
    const Pending<Event> p = pending[i];
    held = held || !finished(p.b);
    if (held) {
      pending[keep++] = p;
    } else {
      add(p);
      give(p.a);
      if (p.last) give(p.b);
    }
    if (p.last) held = false;
  }
  pending.resize(keep);
}

}  // namespace bat
}  // namespace phprng
