// Host side of launches whose blocks meet: which of two sets of polled memory a launch uses.
#pragma once
#include <stdint.h>

namespace adacgd {

// What the blocks of a launch leave for each other is polled, so it must be clear when the launch begins.  It exists twice:
// a launch uses one set and clears the other, which the launch before it has left behind.
//  - A launch that fails has cleared nothing, and whether it left something is not known: both sets are cleared before
//    the next one.
//  - A captured launch may be replayed in any number and cannot rely on the alternation: it is enclosed by clears of both.
struct MeetingSets {
  uint32_t set = 0;      // the one the next launch uses
  bool stale = false;    // the last launch failed
};

// launch(set) enqueues the launch, clear() the clearing of both sets; both return a status whose default value is success.
template <typename Clear, typename Launch>
auto launch_meeting(MeetingSets& m, bool captured, Clear&& clear, Launch&& launch) -> decltype(clear()) {
  using Status = decltype(clear());
  const Status ok{};
  if (captured || m.stale) {
    const Status e = clear();
    if (e != ok) return e;
    m.stale = m.stale && captured;       // (what is captured has not been done)
  }
  const Status e = launch(m.set);
  if (captured) return e == ok ? clear() : e;
  if (e == ok) m.set ^= 1u;
  else m.stale = true;
  return e;
}

}  // namespace adacgd
