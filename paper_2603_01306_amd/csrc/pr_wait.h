// How long a wave has waited, counted while it runs (plain C++, no device
// functions, so that it can be tested on the host).
#pragma once

namespace pr {

// The time between two looks counts up to kWaitStep ticks of the 100 MHz clock,
// which goes on while a process is suspended or its queues are off the device:
// a wave that polls looks every millisecond or so, and what is beyond 10 ms it
// did not spend polling.
constexpr long long kWaitStep = 1000000;

struct WaitClock {
  long long last = 0, spent = 0;
  // now > 0: a look at the clock; true once more than `limit` ticks were waited
  constexpr bool expired(long long now, long long limit) {
    if (last != 0) {
      const long long d = now - last;
      spent += d < kWaitStep ? d : kWaitStep;
    }
    last = now;
    return spent > limit;
  }
};

}  // namespace pr
