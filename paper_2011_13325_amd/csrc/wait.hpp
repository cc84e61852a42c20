// Waiting in host memory for what the device writes there.
#pragma once

#include <thread>

namespace eamg {

// Lets the core's other hardware thread run while this one polls.
struct CoreRest {
  void operator()() const {
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
  }
};

// Polls until ready().  After every kPolls polls, however long the wait, busy() says whether anything
// is left that could still make it ready (it may throw), and the core goes to other threads that
// want it.  Returns whether it is ready.
constexpr int kPolls = 1024;
template <class Ready, class Busy, class Rest = CoreRest>
bool poll_until(Ready &&ready, Busy &&busy, Rest &&rest = Rest()) {
  for (;;) {
    for (int i = 0; i < kPolls; ++i) {
      if (ready()) return true;
      rest();
    }
    if (!busy()) return ready();
    std::this_thread::yield();
  }
}

}  // namespace eamg
