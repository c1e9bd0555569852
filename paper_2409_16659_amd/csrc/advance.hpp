// advance.hpp -- how a call of n time steps is split into launches (host code).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace mlf {

// Advances by `nsteps` steps.  A graph of `graph_steps` steps (0: none) is
// replayed whenever that many remain; it exists for either buffer the
// populations may be in, so that a launch of two steps (which swaps the
// buffers once, like a launch of one) never keeps a later call from it.
// Other launches take as many steps as next(room) says, room the steps left
// until the end or the next guard poll (every `every` > 0 steps; a replay may
// go past a poll, which then follows it).  replay(), launch(n) and poll()
// return a status, 0 to go on.
template <typename Next, typename Replay, typename Launch, typename Poll>
auto advance(int64_t nsteps, int64_t every, int graph_steps, Next&& next, Replay&& replay, Launch&& launch,
             Poll&& poll) -> decltype(replay()) {
  int64_t left = nsteps, since = 0;
  while (left > 0) {
    int64_t adv = graph_steps;
    if (graph_steps > 0 && left >= graph_steps) {
      if (auto s = replay()) return s;
    } else {
      adv = next(every > 0 ? std::min(left, every - since) : left);
      if (auto s = launch((int)adv)) return s;
    }
    left -= adv;
    since += adv;
    if (every > 0 && since >= every && left > 0) {
      since = 0;
      if (auto s = poll()) return s;
    }
  }
  return {};
}

}  // namespace mlf
