// af_slots.hpp -- how many slots of a device-resident step loop to enqueue
// before the host looks again: host arithmetic alone, without HIP.
#pragma once

#include <algorithm>

namespace afi {

// up to `chunk` slots of `rounds` rounds, and no more than `left` steps (at most
// LONG_MAX: a caller who means t_final alone to end the run) need when every
// attempt is accepted: a round with nothing left to do still costs its launches
// (32 rounds for 3 steps of a batch: 750 of its 2460 us)
inline long slots_for(long left, int rounds, long chunk) {
  return left > 0 ? std::min(chunk, (left - 1) / rounds + 1) : 1;
}

}  // namespace afi
