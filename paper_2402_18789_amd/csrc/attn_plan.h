#pragma once
// Which attention kernel a batch's work list takes, how many of its key splits as one, and in which order.  Host arithmetic on the
// maps' sums alone.
#include <algorithm>
#include <cstdint>
#include "flexco.h"

#ifdef __HIPCC__
#define FLEXCO_HOST_DEVICE __host__ __device__
#else
#define FLEXCO_HOST_DEVICE
#endif

namespace flexco {

// The item of the work list that turn `turn` takes where the block of a request of one token takes fold neighbouring key splits as one (turns
// are dealt to the chip's parts one after the other; turns run to turns_of(n_items, fold), those past the last item have none).
// Items at a stride of fold: the ones that are left with work are every fold-th of a request, so in the list's own order requests of a
// multiple of fold splits left all of it to every fold-th part of the chip.  Us, 8 kv heads: 24 requests of 1024 keys in eights 49.9 ->
// 23.9, 4 of 3072 in fours 33.6 -> 19.2, 24 of 4096 in fours 140 -> 80; odd numbers of splits within 5 %.
FLEXCO_HOST_DEVICE inline int turns_of(int n_items, int fold) { return (n_items + fold - 1) / fold * fold; }
FLEXCO_HOST_DEVICE inline int item_of_turn(int turn, int n_items, int fold) {
  const int run = (n_items + fold - 1) / fold;
  return turn % run * fold + turn / run;
}

}  // namespace flexco
