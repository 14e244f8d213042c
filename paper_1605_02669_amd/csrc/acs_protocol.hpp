// How the waves of a block take turns on words they share: the order of their
// reads, writes and barriers, apart from what they compute.  The kernels run
// these functions, and so does a test, with host threads for waves, which can
// hold any one of them back at any point.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define ACS_PROTOCOL __host__ __device__ __forceinline__
#else
#define ACS_PROTOCOL inline
#endif

namespace acs {

// One round of a block whose waves look at the first `heads` entries of a
// queue at the same time, wave w at entry w.
//   examine(word): this wave's entry; a wave that finds something lowers *word
//     to its index (atomically).
//   act(first): on every wave, with the lowest such index (kNoWave: none).  All
//     waves of the block take the same decisions from it.
// Every wave has to read the index that all of them left, and a wave can be
// late by any time: the word of a round is therefore written by nobody between
// the two barriers.  What is reset there is the other word, which the next round
// uses; its readers of the round before have passed two barriers since.
// words: two words, both kNoWave before the first round (0).
constexpr int kNoWave = 64;

template <class Sync, class Examine, class Act>
ACS_PROTOCOL void queue_round(int *words, uint32_t round, int wave, int heads, Sync sync,
                              Examine examine, Act act) {
  int *const word = words + (round & 1);
  if (wave < heads) examine(word);
  sync();
  act(*word);
  if (wave == 0) words[(round + 1) & 1] = kNoWave;
  sync();
}

}  // namespace acs
