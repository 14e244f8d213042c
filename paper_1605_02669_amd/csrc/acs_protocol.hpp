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

// Grid barrier of the synchronous kernels: a flag word says at which barrier its
// writer has arrived, as an epoch: iteration << 17 | barrier, modulo 2^32 (a
// construction has fewer than 2^17 - 1 barriers, from 1 on).
constexpr int kBarrierBits = 17;
ACS_PROTOCOL uint32_t barrier_epoch(uint32_t it, uint32_t bar) { return it << kBarrierBits | bar; }

// Whether the flag's writer has arrived at the barrier of this epoch.  It can be
// one barrier ahead of a block that still waits, never two: the second needs that
// block's own arrival.  Anything else is what an earlier launch left.  Which words
// a launch writes depends on where its blocks are placed, so a word may be any
// number of launches old; only one exactly 32768 iterations old could be taken
// for this epoch, and every kBarrierClear iterations all words are set to
// barrier_epoch(it, 0), which no barrier from there to the next time is.
constexpr uint32_t kBarrierClear = 1u << 14;
ACS_PROTOCOL bool barrier_reached(uint32_t flag, uint32_t epoch) { return flag - epoch <= 1u; }
ACS_PROTOCOL bool barrier_clear_due(uint32_t it) { return it % kBarrierClear == 0; }

}  // namespace acs
