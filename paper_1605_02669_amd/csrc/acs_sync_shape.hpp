// Launch shapes of the synchronous and sequential constructions: which kernel, how
// many ants a block or a group, the words of the grid barrier.  Host arithmetic
// without the GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace acs {

// Ants per block of the synchronous kernels.  Every phase of a step lasts as
// long as its slowest ant, and the waves of a SIMD run it in lockstep, so the
// ants are spread over all compute units (256), at most kSyncMaxAnts per
// block.  (m is a caller's word and may be any int here: a workspace's size is asked
// before it is checked.)
constexpr int kSyncMaxAnts = 16, kSyncBlocks = 256;
inline int sync_ants_per_block(int m) {
  const int64_t a = ((int64_t)m + kSyncBlocks - 1) / kSyncBlocks;
  return a < 1 ? 1 : a < kSyncMaxAnts ? (int)a : kSyncMaxAnts;
}
inline int sync_blocks(int m) {
  return (int)(((int64_t)m + sync_ants_per_block(m) - 1) / sync_ants_per_block(m));
}
// Dense synchronous construction with the candidate entries' pheromone in
// every block's LDS (k_construct_sync_lds).  Its ants per block: about 32
// blocks, up to 64 as long as they hold the ants, at least 4 each; a block then
// has a thread for every ant of the colony.
inline int sync_lds_ants_per_block(int m) {
  const int a = m <= 512 ? (m + 31) / 32 : m <= 64 * kSyncMaxAnts ? (m + 63) / 64 : kSyncMaxAnts;
  return a < 4 ? 4 : a;
}
// It can be taken where 64 blocks hold the ants, n * cl floats and 16 ants' bitmaps
// fit a block's LDS, and the blocks' words (two sets of 128 bytes each) fit the
// place of ctau, which it does not use.
constexpr size_t kSyncLdsBytes = 156 * 1024;
inline bool sync_lds(int n, int m, int cl) {
  const int a = sync_lds_ants_per_block(m);
  return m >= 1 && m <= 64 * kSyncMaxAnts &&
         (size_t)n * cl * 4 + (size_t)kSyncMaxAnts * ((n + 31) / 32) * 4 <= kSyncLdsBytes &&
         (size_t)((m + a - 1) / a) * 256 <= (size_t)n * cl * 4;
}
// It is taken where its blocks also fit the device at once: all blocks of a
// synchronous kernel wait for each other, so all have to be resident.  `resident`:
// blocks the device holds, with this kernel's block size and all of its LDS.  (256
// compute units always hold 64 such blocks; a partition of the card may not, and
// then the kernel below takes the colony.)
inline int sync_lds_blocks(int m) {
  return (int)(((int64_t)m + sync_lds_ants_per_block(m) - 1) / sync_lds_ants_per_block(m));
}
inline bool sync_lds_taken(int n, int m, int cl, int resident) {
  return sync_lds(n, m, cl) && sync_lds_blocks(m) <= resident;
}
// Ants per block of the other kernels on a device that holds `resident` blocks of
// sync_ants_per_block(m): fuller blocks where it does not hold all of those.
inline int sync_ants_per_block_on(int m, int resident) {
  return sync_blocks(m) <= resident ? sync_ants_per_block(m) : kSyncMaxAnts;
}
// Words of the grid barrier: the XCDs' lists and mailboxes, a word per block.
constexpr int kXcds = 8;
inline size_t sync_barrier_words(int m) {
  const size_t g = (size_t)sync_blocks(m);
  return kXcds * (((g + 31) & ~(size_t)31) + 32) + g;
}

// Ants that choose at once in the sequential construction: a multiple of 16, at
// most kSeqGroup.  A round commits the ants before the first whose row an earlier
// one writes, so the fewer cities there are, and the more often steps update, the
// more of a large group's choices are made again.  Best group by measurement (ms
// per iteration with it, with 128, and with the former kernel's rounds of 16 ants;
// cl = 32), update period 1:
//   n = 10, m = 200     16   1.35   2.98   1.69      n = 200, m = 1000    32   35.8   46.4   43.6
//   n = 50, m = 1000    24   15.5   28.1   18.9      n = 300, m = 1000    64   44.6   51.3   57.0
//   n = 100, m = 1000   24   23.9   36.9   28.2      n = 500, m = 500     64   30.6   32.9   43.9
//   n = 150, m = 1000   32   31.3   43.8   36.9      n = 1000, m = 1000   96  110.9  111.6  162.6
// and period 2: n = 50 24 (9.55, 14.9, 12.3), n = 100 32 (15.5, 20.2, 20.7), n = 200
// 64 (23.9, 27.0, 34.5), n = 500 96 (21.4, 21.7, 38.1); at period 16 128 from n = 100
// on.  The line through these is 16 + n * period / 10.
constexpr int kSeqGroup = 128;
inline int seq_group(int n, uint32_t period) {
  const uint64_t g = 16 + (uint64_t)n * period / 10;
  return g >= kSeqGroup ? kSeqGroup : (int)(g + 8) & ~15;
}

}  // namespace acs
