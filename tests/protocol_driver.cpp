// The kernels' shared-word protocols (csrc/acs_protocol.hpp) on host threads,
// one for each wave, with one of them held back at a time, and the launch shapes
// of the synchronous and sequential kernels (csrc/acs_sync_shape.hpp).
#include <pthread.h>
#include <unistd.h>

#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "acs_protocol.hpp"
#include "acs_sync_shape.hpp"

namespace {

int failures = 0;

// Every wave of a block sees the lowest wave that found something, also the one
// that comes late out of the barrier (or late into it).
void queue_rounds() {
  constexpr int kWaves = 4, kRounds = 12;
  // waves that find something, a bit each, and entries in the queue
  const unsigned finds[kRounds] = {8, 0, 1, 14, 2, 0, 0, 12, 15, 4, 6, 0};
  const int heads[kRounds] = {4, 4, 4, 4, 2, 1, 4, 4, 4, 3, 3, 4};
  for (int late = 0; late < kWaves; ++late)
    for (int where = 0; where < 2; ++where) {
      int words[2] = {acs::kNoWave, acs::kNoWave};
      int seen[kWaves][kRounds];
      pthread_barrier_t bar;
      pthread_barrier_init(&bar, nullptr, kWaves);
      std::vector<std::thread> block;
      for (int w = 0; w < kWaves; ++w)
        block.emplace_back([&, w] {
          int syncs = 0;
          auto sync = [&] {
            pthread_barrier_wait(&bar);
            if (w == late && syncs++ % 2 == where) usleep(5000);
          };
          for (int r = 0; r < kRounds; ++r) {
            auto examine = [&](int *word) {
              int old = __atomic_load_n(word, __ATOMIC_RELAXED);
              while ((finds[r] >> w & 1u) && w < old &&
                     !__atomic_compare_exchange_n(word, &old, w, false, __ATOMIC_RELAXED,
                                                  __ATOMIC_RELAXED)) {
              }
            };
            acs::queue_round(words, (uint32_t)r, w, heads[r], sync, examine,
                             [&](int first) { seen[w][r] = first; });
          }
        });
      for (auto &t : block) t.join();
      pthread_barrier_destroy(&bar);
      for (int r = 0; r < kRounds; ++r) {
        int want = acs::kNoWave;
        for (int w = heads[r] - 1; w >= 0; --w)
          if (finds[r] >> w & 1u) want = w;
        for (int w = 0; w < kWaves; ++w)
          if (seen[w][r] != want) {
            std::printf("queue_round %d, wave %d late %s the barrier: wave %d saw %d, not %d\n", r,
                        late, where ? "into" : "out of", w, seen[w][r], want);
            ++failures;
          }
      }
    }
}

// No word that earlier launches left, of whatever age, passes for a barrier of
// this one; a block at the barrier or one ahead does.
void barrier_epochs() {
  const uint32_t bars[] = {1, 2, 3, 1000, 70000, 131069};  // the last: two a step at the largest n
  const uint32_t its[] = {0, 1, 5, 16383, 16384, 16385, 30000, 32767, 32768, 49152, 100000, 1u << 28,
                          0xffffffffu};
  auto expect = [](bool want, uint32_t flag, uint32_t it, uint32_t bar, const char *what) {
    if (acs::barrier_reached(flag, acs::barrier_epoch(it, bar)) == want) return;
    if (failures++ < 8)
      std::printf("barrier %u of iteration %u: %s flag %u\n", bar, it, what, flag);
  };
  for (uint32_t it : its)
    for (uint32_t bar : bars) {
      expect(true, acs::barrier_epoch(it, bar), it, bar, "own");
      expect(true, acs::barrier_epoch(it, bar + 1), it, bar, "next");
      expect(false, acs::barrier_epoch(it, bar - 1), it, bar, "earlier");
      expect(false, acs::barrier_epoch(it, 0), it, bar, "cleared");
      for (uint32_t age = 1; age < 32768 && age <= it; ++age)
        for (uint32_t left : bars) expect(false, acs::barrier_epoch(it - age, left), it, bar, "old");
      // the words as the last clearing left them
      uint32_t cleared = it;
      while (!acs::barrier_clear_due(cleared)) --cleared;
      expect(false, acs::barrier_epoch(cleared, 0), it, bar, "cleared earlier");
      if (it - cleared >= 32768) {
        std::printf("iteration %u: words uncleared for %u iterations\n", it, it - cleared);
        ++failures;
      }
    }
}

// Every block of a synchronous launch is resident on the device, whatever share
// of the card it is.
void sync_residency() {
  auto expect = [](bool ok, int n, int m, int cl, int resident, const char *what) {
    if (ok) return;
    std::printf("n %d, m %d, cl %d, %d blocks resident: %s\n", n, m, cl, resident, what);
    ++failures;
  };
  const int ns[] = {30, 198, 1000, 2392, 20000}, cls[] = {1, 12, 16, 32, 64};
  for (int n : ns)
    for (int cl : cls)
      for (int m = 1; m <= 4096; m += m < 1100 ? 1 : 97)
        for (int resident : {0, 16, 31, 32, 33, 63, 64, 256}) {
          if (acs::sync_lds_taken(n, m, cl, resident))
            expect(acs::sync_lds_blocks(m) <= resident, n, m, cl, resident,
                   "pheromone in LDS, but not all blocks fit");
          if (resident >= 64)
            expect(acs::sync_lds_taken(n, m, cl, resident) == acs::sync_lds(n, m, cl), n, m, cl,
                   resident, "another kernel than on the whole card");
          const int a = acs::sync_ants_per_block_on(m, resident);
          expect((m + a - 1) / a <= resident || a == acs::kSyncMaxAnts, n, m, cl, resident,
                 "more blocks than fit");
          if (resident >= 256)
            expect(a == acs::sync_ants_per_block(m), n, m, cl, resident,
                   "another block size than on the whole card");
        }
}

// The sequential construction's groups: whole waves' worth, small where ants meet
// often, the largest where they rarely do.
void seq_groups() {
  auto expect = [](bool ok, int n, uint32_t period, int g) {
    if (ok) return;
    std::printf("seq_group(%d, %u) = %d\n", n, period, g);
    ++failures;
  };
  const uint32_t periods[] = {1, 2, 3, 16, 250, 65536, 0x7fffffffu, 0xffffffffu};
  for (uint32_t p : periods)
    for (int n = 3, last = 16; n <= 65535; ++n) {
      const int g = acs::seq_group(n, p);
      expect(g >= last && g % 16 == 0 && g <= acs::kSeqGroup, n, p, g);
      last = g;
    }
  // where the largest group was slower than rounds of 16 ants
  for (int n : {10, 30, 50}) expect(acs::seq_group(n, 1) == 16, n, 1, acs::seq_group(n, 1));
  for (int n : {100, 150, 200}) expect(acs::seq_group(n, 1) == 32, n, 1, acs::seq_group(n, 1));
  expect(acs::seq_group(50, 2) <= 32, 50, 2, acs::seq_group(50, 2));
  // where it is the fastest
  for (int n : {1200, 2392, 8000}) expect(acs::seq_group(n, 1) == 128, n, 1, acs::seq_group(n, 1));
  expect(acs::seq_group(100, 16) == 128, 100, 16, acs::seq_group(100, 16));
}

}  // namespace

int main(int argc, char **argv) {
  if (argc == 2 && !std::strcmp(argv[1], "queue_round")) queue_rounds();
  else if (argc == 2 && !std::strcmp(argv[1], "barrier")) barrier_epochs();
  else if (argc == 2 && !std::strcmp(argv[1], "sync_residency")) sync_residency();
  else if (argc == 2 && !std::strcmp(argv[1], "seq_groups")) seq_groups();
  else return 2;
  if (!failures) std::puts("ok");
  return failures ? 1 : 0;
}
