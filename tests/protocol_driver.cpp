// The kernels' shared-word protocols (csrc/acs_protocol.hpp) on host threads,
// one for each wave, with one of them held back at a time.
#include <pthread.h>
#include <unistd.h>

#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "acs_protocol.hpp"

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

}  // namespace

int main(int argc, char **argv) {
  if (argc == 2 && !std::strcmp(argv[1], "queue_round")) queue_rounds();
  else return 2;
  if (!failures) std::puts("ok");
  return failures ? 1 : 0;
}
