// csrc/clear_once.hpp on the CPU: a chip of a few slots, each of which runs one workgroup of one wave after the other to its end;
// two launches that are in flight at once share it, and their workgroups start in an order that is given.  A wave is a thread
// that stands for its lanes.
//   clear_once_model ORDER SLOTS: exit status 0: every word holds what the waves have added to it; 1: not; 2: a wave waited for ever.
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <thread>
#include <vector>
#include <algorithm>
#include <sched.h>
#include <unistd.h>

#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
static uint32_t fetch_max(uint32_t* p, uint32_t v) {
  uint32_t before = __atomic_load_n(p, __ATOMIC_RELAXED);
  while (before < v && !__atomic_compare_exchange_n(p, &before, v, false, __ATOMIC_ACQ_REL, __ATOMIC_RELAXED)) {}
  return before;
}
#define __hip_atomic_fetch_max(p, v, order, scope) fetch_max(p, v)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
static std::atomic<long> waits{0};
static void wait_a_little(int) {
  if (++waits > 2000000) { fprintf(stderr, "a wave waits for ever\n"); _exit(2); }
  sched_yield();
}
#define __builtin_amdgcn_s_sleep(x) wait_a_little(x)
#include "clear_once.hpp"

int main(int argc, char** argv) {
  const char* const order = argv[1];
  const int slots = atoi(argv[2]);
  constexpr uint32_t WORDS = 100, GROUPS = 60;
  struct Launch { uint32_t word = 0, words[WORDS]; } launch[2];
  struct Group { int launch; uint32_t index; };
  std::mt19937 rng(7);
  for (uint32_t done = 2; done <= 2 * 200; done += 2) {
    std::vector<Group> groups;
    for (uint32_t i = 0; i < GROUPS; ++i)
      for (int l = 0; l < 2; ++l) groups.push_back({l, strcmp(order, "ascending") ? GROUPS - 1 - i : i});
    if (!strcmp(order, "random")) std::shuffle(groups.begin(), groups.end(), rng);
    for (Launch& l : launch)
      for (uint32_t& w : l.words) w = rng();              // what the buffer held before
    std::atomic<size_t> next{0};
    waits = 0;
    auto slot = [&]() {
      for (size_t g; (g = next++) < groups.size();) {
        Launch& l = launch[groups[g].launch];
        const uint32_t i = groups[g].index;
        if (i == 0 && fi::take_clearing(&l.word, done, 0)) {
          fi::clear_words(l.words, WORDS, 0, 1);
          fi::clearing_done(&l.word, done, 0);
        }
        if (i % 3 == 2) continue;                         // nothing to write
        uint32_t seen = i % 2 ? __atomic_load_n(&l.word, __ATOMIC_RELAXED) : 0;
        fi::cleared(l.words, WORDS, &l.word, done, seen, 0, 1);
        if (seen < done) return;
        for (uint32_t w = 0; w < WORDS; ++w) __atomic_fetch_add(&l.words[w], i + 1, __ATOMIC_RELAXED);
      }
    };
    std::vector<std::thread> threads;
    for (int s = 0; s < slots; ++s) threads.emplace_back(slot);
    for (std::thread& t : threads) t.join();
    uint32_t sum = 0;
    for (uint32_t i = 0; i < GROUPS; ++i) sum += i % 3 == 2 ? 0 : i + 1;
    for (const Launch& l : launch)
      for (uint32_t w : l.words)
        if (w != sum) { fprintf(stderr, "%u in the place of %u\n", w, sum); return 1; }
  }
  return 0;
}
