// Driver for tests/test_waiting_turn.py: contexts of several threads that take turns (see WaitingTurn).  Every context has at
// most one launch whose decision is not known; a launch takes a few steps of its thread to decide.  Prints how many launches
// waited, how many went without, and the largest number of contexts that had undecided launches at once.
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>

#include "waiting_turn.h"

using moe::WaitingTurn;

static int one_thread() {
  WaitingTurn t;
  uint64_t a = 0, b = 0;  // the contexts' notes: seq in the low half, other things above it
  int bad = 0;
  bad += !t.take(&a, &a, 1);
  bad += !t.take(&a, &a, 2);            // its own launches follow each other on one stream
  bad += t.take(&b, &b, 1);             // not while a's are undecided
  a = (7ull << 32) | 1u;                // the first of them is, the last is not
  bad += t.take(&b, &b, 1);
  a = (7ull << 32) | 2u;
  bad += !t.take(&b, &b, 1);
  bad += t.take(&a, &a, 3);
  b = 5u;                               // later steps of b have been decided too
  bad += !t.take(&a, &a, 3);
  bad += t.take(&b, &b, 6);
  t.give_back(&b);                      // not b's to give back
  bad += t.take(&b, &b, 6);
  t.give_back(&a);
  bad += !t.take(&b, &b, 6);
  b = 0xfffffffeu;
  bad += !t.take(&b, &b, 0xffffffffu);  // the counter wraps
  bad += t.take(&a, &a, 4);
  b = 1u;
  bad += !t.take(&a, &a, 4);
  return bad;
}

int main() {
  const int bad = one_thread();
  WaitingTurn t;
  std::atomic<int> undecided{0}, most{0};
  std::atomic<long> waited{0}, without{0};
  auto work = [&]() {
    uint64_t note = 0;
    for (uint32_t seq = 1; seq <= 20000; ++seq) {
      if (t.take(&note, &note, seq)) {
        const int now = ++undecided;
        int m = most.load();
        while (now > m && !most.compare_exchange_weak(m, now)) {
        }
        ++waited;
        --undecided;  // (decided from here on, said right behind)
        __atomic_store_n(&note, (uint64_t)seq, __ATOMIC_RELEASE);
      } else {
        ++without;
        __atomic_store_n(&note, (uint64_t)seq, __ATOMIC_RELEASE);  // (a step of another form tells its decision too)
      }
    }
    t.give_back(&note);
  };
  std::vector<std::thread> threads;
  for (int i = 0; i < 4; ++i) threads.emplace_back(work);
  for (auto &th : threads) th.join();
  printf("%d %ld %ld %d\n", bad, waited.load(), without.load(), most.load());
  return 0;
}
