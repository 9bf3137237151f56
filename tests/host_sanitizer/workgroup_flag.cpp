// Threads of the host as the threads of a workgroup: what one finds out for all (tdq_workgroup.hpp), asked again and
// again through one word with nothing in between, as workgroups that share a set do between two rounds.
// ThreadSanitizer sees an access that no barrier orders; the answers are checked as well.
#include <pthread.h>

#include <cstdio>
#include <thread>
#include <vector>

struct Index { unsigned x; };
static thread_local Index threadIdx;
static pthread_barrier_t g_barrier;
static void __syncthreads() { pthread_barrier_wait(&g_barrier); }
#define __device__
#define __forceinline__ inline

#include "tdq_workgroup.hpp"

int main() {
  constexpr unsigned kThreads = 6, kAsked = 300;
  static unsigned flag;
  int wrong[kThreads] = {};
  pthread_barrier_init(&g_barrier, nullptr, kThreads);
  std::vector<std::thread> all;
  for (unsigned i = 0; i < kThreads; ++i)
    all.emplace_back([&wrong, i]() {
      threadIdx.x = i;
      for (unsigned n = 0; n < kAsked; ++n) {
        bool asked = false;
        const bool so = tdq::known_to_all(&flag, [&]() { asked = true; return n % 3 == 1; });
        wrong[i] += so != (n % 3 == 1) || asked != (i == 0);
      }
    });
  for (auto& t : all) t.join();
  int n = 0;
  for (int w : wrong) n += w;
  printf("%d wrong\n", n);
  return n != 0;
}
