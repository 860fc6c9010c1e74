// The library's one-workgroup scan on the CPU: every thread of the workgroup is
// a fiber, shuffles run in lockstep within a wavefront, and between two barriers
// the wavefronts run one after another in an order that the test picks, so that
// a word written before all wavefronts have read it gives wrong sums.
// Usage: block_scan <order> <n>; order: up, down, or the seed of random orders.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <random>
#include <vector>

#define __device__
namespace gmp {
constexpr int kWave = 64;
}
constexpr int kThreads = 1024, kWaves = kThreads / gmp::kWave;

enum State { RUN, SHUFFLE, BARRIER, DONE };
struct Fiber {
  ucontext_t ctx;
  State state = RUN;
  std::vector<char> stack;
};
static Fiber fibers[kThreads];
static ucontext_t sched;
static int current;
static int64_t given[kThreads], taken[kThreads];  // shuffle operands, and their copy at the lockstep point
static struct {
  operator int() const { return current; }
} tid;
static struct {
  decltype(tid) x;
} threadIdx;

static void yield(State s) {
  const int me = current;
  fibers[me].state = s;
  swapcontext(&fibers[me].ctx, &sched);
}
static int64_t __shfl_up(int64_t v, int o, int width) {
  const int me = current, lane = me % width;
  given[me] = v;
  yield(SHUFFLE);
  return lane >= o ? taken[me - o] : v;
}
static void __syncthreads() { yield(BARRIER); }
namespace gmp {
inline int lane_id() { return current % kWave; }
}

#include "../../paper_2303_12980_amd/csrc/block_scan.h"

static std::vector<int32_t> in;
static std::vector<int64_t> out;
static int64_t words[gmp::kScanWords];

static void body() {
  gmp::block_scan([](int64_t i) { return (int64_t)in[i]; }, out.data(), (int64_t)in.size(), words);
  fibers[current].state = DONE;
  swapcontext(&fibers[current].ctx, &sched);
}

// one wavefront up to its next barrier (or its end)
static void run_wave(int w) {
  for (;;) {
    int at[4] = {0, 0, 0, 0};
    for (int l = 0; l < gmp::kWave; ++l) {
      current = w * gmp::kWave + l;
      Fiber &f = fibers[current];
      if (f.state == RUN) swapcontext(&sched, &f.ctx);
      ++at[fibers[w * gmp::kWave + l].state];
    }
    if (at[SHUFFLE] == 0) return;
    if (at[SHUFFLE] != gmp::kWave) { fprintf(stderr, "a shuffle in divergent code\n"); exit(3); }
    for (int l = 0; l < gmp::kWave; ++l) {
      const int t = w * gmp::kWave + l;
      taken[t] = given[t];
      fibers[t].state = RUN;
    }
  }
}

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  const int64_t n = atoll(argv[2]);
  in.resize(n);
  out.assign(n + 1, -1);
  for (int64_t i = 0; i < n; ++i) in[i] = (int32_t)((i * 2654435761u) % 1000);
  memset(words, 0x55, sizeof(words));
  for (int t = 0; t < kThreads; ++t) {
    Fiber &f = fibers[t];
    f.stack.resize(32768);
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = f.stack.data();
    f.ctx.uc_stack.ss_size = f.stack.size();
    f.ctx.uc_link = nullptr;
    makecontext(&f.ctx, body, 0);
  }
  std::vector<int> order(kWaves);
  for (int w = 0; w < kWaves; ++w) order[w] = w;
  const bool random = strcmp(argv[1], "up") && strcmp(argv[1], "down");
  std::mt19937 rng(random ? (unsigned)atoi(argv[1]) : 0u);
  if (!strcmp(argv[1], "down")) std::reverse(order.begin(), order.end());
  for (;;) {
    if (random) std::shuffle(order.begin(), order.end(), rng);
    for (int w : order) run_wave(w);
    int done = 0, barrier = 0;
    for (Fiber &f : fibers) {
      done += f.state == DONE;
      barrier += f.state == BARRIER;
    }
    if (done == kThreads) break;
    if (barrier != kThreads) { fprintf(stderr, "a barrier that not every thread reaches\n"); return 3; }
    for (Fiber &f : fibers) f.state = RUN;
  }
  int64_t sum = 0;
  for (int64_t i = 0; i <= n; ++i) {
    if (out[i] != sum) {
      printf("out[%lld] = %lld, expected %lld\n", (long long)i, (long long)out[i], (long long)sum);
      return 1;
    }
    if (i < n) sum += in[i];
  }
  return 0;
}
