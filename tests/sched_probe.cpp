// Test helper: the program of the schedule kernel's wave (gst_sched_tile.h) on
// the CPU.  The 64 lanes are contexts that run in turn up to their next exchange;
// accesses to the staged window are checked and counted.
#include <ucontext.h>

#include <memory>
#include <vector>

#include "gst_sched_tile.h"

namespace {

constexpr int N = 64, STACK = 1 << 16;
ucontext_t main_ctx, lane_ctx[N];
std::vector<char> stacks(N* STACK);
int current = 0, running = 0;
int64_t value[2][N], out_of_range = 0;

void yield() { swapcontext(&lane_ctx[current], &main_ctx); }

struct CpuLanes {
  int id;
  mutable int parity = 0;
  const int64_t* exchange(int64_t v) const {
    int64_t* buf = value[parity];
    parity ^= 1;
    buf[id] = v;
    yield();
    return buf;
  }
  int lane() const { return id; }
  unsigned long long ballot(bool v) const {
    const int64_t* b = exchange(v);
    unsigned long long m = 0;
    for (int i = 0; i < N; ++i) m |= (unsigned long long)(b[i] != 0) << i;
    return m;
  }
  int first(int v) const { return (int)exchange(v)[0]; }
  int64_t from(int64_t v, int lane) const { return exchange(v)[lane]; }
  int from(int v, int lane) const { return (int)exchange(v)[lane]; }
  template <int D>
  uint32_t round(uint32_t v) const {
    return (uint32_t)exchange(v)[(id & 48) | ((id - D) & 15)];
  }
  void sync() const { exchange(0); }
};

struct CheckedWords {
  uint8_t w[gst::SCHED_CHAINS][gst::SCHED_WINDOW] = {};
  bool in(int c, int t) const {
    const bool ok = c >= 0 && c < gst::SCHED_CHAINS && t >= 0 && t < gst::SCHED_WINDOW;
    out_of_range += !ok;
    return ok;
  }
  uint8_t get(int c, int t) const { return in(c, t) ? w[c][t] : 0; }
  void put(int c, int t, uint8_t k) {
    if (in(c, t)) w[c][t] = k;
  }
};

const gst::SchedBuild* build;
int64_t tile_of = 0;
CheckedWords* words_of = nullptr;

void lane_main(int id) {
  gst::sched_tile(*build, tile_of, *words_of, CpuLanes{id});
  --running;
}

}  // namespace

extern "C" int64_t sched_at(int64_t steps_before, int64_t tile) { return gst::sched_at(steps_before, tile); }

// Runs every tile; returns the window accesses out of range.
extern "C" int64_t sched_cpu(const int64_t* off, const uint8_t* gates, const int64_t* order, int64_t S, int K,
                             int tile_seqs, const int64_t* tile_rec, int* tile_n, uint32_t* entries) {
  const gst::SchedBuild a{off, gates, order, S, K, tile_seqs, tile_rec, tile_n, entries};
  build = &a;
  out_of_range = 0;
  for (tile_of = 0; tile_of * tile_seqs < S; ++tile_of) {
    const auto words = std::make_unique<CheckedWords>();
    words_of = words.get();
    running = N;
    bool done[N] = {};
    for (int i = 0; i < N; ++i) {
      getcontext(&lane_ctx[i]);
      lane_ctx[i].uc_stack.ss_sp = &stacks[(size_t)i * STACK];
      lane_ctx[i].uc_stack.ss_size = STACK;
      lane_ctx[i].uc_link = &main_ctx;
      makecontext(&lane_ctx[i], reinterpret_cast<void (*)()>(lane_main), 1, i);
    }
    while (running > 0)
      for (current = 0; current < N; ++current) {
        if (done[current]) continue;
        const int before = running;
        swapcontext(&main_ctx, &lane_ctx[current]);
        done[current] = running < before;
      }
  }
  return out_of_range;
}
