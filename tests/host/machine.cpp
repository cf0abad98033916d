// The machine behind hip/hip_runtime.h: fibers, rendezvous, LDS.
#include <hip/hip_runtime.h>
#include <sanitizer/asan_interface.h>

namespace nwm {
constexpr size_t LDS = 163840, PAST = 4096;
alignas(4096) char host_lds[LDS + PAST];   // dynamic LDS
}  // namespace nwm

extern "C" void wave_switch(void **save, void *load);
asm(R"(
.text
.globl wave_switch
wave_switch:
  push %rbp; push %rbx; push %r12; push %r13; push %r14; push %r15
  mov %rsp, (%rdi)
  mov %rsi, %rsp
  pop %r15; pop %r14; pop %r13; pop %r12; pop %rbx; pop %rbp
  ret
)");

namespace wave {
dim3 thread_idx, block_idx, block_dim, grid_dim;
enum State { READY, WAVE, BLOCK, DONE };
struct Lane {
  void *sp;
  State st;
  int ops;            // cross-lane operations so far
  const char *what;   // the one it waits at
  int line;
};
constexpr size_t STACK = 1 << 19;
static std::vector<char *> stacks;
static std::vector<Lane> lanes;
static std::vector<std::vector<char>> buffers;   // per wave, for two operations in turn
static std::vector<uint64_t> took_part;          // lanes in the wave's last operation
static void *scheduler;
static int cur;
static const std::function<void()> *body;

static void yield(State s) {
  lanes[cur].st = s;
  wave_switch(&lanes[cur].sp, scheduler);
}
static void entry() {
  (*body)();
  yield(DONE);
  std::abort();
}
int lane() { return cur & 63; }
uint64_t live() { return took_part[cur >> 6]; }
char *exchange_buffer() { return buffers[cur >> 6].data() + (lanes[cur].ops & 1) * 64 * 64; }
void sync_wave(const char *what, int line) {
  lanes[cur].what = what;
  lanes[cur].line = line;
  ++lanes[cur].ops;
  yield(WAVE);
}
void sync_block() { yield(BLOCK); }

[[noreturn]] static void stop(const char *kernel, const char *why, const Lane &a, const Lane &b) {
  std::fprintf(stderr, "%s, workgroup %u: %s (%s, line %d; %s, line %d)\n", kernel, block_idx.x, why,
               a.what ? a.what : "barrier", a.line, b.what ? b.what : "barrier", b.line);
  std::abort();
}

// With HOST_ORDER set the waves of a workgroup, and the lanes of a wave, run in
// another order at every turn: a result that depends on it is a race.
static uint64_t turn = 0;
static int place(int k, int n) {   // k-th of n
  if (!turn) return k;
  const uint64_t a = (turn >> 20) % (uint64_t)n;
  return (turn >> 40) & 1 ? (int)((a + n - (uint64_t)k) % n) : (int)((a + (uint64_t)k) % n);
}
static void next_turn() { turn = turn * 6364136223846793005ull + 1442695040888963407ull; }

void launch(const char *name, dim3 g, dim3 b, size_t lds, const std::function<void()> &f) {
  grid_dim = g;
  block_dim = b;
  body = &f;
  const int T = (int)b.x, W = (T + 63) / 64;
  const char *seed = std::getenv("HOST_ORDER");
  turn = seed ? std::strtoull(seed, nullptr, 10) * 0x9E3779B97F4A7C15ull + 1 : 0;
  while ((int)stacks.size() < T) stacks.push_back((char *)aligned_alloc(64, STACK));
  took_part.assign(W, 0);
  buffers.assign(W, std::vector<char>(2 * 64 * 64));
  __asan_unpoison_memory_region(nwm::host_lds, nwm::LDS + nwm::PAST);
  std::memset(nwm::host_lds, 0xA5, nwm::LDS);
  lds = (lds + 7) / 8 * 8;
  __asan_poison_memory_region(nwm::host_lds + lds, nwm::LDS + nwm::PAST - lds);
  for (unsigned blk = 0; blk < g.x; ++blk) {
    block_idx.x = blk;
    lanes.assign(T, Lane{});
    for (int t = 0; t < T; ++t) {
      __asan_unpoison_memory_region(stacks[t], STACK);
      void **sp = (void **)(stacks[t] + STACK - 64);
      *--sp = nullptr;
      *--sp = (void *)entry;
      for (int k = 0; k < 6; ++k) *--sp = nullptr;
      lanes[t].sp = sp;
    }
    for (bool more = true; more;) {
      more = false;
      if (turn) next_turn();
      const uint64_t of_waves = turn;
      for (int v = 0; v < W; ++v) {
        const uint64_t of_lanes = turn;
        turn = of_waves;
        const int w = place(v, W), a = 64 * w, e = std::min(T, a + 64);
        turn = of_lanes;
        for (;;) {
          if (turn) next_turn();
          for (int k = 0; k < e - a; ++k) {
            const int t = a + place(k, e - a);
            if (lanes[t].st == READY) {
              cur = t;
              thread_idx.x = (unsigned)t;
              wave_switch(&scheduler, lanes[t].sp);
            }
          }
          int first = -1, waits = 0;
          for (int t = a; t < e; ++t) {
            const Lane &l = lanes[t];
            if (l.st == BLOCK) ++waits;
            if (l.st != WAVE) continue;
            if (first < 0) first = t;
            else if (l.line != lanes[first].line || l.what != lanes[first].what)
              stop(name, "lanes of a wave at different operations", l, lanes[first]);
          }
          if (first >= 0 && waits > 0) stop(name, "some lanes of a wave at a barrier", lanes[first], Lane{});
          more = more || waits > 0;
          if (first < 0) break;
          took_part[w] = 0;
          for (int t = a; t < e; ++t)
            if (lanes[t].st == WAVE) lanes[t].st = READY, took_part[w] |= 1ull << (t & 63);
        }
      }
      for (Lane &l : lanes)
        if (l.st == BLOCK) l.st = READY;
    }
  }
}
}  // namespace wave

// float -> bfloat16, nearest even (the compiler's own call on this host)
extern "C" __bf16 __truncsfbf2(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  const uint16_t r = (u & 0x7FFFFFFFu) > 0x7F800000u ? (uint16_t)(u >> 16 | 0x40u)
                                                      : (uint16_t)((u + 0x7FFFu + (u >> 16 & 1u)) >> 16);
  __bf16 b;
  std::memcpy(&b, &r, 2);
  return b;
}
