#include <sys/mman.h>

extern "C" void emu_switch(void** save, void* to);
__asm__(R"(
.globl emu_switch
emu_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");

#include "hip/hip_runtime.h"
#undef asm

namespace emu {
namespace {
constexpr size_t kStack = 256 << 10;
struct Wave {
  Fiber lane[64];
  int n = 0;
  const char* what = nullptr;
  bool yielded = false;
  unsigned parity = 0;
  uint64_t value[2][64];
  Operands ops[2];
};
std::vector<Wave> waves;
std::vector<char*> stacks;
void* scheduler_sp;
const std::function<void()>* body;

Wave& my_wave() { return waves[cur->tid.x / 64]; }

void leave(State s) {
  Fiber* me = cur;
  me->state = s;
  emu_switch(&me->sp, scheduler_sp);
}

void entry() {
  (*body)();
  leave(kDone);
  fail("a finished thread ran again");
}
}  // namespace

void fail(const std::string& what) {
  std::fprintf(stderr, "%s\n  in kernel %p, workgroup %u, thread %u\n", what.c_str(),
               launches.empty() ? nullptr : launches.back().first, block_idx.x, cur ? cur->tid.x : 0);
  std::_Exit(3);
}

void wave_sync(const char* what) {
  Wave& w = my_wave();
  for (int l = 0; l < lane(); ++l)
    if (w.lane[l].state == kWave && w.what != what)
      fail(std::string("lanes of a wave apart: ") + w.what + " and " + what);
  w.what = what;
  leave(kWave);
}

void barrier() { leave(kBarrier); }

void yield() {
  my_wave().yielded = true;
  wave_sync("sleep");
}

uint64_t* exchange(uint64_t mine, const char* what) {
  Wave& w = my_wave();
  const unsigned p = w.parity & 1;  // the same for every lane: it changes only when all have arrived
  w.value[p][lane()] = mine;
  wave_sync(what);
  return w.value[p];
}

Operands* operands(const void* a, const void* b, size_t bytes, const char* what) {
  Wave& w = my_wave();
  const unsigned p = w.parity & 1;
  std::memcpy(w.ops[p].a[lane()], a, bytes);
  std::memcpy(w.ops[p].b[lane()], b, bytes);
  wave_sync(what);
  return &w.ops[p];
}

void assembly(const char* text) {
  if (std::strstr(text, "s_barrier")) barrier();
}

void run(const void* kernel_at, dim3 grid, dim3 block, const std::function<void()>& kernel) {
  launches.emplace_back(kernel_at, grid.x);
  body = &kernel;
  grid_dim = grid;
  block_dim = block;
  const int nw = (block.x + 63) / 64;
  while ((int)stacks.size() < (int)block.x)
    stacks.push_back((char*)mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  uint64_t rng = order * 0x9E3779B97F4A7C15ull + 1;
  for (unsigned b = 0; b < grid.x; ++b) {
    block_idx = dim3(b);
    waves.assign(nw, Wave());
    for (unsigned t = 0; t < block.x; ++t) {
      Wave& w = waves[t / 64];
      Fiber& f = w.lane[t % 64];
      w.n = t % 64 + 1;
      f.tid = dim3(t);
      f.state = kRunning;
      void** sp = (void**)(stacks[t] + kStack) - 2;
      *sp = (void*)entry;  // emu_switch returns here; the stack is aligned as after a call
      f.sp = sp - 6;
    }
    for (;;) {
      // Waves that can go on; a wave that waits for another one only when no other can.
      std::vector<int> ready, asleep;
      int live = 0, at_barrier = 0;
      for (int i = 0; i < nw; ++i) {
        Wave& w = waves[i];
        int run_ = 0, wave_ = 0, bar = 0, done = 0;
        for (int l = 0; l < w.n; ++l) {
          run_ += w.lane[l].state == kRunning;
          wave_ += w.lane[l].state == kWave;
          bar += w.lane[l].state == kBarrier;
          done += w.lane[l].state == kDone;
        }
        if (done == w.n) continue;
        ++live;
        if (wave_ > 0 && bar > 0) {
          cur = &w.lane[0];
          fail("lanes of a wave apart: a barrier and a cross-lane operation");
        }
        if (run_ == 0 && bar > 0) ++at_barrier;
        else (w.yielded ? asleep : ready).push_back(i);
      }
      if (live == 0) break;
      if (ready.empty() && asleep.empty()) {  // every live wave is at the barrier
        if (at_barrier != live) fail("the schedule is stuck");
        for (Wave& w : waves)
          for (int l = 0; l < w.n; ++l)
            if (w.lane[l].state == kBarrier) w.lane[l].state = kRunning;
        continue;
      }
      if (ready.empty()) {
        for (int i : asleep) waves[i].yielded = false;
        ready = asleep;
      }
      rng = rng * 6364136223846793005ull + 1442695040888963407ull;
      const int pick = order == 0 ? ready.front() : order == 1 ? ready.back() : ready[(rng >> 33) % ready.size()];
      Wave& w = waves[pick];
      // On to a barrier, the end, or a sleep; in a pseudo-random schedule also anywhere between.
      for (bool on = true; on;) {
        bool any = false;
        for (int l = 0; l < w.n; ++l) any |= w.lane[l].state == kRunning;
        if (!any) {  // all arrived at the cross-lane operation
          ++w.parity;
          for (int l = 0; l < w.n; ++l)
            if (w.lane[l].state == kWave) w.lane[l].state = kRunning;
        }
        bool other = false;
        for (int l = 0; l < w.n; ++l)
          if (w.lane[l].state == kRunning) {
            cur = &w.lane[l];
            emu_switch(&scheduler_sp, cur->sp);
            other |= cur->state != kWave;
          }
        rng = rng * 6364136223846793005ull + 1442695040888963407ull;
        on = !other && !w.yielded && (order <= 1 || (rng >> 33) % 8 != 0);
      }
      cur = nullptr;
    }
  }
}

}  // namespace emu
